"""How few-row units are cut into key pieces (CPU only): about one piece per
workgroup slot of the GPU, never so many that a plan outgrows the static
scratch of the allocation-free entry point when fewer pieces fit."""
import numpy as np
import pytest

import workloads as W
from paper_2606_12688_amd import attn
from tests.helpers import plan_for

SCRATCH = 32 << 20


@pytest.mark.parametrize("d,slots,least", [(128, 768, 256), (64, 1280, 384)])
def test_pieces_fill_the_slots_once(d, slots, least):
    b = W.decode_bf16(seed=2, n=64, hq=28, hkv=4, d=d, pool_pages=None)
    pl = plan_for(b, attn.FLAG_HOST_ONLY)
    it = pl.items(1)
    keys = it[:, 5] - it[:, 4]
    units = 64 * 4
    total = int(keys.sum())
    want = -(-max(least, -(-total // slots)) // 128) * 128
    assert keys.max() == want
    assert len(it) <= slots + units
    pl.destroy()
    small = W.decode_bf16(seed=2, n=2, hq=28, hkv=4, d=d, pool_pages=None)
    pl = plan_for(small, attn.FLAG_HOST_ONLY)
    it = pl.items(1)
    assert (it[:, 5] - it[:, 4]).max() == least
    pl.destroy()


def test_a_plan_that_fits_the_scratch_with_fewer_pieces_gets_fewer():
    """Units of 64 rows that about 1280 pieces would cut into three each at D =
    64, beside a shared-prefix decode whose prefix partials take 7 MB: together
    past the static scratch, so the units are cut into fewer pieces."""
    G, hkv, n, m, prefix = 8, 3, 200, 40, 4096
    q = [8] * n + [1] * m
    # one long unit: near-equal ones would stay whole
    kv = [14000] + [7000] * (n - 1) + [prefix + 16] * m
    segs = [[(0, x, W.SEG_CAUSAL, 0)] for x in kv]
    b = W.custom("scratch", G * hkv, hkv, 64, q, kv, segs, [0] * (n + m))
    for r in range(n + 1, n + m):
        b.block_table[r, :prefix // 16] = b.block_table[n, :prefix // 16]
    b.prefix_groups = [(list(range(n, n + m)), prefix)]
    pl = plan_for(b, attn.FLAG_HOST_ONLY, cascade=True)
    it = pl.items(1)
    keys = it[:, 5] - it[:, 4]
    total = 3 * (14000 + 7000 * (n - 1)) + 16 * m * hkv
    fine = -(-(-(-total // 1280)) // 128) * 128
    pieces = 3 * (n - 1) * -(-7000 // fine) + 3 * -(-14000 // fine)
    prefix_rows = len(pl.items(4))  # 128-row items at most
    assert (pieces * 64 + m * G * hkv * (1 + prefix // 160)) * 260 > SCRATCH > 0 and prefix_rows > 0
    assert keys.max() > fine
    assert 0 < pl.workspace_bytes <= SCRATCH
    pl.destroy()


@pytest.mark.parametrize("d", [64, 128])
def test_a_plan_past_the_scratch_either_way_keeps_its_pieces(d):
    """Decode steps beside a 1200-token chunk over 60000 keys, whose own partials
    take hundreds of megabytes: fewer few-row pieces would not make them fit."""
    q, kv = [1] * 64, [4000] * 64
    keys = []
    for n in (0, 1):
        q, kv = q + [1200] * n, kv + [60000] * n
        b = W.custom("past", 28, 4, d, q, kv, [[(0, x, W.SEG_CAUSAL, 0)] for x in kv], [0] * len(q))
        pl = plan_for(b, attn.FLAG_HOST_ONLY)
        it = pl.items(1)
        keys.append(sorted((it[:, 5] - it[:, 4]).tolist()))
        assert (pl.workspace_bytes > SCRATCH) == bool(n)
        pl.destroy()
    assert keys[0] == keys[1]


@pytest.mark.parametrize("n,whole", [(30, False), (60, True)])
def test_near_equal_units_of_many_rows_split_evenly(n, whole):
    """16-token chunks of 32 rows under one window: equal pieces, no short
    remainder, and none at all once the units alone come close to a round."""
    b = W.stream_window_bf16(seed=1, n=n)
    pl = plan_for(b, attn.FLAG_HOST_ONLY)
    it = pl.items(1)
    keys = it[:, 5] - it[:, 4]
    assert (len(it) == 8 * n) == whole
    assert keys.min() * 4 >= keys.max() * 3
    pl.destroy()
