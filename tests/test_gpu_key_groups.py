"""GPU parity of the tile kernel's key groups: small launches of long items,
whose waves share the keys in runs of tiles; slices with fewer tiles than
groups, runs that do not divide evenly, windows, a pool past 2 GB.

Tolerances as in the other parity tests."""
import pytest

import workloads as W
from paper_2606_12688_amd import attn
from tests.helpers import compare, oracle_of, plan_for, run_gpu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _batch(hq, hkv, d, pool_pages=None):
    q = [700, 130, 150, 90]
    kv = [700, 1500, 666, 817]
    segs = [[(0, 700, W.SEG_CAUSAL, 0)], [(0, 1400, W.SEG_FULL, 0), (1400, 100, W.SEG_BLOCKS, 30)],
            [(0, 666, W.SEG_CAUSAL, 0)], [(0, 817, W.SEG_FULL, 0)]]
    return W.custom("groups", hq, hkv, d, q, kv, segs, [0, 0, 300, 100], seed=hq + d, pool_pages=pool_pages)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(2, 2), (7, 1), (6, 2)])
def test_runs_of_tiles(hq, hkv, d):
    b = _batch(hq, hkv, d)
    pl = plan_for(b, attn.FLAG_HOST_ONLY)
    it = pl.items(0)
    assert len(pl.tile_order()) <= 256 and (it[:, 5] - it[:, 4]).max() >= 640  # the rule for key groups
    pl.destroy()
    t = W.make_tensors_torch(b, DEV, poison_unused=True)
    for flag in (0, attn.FLAG_NO_SPLIT):
        out, lse = run_gpu(b, t, flag, out_fill=float("nan"))
        compare(b, out, lse, *oracle_of(b, t), f"key groups {hq}/{hkv} d{d} flags {flag}")


def test_growing_scores():
    """Keys scaled by position: the groups end with very different references."""
    b = _batch(2, 2, 64)
    t = W.make_tensors_torch(b, DEV)
    k = t["k_pages"]
    for r in range(b.num_seqs):
        for p in range((int(b.seqs[r, 1]) + 15) // 16):
            k[int(b.block_table[r, p])] *= 1 + 0.02 * p
    compare(b, *run_gpu(b, t), *oracle_of(b, t), "key groups, growing scores", rel_o=2.0 ** -8)


def test_pool_past_2_gb():
    import torch

    b = _batch(8, 8, 128, pool_pages=66000)  # 32 KB pages: 2.16 GB of K and of V
    g = torch.Generator(device=DEV).manual_seed(1)
    shape = (b.num_pages, 16, b.num_kv_heads, b.head_dim)
    t = {"q": torch.randn((b.total_q, 8, 128), generator=g, device=DEV).bfloat16(),
         "k_pages": torch.randn(shape, generator=g, device=DEV, dtype=torch.bfloat16),
         "v_pages": torch.randn(shape, generator=g, device=DEV, dtype=torch.bfloat16)}
    out, lse = run_gpu(b, t, attn.FLAG_NO_SPLIT)
    from oracle import oracle_attention

    sb, q, kp, vp, rows = W.extract_requests(b, t, range(b.num_seqs))
    compare(b, out, lse, *oracle_attention(sb, q, kp, vp), "key groups, pool past 2 GB")


@pytest.mark.parametrize("d", [64, 128])
def test_beside_few_row_items(d):
    """Key groups on the caller's stream, a little few-row work on the side stream."""
    b = W.custom("groups_few", 4, 2, d, [900, 1, 1], [900, 300, 77], [[(0, n, W.SEG_CAUSAL, 0)] for n in (900, 300, 77)],
                 [0, 0, 0], seed=d)
    t = W.make_tensors_torch(b, DEV, poison_unused=True)
    for flag in (0, attn.FLAG_SERIAL):
        out, lse = run_gpu(b, t, flag, out_fill=float("nan"))
        compare(b, out, lse, *oracle_of(b, t), f"key groups beside few rows d{d} flags {flag}")


def test_long_pieces_without_groups():
    """Partials of 1024-key pieces would pass the static scratch: longer ones."""
    b = W.custom("long_pieces", 28, 4, 128, [640], [8000], [[(0, 8000, W.SEG_CAUSAL, 0)]], [0], seed=5)
    pl = plan_for(b, attn.FLAG_HOST_ONLY)
    it = pl.items(0)
    assert (it[:, 5] - it[:, 4]).max() > 1024 and (it[:, 6] >= 0).all() and len(pl.tile_order()) > 256
    pl.destroy()
    t = W.make_tensors_torch(b, DEV)
    compare(b, *run_gpu(b, t, out_fill=float("nan")), *oracle_of(b, t), "long pieces")
