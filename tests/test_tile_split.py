"""How multi-row items are cut into key pieces (CPU only).  Pieces longer than
the ordinary ones are for launches whose workgroups share their keys among
groups of waves: at most 256 launch slots, those without rows and few-row items beside them included."""
import itertools

import pytest

import workloads as W
from paper_2606_12688_amd import attn
from tests.helpers import plan_for

HEADS = [(28, 4, 128), (8, 2, 128), (16, 8, 64), (16, 16, 64)]


def _pieces(reqs, hq, hkv, d, flags=0):
    q, kv, win = ([r[k] for r in reqs] for k in range(3))
    b = W.custom("split", hq, hkv, d, q, kv, [[(0, n, W.SEG_CAUSAL, 0)] for n in kv], win)
    pl = plan_for(b, attn.FLAG_HOST_ONLY | flags)
    whole = plan_for(b, attn.FLAG_HOST_ONLY | attn.FLAG_NO_SPLIT)
    span = lambda p: p.items(0)[:, 5] - p.items(0)[:, 4]
    longest, total, units = span(pl).max(), span(whole).sum(), len(whole.items(0))
    slots, few = len(pl.tile_order()), len(pl.items(1))
    ordinary = -(-max(1024, -(-int(total) // 1024)) // 64) * 64
    pl.destroy()
    whole.destroy()
    return int(longest), ordinary, slots, few, units


@pytest.mark.parametrize("reqs,heads", [
    ([(20, 8000, 0)] * 15, (28, 4, 128)), ([(16, 16000, 0)] * 12, (28, 4, 128)), ([(20, 8000, 4000)] * 8, (28, 4, 128)),
    ([(640, 8000, 0)], (28, 4, 128)), ([(640, 20000, 0)], (28, 4, 128)), ([(1100, 32000, 0)], (16, 8, 64))])
def test_launches_without_key_groups_keep_the_ordinary_pieces(reqs, heads):
    longest, ordinary, _, _, _ = _pieces(reqs, *heads)
    assert longest <= ordinary


@pytest.mark.parametrize("hq,hkv,d", HEADS)
@pytest.mark.parametrize("n", [1, 3])
def test_longer_pieces_only_for_key_groups(hq, hkv, d, n):
    for q, kv, win in itertools.product((65, 128, 300, 640, 1100), (1500, 4000, 12000, 32000), (0, 2000)):
        longest, ordinary, slots, few, units = _pieces([(q, max(q, kv), win)] * n, hq, hkv, d)
        if longest > ordinary and units * hq < 512:
            assert slots + few <= 256, (q, kv, win)


def test_long_equal_pieces_for_key_groups():
    """256 rows over 32000 keys at 8/2 heads: 16 pieces of 2048 keys for each
    of two row tiles fill the 256 slots."""
    longest, ordinary, slots, _, _ = _pieces([(256, 32000, 0)], 8, 2, 128)
    assert longest > ordinary and slots == 256


@pytest.mark.parametrize("n,flags,same", [(0, 0, True), (8, 0, False), (8, attn.FLAG_SERIAL, True)])
def test_few_row_work_beside_the_tiles_counts(n, flags, same):
    """Two prompts of 1846 tokens fill the 256 slots whole; decode steps beside
    them leave no CU to each."""
    assert (_pieces([(1846, 1846, 0)] * 2 + [(1, 2000, 0)] * n, 8, 2, 128, flags)[0] == 1846) == same
