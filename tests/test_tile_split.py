"""How multi-row items are cut into key pieces (CPU only): longer pieces than the
ordinary 1024 keys or more are cheaper by the planner's own measure, worked
out here from the plan's items, or keep partials within the static scratch."""
import itertools

import pytest

import workloads as W
from paper_2606_12688_amd import attn
from tests.helpers import plan_for

CUS, SCRATCH = 256, 32 << 20


def cdiv(a, b):
    return -(-a // b)


def _cost(items, hq, hkv, d, few=(0, 0)):
    """(without key groups, with them) of tile items (keys, rows, partial): keys
    walked by a CU's waves together."""
    G = hq // hkv
    wgs = [hkv * (G if r == 128 else cdiv(r * G, 128)) for _, r, _ in items]
    work = sum(n * w for (n, _, _), w in zip(items, wgs))
    rows = sum(r * hq for _, r, partial in items if partial)
    merge = 400 + rows // (70 if d == 64 else 55) if rows else 0
    piece = max(n for n, _, _ in items)
    held = max(0, min(CUS, few[0]) + len(items) * hq - CUS)
    return (max(cdiv(sum(wgs), CUS) * work // sum(wgs), piece + piece // 2) + merge,
            piece + merge + held * (400 + few[1] // 200) // CUS)


def _batch(reqs, hq, hkv, d):
    q, kv, win = ([r[k] for r in reqs] for k in range(3))
    return W.custom("split", hq, hkv, d, q, kv, [[(0, n, W.SEG_CAUSAL, 0)] for n in kv], win)


def _plan(b, flags=0):
    """Tile items (keys, rows, partial), launch slots, few-row items and their
    keys, bytes of partials."""
    pl = plan_for(b, attn.FLAG_HOST_ONLY | flags)
    t, f = pl.items(0).tolist(), pl.items(1)
    got = [(w[5] - w[4], w[3], w[6] >= 0) for w in t], len(pl.tile_order()), (len(f), int((f[:, 5] - f[:, 4]).sum())), \
        pl.workspace_bytes
    pl.destroy()
    return got


def _ordinary(units):
    """The units in equal pieces of about 1024 keys."""
    chunk = cdiv(max(1024, cdiv(sum(n for n, _, _ in units), 1024)), 64) * 64
    out = []
    for n, r, _ in units:
        if n > chunk:
            size = cdiv(cdiv(n, cdiv(n, chunk)), 64) * 64
            out += [(min(size, n - at), r, True) for at in range(0, n, size)]
        else:
            out.append((n, r, False))
    return out


def _check(reqs, hq, hkv, d):
    b = _batch(reqs, hq, hkv, d)
    items, slots, few, _ = _plan(b)
    units = _plan(b, attn.FLAG_NO_SPLIT)[0]
    if len(units) * hq >= 512:
        assert sorted(items) == sorted(units)
        return
    ordinary = _ordinary(units)
    if sorted(items) == sorted(ordinary):
        return
    limit = _cost(ordinary, hq, hkv, d)[0]
    plain, groups = _cost(items, hq, hkv, d, few)
    bytes_ordinary = sum(r * hq for _, r, p in ordinary if p) * (d + 1) * 4
    assert plain <= limit or (slots <= CUS and groups < limit) or bytes_ordinary > SCRATCH // 2, \
        (reqs, plain, groups, limit, slots)


@pytest.mark.parametrize("reqs,heads", [
    ([(20, 8000, 0)] * 15, (28, 4, 128)), ([(16, 16000, 0)] * 12, (28, 4, 128)), ([(20, 8000, 4000)] * 8, (28, 4, 128)),
    ([(128, 6000, 0)] * 3, (28, 4, 128)), ([(300, 12000, 0)], (16, 8, 64)),
    ([(1829, 1829, 0)] + [(1, 4000, 0)] * 64, (16, 8, 64))])
def test_longer_pieces_are_cheaper(reqs, heads):
    _check(reqs, *heads)


@pytest.mark.parametrize("hq,hkv,d", [(28, 4, 128), (8, 2, 128), (16, 8, 64), (16, 16, 64)])
@pytest.mark.parametrize("n", [1, 3])
def test_longer_pieces_are_cheaper_over_lengths(hq, hkv, d, n):
    for q, kv, win in itertools.product((65, 128, 300, 640, 1100), (1500, 4000, 12000, 32000), (0, 2000)):
        _check([(q, max(q, kv), win)] * n, hq, hkv, d)


@pytest.mark.parametrize("reqs,heads", [
    ([(640, 8000, 0)], (28, 4, 128)), ([(640, 20000, 0)], (28, 4, 128)), ([(1100, 32000, 0)], (16, 8, 64)),
    ([(1327, 8881, 0), (162, 3774, 2000)], (16, 8, 128))])
def test_long_units_are_cut_evenly_within_the_scratch(reqs, heads):
    """Requests whose pieces of 1024 keys would write 40-190 MB of partials:
    pieces that fit the scratch, several workgroups for each CU."""
    items, slots, _, workspace = _plan(_batch(reqs, *heads))
    assert workspace <= SCRATCH and slots > CUS
    n = [k for k, _, _ in items]
    assert max(n) < 9000 and max(n) * len(n) <= 1.4 * sum(n)


def test_long_equal_pieces_for_key_groups():
    """256 rows over 32000 keys at 8/2 heads: 16 pieces of 2048 keys for each
    of two row tiles fill the 256 slots."""
    items, slots, _, _ = _plan(_batch([(256, 32000, 0)], 8, 2, 128))
    assert max(n for n, _, _ in items) == 2048 and slots == 256
