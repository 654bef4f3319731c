"""GPU parity of tile items that are not full: their (query row, head) pairs
are shared out as 128-row slices of a KV head's group, with slices that end
inside a query row's heads, empty last slices, windows that move a slice's
first key, and key pieces that a slice does not reach.

Tolerances as in the other parity tests."""
import pytest

import workloads as W
from paper_2606_12688_amd import attn
from tests.helpers import compare, oracle_of, run_gpu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("flag", [0, attn.FLAG_FORCE_SPLIT, attn.FLAG_NO_SPLIT])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(2, 1), (14, 2), (5, 1), (33, 1), (4, 4)])
def test_slices(hq, hkv, d, flag):
    G = hq // hkv
    q = [64 // G + 1, 128 // G, 128 // G + 1, 127, 129, 100, 70]
    q = [max(65, x) if G == 1 else x for x in q]
    kv = [q[0], q[1] + 37, q[2] + 400, 127, 129 + 64, 900, 333]
    segs = [[(0, n, W.SEG_CAUSAL, 0)] for n in kv]
    segs[5] = [(0, 500, W.SEG_FULL, 0), (500, 400, W.SEG_BLOCKS, 48)]
    b = W.custom("packed", hq, hkv, d, q, kv, segs, [0, 0, 50, 0, 20, 0, 200], seed=hq + d,
                 pool_pages=sum((n + 15) // 16 for n in kv) + 3)
    t = W.make_tensors_torch(b, DEV, poison_unused=True)
    out, lse = run_gpu(b, t, flag, out_fill=float("nan"))
    compare(b, out, lse, *oracle_of(b, t), f"packed tiles {hq}/{hkv} d{d} flags {flag}")


@pytest.mark.parametrize("hq", [4096, 4097])
def test_largest_group_of_the_reciprocal_and_one_more(hq):
    """Groups above 4096 heads keep one head per workgroup."""
    b = W.custom("packed_group", hq, 1, 64, [1, 2], [40, 33],
                 [[(0, 40, W.SEG_CAUSAL, 0)], [(0, 33, W.SEG_CAUSAL, 0)]], [0, 0], seed=1)
    t = W.make_tensors_torch(b, DEV)
    compare(b, *run_gpu(b, t, out_fill=float("nan")), *oracle_of(b, t), f"packed tiles group {hq}")
