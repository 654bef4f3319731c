"""kv_append on either side of the size from which new rows are stored the
ordinary way: bitwise equal to an indexed assignment, also for the attention that reads
them on the same stream right after."""
import numpy as np
import pytest

import workloads as W
from paper_2606_12688_amd import attn
from tests.helpers import plan_for, run_gpu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows", [1, 17, 8192, 8193])  # 4 KB per row and step: 32 MB is 8192 rows
def test_both_store_paths(rows):
    import torch

    b = W.custom("append_sizes", 8, 8, 128, [rows], [rows + 50], [[(0, rows + 50, W.SEG_CAUSAL, 0)]], [64], seed=rows)
    t = W.make_tensors_torch(b, DEV)
    shape = (rows, 8, 128)
    g = torch.Generator(device=DEV).manual_seed(rows)
    kn, vn = (torch.randn(shape, generator=g, device=DEV).bfloat16() for _ in range(2))
    bt = torch.from_numpy(np.ascontiguousarray(b.block_table)).to(DEV)
    want = {n: t[n].clone() for n in ("k_pages", "v_pages")}
    pos = torch.arange(50, 50 + rows, device=DEV)
    page = bt[0].long()[pos // 16]
    want["k_pages"][page, pos % 16], want["v_pages"][page, pos % 16] = kn, vn
    pl = plan_for(b)
    out, lse = torch.empty_like(t["q"]), torch.empty(t["q"].shape[:2], device=DEV)
    attn.kv_append(pl, kn, vn, bt, t["k_pages"], t["v_pages"])
    attn.fwd(pl, t["q"], t["k_pages"], t["v_pages"], bt, out, lse, attn.workspace(pl, DEV))
    assert attn.check(pl) == 0
    for n in want:
        assert torch.equal(t[n].view(torch.int16), want[n].view(torch.int16))
    ref, ref_lse = run_gpu(b, dict(t, **want))
    assert torch.equal(out, ref) and torch.equal(lse, ref_lse)
