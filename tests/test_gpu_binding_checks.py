"""The binding refuses every tensor that does not match the plan, whichever
argument it is, and takes the calls that do."""
import numpy as np
import pytest

import workloads as W
from paper_2606_12688_amd import attn
from tests.helpers import plan_for

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FWD = ["q", "k_pages", "v_pages", "block_table", "out", "lse"]
APPEND = ["k_new", "v_new", "block_table", "k_pages", "v_pages"]


def _wrong(t):
    import torch

    yield "device", t.cpu()
    yield "shape", torch.cat([t, t])
    yield "strides", torch.stack([t, t], -1)[..., 0]
    yield "dtype", t.to(torch.float16 if t.is_floating_point() else torch.int64)


@pytest.mark.parametrize("call,names", [("fwd", FWD), ("fwd_noalloc", FWD), ("kv_append", APPEND)])
def test_every_mismatch_is_refused(call, names):
    import torch

    b = W.reduced("decode_bf16")
    t = W.make_tensors_torch(b, DEV)
    pl = plan_for(b)
    ws = attn.workspace(pl, DEV)
    new = torch.zeros((b.total_q, b.num_kv_heads, b.head_dim), dtype=torch.bfloat16, device=DEV)
    good = dict(t, block_table=torch.from_numpy(np.ascontiguousarray(b.block_table)).to(DEV), k_new=new, v_new=new,
                out=torch.empty_like(t["q"]), lse=torch.empty(t["q"].shape[:2], device=DEV))
    extra = (ws,) if call == "fwd" else ()
    fn = getattr(attn, call)
    fn(pl, *(good[n] for n in names), *extra)
    for n in names:
        for what, bad in _wrong(good[n]):
            with pytest.raises(ValueError):
                fn(pl, *(bad if m == n else good[m] for m in names), *extra)
                pytest.fail(f"{call}: {n} with the wrong {what} was taken")
    assert attn.check(pl) == 0
    pl.destroy()
    with pytest.raises(ValueError):
        fn(pl, *(good[n] for n in names), *extra)
