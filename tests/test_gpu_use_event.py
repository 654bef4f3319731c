"""Every kind of call marks its plan's device buffer as in use until its last
kernel is done: behind a stream that is held up, a plan is used and destroyed
at once, and another plan that takes its buffer is uploaded on another stream
meanwhile.  Without the mark the upload would overwrite the first plan's work
list before its kernels read it."""
import numpy as np
import pytest

import workloads as W
from paper_2606_12688_amd import attn
from tests.helpers import plan_for, run_gpu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# the last kernel of the call: tiles, few-row, fp32, merge, cascade + merge,
# the wait for the side stream (tiles beside few-row items, nothing merged)
KINDS = {"tiles": ("text_latent_bf16", attn.FLAG_NO_SPLIT, False), "few": ("decode_bf16", attn.FLAG_NO_SPLIT, False),
         "f32": ("tiny_causal_f32", 0, False), "merge": ("decode_bf16", attn.FLAG_FORCE_SPLIT, False),
         "cascade": ("shared_prefix_decode_bf16", 0, True), "forked": ("mixed", attn.FLAG_NO_SPLIT, False),
         "append": ("decode_bf16", attn.FLAG_NO_SPLIT, False)}


def _other(name):
    """Another batch for the same buffer whose work list differs: where the seed
    does not change it, one of a little less work."""
    if name == "text_latent_bf16":
        return W.text_latent_bf16(7, n=2, text=29, latent=290)
    if name == "tiny_causal_f32":
        lens = [int(n) - 1 for n in W.reduced(name).seqs[:, 1]]
        return W.custom("tiny_other", 2, 1, 64, lens, lens, [[(0, n, W.SEG_CAUSAL, 0)] for n in lens], [0] * len(lens),
                        dtype="f32")
    if name == "shared_prefix_decode_bf16":
        return W.shared_prefix_decode_bf16(7, n=36, prefix=320, own_min=1, own_max=150, hq=8, hkv=2)
    return W.reduced(name, seed=7)


def _work(b, flags, cascade):
    """The items of every kind of a plan whose device buffer has the smallest size."""
    pl = plan_for(b, flags | attn.FLAG_HOST_ONLY, cascade=cascade)
    assert pl.stats()["device_bytes"] <= 64 << 10
    lists = [pl.items(k) for k in range(5)]
    pl.destroy()
    return lists


@pytest.mark.parametrize("kind", list(KINDS))
def test_next_plan_waits_for_the_last_kernel(kind):
    import torch

    name, flags, cascade = KINDS[kind]
    b = W.reduced(name)
    other = _other(name)
    mine, others = (_work(x, flags, cascade) for x in (b, other))
    # the items that the call's last kernels read (the append's follow from the requests)
    last = {"tiles": 0, "few": 1, "f32": 2, "merge": 3, "cascade": 3, "forked": 1}
    if kind == "append":
        assert (b.seqs != other.seqs).any()
    else:
        assert not np.array_equal(mine[last[kind]], others[last[kind]])
    t = W.make_tensors_torch(b, DEV)
    ref, ref_lse = run_gpu(b, t, flags, cascade=cascade)
    stream, upload = torch.cuda.current_stream(), torch.cuda.Stream()
    bt = torch.from_numpy(np.ascontiguousarray(b.block_table)).to(DEV)
    out, lse = torch.zeros_like(ref), torch.zeros_like(ref_lse)
    shape = (b.total_q, b.num_kv_heads, b.head_dim)
    kn, vn = (torch.randn(shape, device=DEV).to(t["q"].dtype) for _ in range(2))
    pages = [t["k_pages"].clone(), t["v_pages"].clone()]
    pl = plan_for(b, flags, stream, cascade=cascade)
    if kind == "append":
        attn.kv_append(pl, kn, vn, bt, *pages)
        want = [x.clone() for x in pages]
        pages[0].copy_(t["k_pages"]), pages[1].copy_(t["v_pages"])
    ws = attn.workspace(pl, DEV)
    torch.cuda.synchronize()
    torch.cuda._sleep(20_000_000)  # some 10 ms
    if kind == "append":
        attn.kv_append(pl, kn, vn, bt, *pages)
    else:
        attn.fwd(pl, t["q"], t["k_pages"], t["v_pages"], bt, out, lse, ws, stream)
    pl.destroy()
    nxt = plan_for(other, flags, upload, cascade=cascade)
    torch.cuda.synchronize()
    nxt.destroy()
    if kind == "append":
        assert all(torch.equal(x.view(torch.int16), y.view(torch.int16)) for x, y in zip(pages, want))
    else:
        assert torch.equal(out, ref) and torch.equal(lse, ref_lse)
