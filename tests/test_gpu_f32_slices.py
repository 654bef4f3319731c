"""GPU parity of the fp32 kernel at the edges of its work split: 16-row slices
of (query row, head) pairs, 16-key steps dealt to four waves, page indices held
64 steps at a time.

Tolerances as in the other parity tests: 1e-5 (out) and 1e-3 (lse) on
unit-variance inputs."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import compare, host64, oracle_of, run_gpu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _batch(name, hq, hkv, d, q_lens, kv_lens, windows, seed=0):
    segs = [[(0, n // 3, W.SEG_CAUSAL, 0), (n // 3, n - n // 3, W.SEG_BLOCKS, 5)] if k % 2 else
            [(0, n, W.SEG_CAUSAL, 0)] for k, n in enumerate(kv_lens)]
    return W.custom(name, hq, hkv, d, q_lens, kv_lens, segs, windows, seed=seed, dtype="f32",
                    pool_pages=sum((n + 15) // 16 for n in kv_lens) + 5)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(2, 2), (3, 1), (14, 2), (17, 1)])
def test_slices_and_steps(hq, hkv, d):
    q = [1, 15, 16, 17, 33, 1, 40]
    kv = [1, 15, 16, 49, 33, 130, 300]
    b = _batch("f32_slices", hq, hkv, d, q, kv, [0, 0, 0, 7, 0, 40, 64])
    t = W.make_tensors_torch(b, DEV, poison_unused=True)
    compare(b, *run_gpu(b, t, out_fill=float("nan")), *oracle_of(b, t), f"f32 slices {hq}/{hkv} d{d}")


def test_more_steps_than_one_page_window():
    """A wave takes every fourth page: 64 steps of it span 4096 keys."""
    b = _batch("f32_long", 4, 2, 64, [1, 20], [4097, 8300], [0, 0])
    t = W.make_tensors_torch(b, DEV, poison_unused=True)
    compare(b, *run_gpu(b, t), *oracle_of(b, t), "f32 long")


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("d", [64, 128])
def test_values_of_hidden_keys_stay_out(d, bad):
    """A value that is not finite reaches exactly the rows that see its key,
    although rows that do not share its matrix products."""
    n, at, window = 40, 21, 9
    b = W.custom("f32_hidden", 4, 2, d, [n], [n], [[(0, n, W.SEG_CAUSAL, 0)]], [window], seed=3, dtype="f32")
    t = W.make_tensors_torch(b, DEV)
    clean = dict(t, v_pages=t["v_pages"].clone())
    page = int(b.block_table[0, at // 16])
    clean["v_pages"][page, at % 16] = 0.0
    t["v_pages"][page, at % 16] = bad
    out, lse = run_gpu(b, t)
    ro, rl = oracle_of(b, clean)
    sees = np.array([at <= i < at + window for i in range(n)])
    o = host64(out)
    assert not np.isfinite(o[sees]).any()
    assert np.abs(o[~sees] - ro[~sees]).max() <= 1e-5
    assert np.abs(host64(lse) - rl).max() <= 1e-3


@pytest.mark.parametrize("scale", [1e3, 1e5, 1e8])
def test_scores_far_past_the_exponent_of_exp2(scale):
    """Scores of 1e6 to 1e16: one key takes all of a row's weight, wherever the
    roundings of the scores lie."""
    n, d = 300, 64
    b = W.custom("f32_large_scores", 4, 2, d, [40], [n], [[(0, n, W.SEG_CAUSAL, 0)]], [0], seed=3, dtype="f32")
    t = W.make_tensors_torch(b, DEV)
    t["q"] *= scale
    t["k_pages"] *= scale
    out, lse = (host64(x) for x in run_gpu(b, t))
    ro, rl = oracle_of(b, t)
    q, k = host64(t["q"]), host64(t["k_pages"])[b.block_table[0]].reshape(-1, 2, d)[:n]
    for i in range(40):
        for h in range(4):
            s = np.sort(k[:n - 40 + i + 1, h // 2] @ q[i, h]) * b.sm_scale
            err = d * 2.0 ** -24 * np.abs(k[:n - 40 + i + 1, h // 2] * q[i, h]).sum(-1).max() * b.sm_scale
            if s[-1] - s[-2] < 20 + 2 * err:  # not decided within an fp32 dot product's error
                continue
            assert np.abs(out[i, h] - ro[i, h]).max() <= 1e-5, (i, h)
            assert abs(lse[i, h] - rl[i, h]) <= err + 2.0 ** -22 * abs(rl[i, h]), (i, h)
    assert np.isfinite(out).all() and np.isfinite(lse).all()


@pytest.mark.parametrize("d", [64, 128])
def test_values_near_the_largest_float(d):
    """Values of 1e37 under scores that grow along the keys: no sum of weighted
    values passes the largest float, since no weight passes 1."""
    n = 300
    b = W.custom("f32_large_values", 4, 2, d, [40], [n], [[(0, n, W.SEG_CAUSAL, 0)]], [0], seed=4, dtype="f32")
    t = W.make_tensors_torch(b, DEV)
    for p in range((n + 15) // 16):
        t["k_pages"][int(b.block_table[0, p])] *= 1 + 0.2 * p
    ref, ref_lse = run_gpu(b, t)  # the same weights over values of unit size
    t["v_pages"] *= 1e37
    out, lse = run_gpu(b, t)
    # both round each product and sum once more or less: 300 terms of 2^-24
    assert np.abs(host64(out) / 1e37 - host64(ref)).max() <= 300 * 2.0 ** -24 * float(t["v_pages"].abs().max()) / 1e37
    assert np.array_equal(host64(lse), host64(ref_lse))
