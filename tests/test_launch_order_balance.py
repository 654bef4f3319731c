"""The multi-row launch order loads the eight XCDs evenly whatever the number
and the sizes of the (request, KV head) groups are (CPU only)."""
import pytest

import workloads as W
from paper_2606_12688_amd import attn
from tests.helpers import plan_for
from tests.test_abi_host import _check_xcd_runs


def _prompts(lens):
    return W.custom("prompts", 28, 4, 128, lens, lens, [[(0, n, W.SEG_CAUSAL, 0)] for n in lens], [0] * len(lens))


@pytest.mark.parametrize("b", [W.cfg_labels_bf16(n=1), W.text_latent_bf16(n=1), W.text_latent_bf16(n=3),
                               _prompts([1900, 900, 500, 300]), _prompts([4000, 129]), _prompts([130]),
                               W.rollout_bf16(n=5, hq=3, hkv=3)], ids=lambda b: f"{b.name}-{b.num_seqs}")
def test_xcd_loads_are_even(b):
    pl = plan_for(b, attn.FLAG_HOST_ONLY)
    items, order = pl.items(0), pl.tile_order()
    G = b.num_qo_heads // b.num_kv_heads
    real = [(i, h) for i, h in order.tolist() if i >= 0]
    assert sorted(real) == sorted((i, h) for i in range(len(items)) for h in range(b.num_qo_heads))
    _check_xcd_runs(order, items, G, balanced=False)

    def pairs(w):  # visible pairs of an item for one head; causal and full segments without windows
        seq, _, row0, nrows, kb, ke = (int(x) for x in w[:6])
        q, kv, _ = (int(x) for x in b.seqs[seq])
        n = 0
        for i in range(row0, row0 + nrows):
            p = kv - q + i
            for start, ln, kind, block in b.seq_segments(seq).tolist():
                if start <= p < start + ln:
                    hi = {W.SEG_CAUSAL: p + 1, W.SEG_FULL: start + ln}.get(kind)
                    if hi is None:
                        hi = min(start + ((p - start) // block + 1) * block, start + ln)
            n += max(0, min(hi, ke) - kb)
        return n

    cost = [pairs(w) + 1 for w in items]  # per workgroup
    load = [0] * 8
    for wg, (i, _) in enumerate(order.tolist()):
        if i >= 0:
            load[wg % 8] += cost[i]
    share = sum(load) / 8
    # cuts fall on whole items (G workgroups each), to the nearest one
    assert max(load) <= share * (1 + 1 / 64) + G * max(cost)
    pl.destroy()
