"""bf16 forward and dQ where the four waves of a workgroup take four heads of a kv group on the same 32 queries (groups of a
multiple of four heads, more than 512 workgroups), against the oracle, where leaving out tiles that only other queries of the
q-tile of 128 read can go wrong: blocks of 32 queries that end on, before and behind a sample's end, blocks of several samples,
a response's hidden range that covers whole tiles, blocks of padding alone, a clipped last block, lists longer than one 64-entry
window; and the largest grid on either side of the line.  Bars as in test_gpu_parity.py."""
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W
from gpu_util import run_gpu
from test_gpu_parity import compare_full

pytestmark = pytest.mark.gpu

CASES = {
    "block_edges": dict(samples=[(16, 8, 8), (20, 5, 6), (17, 8, 8), (95, 1, 1), (31, 32, 33)] * 12, hq=32, hkv=8),
    "tiny_samples": dict(samples=[(3, 2, 1), (1, 0, 4), (0, 5, 2)] * 100, hq=48, hkv=12),
    "hidden_tiles": dict(samples=[(70, 300, 260), (64, 128, 96)], hq=80, hkv=10),
    "padding": dict(samples=[(40, 20, 33), (130, 40, 70), (5, 3, 2)], offsets=[7, 260, 640], T=1077, hq=64, hkv=16),
    "long_list": dict(samples=[(4100, 150, 33), (30, 20, 10)], offsets=[9, 4300], T=4371, hq=16, hkv=4),
    "line_512": dict(samples=[(100, 80, 90), (90, 60, 75)], hq=128, hkv=16),           # 495 tokens: 4 q-tiles
    "line_above": dict(samples=[(100, 80, 90), (90, 60, 95)], hq=108, hkv=9),          # 515 tokens: 5 q-tiles, 540 workgroups
}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", sorted(CASES))
def test_four_heads_on_the_same_queries(case, d):
    c = CASES[case]
    w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=c["hq"], hkv=c["hkv"], d=d,
                          dtype="bf16", seed=324)
    assert ((w.total_tokens + 127) // 128 * c["hq"] > 512) == (case != "line_512")
    tens = W.make_tensors(w)
    out, meta = run_gpu(w, tens)
    assert meta.uses_mfma(ps.BF16, d, w.scale, backward=True)
    compare_full(w, tens, out, "bf16", what="shared queries %s d %d" % (case, d))
