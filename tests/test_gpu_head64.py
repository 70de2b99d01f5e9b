"""The bf16 matrix-core kernels at head_dim 64 against the oracle, where they can go wrong: one token, ragged tails
around the 64- and 128-token tiles, padding inside and behind, responses that end on a tile edge, head groupings, tile
lists longer than one 64-entry window.  Bars as for head_dim 128 (tests/test_gpu_parity.py)."""
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W
from gpu_util import run_gpu
from test_gpu_parity import compare_full

pytestmark = pytest.mark.gpu

CASES = {
    "one_token": dict(samples=[(1, 0, 0)], hq=1, hkv=1),
    "below_tile": dict(samples=[(31, 15, 17)], hq=2, hkv=1),          # 63 tokens
    "tile_edges": dict(samples=[(64, 64, 64), (63, 1, 1)], hq=4, hkv=2),
    "behind_edges": dict(samples=[(65, 63, 129), (1, 127, 1)], hq=4, hkv=4),
    "padding": dict(samples=[(150, 40, 70), (30, 90, 10)], offsets=[5, 300], T=450, hq=6, hkv=2),
    "no_prompt": dict(samples=[(0, 70, 90), (64, 0, 64)], hq=8, hkv=1),
    "long_list": dict(samples=[(4100, 150, 33)], offsets=[9], T=4300, hq=2, hkv=1),  # lists of 67 entries
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_head64_parity(case):
    c = CASES[case]
    w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=c["hq"], hkv=c["hkv"], d=64,
                          dtype="bf16", seed=641)
    tens = W.make_tensors(w)
    out, meta = run_gpu(w, tens)
    assert meta.uses_mfma(ps.BF16, 64, w.scale, backward=True)
    compare_full(w, tens, out, "bf16", what="head64 " + case)
