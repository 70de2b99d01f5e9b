"""Backward of the fp32 kernels in one launch and in two (head groups beyond four go in two), against the oracle: block
edges of 16, one token, padding, several heads.  Bars as in test_gpu_parity.py."""
import pytest

import psattn_workloads as W
from gpu_util import run_gpu
from test_gpu_parity import compare_full

pytestmark = pytest.mark.gpu

CASES = {
    "one_token": dict(samples=[(1, 0, 0)], hq=1, hkv=1),
    "block_edges": dict(samples=[(16, 16, 15), (17, 1, 16)], hq=4, hkv=1),
    "padding": dict(samples=[(50, 20, 33), (30, 9, 10)], offsets=[5, 130], T=200, hq=4, hkv=4),
    "two_launches": dict(samples=[(40, 20, 33)], hq=5, hkv=1),
}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", sorted(CASES))
def test_one_launch(case, d):
    c = CASES[case]
    w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=c["hq"], hkv=c["hkv"], d=d,
                          dtype="f32", seed=16)
    tens = W.make_tensors(w)
    out, _ = run_gpu(w, tens)
    compare_full(w, tens, out, "f32", what="one launch %s d %d" % (case, d))
