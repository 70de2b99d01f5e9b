"""dK/dV where a row's walk is shared by two groups of waves (launches bound by their longest row), against the oracle:
odd and even numbers of steps, group sizes that do not divide by two, a k-tile whose second half lies past the end or holds
padding only, lists longer than one 64-entry window, rotary embedding.  Bars as in test_gpu_parity.py."""
import numpy as np
import pytest

import psattn_workloads as W
from gpu_util import run_gpu
from test_gpu_parity import compare_full

pytestmark = pytest.mark.gpu

CASES = {
    "group_of_1": dict(samples=[(700, 50, 33)], hq=2, hkv=2),
    "group_of_3": dict(samples=[(300, 129, 65)], hq=3, hkv=1),
    "group_of_7": dict(samples=[(150, 40, 70)], hq=14, hkv=2),
    "short_last_tile": dict(samples=[(500, 100, 50)], hq=4, hkv=2),                            # 650 tokens: 10 in the last k-tile
    "padding": dict(samples=[(150, 40, 70), (330, 90, 10)], offsets=[5, 300], T=900, hq=8, hkv=2),
    "long_list": dict(samples=[(4100, 150, 33)], offsets=[9], T=4300, hq=1, hkv=1),            # lists of 67 entries
}


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("case", sorted(CASES))
def test_split_rows(case, d):
    c = CASES[case]
    w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=c["hq"], hkv=c["hkv"], d=d,
                          dtype="bf16", seed=128)
    tens = W.make_tensors(w)
    out, meta = run_gpu(w, tens)
    import paper_2410_20305_amd as ps
    row_ptr, _, _ = meta.csr(ps.GRID_BWD)
    chain = int(np.diff(row_ptr).max()) * (c["hq"] // c["hkv"])
    assert chain >= 8 and 10 * chain * 256 >= 16 * int(row_ptr[-1]) * c["hq"]  # the launch rules' conditions
    compare_full(w, tens, out, "bf16", what="split %s d %d" % (case, d))
