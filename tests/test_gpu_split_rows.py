"""dK/dV where a row's walk is shared by two groups of waves (launches bound by their longest row), against the oracle:
odd and even numbers of steps, group sizes that do not divide by two, a k-tile whose second half lies past the end or holds
padding only, lists longer than one 64-entry window; and tables on either side of the line.  Bars as in test_gpu_parity.py."""
import numpy as np
import pytest

import paper_2410_20305_amd as ps
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
    assert _splits(meta, c["hq"], c["hkv"])  # at head_dim 64 too, whose line is one share
    compare_full(w, tens, out, "bf16", what="split %s d %d" % (case, d))


def _splits(meta, hq, hkv):
    """The launch rule at head_dim 128: the longest chain of steps against a CU's share of all steps."""
    row_ptr, _, _ = meta.csr(ps.GRID_BWD)
    chain, steps = int(np.diff(row_ptr).max()) * (hq // hkv), int(row_ptr[-1]) * hq
    return chain >= 8 and (10 * chain * 256 >= 16 * steps or 10 * (chain - 8) * 256 >= 13 * steps)


LINE = {  # ratio of the longest chain to a CU's share, and the side
    "1.18": (dict(samples=[(150, 40, 70)] * 2, hq=256, hkv=64), False),
    "1.30": (dict(samples=[(300, 100, 50)], hq=312, hkv=78), False),                           # 32 steps
    "1.33_group_of_2": (dict(samples=[(500, 60, 40)], hq=128, hkv=64), False),                 # 20 steps
    "1.40_below": (dict(samples=[(500, 60, 40)], hq=488, hkv=61), False),                      # 80 steps, 5.7 above 1.3 shares
    "1.50_above": (dict(samples=[(500, 60, 40)], hq=456, hkv=57), True),                       # 80 steps, 10.5
    "1.60_group_of_4": (dict(samples=[(300, 100, 50)], hq=256, hkv=64), True),                 # 32 steps, 6 above 1.3 shares
    "1.5_padding": (dict(samples=[(300, 100, 50), (20, 10, 5)], offsets=[7, 500], T=600, hq=434, hkv=62), False),   # 56 steps, 7.5
    "1.57_padding": (dict(samples=[(300, 100, 50), (20, 10, 5)], offsets=[7, 500], T=600, hq=413, hkv=59), True),   # 56 steps, 9.9
}


@pytest.mark.parametrize("case", sorted(LINE))
def test_either_side_of_the_line(case):
    c, split = LINE[case]
    w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=c["hq"], hkv=c["hkv"], d=128,
                          dtype="bf16", seed=129)
    tens = W.make_tensors(w)
    out, meta = run_gpu(w, tens)
    assert _splits(meta, c["hq"], c["hkv"]) == split
    compare_full(w, tens, out, "bf16", what="line %s" % case)
