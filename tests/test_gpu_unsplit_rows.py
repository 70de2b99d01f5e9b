"""Kernels that small test tables do not reach: dK/dV at head_dim 64 with a row held by one workgroup (a CU's share of all
steps exceeds the longest row), and the generic backward of bf16 in two launches (head groups beyond four).  Against the
oracle; bars as in test_gpu_parity.py."""
import numpy as np
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W
from gpu_util import run_gpu
from test_gpu_parity import compare_full

pytestmark = pytest.mark.gpu

CASES = {
    "even": dict(samples=[(64, 40, 24)] * 33, hq=8, hkv=8),                                                   # every tile a sample's own
    "ragged_tail": dict(samples=[(50, 33, 44)] * 35 + [(3, 1, 2)], hq=8, hkv=8),                              # tiles of two samples, 6 tokens in the last
    "padding": dict(samples=[(60, 20, 41)] * 30, offsets=[7 + 133 * i for i in range(30)], T=4100, hq=16, hkv=16),
    "group_of_3": dict(samples=[(64, 64, 64), (90, 20, 30)] * 20, hq=24, hkv=8),
    "long_list": dict(samples=[(4200, 60, 40)] * 3, hq=6, hkv=6),                                             # lists of 67 entries
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_rows_of_one_workgroup_head64(case):
    c = CASES[case]
    w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=c["hq"], hkv=c["hkv"], d=64,
                          dtype="bf16", seed=64)
    meta = ps.psattn_build_meta(w.offset, w.prefix_len, w.chosen_len, w.rejected_len, w.total_tokens, host_only=True)
    row_ptr, _, _ = meta.csr(ps.GRID_BWD)
    chain = int(np.diff(row_ptr).max()) * (c["hq"] // c["hkv"])
    assert chain * 256 < int(row_ptr[-1]) * c["hq"]  # the launch rule's other side
    tens = W.make_tensors(w)
    out, meta = run_gpu(w, tens)
    assert meta.uses_mfma(ps.BF16, 64, w.scale, backward=True)
    compare_full(w, tens, out, "bf16", what="one workgroup " + case)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(5, 1), (12, 2), (4, 2)])
def test_bf16_generic_backward(hq, hkv, d):
    w = W.custom_workload([(40, 17, 25), (9, 30, 0)], offsets=[2, 90], total_tokens=131, hq=hq, hkv=hkv, d=d, dtype="bf16", seed=33)
    tens = W.make_tensors(w)
    out, meta = run_gpu(w, tens, (64, 64, 64, 64))
    assert not meta.uses_mfma(ps.BF16, d, w.scale) and not meta.uses_mfma(ps.BF16, d, w.scale, backward=True)
    one = hq <= 4 * hkv
    assert ps.psattn_kernel_name(ps.BF16, 0) == "generic_fwd"
    assert ps.psattn_kernel_name(ps.BF16, 2) == ("generic_bwd" if one else "generic_dq")
    assert ps.psattn_kernel_name(ps.BF16, 3) == ("generic_bwd" if one else "generic_dkdv")
    compare_full(w, tens, out, "bf16", what="generic backward %d/%d d %d" % (hq, hkv, d))
