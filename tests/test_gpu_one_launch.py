"""Backward of the fp32 kernels in one launch and in two (head groups beyond four go in two), against the oracle: block
edges of 16, one token, padding, several heads.  Bars as in test_gpu_parity.py."""
import numpy as np
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W
from gpu_util import run_gpu, to_dev, to_np
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


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("tiles", [(0, 0, 0, 0), (64, 64, 64, 64)])
def test_outputs_in_the_memory_of_inputs(dtype, d, tiles):
    """O in Q's memory; dQ in O's, dK in K's and dV in V's: bit for bit what separate buffers give with the same kernels.  One
    launch would read O, K and V while they are overwritten, so such calls take two."""
    w = W.custom_workload([(50, 20, 33), (30, 9, 10), (150, 40, 70)], offsets=[5, 130, 190], total_tokens=470, hq=4, hkv=2, d=d, dtype=dtype, seed=17)
    tens = W.make_tensors(w)
    meta = ps.psattn_build_meta(w.offset, w.prefix_len, w.chosen_len, w.rejected_len, w.total_tokens, *tiles)
    Q, K, V, dO = (to_dev(tens[n], dtype) for n in ("Q", "K", "V", "dO"))
    O, LSE = ps.psattn_fwd(meta, Q, K, V, w.scale)
    Q2 = Q.clone()
    _, LSE2 = ps.psattn_fwd(meta, Q2, K, V, w.scale, O=Q2)
    assert np.array_equal(to_np(Q2), to_np(O)) and np.array_equal(to_np(LSE2), to_np(LSE))
    dQ, dK, dV = ps.psattn_bwd(meta, Q, K, V, O, dO, LSE, w.scale)
    mfma = meta.uses_mfma(ps.BF16, d, w.scale, backward=True) and dtype == "bf16"
    code = ps.F32 if dtype == "f32" else ps.BF16
    assert ps.psattn_kernel_name(code, 2) == ("psattn_dq_bf16_mfma" if mfma else "generic_bwd")
    O2, K2, V2 = O.clone(), K.clone(), V.clone()
    ps.psattn_bwd(meta, Q, K2, V2, O2, dO, LSE, w.scale, dQ=O2, dK=K2, dV=V2)
    assert ps.psattn_kernel_name(code, 2) == ("psattn_dq_bf16_mfma" if mfma else "generic_dq")
    for got, ref in ((O2, dQ), (K2, dK), (V2, dV)):
        assert np.array_equal(to_np(got), to_np(ref))


def test_profiling_times_the_kernels_that_run_without_it():
    w = W.custom_workload([(50, 20, 33)], hq=4, hkv=2, d=64, dtype="f32", seed=18)
    tens = W.make_tensors(w)
    ps.psattn_profile_enable(True)
    try:
        ps.psattn_profile_read()
        run_gpu(w, tens)
        ms, count = ps.psattn_profile_read()
    finally:
        ps.psattn_profile_enable(False)
    assert ps.psattn_kernel_name(ps.F32, 3) == "generic_bwd"
    assert count.tolist() == [1, 0, 0, 1] and ms[0] > 0 and ms[3] > 0
