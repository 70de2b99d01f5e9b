"""delta = rowsum(dO o O) that the bf16 dQ kernel leaves in the workspace (negated), bit for bit: two chains of fp32 sums over a
row, head dims 16 t .. 16 t + 7 and 16 t + 8 .. 16 t + 15 for ascending t, added at the end.  The order is pinned because a delta that
is off by one bit turns the bf16 rounding of a score gradient now and then, and with it bits of dQ, dK and what is computed from
them.  One and four heads per workgroup, clipped blocks, padding."""
import numpy as np
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W

pytestmark = pytest.mark.gpu


def _fma(a, b, c):
    # products of bf16 values are exact in fp32, and their sum with an fp32 value is as good as exact in fp64
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


def _delta(dO, O):
    T, H, d = O.shape
    half = [np.zeros((T, H), dtype=np.float32), np.zeros((T, H), dtype=np.float32)]
    for t in range(d // 16):
        for g in range(2):
            for k in range(16 * t + 8 * g, 16 * t + 8 * g + 8):
                half[g] = _fma(O[:, :, k], dO[:, :, k], half[g])
    return half[0] + half[1]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv,T", [(4, 2, 360), (3, 1, 383), (48, 12, 1430)])
def test_delta_bits(d, hq, hkv, T):
    import torch
    w = W.custom_workload([(50, 20, 33), (30, 9, 10), (90, 40, 30)], offsets=[5, 130, 190], total_tokens=T, hq=hq, hkv=hkv, d=d,
                          dtype="bf16", seed=23)
    t = {n: torch.from_numpy(x).to("cuda").to(torch.bfloat16) for n, x in W.make_tensors(w).items()}
    meta = ps.psattn_build_meta(w.offset, w.prefix_len, w.chosen_len, w.rejected_len, w.total_tokens)
    O, LSE = ps.psattn_fwd(meta, t["Q"], t["K"], t["V"], w.scale)
    ws = torch.zeros(ps.psattn_bwd_workspace_bytes(meta, hq, hkv, d), dtype=torch.uint8, device="cuda")
    assert ws.data_ptr() % 256 == 0
    ps.psattn_bwd(meta, t["Q"], t["K"], t["V"], O, t["dO"], LSE, w.scale, workspace=ws)
    torch.cuda.synchronize()
    assert ps.psattn_kernel_name(ps.BF16, 2) == "psattn_dq_bf16_mfma"
    got = ws.cpu().numpy().view(np.float32)[:hq * w.total_tokens].reshape(hq, w.total_tokens).T
    want = -_delta(t["dO"].float().cpu().numpy(), O.float().cpu().numpy())
    assert np.array_equal(got, want), (np.abs(got - want).max(), (got != want).mean())
