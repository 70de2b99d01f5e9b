"""bf16 forward at head_dim 128 with a Q that does not start on a 16-byte boundary: its rows are loaded without the asynchronous
copies that take 16-byte groups, and the result is the aligned one bit for bit.  (Rows that pass through LDS are covered by the
parity tests: clipped blocks, padding, every head grouping.)"""
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,T", [(4, 2, 360), (48, 12, 1430), (768, 192, 360)])  # one and four heads per workgroup, three workgroups to a CU
@pytest.mark.parametrize("off", [1, 2, 5])
def test_forward_of_unaligned_q(off, hq, hkv, T):
    import torch
    w = W.custom_workload([(50, 20, 33), (30, 9, 10), (90, 40, 30)], offsets=[5, 130, 190], total_tokens=T, hq=hq, hkv=hkv, d=128, dtype="bf16", seed=19)
    t = {n: torch.from_numpy(x).to("cuda").to(torch.bfloat16) for n, x in W.make_tensors(w).items()}
    meta = ps.psattn_build_meta(w.offset, w.prefix_len, w.chosen_len, w.rejected_len, w.total_tokens)
    O, LSE = ps.psattn_fwd(meta, t["Q"], t["K"], t["V"], w.scale)
    buf = torch.full((t["Q"].numel() + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    Q = buf[off:off + t["Q"].numel()].view(t["Q"].shape).copy_(t["Q"])
    O2, LSE2 = ps.psattn_fwd(meta, Q, t["K"], t["V"], w.scale)
    torch.cuda.synchronize()
    assert ps.psattn_kernel_name(ps.BF16, 0) == "psattn_fwd_bf16_mfma"
    assert torch.equal(O, O2) and torch.equal(LSE, LSE2)
