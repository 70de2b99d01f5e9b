"""Tensors that start off a 16-byte boundary (views into a larger buffer): fp32 and bf16 with head_dim 64, default and other
tile grids, against the oracle.  Bars as in test_gpu_parity.py."""
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W
from gpu_util import to_np
from test_gpu_parity import compare_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,tiles", [("f32", 64, (0, 0, 0, 0)), ("f32", 128, (0, 0, 0, 0)), ("bf16", 64, (0, 0, 0, 0)),
                                           ("bf16", 64, (32, 16, 16, 32)), ("bf16", 128, (32, 16, 16, 32))])
@pytest.mark.parametrize("off", [1, 2, 5])
def test_unaligned_tensors(dtype, d, tiles, off):
    import torch
    w = W.custom_workload([(50, 20, 33), (30, 9, 10), (90, 40, 30)], offsets=[5, 130, 190], total_tokens=360, hq=4, hkv=2, d=d, dtype=dtype, seed=19)
    tens = W.make_tensors(w)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16

    def at(shape):
        n = shape[0] * shape[1] * shape[2]
        buf = torch.full((n + 64,), float("nan"), dtype=dt, device="cuda")
        return buf, buf[off:off + n].view(*shape)
    ins = {n: at(tens[n].shape) for n in ("Q", "K", "V", "dO")}
    for n, (_, x) in ins.items():
        x.copy_(torch.from_numpy(tens[n]))
    outs = {n: at(tens[like].shape) for n, like in (("O", "Q"), ("dQ", "Q"), ("dK", "K"), ("dV", "V"))}
    x = {n: t for n, (_, t) in list(ins.items()) + list(outs.items())}
    meta = ps.psattn_build_meta(w.offset, w.prefix_len, w.chosen_len, w.rejected_len, w.total_tokens, *tiles)
    _, LSE = ps.psattn_fwd(meta, x["Q"], x["K"], x["V"], w.scale, O=x["O"])
    ps.psattn_bwd(meta, x["Q"], x["K"], x["V"], x["O"], x["dO"], LSE, w.scale, dQ=x["dQ"], dK=x["dK"], dV=x["dV"])
    torch.cuda.synchronize()
    code = ps.F32 if dtype == "f32" else ps.BF16
    assert ps.psattn_kernel_name(code, 0) == "generic_fwd" and ps.psattn_kernel_name(code, 3).startswith("generic")
    out = {n: to_np(x[n]) for n in ("O", "dQ", "dK", "dV")}
    out["LSE"] = to_np(LSE)
    compare_full(w, tens, out, dtype, what="unaligned by %d" % off)
    for n, (buf, view) in outs.items():  # nothing is written beside the tensor
        assert bool(torch.isnan(buf[:off]).all()) and bool(torch.isnan(buf[off + view.numel():]).all()), n
