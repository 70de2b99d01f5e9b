"""The bf16 forward with three workgroups to a CU (head_dim 128, grids of 768 workgroups and more that no few long rows bind): where its
single V buffer and the clipped last tile, which stands for the last 64 rows of the buffer, can go wrong.  Lengths around multiples of 64 from the
smallest buffer on, waves that sit out a tile beside others that do not, padding, hidden ranges, heads that share their queries and
heads that do not, either side of the line, rotary embedding; against the oracle with the bars of test_gpu_parity.py.  On the CPU,
the compiled kernel: 168 registers and a third of the LDS at most, nothing spilled, no copy waited for but by the kernel itself."""
import re

import numpy as np
import pytest
import torch

import paper_2410_20305_amd as ps
import psattn_workloads as W
from gpu_util import run_gpu
from oracle import psattn_oracle as orc
from test_gpu_parity import compare_full
from test_gpu_rope import run_rope_case
from test_kernel_build import _asm, _kernels, _no_spills, _outside_asm

CASES = {
    "t63": dict(samples=[(30, 20, 13)], hq=768, hkv=192),           # below the smallest buffer: two to a CU
    "t64": dict(samples=[(30, 20, 14)], hq=768, hkv=192),
    "t65": dict(samples=[(30, 20, 15)], hq=768, hkv=192),           # the clipped tile is one row, the 63 before it are masked
    "t127": dict(samples=[(60, 30, 37)], hq=772, hkv=193),
    "t129": dict(samples=[(40, 20, 30), (20, 9, 10)], hq=384, hkv=384),
    "below": dict(samples=[(100, 60, 67), (50, 30, 40)], hq=255, hkv=51),    # 347 tokens: 765 workgroups
    "hidden": dict(samples=[(70, 300, 260), (64, 128, 101)], hq=100, hkv=25),
    "padding": dict(samples=[(40, 20, 33), (130, 40, 70), (5, 3, 2)], offsets=[7, 260, 640], T=1077, hq=96, hkv=12),
    "long": dict(samples=[(2200, 150, 33), (30, 20, 10)], offsets=[9, 2400], T=2463, hq=40, hkv=10),   # bound by its long rows: two
    "long_many": dict(samples=[(2200, 150, 33), (30, 20, 10)], offsets=[9, 2400], T=2463, hq=100, hkv=25),
}


def three(meta, T, hq):
    """The launch rule: workgroups, and the longest row against a slot's share of all k-tiles."""
    n = np.diff(meta.csr(ps.GRID_FWD)[0])
    return T >= 64 and len(n) * hq >= 768 and (n.max() < 12 or 100 * 768 * n.max() <= 85 * n.sum() * hq)


@pytest.mark.gpu
@pytest.mark.parametrize("case", sorted(CASES))
def test_against_oracle(case):
    c = CASES[case]
    w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=c["hq"], hkv=c["hkv"], d=128,
                          dtype="bf16", seed=731)
    tens = W.make_tensors(w)
    out, meta = run_gpu(w, tens)
    assert three(meta, w.total_tokens, c["hq"]) == (case not in ("t63", "below", "long"))
    assert meta.uses_mfma(ps.BF16, 128, w.scale, backward=True)
    compare_full(w, tens, out, "bf16", what="three to a CU %s" % case)


@pytest.mark.gpu
def test_rotary_rows_leave_whole():
    """Q is turned, saved and used in one go: the output equals that of a call on the rows that were saved (which
    test_rotary_embedding compares with rows turned by the oracle)."""
    w = W.custom_workload([(150, 40, 70), (130, 90, 51)], hq=160, hkv=40, d=128, dtype="bf16", seed=5)
    t = W.make_tensors(w)
    dev = lambda x: torch.from_numpy(x).to("cuda").to(torch.bfloat16)
    Q, K, V = (dev(t[n]) for n in ("Q", "K", "V"))
    meta = ps.psattn_build_meta(w.offset, w.prefix_len, w.chosen_len, w.rejected_len, w.total_tokens)
    assert three(meta, w.total_tokens, 160)
    rope = ps.Rope(128, 10000.0, meta.positions()[1])
    O, LSE, Qr, Kr = ps.psattn_fwd_rope(meta, rope, Q, K, V, w.scale)
    O2, LSE2 = ps.psattn_fwd(meta, Qr, Kr, V, w.scale)
    assert torch.equal(O, O2) and torch.equal(LSE, LSE2)
    Ic, Ir, D = orc.index_arrays(w.offset, w.prefix_len, w.chosen_len, w.rejected_len, w.total_tokens)
    f = lambda x: x.float().cpu().numpy().astype(np.float64)
    ref = orc.forward(f(Qr), f(Kr), t["V"].astype(np.float64), w.scale, Ic, Ir, D)
    assert np.abs(f(O) - ref[0]).max() <= 1.3e-2   # 1e-2 below 2, half a bf16 ulp (0.0078) + 5e-3 on [2, 4)


@pytest.mark.gpu
def test_rotary_embedding():
    """Saved rows, output and gradients against the oracle, which turns the original rows by its own position ids."""
    assert (900 + 127) // 128 * 160 >= 768
    run_rope_case([5, 460], [150, 130], [0, 2, 5], [40, 70, 90, 51, 33], 900, 160, 40, 10000.0, 6)


def test_compiled_kernel(tmp_path):
    for name, body, meta in _kernels(_asm(tmp_path, "psattn_mfma_fwd3.hip"), "psattn_fwd_bf16_mfma", 1):
        assert int(meta["vgpr_count"]) <= 168 and int(meta["agpr_count"]) == 0, name
        assert int(meta["group_segment_fixed_size"]) <= 160 * 1024 // 3, name
        _no_spills(name, meta)
        for code in _outside_asm(body):
            assert not re.search(r"\bm0\b", code), code
        first, last = body.index("global_load_lds_dwordx4"), body.rindex("global_load_lds_dwordx4")
        loads = [c for c in _outside_asm("#ASMSTART\n" + body[first:last]) if re.match(r"(global|buffer|flat|scratch)_load", c)]
        assert all(c.startswith("global_load_dword ") for c in loads), loads
