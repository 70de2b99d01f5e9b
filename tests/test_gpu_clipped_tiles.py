"""bf16 kernels on buffers whose length is no multiple of a tile: rows of the last tile past the end of the buffer re-read its last
row and are masked; the forward with three workgroups to a CU (heads by the hundred here) takes the last 64 rows of the buffer instead,
of which the ones before the tile's own first are masked.  Lengths on either side of multiples of 32, 64 and 128, with one sample, with
several in the last 64 rows, and with padding at the end; dK/dV rows in one piece and split.  Against the oracle, bars as in
test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import paper_2410_20305_amd as ps
import psattn_workloads as W
from gpu_util import BF16_LSE_TOL, oracle_arrays, run_gpu, to_dev, to_np
from oracle import psattn_oracle as orc
from test_gpu_parity import compare_full

pytestmark = pytest.mark.gpu

LAYOUTS = {
    "one": lambda T: dict(samples=[(T - T // 3 - T // 4, T // 3, T // 4)]),
    "several": lambda T: dict(samples=[(T - T // 2 - 2 * (T // 5), T // 5, T // 5), (T // 2 - 2 * (T // 6), T // 6, T // 6)]),
    "padding": lambda T: dict(samples=[(T // 2, T // 8, T // 8)], offsets=[T // 16], T=T),
}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(2, 2), (8, 1)])
@pytest.mark.parametrize("layout", sorted(LAYOUTS))
def test_lengths(layout, hq, hkv, d):
    for T in (1, 2, 31)[0 if layout == "one" else 2:] + (33, 63, 64, 65, 95, 97, 127, 128, 129, 191, 193, 320, 383):
        c = LAYOUTS[layout](T)
        w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=hq, hkv=hkv, d=d, dtype="bf16", seed=T)
        assert w.total_tokens == T
        tens = W.make_tensors(w)
        out, meta = run_gpu(w, tens)
        assert meta.uses_mfma(ps.BF16, d, w.scale, backward=True)
        compare_full(w, tens, out, "bf16", what="clipped %s T %d d %d" % (layout, T, d))


@pytest.mark.parametrize("layout", sorted(LAYOUTS))
def test_lengths_three_to_a_cu(layout):
    """The forward alone.  Millions of outputs meet the worst case of rounding, so the bar is its bound: weights are rounded to bf16 (2^-8 of
    each, against their sum before rounding; scores and sums in fp32 add less than 2^-14), then the output is (half an ulp, 2^-8)."""
    for T in (65, 95, 97, 127, 129, 191, 193):
        c = LAYOUTS[layout](T)
        w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=768, hkv=192, d=128, dtype="bf16", seed=T)
        assert w.total_tokens == T
        t = W.make_tensors(w)
        Ic, Ir, D = oracle_arrays(w)
        ref, lse = orc.forward(t["Q"], t["K"], t["V"], w.scale, Ic, Ir, D)[:2]
        size = orc.forward(t["Q"], t["K"], np.abs(t["V"]), w.scale, Ic, Ir, D)[0]
        meta = ps.psattn_build_meta(w.offset, w.prefix_len, w.chosen_len, w.rejected_len, T)
        Q, K, V = (to_dev(t[n], "bf16") for n in ("Q", "K", "V"))
        O, LSE = torch.full_like(Q, float("nan")), torch.full((768, T), float("nan"), device="cuda")
        ps.psattn_fwd(meta, Q, K, V, w.scale, O=O, LSE=LSE)
        weights = (2.0 ** -8 + 2.0 ** -14) * size
        err = np.abs(to_np(O) - ref) - weights - 2.0 ** -8 * (np.abs(ref) + weights)
        assert err.max() <= 0, (layout, T, err.max(), np.unravel_index(err.argmax(), err.shape))
        real = D != orc.PAD_DOC
        assert np.all(to_np(O)[~real] == 0) and np.all(np.isneginf(to_np(LSE)[:, ~real]))
        assert np.abs(to_np(LSE)[:, real] - lse[:, real]).max() <= BF16_LSE_TOL, (layout, T)
