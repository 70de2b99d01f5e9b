"""NaN and inf in padding, in another sample of the same tile or at a later token reach no row that may not read them, on
the fp32 kernels and wherever else the exact zeros of a matrix product could carry them.  Rows that do not depend on a
poisoned token match the oracle on clean inputs (bars as in test_gpu_parity.py), padding stays exact zeros, and what does
depend on one is not finite."""
import numpy as np
import pytest

import psattn_workloads as W
from gpu_util import (BF16_LSE_TOL, F32_TOL, check_grad, check_o, check_padding_zero, dq_delta_floor, oracle_arrays, run_gpu)
from oracle import psattn_oracle as orc

pytestmark = pytest.mark.gpu

SMALL = dict(samples=[(23, 9, 14), (5, 0, 11), (20, 7, 13)], offsets=[3, 52, 70], T=125)
FEW = dict(samples=[(23, 9, 14), (0, 0, 6), (20, 7, 13)], offsets=[0, 52, 58], T=98)  # eight runs: travels with the kernels' arguments
TILES = dict(samples=[(150, 40, 70), (30, 90, 10), (100, 33, 65)], offsets=[5, 300, 430], T=700)
MANY = dict(samples=[(70, 30, 28)] * 40, offsets=[5 + 130 * i for i in range(40)], T=5300)  # dK/dV rows held by one workgroup each
# kernels: dtype, d, heads, tiles, layout
PATHS = {
    "f32_64": ("f32", 64, 2, 1, (0, 0, 0, 0), SMALL),
    "f32_128": ("f32", 128, 4, 2, (0, 0, 0, 0), SMALL),
    "f32_two_launches": ("f32", 64, 5, 1, (0, 0, 0, 0), SMALL),
    "f32_tiles": ("f32", 64, 2, 2, (0, 0, 0, 0), TILES),
    "bf16_generic_64": ("bf16", 64, 4, 2, (7, 5, 3, 9), SMALL),
    "bf16_64": ("bf16", 64, 4, 2, (0, 0, 0, 0), TILES),
    "bf16_64_many": ("bf16", 64, 16, 16, (0, 0, 0, 0), MANY),
    "bf16_64_small": ("bf16", 64, 3, 1, (0, 0, 0, 0), SMALL),
    "bf16_64_shared": ("bf16", 64, 16, 4, (0, 0, 0, 0), MANY),  # four heads on the same queries
    "f32_64_in_args": ("f32", 64, 2, 1, (0, 0, 0, 0), FEW),
    "f32_128_in_args": ("f32", 128, 4, 2, (0, 0, 0, 0), FEW),
    "f32_two_launches_in_args": ("f32", 64, 5, 1, (0, 0, 0, 0), FEW),
    "bf16_64_in_args": ("bf16", 64, 4, 2, (0, 0, 0, 0), FEW),
    "bf16_generic_128": ("bf16", 128, 5, 1, (32, 16, 16, 32), SMALL),
}


@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("path", sorted(PATHS))
def test_poison_stays_where_it_is_read(path, value):
    dtype, d, hq, hkv, tiles, lay = PATHS[path]
    w = W.custom_workload(lay["samples"], offsets=lay["offsets"], total_tokens=lay["T"], hq=hq, hkv=hkv, d=d, dtype=dtype, seed=77)
    tens = W.make_tensors(w)
    Ic, Ir, D = oracle_arrays(w)
    mask, real = orc.dense_mask(Ic, Ir, D), D != orc.PAD_DOC
    poison = ~real
    o, p, c = int(w.offset[0]), int(w.prefix_len[0]), int(w.chosen_len[0])
    poison[o + p:o + p + c] = True                             # a whole response
    poison[int(w.offset[2]) + int(w.prefix_len[2]) - 1] = True  # the last token of a prompt
    bad = {n: x.copy() for n, x in tens.items()}
    for x in bad.values():
        x[poison] = value
    out, meta = run_gpu(w, bad, tiles)
    assert (meta.device_bytes() == 0) == path.endswith("_in_args")
    check_padding_zero(out, D)
    q_bad = real & (poison | (mask & poison[None, :]).any(axis=1))
    k_bad = real & (poison | (mask & q_bad[:, None]).any(axis=0))
    q_ok, k_ok = real & ~q_bad, real & ~k_bad
    assert q_ok.any() and k_ok.any() and q_bad.any()
    if np.isnan(value):
        for n in ("O", "dQ"):
            assert np.all(~np.isfinite(out[n][q_bad]).all(axis=-1)), n
    clean = {n: np.where(poison[:, None, None], 0.0, x) for n, x in tens.items()}
    ref = orc.backward(clean["Q"], clean["K"], clean["V"], clean["dO"], w.scale, Ic, Ir, D)
    for n, rows in (("O", q_ok), ("dQ", q_ok), ("dK", k_ok), ("dV", k_ok)):
        got, want = out[n][rows], ref[n][rows]
        assert np.all(np.isfinite(got)), n
        if dtype == "f32":
            assert np.abs(got - want).max() <= F32_TOL, (n, np.abs(got - want).max())
        elif n == "O":
            check_o(got, want, path)
        else:
            check_grad(got, want, n, path, dq_delta_floor(clean["dO"][rows], ref["O"][rows], clean["K"], w.scale) if n == "dQ" else None)
    err = np.abs(out["LSE"][:, q_ok] - ref["LSE"][:, q_ok]).max()
    assert err <= (F32_TOL if dtype == "f32" else BF16_LSE_TOL)
