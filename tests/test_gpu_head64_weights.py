"""bf16 with head_dim 64 keeps probabilities and score gradients in fp32 up to the sums that they weight: what separates the
outputs from 64-bit arithmetic is the rounding of the outputs and fp32 sums, not a rounding of the weights (2^-9 each, which
shows on every row of few keys).  delta = rowsum(dO o O) takes the forward's bf16 O, as the backward does."""
import numpy as np
import pytest

import psattn_workloads as W
from gpu_util import bf16_half_ulp, check_padding_zero, oracle_arrays, run_gpu
from oracle import psattn_oracle as orc

pytestmark = pytest.mark.gpu

# Relative to the sum of the magnitudes of the terms.  A score is off by 64 products' fp32 rounding, at most 64 2^-24 of their
# magnitudes, the exponent (below 2^4 in magnitude) by 4 roundings of it, an output sum of n <= 460 terms by n 2^-24:
# together below 2^-18 + 2^-18 + 2^-15.1.
EPS = 2.0 ** -14

CASES = {
    "one_token": dict(samples=[(1, 0, 0)], hq=1, hkv=1),
    "tile_edges": dict(samples=[(64, 64, 64), (63, 1, 1)], hq=4, hkv=2),
    "padding": dict(samples=[(150, 40, 70), (30, 90, 10)], offsets=[5, 300], T=450, hq=6, hkv=2),
    "ragged": dict(samples=[(300, 96, 64)], hq=2, hkv=1),
}


def near(got, ref, mag, what):
    bar = bf16_half_ulp(np.abs(ref) + EPS * mag) + EPS * mag
    err = np.abs(got - ref)
    at = np.unravel_index(np.argmax(err / np.maximum(bar, 1e-300)), err.shape)
    assert np.all(err <= bar), (what, at, float(err[at]), float(ref[at]), float(bar[at]), float((err > bar).mean()))


@pytest.mark.parametrize("case", sorted(CASES))
def test_weights_keep_their_bits(case):
    c = CASES[case]
    w = W.custom_workload(c["samples"], offsets=c.get("offsets"), total_tokens=c.get("T"), hq=c["hq"], hkv=c["hkv"], d=64,
                          dtype="bf16", seed=645)
    tens = W.make_tensors(w)
    out, _ = run_gpu(w, tens)
    Ic, Ir, D = oracle_arrays(w)
    check_padding_zero(out, D)
    mask, real = orc.dense_mask(Ic, Ir, D), D != orc.PAD_DOC
    G = w.n_q_heads // w.n_kv_heads
    f = {n: np.where(real[:, None, None], tens[n].astype(np.float64), 0.0) for n in ("Q", "K", "V", "dO")}
    grads = {n: np.zeros((2,) + f[n[1]].shape) for n in ("dK", "dV")}  # sums and sums of magnitudes
    for h in range(w.n_q_heads):
        q, k, v, g, o = f["Q"][:, h], f["K"][:, h // G], f["V"][:, h // G], f["dO"][:, h], out["O"][:, h]
        s = np.where(mask, w.scale * (q @ k.T), -np.inf)
        top = np.where(real, s.max(axis=1, initial=-np.inf), 0.0)
        p = np.exp(s - top[:, None])
        p /= np.where(real, p.sum(axis=1), 1.0)[:, None]
        near(o, p @ v, p @ np.abs(v), (case, "O", h))
        ds = p * (g @ v.T - (g * o).sum(axis=1)[:, None])
        ds_mag = p * (np.abs(g) @ np.abs(v).T + (np.abs(g) * np.abs(o)).sum(axis=1)[:, None])
        near(out["dQ"][:, h], w.scale * (ds @ k), w.scale * (ds_mag @ np.abs(k)), (case, "dQ", h))
        for n, x, mag, y in (("dK", w.scale * ds, w.scale * ds_mag, q), ("dV", p, p, g)):
            grads[n][0, :, h // G] += x.T @ y
            grads[n][1, :, h // G] += mag.T @ np.abs(y)
    for n, (ref, mag) in grads.items():
        near(out[n], ref, mag, (case, n))
