"""Block masks that travel with the kernels' arguments (up to 1 024 tokens, 8 runs of equal descriptors, 8 rows of tiles) against the
same masks in device memory: the samples once more in a longer buffer, whose further tokens are padding, give the same outputs
bit for bit.  Which form a mask takes is asserted.  Sizes on both sides of every line, empty and one-token segments, padding in front, between and behind."""
import numpy as np
import pytest

import paper_2410_20305_amd as ps

pytestmark = pytest.mark.gpu

# offsets, prompts, responses of each sample, tokens of the buffer
CASES = {
    "one_token": ([0], [1], [[]], 1),
    "one_sample": ([0], [100], [[40, 37]], 177),
    "tile_edges": ([0], [64], [[64, 64]], 192),
    "padding_around": ([5, 130], [40, 33], [[20, 30], [9, 11]], 250),     # 9 runs: in device memory either way
    "nine_runs": ([3, 70], [20, 31], [[10, 12], [7, 8]], 140),            # with padding in front, between and behind
    "eight_runs": ([3, 70], [20, 31], [[10, 12], [7, 8]], 116),           # in front and between
    "eight_runs_full": ([0, 40, 77], [20, 31, 9], [[10, 10], [6], [5, 4]], 95),
    "no_prompt": ([0], [0], [[70, 90, 33]], 193),
    "six_responses": ([0], [90], [[30, 1, 64, 17, 5, 80]], 300),
    "longest": ([0], [700], [[200, 124]], 1024),
    "one_too_long": ([0], [700], [[200, 125]], 1025),
    "all_padding_rows": ([900], [50], [[30, 20]], 1010),
}
IN_MEMORY = ("padding_around", "nine_runs", "one_too_long")


def _tables(case):
    off, p, r, T = CASES[case]
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in r])]).astype(np.int32)
    return off, p, ptr, np.array([x for y in r for x in y], dtype=np.int32), T


def _step(case, T, tens, scale, in_args, theta=None):
    import torch
    off, p, ptr, resp, _ = _tables(case)
    meta = ps.psattn_build_meta_multi(off, p, ptr, resp, T)
    assert (meta.device_bytes() == 0) == in_args
    t = {n: torch.zeros((T,) + tuple(x.shape[1:]), dtype=x.dtype, device="cuda") for n, x in tens.items()}
    for n, x in tens.items():
        t[n][:x.shape[0]] = x
    if theta is None:
        O, LSE = ps.psattn_fwd(meta, t["Q"], t["K"], t["V"], scale)
        grads = ps.psattn_bwd(meta, t["Q"], t["K"], t["V"], O, t["dO"], LSE, scale)
        out = (O, LSE.T) + tuple(grads)
    else:
        rope = ps.Rope(128, theta, meta.positions()[1])
        O, LSE, Qr, Kr = ps.psattn_fwd_rope(meta, rope, t["Q"], t["K"], t["V"], scale)
        out = (O, LSE.T, Qr, Kr) + tuple(ps.psattn_bwd_rope(meta, rope, Qr, Kr, t["V"], O, t["dO"], LSE, scale))
    torch.cuda.synchronize()
    n = tens["Q"].shape[0]
    return [x[:n] for x in out]


@pytest.mark.parametrize("dtype,d,theta", [("bf16", 128, None), ("bf16", 128, 10000.0), ("bf16", 64, None), ("f32", 64, None), ("f32", 128, None)])
@pytest.mark.parametrize("case", sorted(CASES))
def test_mask_in_arguments(case, dtype, d, theta):
    import torch
    T = CASES[case][3]
    gen = torch.Generator(device="cuda").manual_seed(8)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    tens = {n: torch.randn((T, h, d), generator=gen, device="cuda").to(dt) for n, h in (("Q", 4), ("K", 2), ("V", 2), ("dO", 4))}
    a = _step(case, T, tens, d ** -0.5, case not in IN_MEMORY, theta)
    b = _step(case, 1300, tens, d ** -0.5, False, theta)
    for x, y in zip(a, b):
        assert torch.equal(x, y)
