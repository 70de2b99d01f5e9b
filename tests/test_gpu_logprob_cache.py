"""The log-sum-exp reads its rows by non-temporal loads where those with a target hold more than 256 MB: either side of that line,
rows of whole and of odd 16-byte groups, every row of the gradient against 64-bit sums by plain torch operations."""
import numpy as np
import pytest
import torch

import paper_2410_20305_amd as ps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,vocab,resp", [(torch.bfloat16, 50257, 1300), (torch.bfloat16, 50257, 1350), (torch.float32, 32000, 1040),
                                              (torch.float32, 32000, 1060)])
def test_every_row(dtype, vocab, resp):
    off, P, ptr, rl, T = [3, 2 * resp + 20], [10, 0], [0, 2, 3], [resp, resp, 5], 2 * resp + 40
    size = 4 if dtype == torch.float32 else 2
    rows = 1 + 2 * (resp - 1) + 4
    assert (rows * vocab * size > 256 << 20) == (resp in (1350, 1060))
    gen = torch.Generator(device="cuda").manual_seed(resp)
    logits = (3 * torch.randn(T, vocab, generator=gen, device="cuda")).to(dtype)
    ids = torch.randint(0, vocab, (T,), generator=gen, device="cuda", dtype=torch.int32)
    plan = ps.LogprobPlan(off, P, ptr, rl, T)
    row_lse, _ = ps.psattn_logprob_fwd(plan, logits, ids)
    d_logp = torch.tensor([0.7, -1.3, 0.4], device="cuda")
    g = ps.psattn_logprob_bwd(plan, logits, ids, row_lse, d_logp)
    target = np.full((T, 2), -1)       # token that the row predicts, its response
    for j, first in enumerate((13, 13 + resp, 2 * resp + 20)):
        for u in range(1, rl[j]):
            target[first + u - 1, 0] = first + u
            target[first + u - 1, 1] = j
    for t in range(0, T, 256):
        n = min(256, T - t)
        want = torch.zeros(n, vocab, dtype=torch.float64, device="cuda")
        soft = torch.softmax(logits[t:t + n].double(), dim=1)
        for i in range(n):
            items = [(13, 0), (13 + resp, 1)] if t + i == 12 else [tuple(target[t + i])] if target[t + i, 0] >= 0 else []
            for tok, j in items:
                want[i] -= d_logp[j].double() * soft[i]
                want[i, ids[tok].long()] += d_logp[j].double()
        err = (g[t:t + n].double() - want).abs()
        # half a bf16 ulp, the error of one fp32 exponential of a difference of magnitude 30, and of coef * softmax (as in test_gpu_logprob.py)
        bar = want.abs() * (2.0 ** -8 if dtype == torch.bfloat16 else 0) + 1e-6
        assert bool((err <= bar).all()), (t, float((err - bar).max()))
        silent = (want == 0).all(dim=1)
        assert bool((g[t:t + n][silent] == 0).all())
