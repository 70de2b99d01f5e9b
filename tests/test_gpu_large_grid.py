"""More 16-row blocks than one grid of the fp32 / generic kernels may hold (2^23 workgroups of 512 threads), forward and
backward, on one-token samples: O is V of the token, LSE the one score, dV the sum of dO over the heads of the group."""
import numpy as np
import pytest

import paper_2410_20305_amd as ps

pytestmark = pytest.mark.gpu


def test_more_blocks_than_one_grid_holds():
    import torch
    T, hq, d, scale = 1 << 22, 32, 64, 0.125
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of device memory")
    one, zero = np.ones(T, np.int32), np.zeros(T, np.int32)
    meta = ps.psattn_build_meta(np.arange(T, dtype=np.int32), one, zero, zero, T, 64, 64, 64, 64)
    assert not meta.uses_mfma(ps.BF16, d, scale)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    Q = torch.randn((T, hq, d), generator=gen, device="cuda", dtype=torch.bfloat16)  # dO as well
    K, V = (torch.randn((T, 1, d), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    O, LSE = torch.full_like(Q, float("nan")), torch.full((hq, T), float("nan"), device="cuda")
    ps.psattn_fwd(meta, Q, K, V, scale, O=O, LSE=LSE)
    dQ, dK, dV = torch.full_like(Q, float("nan")), torch.full_like(K, float("nan")), torch.full_like(V, float("nan"))
    ps.psattn_bwd(meta, Q, K, V, O, Q, LSE, scale, dQ=dQ, dK=dK, dV=dV)
    for t in range(0, T, 1 << 18):
        s = slice(t, t + (1 << 18))
        q, k, v = Q[s].float(), K[s].float(), V[s].float()
        assert torch.equal(O[s], V[s].expand(-1, hq, -1)), t
        # 64 products of 2^-24 relative error and magnitude up to 4^2, times the scale
        assert float((LSE[:, s] - scale * (q * k).sum(-1).t()).abs().max()) <= 64 * 16 * scale * 2.0 ** -24, t
        # dS = dO V - delta, the same 64 products summed in two orders; times the scale and |K| <= 8
        bar = 2 * 64 * 32 * 2.0 ** -24 * scale * 8
        assert float(dQ[s].float().abs().max()) <= bar and float(dK[s].float().abs().max()) <= hq * bar, t
        ref = q.sum(1, keepdim=True)  # |sum| up to 64: half a bf16 ulp there is 2^-3
        assert float((dV[s].float() - ref).abs().sub(ref.abs() * 2.0 ** -8).max()) <= 1e-4, t
    meta.free()
