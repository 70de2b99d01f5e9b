"""Logits rows whose 16-byte groups start anywhere: head, groups and tail of a row, the unrolled loop's remainder, buffers
that start off a 16-byte boundary (logits and gradient alike and differently), and logits of -inf.  Bars as in
test_gpu_logprob.py."""
import numpy as np
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W
from oracle import psattn_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("vocab,x_off,g_off", [(1, 0, 0), (7, 0, 0), (8, 3, 3), (255, 0, 0), (4096, 1, 1), (4099, 0, 0),
                                               (8191, 0, 0), (8193, 2, 5), (16390, 0, 0), (1000, 0, 1)])
def test_rows(dtype, vocab, x_off, g_off):
    import torch
    rng = np.random.default_rng(vocab)
    off, P, ptr, rl, T = [2, 20], [5, 0], [0, 2, 4], [4, 3, 2, 5], 29
    logits = (rng.standard_normal((T, vocab)) * 3).astype(np.float32)
    if dtype == "bf16":
        logits = W.bf16_round(logits)
    if vocab > 8:  # leading logits of -inf: a lane's first groups hold nothing else
        logits[:, : vocab // 2] = -np.inf
    ids = rng.integers(vocab // 2, vocab, size=T).astype(np.int32)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def at(offset):
        whole = torch.full((T * vocab + 64,), float("nan"), dtype=dt, device="cuda")
        return whole, whole[16 + offset:16 + offset + T * vocab].view(T, vocab)
    (_, x), (whole, g) = at(x_off), at(g_off)
    x.copy_(torch.from_numpy(logits))
    plan = ps.LogprobPlan(off, P, ptr, rl, T)
    tid = torch.from_numpy(ids).cuda()
    d_logp = rng.standard_normal(len(rl)).astype(np.float32)
    row_lse, logp = ps.psattn_logprob_fwd(plan, x, tid)
    ps.psattn_logprob_bwd(plan, x, tid, row_lse, torch.from_numpy(d_logp).cuda(), dlogits=g)
    torch.cuda.synchronize()
    fin = np.maximum(logits, -1e30)  # the oracle's stand-in for -inf: the same exponential, zero
    ref = orc.response_logprobs(fin, ids, off, P, ptr, rl)
    assert np.abs(logp.cpu().numpy().astype(np.float64) - ref).max() <= 1e-4
    gref = orc.response_logprobs_grad(fin, ids, off, P, ptr, rl, d_logp.astype(np.float64))
    got = g.float().cpu().numpy().astype(np.float64)
    tol = 1e-6 if dtype == "f32" else 2.0 ** -8 * np.abs(gref) + 1e-6
    assert np.all(np.isfinite(got)) and float((np.abs(got - gref) - tol).max()) <= 0
    outside = torch.cat([whole[:16 + g_off], whole[16 + g_off + T * vocab:]])
    assert outside.numel() == 64 and bool(torch.isnan(outside).all())  # nothing is stored beside the rows
    plan.free()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("vocab", [8, 16, 2048, 4096, 5120, 10240, 16392])
def test_whole_rows(dtype, vocab):
    """Rows that start on a boundary and are whole numbers of 16 bytes, on either side of the thread counts' lines."""
    test_rows(dtype, vocab, 0, 0)


def test_more_rows_than_a_grid_of_wide_rows_holds():
    """2^22 + 3 rows of 20 480 bytes: the gradient of the few rows that predict something, zeros everywhere else.  Logits,
    token ids and row sums are read at predicting rows only, so they are given for the first rows alone."""
    import torch
    T, vocab, head = (1 << 22) + 3, 10240, 32
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of device memory")
    off, P, ptr, rl = [2, 20], [5, 0], [0, 2, 4], [4, 3, 2, 5]
    rng = np.random.default_rng(3)
    logits = W.bf16_round((rng.standard_normal((head, vocab)) * 3).astype(np.float32))
    ids = rng.integers(0, vocab, size=head).astype(np.int32)
    d_logp = rng.standard_normal(len(rl)).astype(np.float32)
    small, plan = ps.LogprobPlan(off, P, ptr, rl, head), ps.LogprobPlan(off, P, ptr, rl, T)
    x, tid, dl = torch.from_numpy(logits).cuda().to(torch.bfloat16), torch.from_numpy(ids).cuda(), torch.from_numpy(d_logp).cuda()
    row_lse, _ = ps.psattn_logprob_fwd(small, x, tid)
    g = torch.full((T, vocab), float("nan"), dtype=torch.bfloat16, device="cuda")
    st = ps.load_library().psattn_logprob_bwd(plan.handle, ps.BF16, vocab, x.data_ptr(), tid.data_ptr(), row_lse.data_ptr(),
                                              dl.data_ptr(), g.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    gref = orc.response_logprobs_grad(logits, ids, off, P, ptr, rl, d_logp.astype(np.float64))
    got = g[:head].float().cpu().numpy().astype(np.float64)
    assert float((np.abs(got - gref) - 2.0 ** -8 * np.abs(gref)).max()) <= 1e-6
    for t in range(head, T, 1 << 17):
        assert int(torch.count_nonzero(g[t:t + (1 << 17)].view(torch.int16))) == 0, t
    small.free()
    plan.free()
