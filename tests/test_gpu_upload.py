"""The block mask as the kernels read it: token descriptors are expanded on the device from runs of equal ones, 1024
tokens to a workgroup, up to 256 runs fetched at once and more through a per-workgroup index.  Checked through forward
and backward against the oracle on tables that reach both ways and their edges."""
import numpy as np
import pytest

import psattn_workloads as W
from gpu_util import run_gpu
from test_gpu_parity import compare_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,gap,T,dtype", [(63, 1, 1024, "f32"),     # 252 runs and a tail, one workgroup exactly
                                           (85, 0, 1025, "bf16"),    # 255 runs and a tail; one token behind a workgroup's end
                                           (64, 1, 1500, "bf16"),    # 256 runs and a tail: the index
                                           (400, 1, 2900, "f32"),    # 1600 runs, some 550 to a workgroup
                                           (1, 5, 4097, "f32")])     # few runs, mostly padding
def test_many_runs_of_descriptors(n, gap, T, dtype):
    rng = np.random.default_rng(n)
    samples, offsets, at = [], [], 0
    for _ in range(n):
        s = tuple(int(x) for x in rng.integers(1, 4, 3)) if n > 1 else (700, 300, 200)
        at += gap
        samples.append(s)
        offsets.append(at)
        at += sum(s)
    assert at <= T
    w = W.custom_workload(samples, offsets=offsets, total_tokens=T, hq=2, hkv=1, d=64 if dtype == "f32" else 128, dtype=dtype, seed=n)
    tens = W.make_tensors(w)
    out, _ = run_gpu(w, tens)
    compare_full(w, tens, out, dtype, what="runs of descriptors")
