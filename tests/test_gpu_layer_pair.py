"""The layer's dWk and dWv as one batch of two or one by one: the rule's two lines (CPU only: checked at compile time), and both ways
against the oracle at the token counts on either side of the room, bar as in test_gpu_layer.py.  The gradients come out of
one workspace twice, and both times with the same bytes."""
import os
import subprocess

import numpy as np
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W
from oracle import psattn_oracle as orc
from paper_2410_20305_amd import build

HIDDEN, HQ, HKV, D = 256, 4, 2, 128


def room(T):  # places of the unrotated Q and K, each a whole number of 256 bytes
    return T * (HQ + HKV) * D * 2


def test_rule(tmp_path):
    src = tmp_path / "rule.cpp"
    src.write_text("""#include "%s"
constexpr size_t kAll = ~size_t{0};
static_assert(!weights_as_pair(%d, %d, %d) && weights_as_pair(%d, %d, %d), "room");
static_assert(weights_as_pair(1024, 8192, kAll) && weights_as_pair(2048, 4096, kAll) && weights_as_pair(128, 1, kAll), "half the chip");
static_assert(!weights_as_pair(1024, 8193, kAll) && !weights_as_pair(2176, 4096, kAll) && !weights_as_pair(3072, 3072, kAll), "more than half");
static_assert(!weights_as_pair(4096, 4096, kAll), "32 / 32 heads at hidden 4096");
static_assert(!weights_as_pair(128, 5, 2559) && weights_as_pair(128, 5, 2560) && !weights_as_pair(129, 5, 1536 + 1289) && weights_as_pair(129, 5, 1536 + 1290), "the second result starts on a multiple of 256 bytes");
""" % (os.path.join(build.CSRC, "psattn_layer.cpp"), HKV * D, HIDDEN, room(170), HKV * D, HIDDEN, room(171)))
    subprocess.check_call([build.hipcc(), "--offload-arch=gfx950", "-std=c++17", "-x", "hip", "-fsyntax-only", "-w", "-I",
                           os.path.join(build.ROOT, "include"), str(src)])


@pytest.mark.gpu
@pytest.mark.parametrize("T", [170, 171])
def test_both_ways(T):
    import torch
    from gpu_util import rel_l2, to_np
    from paper_2410_20305_amd.layer import Layer
    off, P, ptr, rl, theta, scale = [2], [T - 92], [0, 2], [50, 37], 10000.0, 1.0 / np.sqrt(D)
    rng = np.random.default_rng(T)
    bf = lambda x: W.bf16_round(x.astype(np.float32))
    X, dY = bf(rng.standard_normal((T, HIDDEN))), bf(rng.standard_normal((T, HIDDEN)))
    Wq, Wk, Wv = (bf(rng.standard_normal((h * D, HIDDEN)) / np.sqrt(HIDDEN)) for h in (HQ, HKV, HKV))
    Wo = bf(rng.standard_normal((HIDDEN, HQ * D)) / np.sqrt(HQ * D))
    meta = ps.psattn_build_meta_multi(off, P, ptr, rl, T)
    rope = ps.Rope(D, theta, meta.positions()[1])
    layer = Layer(HIDDEN, HQ, HKV, D)
    args = (meta, rope, scale) + tuple(torch.from_numpy(a).to("cuda").to(torch.bfloat16) for a in (X, Wq, Wk, Wv, Wo))
    tdY = torch.from_numpy(dY).to("cuda").to(torch.bfloat16)
    ws = torch.empty(layer.workspace_bytes(meta), dtype=torch.uint8, device="cuda")
    layer.forward(*args, ws)
    grads = layer.backward(*args, tdY, ws)
    again = layer.backward(*args, tdY, ws)
    assert all(torch.equal(a, b) for a, b in zip(grads, again))
    Dd, B = orc.branch_arrays(off, P, ptr, rl, T)
    ref = orc.layer_backward(X, Wq, Wk, Wv, Wo, dY, scale, theta, Dd, B, lambda *a: orc.dense_branch_mask(Dd, B, *a), HQ, HKV,
                             round_act=lambda x: bf(x).astype(np.float64))
    for name, g in zip(("dX", "dWq", "dWk", "dWv", "dWo"), grads):
        e = rel_l2(to_np(g), ref[name])
        assert np.all(np.isfinite(to_np(g))) and e <= 2e-2, (name, e)
    layer.free()
    rope.free()
    meta.free()
