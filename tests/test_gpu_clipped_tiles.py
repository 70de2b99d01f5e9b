"""bf16 kernels on buffers whose length is no multiple of a tile: the last tile of either grid stands for the last 64 rows of the
buffer, of which the ones before its own first are masked, and a buffer of fewer than 64 rows re-reads its last one.  Lengths on
either side of multiples of 32, 64 and 128, with one sample, with several in the last 64 rows, with padding at the end and with a
hidden range that ends in the last tile; dK/dV rows in one piece and split.  Against the oracle, bars as in test_gpu_parity.py."""
import pytest

import paper_2410_20305_amd as ps
import psattn_workloads as W
from gpu_util import run_gpu
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
