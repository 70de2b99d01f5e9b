"""Lines between two forms of a bf16 kernel at head_dim 128 (CPU only: the rules are checked at compile time, on the counts that the
host's block mask gives for tables on either side)."""
import os
import subprocess

import numpy as np
import pytest

import paper_2410_20305_amd as ps
from paper_2410_20305_amd import build


def lists(samples, grid):
    """(rows, entries of the longest row, entries of all rows)."""
    p, c, r = (np.array(x, dtype=np.int32) for x in zip(*samples))
    off = np.concatenate([[0], np.cumsum(p + c + r)]).astype(np.int32)
    m = ps.psattn_build_meta(off[:-1], p, c, r, int(off[-1]), host_only=True)
    n = np.diff(m.csr(grid)[0])
    return int(off[-1]), len(n), int(n.max()), int(n.sum())


def check(tmp_path, source, lines):
    src = tmp_path / "rule.hip"
    src.write_text("#include \"%s\"\nusing namespace psattn;\n%s\n" % (os.path.join(build.CSRC, source), "\n".join(lines)))
    subprocess.check_call([build.hipcc(), "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-x", "hip", "-fsyntax-only", "-w", "-I",
                           os.path.join(build.ROOT, "include"), "-I", build.CSRC, str(src)])


FORWARD = [  # samples, q heads, three workgroups to a CU or two
    ([(6000, 20, 20)], 16, False),         # 768 workgroups, the longest row 95 tiles, twice a slot's share
    ([(6000, 20, 20)], 32, False),         # 1 536
    ([(6000, 20, 20)], 64, True),          # 3 072: half a share
    ([(1500, 200, 200)] * 3, 32, False),
    ([(1500, 200, 200)] * 12, 32, True),
    ([(600, 100, 60)] * 2, 64, False),     # 13 tiles
    ([(128, 64, 64)] * 24, 16, True),      # short rows, 768 workgroups
    ([(128, 64, 64)] * 23, 16, False),     # 736
    ([(30, 20, 13)], 768, False),          # 63 tokens
    ([(30, 20, 14)], 768, True),
]


def test_forward(tmp_path):
    lines = []
    for samples, hq, three in FORWARD:
        T, rows, longest, tiles = lists(samples, ps.GRID_FWD)
        lines.append("static_assert(three_to_a_cu(%d, %d, %d, %d) == %s, \"\");" % (T, rows * hq, longest, tiles * hq, str(three).lower()))
    check(tmp_path, "psattn_mfma_fwd3.hip", lines)


BACKWARD = [  # samples, q heads, kv heads, rows split or not
    ([(10, 8, 7)] * 220, 28, 4, False),      # 21 steps, 172 workgroups of one length
    ([(40, 15, 15)], 768, 192, False),       # 8 steps, 192 workgroups
    ([(1024, 128, 128)] * 4, 32, 8, True),   # 80 steps, 1.48 shares
    ([(1200, 100, 50)] * 5, 32, 8, False),   # 92 steps, 1.09 shares
    ([(2000, 100, 50)] * 2, 32, 8, True),    # 144 steps, 1.78 shares
    ([(110, 50, 40)], 4, 4, False),          # 4 steps
    ([(110, 50, 40)], 8, 4, True),           # 8 steps
]


def test_backward(tmp_path):
    lines = []
    for samples, hq, hkv, split in BACKWARD:
        _, _, longest, tiles = lists(samples, ps.GRID_BWD)
        lines.append("static_assert(split_rows(%d, %d) == %s, \"\");" % (longest * (hq // hkv), tiles * hq, str(split).lower()))
    check(tmp_path, "psattn_mfma_dkdv.hip", lines)
