"""Lanes of a wave hand rows to each other through LDS without a workgroup barrier (CPU only: the compiled gfx950 code is read).  LDS
is in order within a wave, but the compiler may move a lane's read above its write wherever the two addresses differ, so
every read that follows a write has to stand behind a workgroup or a wave barrier."""
import re

import pytest

from test_kernel_build import _asm, _kernels


@pytest.mark.parametrize("src,count", [("psattn_mfma_fwd.hip", 1), ("psattn_mfma_fwd64.hip", 1), ("psattn_mfma_fwd3.hip", 1), ("psattn_mfma_bwd.hip", 2),
                                       ("psattn_mfma_dkdv.hip", 2), ("psattn_mfma_dkdv64.hip", 2)])
def test_reads_behind_a_barrier(tmp_path, src, count):
    for name, body, _ in _kernels(_asm(tmp_path, src), "_mfma", count):
        written = None
        for ln in body.splitlines():
            if "s_barrier" in ln or "; wave barrier" in ln:
                written = None
            elif re.search(r"\bds_write", ln):
                written = ln.strip()
            elif re.search(r"\bds_read", ln):
                assert written is None, (name, written, ln.strip())
