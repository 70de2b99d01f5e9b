"""Rows with a target that do not fit the last-level cache are read by non-temporal loads (CPU only: the compiled gfx950 code is
read): log-probabilities that no gradient follows take 11 - 14 % longer by ordinary ones."""
import re

from test_kernel_build import _asm, _kernels


def test_rows_have_a_non_temporal_way(tmp_path):
    kernels = _kernels(_asm(tmp_path, "psattn_logprob.hip"), "psattn_lp_row_lse", 8)  # both types, whole and odd rows, both ways
    ways = []
    for name, body, _ in kernels:
        loads = [ln.split(";")[0] for ln in body.splitlines() if re.search(r"\bglobal_load_dwordx4\b", ln)]
        assert len(loads) >= 5, name  # four in flight and one
        nt = [bool(re.search(r"\bnt\b", ln)) for ln in loads]
        assert len(set(nt)) == 1, (name, loads)
        ways.append(nt[0])
    assert sorted(ways) == [False] * 4 + [True] * 4, ways
