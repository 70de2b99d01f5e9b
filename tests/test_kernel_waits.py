"""A block mask in the kernels' arguments is searched while the first copies are in flight (CPU only: the compiled gfx950 code is
read).  The compiler does not count those copies, so a wait for a vector load that it places there would be a wait for all of
them: the blocks that search (they take the 11-bit fields of the packed runs apart) hold none."""
import re

import pytest

from test_kernel_build import _asm, _kernels


@pytest.mark.parametrize("src,count", [("psattn_mfma_fwd.hip", 1), ("psattn_mfma_fwd64.hip", 1), ("psattn_mfma_fwd3.hip", 1), ("psattn_mfma_bwd.hip", 2),
                                       ("psattn_mfma_dkdv.hip", 2), ("psattn_mfma_dkdv64.hip", 2)])
def test_search_waits_for_no_copy(tmp_path, src, count):
    for name, body, _ in _kernels(_asm(tmp_path, src), "_mfma", count):
        body = body[body.index("global_load_lds_dwordx4"):body.index("v_mfma")]
        searches = [b for b in re.split(r"\n\.LBB\w+:", body) if "0x7ff\n" in b or "0x7ff," in b]
        assert searches, name
        for b in searches:
            assert not re.search(r"s_waitcnt[^\n]*vmcnt", b), (name, re.findall(r"s_waitcnt[^\n]*", b))
