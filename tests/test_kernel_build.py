"""Static checks on the compiled MFMA kernels (CPU only: hipcc cross-compiles gfx950).

The dK/dV kernel keeps dK, dV and its K/V fragments in the accumulation registers
a[0:191] and addresses them by name from inline assembly.  That is only sound while the
compiler itself never touches an accumulation register in that kernel and spills nothing,
which is what these tests pin down, together with the absence of spills in the other two
kernels (a spill there costs scratch traffic in the hot loop).
"""
import os
import re
import subprocess

import pytest

from paper_2410_20305_amd import build


def _asm(tmp_path, src):
    return build.device_asm(src, str(tmp_path / (src + ".s")))


def _kernels(text, kernel, count):
    """Every instantiation of `kernel` in the file: (name, device code, metadata scalars).  `count` pins how many there are."""
    meta = {}
    for b in re.split(r"\n  - \.agpr_count:", text)[1:]:
        d = dict(re.findall(r"\.([a-z_]+):\s+(\S+)", ".agpr_count:" + b))
        meta[d["name"]] = d
    out = []
    for name in re.findall(r"\.amdhsa_kernel (\S+)", text):
        start, end = text.index("\n" + name + ":"), text.index(".amdhsa_kernel " + name + "\n")
        if kernel in name:
            out.append((name, text[start:end], meta[name]))
    assert len(out) == count, (kernel, [n for n, _, _ in out])
    return out


def _outside_asm(body):
    """Instruction lines that the compiler itself emitted."""
    inside = False
    for ln in body.splitlines():
        if "#ASMSTART" in ln:
            inside = True
        elif "#ASMEND" in ln:
            inside = False
        elif not inside:
            code = ln.split(";")[0].strip()
            if code and not code.startswith(".") and not code.endswith(":"):
                yield code


def _no_spills(name, meta):
    assert int(meta["vgpr_spill_count"]) == 0 and int(meta["sgpr_spill_count"]) == 0, name
    assert int(meta["private_segment_fixed_size"]) == 0, name


def test_dkdv_accumulation_registers_belong_to_the_assembly(tmp_path):
    text = _asm(tmp_path, "psattn_mfma_dkdv.hip")
    for name, body, meta in _kernels(text, "psattn_dkdv_bf16_mfma", 2):
        offenders = [c for c in _outside_asm(body) if re.search(r"accvgpr|\ba\[|[ ,\[]a\d+\b", c)]
        assert not offenders, (name, offenders[:5])
        assert int(meta["agpr_count"]) == 192, name
        _no_spills(name, meta)
        # one wave per SIMD: ordinary + accumulation registers of one lane
        assert int(meta["vgpr_count"]) <= 512, name


@pytest.mark.parametrize("src,kernel,count,waves", [("psattn_mfma_fwd.hip", "psattn_fwd_bf16_mfma", 1, [2]),
                                                    ("psattn_mfma_fwd64.hip", "psattn_fwd_bf16_mfma", 1, [3]),
                                                    ("psattn_mfma_bwd.hip", "psattn_dq_bf16_mfma", 2, [2, 3])])
def test_two_workgroups_per_cu_without_spills(tmp_path, src, kernel, count, waves):
    for (name, _, meta), n in zip(_kernels(_asm(tmp_path, src), kernel, count), waves):
        assert int(meta["vgpr_count"]) <= 512 // n // 8 * 8, name   # n waves per SIMD, registers in eights
        assert int(meta["agpr_count"]) == 0, name
        _no_spills(name, meta)
        assert int(meta["group_segment_fixed_size"]) <= 160 * 1024 // n, name  # n workgroups in 160 KB of LDS


@pytest.mark.parametrize("src,count", [("psattn_mfma_fwd.hip", 1), ("psattn_mfma_fwd64.hip", 1), ("psattn_mfma_bwd.hip", 2),
                                       ("psattn_mfma_dkdv.hip", 2), ("psattn_mfma_dkdv64.hip", 2)])
def test_compiler_keeps_m0_and_the_copy_counter_free(tmp_path, src, count):
    """The asynchronous global -> LDS copies are issued from inline assembly that writes M0
    and counts its own outstanding copies (vmcnt).  Sound only while compiled code never
    keeps a value in M0, and while the only vector-memory loads the compiler issues between
    the first and the last copy are the one-dword tile-list refills."""
    for name, body, _ in _kernels(_asm(tmp_path, src), "_mfma", count):
        for code in _outside_asm(body):
            assert not re.search(r"\bm0\b", code), (name, code)
        first, last = body.index("global_load_lds_dwordx4"), body.rindex("global_load_lds_dwordx4")
        loop = "#ASMSTART\n" + body[first:last]  # the slice starts in the middle of an assembly statement
        for code in _outside_asm(loop):
            m = re.match(r"(global_load|buffer_load|flat_load|scratch_load)\w*", code)
            if m:
                assert m.group(0) == "global_load_dword", (name, code)


def test_dkdv64_two_waves_per_simd_without_spills(tmp_path):
    """The head_dim 64 dK/dV kernel is left to the compiler: two waves per SIMD, nothing spilled, M0 untouched."""
    for name, body, meta in _kernels(_asm(tmp_path, "psattn_mfma_dkdv64.hip"), "psattn_dkdv64_bf16_mfma", 2):
        assert int(meta["vgpr_count"]) <= 256 and int(meta["agpr_count"]) == 0, name
        _no_spills(name, meta)
        for code in _outside_asm(body):
            assert not re.search(r"\bm0\b", code), (name, code)


@pytest.mark.parametrize("kernel,count", [("generic_fwd", 4), ("generic_dq", 4), ("generic_dkdv", 4), ("generic_bwd", 4)])
def test_generic_kernels_without_spills(tmp_path, kernel, count):
    for name, _, meta in _kernels(_asm(tmp_path, "psattn_generic.hip"), kernel, count):
        _no_spills(name, meta)
        assert int(meta["vgpr_count"]) <= 256, name  # eight waves to a workgroup


def test_upload_blocks_up_to_the_largest_buffer(tmp_path):
    """Workgroups that expand the token descriptors, for every T that total_tokens can name: rounding up must not leave int32,
    and the last workgroup's token numbers (1024 per workgroup) must not either."""
    src = tmp_path / "blocks.hip"
    src.write_text("""#include "psattn_internal.h"
using namespace psattn;
static_assert(upload_blocks(0) == 0 && upload_blocks(1) == 1 && upload_blocks(1024) == 1 && upload_blocks(1025) == 2, "");
static_assert(upload_blocks(INT32_MAX) == 1 << 21 && upload_blocks(INT32_MAX - 1023) == (1 << 21) - 1, "");
static_assert(int64_t{upload_blocks(INT32_MAX)} * kUploadTokens - 1 == INT32_MAX, "");
""")
    subprocess.check_call([build.hipcc(), "--offload-arch=gfx950", "-std=c++17", "-x", "hip", "-fsyntax-only", "-w", "-I",
                           os.path.join(build.ROOT, "include"), "-I", build.CSRC, str(src)])
