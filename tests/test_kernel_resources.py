"""Build-time guard (no GPU): the hot kernels must not touch scratch memory.  A spill or a stack object in one of
them costs more than any tuning gains (a lone wave per SIMD cannot hide scratch latency), and it happens silently
when a change makes the register allocator give up."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_17834_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

HOT = {
    "asp_bcsr_wide.hip": ["bcsr_spmm_wide_kernel"],
    "asp_bcsr.hip": ["bcsr_spmm_kernel"],
    "asp_bcsr_dma.hip": ["bcsr_spmm_dma_kernel"],
    "asp_bcsr_strip.hip": ["bcsr_strip_kernel"],
    "asp_bcsr_xt.hip": ["bcsr_xt_strip_kernel", "bcsr_xt_staged_kernel", "bcsr_xt_decode_kernel"],
    "asp_bcsr_f32.hip": ["bcsr_f32_spmm_kernel"],
    "asp_wcsr.hip": ["wcsr16_spmm_kernel", "wcsr32_spmm_kernel"],
    "asp_wcsr_rows.hip": ["wcsr_rows_kernel"],
    "asp_wcsr_groups.hip": ["wcsr_groups_kernel"],
    "asp_wcsr_dense.hip": ["wcsr_dense_kernel"],
    "asp_wcsr_bf16.hip": ["wcsr_bf16_spmm_kernel"],
}


@functools.lru_cache(maxsize=4)
def _compiled(source, *options):
    """What the compiler makes of a source's device code, as text."""
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        subprocess.check_call([HIPCC, "-O3", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                               "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                               "-S", "--cuda-device-only", *options, "-o", out, os.path.join(CSRC, source)],
                              stderr=subprocess.DEVNULL)
        return open(out).read()


@pytest.mark.parametrize("source", sorted(HOT))
def test_hot_kernels_use_no_scratch(source):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    text = _compiled(source)
    seen = set()
    for m in re.finditer(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)", text):
        name, scratch = m.group(1), int(m.group(2))
        kernels = [k for k in HOT[source] if k in name]
        if kernels:
            seen.update(kernels)
            assert scratch == 0, "%s uses %d bytes of scratch per lane" % (name, scratch)
    assert seen == set(HOT[source])


def test_groups_leave_room_for_three_workgroups():
    """wcsr_groups_kernel: the waves of an XCD's column tile have to be resident at once, and half of a second tile's: three
    workgroups of four waves to a compute unit, so at most 512 / 3 registers a lane."""
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    found = re.findall(r"\.name:\s+(\S*wcsr_groups_kernel\S*)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)", _compiled("asp_wcsr_groups.hip"))
    assert len(found) == 2 and all(int(n) <= 168 for _, n in found), found


def _registers(kind, operands):
    found = set()
    for first, last in re.findall(r"\b%s\[?(\d+)(?::(\d+))?" % kind, operands):
        found |= set(range(int(first), int(last or first) + 1))
    return found


def test_staged_strips_wait_for_their_last_products():
    """bcsr_xt_staged_kernel multiplies in inline assembly, which the compiler's waits do not cover: its own wait has to hold all
    accumulators, so that nothing reads them before it, and no VALU result may be an operand in the next two instructions."""
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    ir = _compiled("asp_bcsr_xt.hip", "-emit-llvm")
    waits = re.findall(r'asm sideeffect "s_nop 15[^"]*", "([^"]*)"', ir)
    assert sorted(w.count("=a") for w in waits) == [4, 4, 8]     # 64-row strips of both block sizes, 128-row strips
    kernels = [k for k in re.split(r"(?m)^(?=_ZN\S+:)", _compiled("asp_bcsr_xt.hip")) if k.startswith("_ZN3asp21bcsr_xt_staged_kernel")]
    assert len(kernels) == 3
    for k in kernels:
        code = [l.split(";")[0].split() for l in k[:k.index("s_endpgm")].splitlines()]
        code = [l for l in code if l and re.match(r"[a-z]+_", l[0])]
        last = max(i for i, l in enumerate(code) if l[0].startswith("v_mfma"))
        wait = next(i for i in range(last, len(code)) if code[i] == ["s_nop", "15"])
        sums = set().union(*(_registers("a", l[1]) for l in code if l[0].startswith("v_mfma")))
        assert len(sums) in (64, 128) and not any(sums & _registers("a", " ".join(l[1:])) for l in code[last + 1:wait])
        for i, l in enumerate(code):
            if l[0].startswith("v_mfma") and code[i - 1][0] != "s_nop":
                read = _registers("v", " ".join(l[1:]))
                for w in code[i - 2:i]:
                    if w[0].startswith("v_") and not w[0].startswith("v_mfma"):
                        assert not read & _registers("v", w[1]), (w, l)


def test_decode_kernels_that_are_built_are_reached():
    """bcsr_xt_decode_kernel: the waves and tokens that decode_waves gives each block size, and no others."""
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    found = re.findall(r"\.name:\s+\S*bcsr_xt_decode_kernelILi(\d+)ELi(\d+)ELi(\d+)E", _compiled("asp_bcsr_xt.hip"))
    shapes = {(int(a), int(b), int(c)) for a, b, c in found}
    assert shapes == {(32, 1, 8), (64, 1, 4), (64, 1, 8), (64, 2, 8), (128, 1, 4), (128, 1, 8), (128, 2, 8)}
