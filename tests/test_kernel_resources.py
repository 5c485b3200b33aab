"""What the kernels' code must and must not hold, read from the assembly that the library's compiler and flags
make of their sources; no GPU.

The lossless calls use no memory besides their buffers (include/zc.h): none of their kernels keeps anything in
scratch memory, which the runtime would have to allocate.  Kernels that just fit a number of wavefronts per SIMD do not
outgrow it.  And inline assembly, whose waits the compiler does not know of, keeps away from matrix
instructions and is not waited for where it is."""
import os
import re
import subprocess

import pytest

from paper_2409_02423_amd import build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """The assembly of each source by its name, all of them made side by side."""
    work = tmp_path_factory.mktemp("asm")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    running = []
    for source in build.SOURCES:
        out = str(work / (os.path.basename(source) + ".s"))
        running.append((os.path.basename(source), out, subprocess.Popen(
            [build.HIPCC] + flags + ["-S", "--cuda-device-only", source, "-o", out], stderr=subprocess.DEVNULL)))
    texts = {}
    for name, out, process in running:
        assert process.wait() == 0, name
        with open(out) as f:
            texts[name] = f.read()
    return texts


def test_lossless_kernels_use_no_scratch(assembly):
    text = assembly["zl_kernels.hip"]
    kernels = re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", text, flags=re.S)
    assert sum("zl_compress_kernel" in name for name, _ in kernels) == 2
    for name, meta in kernels:
        assert re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", meta).group(1) == "0", name


# Kernels whose registers are just few enough for so many wavefronts per SIMD: template arguments as they are mangled.
@pytest.mark.parametrize("source, kernel, waves", [
    ("zc_kernels.hip", "reduce_kernelILi12ELi2ELb0ELb1ELi0E", 8),
    ("zc_kernels.hip", "reduce_kernelILi24ELi2ELb1ELb0ELi0E", 8),
    ("zc_kernels.hip", "reduce_kernelILi28ELi2ELb0ELb1ELi0E", 8),
    ("zc_kernels.hip", "reduce_kernelILi32ELi2ELb0ELb1ELi0E", 8),
    ("zc2d_kernels.hip", "reduce2d_kernelILi2ELb1ELb0ELi512E", 6),
    ("zc2d_kernels.hip", "reduce2d_kernelILi4ELb1ELb0ELi512E", 6),
    ("zc2d_kernels.hip", "reduce2d_kernelILi8ELb1ELb0ELi512E", 6),
])
def test_kernels_that_just_fit_do(assembly, source, kernel, waves):
    m = re.search(r"^_Z\w*%s\w*:.*?; Occupancy: (\d+)" % kernel, assembly[source], flags=re.S | re.M)
    assert int(m.group(1)) >= waves


# What few wavefronts need is branched around (materialise_seldom in zc_codec.h), for zero blocks' sake.
@pytest.mark.parametrize("kernel", ["reduce_kernelILi12ELi2ELb0ELb1ELi2E", "reduce_kernelILi16ELi2ELb0ELb1ELi0E"])
def test_seldom_wanted_counts_are_branched_around(assembly, kernel):
    code = re.search(r"^_Z\w*%s\w*:.*?s_endpgm" % kernel, assembly["zc_kernels.hip"], flags=re.S | re.M).group(0)
    around = re.findall(r"s_cbranch_\w+ (\.LBB\w+)\n(?:(?!\.LBB|\s+s_cbranch).*\n)+?\s+; seldom\n\s+;;#ASMEND\n\1:", code)
    assert 0 < len(around) == code.count("; seldom")


# The step through a block's planes waits for nothing between the window's shift, which is inline assembly, and the
# next look-up: what reads such a result at once gets an idle cycle in front of it.
@pytest.mark.parametrize("kernel", ["reduce2d_kernelILi4ELb0ELb0ELi256E", "reduce2d_kernelILi4ELb0ELb0ELi512E"])
def test_nothing_waits_for_the_windows_shift(assembly, kernel):
    code = re.search(r"^_Z\w*%s\w*:.*?s_endpgm" % kernel, assembly["zc2d_kernels.hip"], flags=re.S | re.M).group(0)
    lines = [l.strip() for l in code.splitlines() if l.strip() and not l.strip().startswith((";", "."))]
    after = [b for a, b in zip(lines, lines[1:]) if a.startswith("v_lshrrev_b64")]
    assert after and not any(b.startswith("s_nop") for b in after)


def _registers(operand):
    m = re.fullmatch(r"[-|]*v\[(\d+):(\d+)\][|]*", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"[-|]*v(\d+)[|]*", operand)
    return {int(m.group(1))} if m else set()


# How long a matrix instruction and its neighbours have to wait for each other, the compiler sees to for the instructions that it
# knows.  Inline assembly reads no matrix result, writes no operand of a matrix instruction within the last few
# instructions before it, and none of its operands or results within the time that it takes.
kBefore, kAfter = 4, 20


@pytest.mark.parametrize("source, least", [("zc_kernels.hip", 16), ("zc2d_kernels.hip", 8)])
def test_inline_assembly_keeps_away_from_matrix_instructions(assembly, source, least):
    from_matrix, inline, products, blocks, at = set(), False, 0, 0, 0
    written, busy = [], []   # (place, registers) of what inline assembly wrote, and of matrix instructions
    for line in assembly[source].splitlines():
        line = line.strip()
        if line in (";;#ASMSTART", ";;#ASMEND"):
            inline = line == ";;#ASMSTART"
            continue
        if not re.match(r"[a-z]\w+(\s|$)", line):
            continue
        at += 1
        m = re.match(r"(v_\w+|ds_read\w*|global_load\w*|scratch_load\w*)\s+([^;]*)", line)
        if not m:
            continue
        operands = [_registers(o.strip().split(" ")[0]) for o in m.group(2).split(",")]
        if inline:
            blocks += 1
            assert not any(o & from_matrix for o in operands[1:]), line
            busy = [(p, r) for p, r in busy if at - p <= kAfter]
            assert not any(operands[0] & r for _, r in busy), line
            written.append((at, operands[0]))
        if m.group(1).startswith("v_mfma"):
            products += 1
            written = [(p, r) for p, r in written if at - p <= kBefore]
            assert not any(o & r for o in operands[1:] for _, r in written), line
            busy.append((at, set().union(*operands)))
            from_matrix |= operands[0]
        elif not m.group(1).startswith("v_cmp"):
            from_matrix -= operands[0]
    assert products >= least and blocks > 0
