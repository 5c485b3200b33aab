"""What the kernels' code must and must not hold, read from the assembly that the library's compiler and flags
make of their sources; no GPU.

The lossless calls use no memory besides their buffers (include/zc.h): none of their kernels keeps anything in
scratch memory, which the runtime would have to allocate.  And no inline assembly of the 4 x 4 kernels reads a
register that a matrix instruction wrote: how long a reader has to wait for it, the compiler sees to for the
instructions that it knows only."""
import re
import subprocess

from paper_2409_02423_amd import build


def _assembly(tmp_path, name):
    source = [s for s in build.SOURCES if s.endswith(name)][0]
    out = str(tmp_path / "kernels.s")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([build.HIPCC] + flags + ["-S", "--cuda-device-only", source, "-o", out],
                          stderr=subprocess.DEVNULL)
    return open(out).read()


def test_lossless_kernels_use_no_scratch(tmp_path):
    text = _assembly(tmp_path, "zl_kernels.hip")
    kernels = re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", text, flags=re.S)
    assert sum("zl_compress_kernel" in name for name, _ in kernels) == 2
    for name, meta in kernels:
        assert re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", meta).group(1) == "0", name


def _registers(operand):
    m = re.fullmatch(r"[-|]*v\[(\d+):(\d+)\][|]*", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"[-|]*v(\d+)[|]*", operand)
    return {int(m.group(1))} if m else set()


def test_inline_assembly_reads_no_matrix_results(tmp_path):
    from_matrix, inline, products, blocks = set(), False, 0, 0
    for line in _assembly(tmp_path, "zc2d_kernels.hip").splitlines():
        line = line.strip()
        if line in (";;#ASMSTART", ";;#ASMEND"):
            inline = line == ";;#ASMSTART"
            continue
        m = re.match(r"(v_\w+|ds_read\w*|global_load\w*|scratch_load\w*)\s+([^;]*)", line)
        if not m:
            continue
        operands = [o.strip().split(" ")[0] for o in m.group(2).split(",")]
        if inline:
            blocks += 1
            assert not any(_registers(o) & from_matrix for o in operands[1:]), line
        if m.group(1).startswith("v_mfma"):
            products += 1
            from_matrix |= _registers(operands[0])
        elif not m.group(1).startswith("v_cmp"):
            from_matrix -= _registers(operands[0])
    assert products >= 8 and blocks > 0
