"""The lossless calls use no memory besides their buffers (include/zc.h): none of their kernels keeps
anything in scratch memory, which the runtime would have to allocate.  Read from the assembly that the
library's compiler and flags make of csrc/zl_kernels.hip; no GPU."""
import re
import subprocess

from paper_2409_02423_amd import build


def test_lossless_kernels_use_no_scratch(tmp_path):
    source = [s for s in build.SOURCES if s.endswith("zl_kernels.hip")][0]
    out = str(tmp_path / "zl.s")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([build.HIPCC] + flags + ["-S", "--cuda-device-only", source, "-o", out],
                          stderr=subprocess.DEVNULL)
    text = open(out).read()
    kernels = re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", text, flags=re.S)
    assert sum("zl_compress_kernel" in name for name, _ in kernels) == 2
    for name, meta in kernels:
        assert re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", meta).group(1) == "0", name
