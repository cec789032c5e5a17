"""Dynamic LDS that a kernel reads or writes 16 bytes at a time has to be declared
16-byte aligned: it starts after the kernel's static LDS, whose size is only a
multiple of 8.  Looked up in the compiler's own record of every dynamic LDS array
of the batched kernels (no GPU needed)."""
import os
import re
import subprocess

from paper_1401_2720_amd import build


def test_dynamic_lds_is_aligned_for_16_byte_accesses(tmp_path):
    out = tmp_path / "batched.ll"
    subprocess.run([build.HIPCC, *[f for f in build.FLAGS if f != "-O3"], "-O0", "-w",
                    "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-x", "hip",
                    "--cuda-device-only", "-S", "-emit-llvm",
                    os.path.join(build.CSRC, "jsvd_batched.hip"), "-o", str(out)], check=True)
    arrays = re.findall(r"^@(\S+) = external addrspace\(3\) global \[0 x double\], align (\d+)",
                        out.read_text(), re.M)
    assert arrays and all(int(a) >= 16 for _, a in arrays), arrays
