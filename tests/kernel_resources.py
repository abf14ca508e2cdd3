"""What the compiler gives a source's kernels: registers, LDS and scratch of each, from the generated code (not collected by pytest)."""
import functools
import os
import re
import subprocess
import tempfile

from paper_2408_16978_amd import build as lib_build


@functools.lru_cache(maxsize=None)
def kernels(source):
    """{name: (vector registers, bytes of LDS, bytes of scratch)}"""
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "x.s")
        subprocess.run([lib_build.HIPCC] + lib_build.FLAGS + ["-S", "--cuda-device-only", os.path.join(lib_build.SRC_DIR, source), "-o", out],
                       check=True, capture_output=True)
        with open(out) as f:
            text = f.read()
    found = {}
    for m in re.finditer(r"\.group_segment_fixed_size: (\d+)(.*?)\.vgpr_count:\s+(\d+)", text, re.S):
        name = re.search(r"\.name:\s+(\S+)", m.group(2)).group(1)
        name = subprocess.run(["c++filt", name], capture_output=True, text=True, check=True).stdout
        scratch = re.search(r"\.private_segment_fixed_size: (\d+)", m.group(2)).group(1)
        # "void fpdt::(anonymous namespace)::kernel<..>(fpdt::(anonymous namespace)::Args)": up to the parameters
        key = re.split(r"[ :](?=\w+(?:<[^()]*>)?\()", name.replace("(anonymous namespace)::", ""), maxsplit=1)[-1].split("(")[0]
        found[key] = int(m.group(3)), int(m.group(1)), int(scratch)
    return found


def workgroups_per_cu(source, kernel, waves):
    """Of `waves` waves each: 512 registers a lane (in steps of 8) for the waves of a SIMD, 160 KiB of LDS."""
    regs, lds, scratch = kernels(source)[kernel]
    assert scratch == 0, kernel
    by_regs = 512 // (-(-regs // 8) * 8) * 4 // waves
    return min(by_regs, 163840 // lds if lds else 99, 32 // waves)
