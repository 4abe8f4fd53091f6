"""Order of the loads in the quantize-on-write kernels, from the assembly of a
compile of the shipped source: a wave issues the loads of its K row (4 at head
size 128, bf16) before it reads its page-table entry (the kernel's first 4-byte
load), so that the row's latency overlaps the lookup instead of following it."""
import os
import re
import subprocess

import pytest

from paper_2606_20474_amd import build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "quantize.txt")
    flags = [f for f in build.FLAGS if f != "-shared"]
    src = os.path.join(build.CSRC, "uq_quantize.hip")
    subprocess.run([build.HIPCC, *flags, "--cuda-device-only", "-S", src, "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


# 16-byte loads of a K row per lane: D = 32 NG channels over 4 lanes, or 256 over 16
@pytest.mark.parametrize("kernel,loads", [
    ("quantize_kv_kernelILi0ELi2E", 4), ("quantize_kv_kernelILi1ELi2E", 2), ("quantize_kv_kernelILi1ELi4E", 4),
    ("quantize_kv_kernelILi2ELi4E", 4), ("quantize_kv_kernelILi0ELi4E", 8), ("quantize_kv_d256_kernelILi0E", 4),
    ("quantize_kv_d256_kernelILi1E", 2)])
def test_k_row_is_loaded_before_the_page_table(assembly, kernel, loads):
    body = re.search(r"^_ZN2uq\d+%s\w*:.*?s_endpgm" % kernel, assembly, re.S | re.M).group(0)
    before = body[:re.search(r"global_load_dword ", body).start()]
    assert before.count("global_load_dwordx4") >= loads
