"""The assembly lists' packed entries at the ends of their ranges: elements from 2^25
on (beyond a 32-bit element << 6 | corners), blocks and first contributions up to
2^32 - 1, with each flag and count.  The header of the tables is compiled for the
host alone.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include "tables.hpp"
#include <cstdio>
using namespace pufe;
int main() {
    const int64_t elems[] = {0, 1, (1LL << 25) - 1, 1LL << 25, (1LL << 31) - 1};
    for (int64_t e : elems)
        for (int c = 0; c < 64; ++c) {
            const int64_t k = contr_pack(e, c >> 3, c & 7);
            if (contr_elem(k) != e || contr_corners(k) != c) return 1;
        }
    const int64_t top = (1LL << 32) - 1, idx[] = {0, 1, (1LL << 31) - 1, 1LL << 31, top};
    for (int64_t b : idx)
        for (int n = 0; n <= 8; ++n)
            for (int p = 0; p < 2; ++p)
                for (int problem : {0, 7, kBlockProjected - 1}) {
                    int4 e = block_pack(b, top - b, b, n, p != 0);
                    e.w |= problem;
                    if (block_index(e) != b || block_mirror(e) != top - b || block_first(e) != b || block_count(e) != n ||
                        block_projected(e) != (p != 0) || (e.w & (kBlockProjected - 1)) != problem)
                        return 2;
                }
    std::puts("packed");
}
"""


def test_entries_survive_packing(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    include = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc))), "include")
    if not shutil.which("g++") or not os.path.exists(os.path.join(include, "hip")):
        pytest.skip("no host compiler or HIP headers")
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", include, "-I",
                           os.path.join(ROOT, "paper_1611_00731_amd", "csrc"), str(src), "-o", str(exe)])
    assert subprocess.check_output([str(exe)]).decode().strip() == "packed"
