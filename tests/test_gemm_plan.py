"""Host rules of the GEMM launches (csrc/gemm_plan.h), compiled here for the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_13304_amd", "csrc")


def run(tmp_path, body):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text('#include <cstdio>\n#include <climits>\n#include "gemm_plan.h"\nusing namespace dp;\n'
                   "int main()\n{\n" + body + "\nreturn 0;\n}\n")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_operands_with_32_bit_offsets_are_in_their_range(tmp_path):
    """The furthest element of a 128 x 64 tile (rows x k), either way round."""
    run(tmp_path, """
    long long lds[] = {8, 72, 1 << 20, (1 << 24) - 8, 1 << 24, (1 << 24) + 8, 34087040, 1 << 25, 1 << 28, INT_MAX - 7};
    for (long long ld : lds)
        for (int kc = 0; kc < 2; ++kc) {
            const Vec v = dense_vec(kc, 64, 64, (int)ld, 4096);
            const long long last = 127 * ld + 127;  // element
            const bool fits = last <= INT_MAX && 2 * last + 16 <= 0xFFFFFFFFll;
            if (v == kWhole && !fits) { printf("ld %lld: offsets wrap\\n", ld); return 1; }
            if (v != kWhole && ld <= 1 << 23) { printf("ld %lld: not vectorised\\n", ld); return 1; }
            if (v == kElems) { printf("ld %lld: element by element\\n", ld); return 1; }
        }
    """)


@pytest.mark.parametrize("kc,rows,k,ld,ptr,want", [
    (1, 5, 64, 64, 4096, "kWhole"), (1, 5, 60, 64, 4096, "kRagged"), (0, 64, 5, 64, 4096, "kWhole"),
    (0, 60, 5, 64, 4096, "kRagged"), (1, 64, 64, 65, 4096, "kElems"), (1, 64, 64, 64, 4098, "kElems")])
def test_operand_forms(tmp_path, kc, rows, k, ld, ptr, want):
    run(tmp_path, f"return dense_vec({kc}, {rows}, {k}, {ld}, {ptr}) != {want};")
