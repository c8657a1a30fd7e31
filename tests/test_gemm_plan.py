"""Host rules of the GEMM launches (csrc/gemm_plan.h), compiled here for the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_13304_amd", "csrc")


def run(tmp_path, body):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text('#include <cstdio>\n#include <climits>\n#include <vector>\n#include "gemm_plan.h"\nusing namespace dp;\n'
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


def test_every_tile_of_a_launch_is_one_block(tmp_path):
    """Including products with more blocks than a launch takes along x."""
    run(tmp_path, r"""
    const long long sizes[][2] = {{1, 1}, {1, 256}, {7, 3}, {8, 1}, {9, 4}, {1025, 2}, {1 << 23, 2}, {(1 << 23) + 1, 3}};
    for (auto& s : sizes) {
        const Groups gr((int)s[0], (int)s[1]);
        const Grid grid = gemm_grid(gr.blocks());
        if ((uint64_t)grid.x * 256 >= 1ull << 32 || grid.y > 65535 || (uint64_t)grid.x * grid.y < gr.blocks()) {
            printf("grid %u x %u\n", grid.x, grid.y);
            return 1;
        }
        std::vector<bool> seen(s[0] * s[1]);
        uint64_t n = 0;
        for (uint64_t b = 0; b < (uint64_t)grid.x * grid.y; ++b) {
            int g, m;
            if (!gr.get((unsigned)b, g, m)) continue;
            if (g < 0 || g >= s[0] || m < 0 || m >= s[1] || seen[g * s[1] + m]) {
                printf("%lld x %lld: block %llu\n", s[0], s[1], (unsigned long long)b);
                return 1;
            }
            seen[g * s[1] + m] = true;
            ++n;
        }
        if (n != (uint64_t)(s[0] * s[1])) { printf("%lld x %lld: %llu tiles\n", s[0], s[1], (unsigned long long)n); return 1; }
    }
    """)


def test_every_tile_of_a_product_is_one_block(tmp_path):
    """Row tiles from one to many, column tiles, split-K ranges; no XCD gets more than
    its share of the groups (about 5 %, or one group where there are few tiles)."""
    run(tmp_path, r"""
    for (int tm : {1, 2, 3, 7, 8, 9, 31, 129, 1000})
        for (int tn : {1, 2, 3, 5, 64, 625})
            for (int z : {1, 2, 3, 13, 104}) {
                if ((long long)tm * tn * z > 2000000) continue;
                const TileMap map(tm, tn, z);
                const Grid grid = gemm_grid(map.gr.blocks());
                std::vector<bool> seen((size_t)tm * tn * z);
                long long n = 0, xcd[8] = {};
                for (uint64_t b = 0; b < (uint64_t)grid.x * grid.y; ++b) {
                    int r, c, q;
                    if (!map.get((unsigned)b, r, c, q)) continue;
                    const long long at = ((long long)q * tm + r) * tn + c;
                    if (r < 0 || r >= tm || c < 0 || c >= tn || q < 0 || q >= z || seen[at]) {
                        printf("%d x %d x %d: block %llu\n", tm, tn, z, (unsigned long long)b);
                        return 1;
                    }
                    seen[at] = true;
                    ++n;
                    ++xcd[b & 7];
                }
                long long most = 0;
                for (long long x : xcd) most = x > most ? x : most;
                const double fair = (double)n / 8;
                if (n != (long long)tm * tn * z || most > 1.3 * fair + map.gr.size) {
                    printf("%d x %d x %d: %lld tiles, %lld on an XCD\n", tm, tn, z, n, most);
                    return 1;
                }
            }
    """)
