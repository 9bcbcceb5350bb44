"""The batched symmetric product loads from the matrix's lower triangle only:
its index rules (csrc/sym_rows.h) over every block and element of the orders
around one, two and three blocks, compiled for the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROG = r"""
#include <cstdio>
#include "sym_rows.h"
int main()
{
    for (int n = 1; n <= 98; ++n) {
        const int nb = (n + 31) / 32;
        auto get = [&](int r, int c) {  // a load
            if (r < c || r >= n || c < 0 || c >= n) { printf("n=%d loads (%d, %d)\n", n, r, c); return -1e9; }
            return 1000.0 * r + c + 1;
        };
        for (int J = 0; J < nb; ++J)
            for (int I = J; I < nb; ++I)
                for (int i = 32 * I; i < 32 * I + 32; i += 2)
                    for (int j = 32 * J; j < 32 * J + 32; ++j) {
                        const int c = j < n ? j : n - 1;
                        const bool end = J == nb - 1, trim = I == J || 32 * I + 32 > n;
                        const int r = sym_first(i, c, n, I == J);
                        const double v0 = end ? get(sym_row(i, c, n), c) : get(r, c);
                        const double v1 = end ? get(sym_row(i + 1, c, n), c) : get(r + 1, c);
                        const double x = trim ? sym_even(v0, v1, i, j, n, end) : v0;
                        const double y = trim ? sym_odd(v0, v1, i, j, n, I == J, end) : v1;
                        auto want = [&](int r) { return r >= n || j >= n || r < j ? 0.0 : (r == j ? 0.5 : 1.0) * (1000.0 * r + j + 1); };
                        if (x != want(i) || y != want(i + 1)) printf("n=%d (%d, %d): %g %g\n", n, i, j, x, y);
                    }
    }
}
"""


def test_only_the_lower_triangle_is_loaded(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROG)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1405_4644_amd", "csrc"), "-o", str(exe),
                    str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout
    assert out == "", out[:2000]
