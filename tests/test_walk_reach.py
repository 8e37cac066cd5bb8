"""The traceback's walk reads only what its fetch has filled: a host program over
the reach of every shape (lanes per pair, rows per lane) and every end cell in
the first rows and columns of a pair (no GPU)."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "walk_reach.hpp"
using namespace pastis;
int main() {
    long looked = 0;
    for (int W : {8, 16, 32})
        for (int RP = 1; RP <= 16; ++RP)
            for (int multi = 0; multi <= 1; ++multi) {
                const int slots = walk_slots(RP, multi != 0), cols = walk_cols(W), rows = slots * RP;
                for (int la = 1; la <= 3 * rows; ++la)
                    for (int i = 0; i < la; ++i)
                        for (int j0 : {0, 1, cols - 2, cols - 1, cols, 3 * cols}) {
                            if (j0 < 0) continue;
                            const int r0 = walk_first_row(i / RP, RP, slots);
                            std::vector<char> row(rows), col(cols);
                            for (int r = 0; r < rows; ++r) row[r] = walk_holds_row(r0, r, la);
                            for (int c = 0; c < cols; ++c) col[c] = j0 - c >= 0;
                            const int cend = cols < j0 + 1 ? cols : j0 + 1;
                            // every cell of the fetch a run of diagonal cells can begin at
                            for (int x = 0; x < (i - r0 + 1) * cend; ++x)
                                for (int lane = 0; lane < W; ++lane) {
                                    const int rr = x / cend - lane, cc = x % cend + lane;
                                    if (!walk_reads(r0, rr, cc, cend)) continue;
                                    ++looked;
                                    if (rr < 0 || rr >= rows || !row[rr] || cc >= cols || !col[cc]) {
                                        std::printf("W %d RP %d multi %d la %d i %d j0 %d: row %d column %d is not filled\n",
                                                    W, RP, multi, la, i, j0, r0 + rr, j0 - cc);
                                        return 1;
                                    }
                                }
                            for (int r = 0; r < rows; ++r)
                                if (row[r] && !walk_reads(r0, r, 0, cend)) return 2;
                        }
            }
    return looked > 0 ? 0 : 3;
}
"""


def test_walk_reads_only_filled_cells(tmp_path):
    src, exe = tmp_path / "reach.cpp", tmp_path / "reach"
    src.write_text(PROGRAM)
    inc = os.path.join(ROOT, "paper_2009_14467_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", inc, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
