"""Rows staged four elements to a load, compiled for the host with the shifts checked: every load stays inside the rows, every element of a row
comes to its column, and no shift is as wide as the word it shifts."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2305_02299_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "ragged_rows.h"
int main() {
    const int unit = 32;                                        // columns a tile is staged in, at most
    for (int d_in = 1; d_in <= 200; ++d_in)
        for (int rows : {1, 2, 7}) {
            const int total = rows * d_in;
            if (total < 4) continue;
            for (int r = 0; r < rows; ++r)
                for (int c = 0; c < (d_in + unit - 1) / unit * unit; c += 4) {
                    const unsigned e = (unsigned)(r * d_in + c);
                    const int shift = srigl::ragged_shift(e, total), start = (int)e - shift;
                    uint64_t four = 0;
                    for (int i = 0; i < 4; ++i) {
                        if (start + i < 0 || start + i >= total) { printf("%d columns, %d rows: element %d read\n", d_in, rows, start + i); return 1; }
                        four |= (uint64_t)(uint16_t)(start + i) << (16 * i);
                    }
                    four = srigl::move_halves(four, shift);
                    for (int i = 0; i < 4 && c + i < d_in; ++i)
                        if ((uint16_t)(four >> (16 * i)) != (uint16_t)(e + i)) { printf("%d columns: row %d, column %d\n", d_in, r, c + i); return 1; }
                }
        }
    printf("rows ok\n");
}
"""


def test_rows_that_end_inside_a_load(tmp_path):
    src = tmp_path / "rows.cpp"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=shift,signed-integer-overflow", "-fno-sanitize-recover=all", "-I", CSRC,
                    "-o", str(tmp_path / "rows"), str(src)], check=True)
    r = subprocess.run([str(tmp_path / "rows")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "rows ok" in r.stdout, (r.stdout + r.stderr)[-500:]
