"""Index arithmetic of the passes of a connectivity update at the largest layers the call accepts (fewer than 2^32 elements), compiled for the
host: every worker ends, the workers together visit each element once, and places behind the last row are no rows."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2305_02299_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "scan_tail.h"
int main() {
    const uint32_t sizes[] = {1u, 7u, 4097u, 0xfffc0000u, 0xfffc0001u, 0xfffffffcu, 0xffffffffu};
    for (uint32_t n : sizes)
        for (uint32_t n4 : {0u, n / 4}) {
            const uint32_t workers = 256 * 1024;   // the launch's largest grid
            const uint64_t first = 4 * (uint64_t)n4, left = n - first;
            for (uint32_t w : {0u, 1u, 3u, 1024u, workers / 2, workers - 4, workers - 1}) {
                const uint64_t want = left > w ? (left - w + workers - 1) / workers : 0;
                uint64_t seen = 0, next = first + w;
                srigl::each_of_tail(n, n4, w, workers, [&](uint32_t i) {
                    if (i != next || i >= n || ++seen > want) { printf("n %u n4 %u worker %u: %u instead of %llu\n", n, n4, w, i, (unsigned long long)next); exit(1); }
                    next += workers;
                });
                if (seen != want) { printf("n %u n4 %u worker %u: %llu of %llu\n", n, n4, w, (unsigned long long)seen, (unsigned long long)want); exit(1); }
            }
        }
    // rows: every row of the layer has a place in the launch, and no place behind the last row is taken for one
    for (int32_t d_out : {1, 4, 31, 32, 33, 3072, 0x7fffffe0, 0x7fffffe1, 0x7ffffffd, 0x7fffffff})
        for (uint32_t each : {1u, 4u}) {
            const uint64_t places = (uint64_t)srigl::row_workgroups(d_out, each) * each;
            if (places < (uint64_t)d_out || places >= (uint64_t)d_out + 8 * each || places > 0xffffffffull || srigl::row_workgroups(d_out, each) % 8) {
                printf("%d rows, %u each: %llu places\n", d_out, each, (unsigned long long)places);
                return 1;
            }
            for (uint64_t r = (uint64_t)d_out > 40 ? d_out - 40 : 0; r < places; ++r)
                if (srigl::is_row((uint32_t)r, d_out) != (r < (uint64_t)d_out)) { printf("%d rows: row %llu\n", d_out, (unsigned long long)r); return 1; }
        }
    printf("bounds ok\n");
}
"""


def test_elements_taken_one_by_one(tmp_path):
    src = tmp_path / "bounds.cpp"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(tmp_path / "bounds"), str(src)], check=True)
    r = subprocess.run([str(tmp_path / "bounds")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "bounds ok" in r.stdout, r.stdout[-500:]
