"""Host test of the out-of-range byte offsets of the kernels' buffer loads: a
column outside its row stays outside every buffer whatever row it is moved to,
and the sums are defined (compiled with the undefined-behaviour sanitizer)."""

import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_07515_amd", "csrc")

PROGRAM = """
#include "offsets.h"
#include <cstdio>
#include <initializer_list>
using namespace fdkod;
int main() {
    for (int n : {2, 3, 63, 500, 4095, 4096})
        for (int es : {2, 4}) {
            const int rowb = n * es;
            const uint32_t plane = (uint32_t)n * (uint32_t)rowb;
            for (int row = -2; row <= n + 64; ++row)        // rows above and below the detector, a band's last tasks
                for (int col : {-n, -1, 0, n - 1, n, 2 * n}) {
                    const bool inside = (unsigned)col < (unsigned)n;
                    const uint32_t off = moved(column_offset(inside, col * es), row * rowb);
                    const uint32_t next = moved(column_offset(inside, col * es), row * rowb + rowb);
                    const bool hit = inside && row >= 0 && row < n, hit1 = inside && row + 1 >= 0 && row + 1 < n;
                    if ((off < plane) != hit || (next < plane) != hit1) {
                        std::printf("n %d row %d col %d\\n", n, row, col);
                        return 1;
                    }
                    if (hit && off != (uint32_t)(row * rowb + col * es)) return 2;
                }
            // mirrored footprints: up to 63 rows below an offset
            for (int q = 0; q < 64; ++q)
                if (moved(kOutside, -q * rowb) < plane) return 3;
        }
    return 0;
}
"""


def test_offsets_outside_stay_outside(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert out.returncode == 0, out.stdout
