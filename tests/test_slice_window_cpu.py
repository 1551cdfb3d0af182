"""Every byte that a ring GEMM's copy of a slice can touch lies in the operand tile, whether the hardware adds the scalar
offset before its bounds check or (as the instruction is specified) behind it.  The rule is plain C++ and is compiled here."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_07203_amd", "csrc")

PROGRAM = r"""
#include "slice_window.h"
#include <cstdio>
int main() {
    const int slice = 128;
    for (int kt = 1; kt <= 9; ++kt)
        for (int tail = 0; tail <= 16; tail += 16)                    // pitch beyond the last slice
            for (int rows = 1; rows <= 40; rows += 13) {              // rows that exist of a tile of 64
                const long pitch = (long)kt * slice + tail, tile = rows * pitch;
                for (int s = 0; s < kt + 9; ++s) {                    // a ring runs up to 7 slices ahead
                    const po::SliceWindow w = po::slice_window(s, kt, (unsigned)tile, slice);
                    for (int row = 0; row < 64; ++row)
                        for (int seg = 0; seg < 8; ++seg) {
                            const long lane = row * pitch + seg * 16, end = lane + w.offset + 16;
                            const bool read = lane < (long)w.bytes;
                            if (read && (end > tile || s >= kt)) return std::printf("s %d of %d row %d: read ends at %ld of %ld\n", s, kt, row, end, tile), 1;
                            if (!read && s < kt && row < rows) return std::printf("s %d of %d row %d is not read\n", s, kt, row), 1;
                        }
                }
            }
    return 0;
}
"""


def test_copies_stay_inside_the_tile(tmp_path):
    src, exe = tmp_path / "window.cpp", tmp_path / "window"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout

