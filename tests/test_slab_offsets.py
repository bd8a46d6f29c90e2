"""Offsets of the TRSM into an X slab, at the row counts that outgrow 32 bits (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "device.hpp"
using namespace scasm;

int main() {
    int bad = 0;
    // every row that a plan accepts (below 2^27), the element index not negative (that means: no row)
    for (int k = 0; k < 27; ++k)
        for (long long row : {(1ll << k) - 1, 1ll << k, (1ll << k) + 1, (1ll << 27) - 1})
            for (int col : {0, 63}) {
                const long long at = row * kTile + col;
                if (slab_offset<double, true>((int)row, col) != at || slab_offset<float, true>((int)row, col) != at) {
                    std::printf("row %lld column %d\n", row, col);
                    ++bad;
                }
                // smaller slabs: bytes, unsigned
                if (at * 8 < kTrsmSlabBytes && (uint32_t)slab_offset<double, false>((int)row, col) != at * 8) ++bad;
                if (at * 4 < kTrsmSlabBytes && (uint32_t)slab_offset<float, false>((int)row, col) != at * 4) ++bad;
            }
    return bad != 0;
}
"""


def test_slab_offsets_span_every_row_count(tmp_path):
    """Slabs of 2^25 rows and more hold 2^31 elements and more: their element
    indices are 64 bits wide; those of smaller ones are unsigned byte offsets."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2509_21037_amd", "csrc"), str(src), "-o",
                           str(exe)])
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
