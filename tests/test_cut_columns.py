"""Which floats the fused kernel loads of a tile that component edges cut: none but the tile's.  The kernel's own arithmetic
(csrc/gbmuf_cut.h), compiled for the host and run over every tile of small components."""
import os
import subprocess

from paper_1909_09010_amd import build

PROGRAM = r"""
#include "gbmuf_cut.h"
#include <initializer_list>
#include <stdio.h>
using namespace gbmuf;

// Tile g of T columns, as far as the component [a, b) has it; blocks of 2^logB floats.  0 if all is well.
static int look(int64_t a, int64_t b, int64_t T, int64_t g, int logB, bool whole_blocks)
{
    const int64_t lo = g * T * 4 > a ? g * T * 4 : a, hi = (g + 1) * T * 4 < b ? (g + 1) * T * 4 : b;
    if (lo >= hi) return 0;
    const int n = static_cast<int>(hi - lo);
    if (is_thin(lo, n, logB)) return whole_blocks && n >= 4 ? 1 : 0;            // only for what it is there for
    if ((lo >> logB) != ((lo + 3) >> logB) || lo + 4 > hi) return 2;            // what threads without a row load
    int64_t owned = 0;
    for (int64_t e = lo & ~static_cast<int64_t>(3); e < (g + 1) * T * 4; e += 4) {
        const CutColumn c = cut_column(e, lo, n);
        for (int i = 0; i < 4; ++i) {
            const bool mine = e + i >= lo && e + i < hi;
            if (((c.mine >> i) & 1) != mine) return 3;
            if (mine && (i < c.from || i >= c.from + 4)) return 4;              // not among what was loaded
            if (c.mine && (e + c.from + i < lo || e + c.from + i >= hi)) return 5;      // beside the tile
            if (c.mine && ((e + c.from + i) >> logB) != (e >> logB)) return 6;  // in another block
            owned += mine;
        }
    }
    return owned == n ? 0 : 7;
}

int main()
{
    long tiles = 0;
    for (int64_t T = 2; T <= 32; T *= 4)
        for (int logB : {62, 3, 5, 7, 10})
            for (int64_t a = 0; a < 4 * T + 9; ++a)
                for (int64_t b = a + 1; b < a + 8 * T + 10; ++b)
                    for (int64_t g = 0; g * T * 4 < b; ++g, ++tiles)
                        if (const int bad = look(a, b, T, g, logB, (int64_t{1} << logB) >= 4 * T)) {
                            printf("%d: [%ld, %ld), T %ld, tile %ld, blocks of 2^%d\n", bad, a, b, T, g, logB);
                            return 1;
                        }
    printf("%ld\n", tiles);
    return 0;
}
"""


def test_a_cut_tile_loads_no_float_beside_it(tmp_path):
    src, exe = tmp_path / "cut.cpp", tmp_path / "cut"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-I", build.CSRC, "-o", str(exe), str(src)], check=True)
    got = subprocess.run([str(exe)], capture_output=True, text=True)
    assert got.returncode == 0, got.stdout
    assert int(got.stdout) > 100_000
