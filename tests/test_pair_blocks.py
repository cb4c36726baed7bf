"""CPU-only check of where the pair products read the caller's X: the geometry functions of the kernel's own
header, compiled for the host, over every tile, wavefront, block and lane of the three tile shapes."""
import ctypes
import os
import subprocess

import paper_2605_16184_amd.build as build

SOURCE = r"""
#include "root_products.h"
using namespace asteria;

// reads that reach beyond a dense n x n matrix, and elements of the lower triangle that no block brings
template <int WGM, int WGN, int MI, int NJ, int ST>
static long stray(int n, unsigned char *seen)
{
    using SH = PairShape<WGM, WGN, MI, NJ, ST>;
    long bad = 0;
    for (int i = 0; i < n * n; ++i) seen[i] = 0;
    for (int row0 = 0; row0 < n; row0 += SH::TM)
        for (int col0 = 0; col0 <= row0; col0 += SH::TN)
            for (int br = row0; br < row0 + SH::TM; br += 32)
                for (int bc = col0; bc < col0 + SH::TN; bc += 32) {
                    if (!pair_block_live(br, bc, n)) continue;
                    for (int lane = 0; lane < 64; ++lane)
                        for (int v = 0; v < 16; ++v) {
                            const int row = pair_elem_row(br, v, lane), col = pair_elem_col(bc, v, lane);
                            if (pair_x_whole(bc, n, true)) bad += col >= n;    // 4 columns in one load, the row kept inside the matrix
                            if (row < n && col <= row) seen[row * n + col] = 1;
                        }
                }
    for (int i = 0; i < n; ++i)
        for (int j = 0; j <= i; ++j) bad += !seen[i * n + j];
    return bad;
}

extern "C" long stray_reads(int shape, int n, unsigned char *seen)
{
    if (shape == 64) return stray<2, 2, 2, 2, 4>(n, seen);
    if (shape == 128) return stray<2, 2, 4, 4, 2>(n, seen);
    return stray<4, 2, 4, 8, 2>(n, seen);
}
"""


def test_products_read_inside_the_callers_matrix(tmp_path):
    src, lib = str(tmp_path / "pair_blocks.hip"), str(tmp_path / "pair_blocks.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-host-only", "-shared", "-I", build.CSRC, src, "-o", lib], check=True,
                   capture_output=True)
    stray_reads = ctypes.CDLL(lib).stray_reads
    stray_reads.restype = ctypes.c_long
    seen = (ctypes.c_ubyte * (600 * 600))()
    for shape in (64, 128, 256):
        for n in [*range(1, 300, 7), *range(44, 132), 200, 252, 260, 284, 508, 516, 520, 540, 600]:
            assert stray_reads(shape, n, seen) == 0, (shape, n)
