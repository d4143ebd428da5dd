"""Addresses of the epilogue of the 256 x 256 block kernel (host build of the kernel's own index functions)."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2201_05587_amd", "csrc")

# Every block of matrices whose last block row and column have 8 to 256 rows and columns: each vector of 8 residuals
# that a lane of a quadrant fetches lies inside the residual, whether the lane is inside the matrix or not.
SOURCE = r"""
#include <cstdio>
#include <initializer_list>
#include "tt_internal.h"
using namespace tt;
int main()
{
    long fetched = 0;
    for (int last_m : {1, 8, 100, 120, 127, 128, 129, 136, 255, 256})
        for (int last_n : {8, 120, 128, 136, 248, 256})
            for (int bm = 0; bm < 2; ++bm)
                for (int bn = 0; bn < 2; ++bn) {
                    const int M = 256 + last_m, N = 256 + last_n;
                    TileCoord block = {};
                    block.m0 = 256 * bm, block.n0 = 256 * bn;
                    for (int k = 0; k < 2; ++k)
                        for (int h = 0; h < 2; ++h) {
                            TileCoord q;
                            if (!block_quadrant(block, M, N, h, k, &q)) {
                                if (block.m0 + 128 * h < M && block.n0 + 128 * k < N) return printf("left out\n"), 1;
                                continue;
                            }
                            for (int row = 0; row < 128; ++row)
                                for (int col = 0; col < 128; col += 8) {
                                    const int m = q.m0 + row, first = q.n0 + col;
                                    const int64_t at = residual_element(q, M, N, m < M && first < N, m, first);
                                    ++fetched;
                                    if (at < 0 || at + 8 > (int64_t)M * N) {
                                        printf("%d x %d block %d %d quadrant %d %d row %d column %d: %lld\n", M, N, bm, bn, h, k,
                                               row, col, (long long)at);
                                        return 1;
                                    }
                                }
                        }
                }
    return fetched > 0 ? 0 : 1;
}
"""


def test_every_residual_a_block_fetches_lies_inside_the_residual(tmp_path):
    src, exe = tmp_path / "block_epilogue.cpp", tmp_path / "block_epilogue"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, "-I", os.path.join(CSRC, "..", "..", "include"), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, universal_newlines=True)
    assert r.returncode == 0, r.stdout
