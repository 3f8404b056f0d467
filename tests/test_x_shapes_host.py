"""Launch geometry of the x passes (csrc/pipeline.h, csrc/llg_internal.h),
from a host program compiled against those headers: the shapes and block
counts that the GPU tests' grids are chosen for."""

import os
import subprocess

import pytest

from paper_2607_15290_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "llg_internal.h"
using namespace llg;
int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4) {
    const int eb = atoi(argv[i]), nh = atoi(argv[i + 1]) / 2;
    const long long lines = atoll(argv[i + 2]) * atoll(argv[i + 3]);
    const int s = x_shape(eb, nh, lines);
    printf("%d %u %d %d\n", s, x_blocks(eb, nh, lines, s), x_lx(eb, nh, s), kRedBlocksMax);
  }
}
"""
NAMES = {0: "wide", 1: "mid", 2: "small"}


@pytest.fixture(scope="module")
def geometry(tmp_path_factory):
    """geometry(elem_bytes, (nx, ny, nz)) -> (shape, blocks, lines per block, partial rows)"""
    d = tmp_path_factory.mktemp("geometry")
    src, exe = d / "geometry.hip", d / "geometry"
    src.write_text(PROGRAM)
    subprocess.run([B.hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-I", B.CSRC, "-I",
                    os.path.join(os.path.dirname(B.HERE), "include"), str(src), "-o", str(exe)],
                   check=True, capture_output=True)

    def ask(elem_bytes, grid):
        out = subprocess.run([str(exe)] + [str(v) for v in (elem_bytes, *grid)], check=True, capture_output=True,
                             text=True).stdout.split()
        return NAMES[int(out[0])], int(out[1]), int(out[2]), int(out[3])

    return ask


def test_largest_grid_has_more_blocks_than_partial_rows(geometry):
    """512 x 384 x 384, the grid of the solve whose float64 products fall back to
    the separate pass: more x-inverse blocks than partial rows in float64, not
    in float32."""
    shape, blocks, lx, rows = geometry(8, (512, 384, 384))
    assert (shape, lx) == ("wide", 2) and blocks == 73728 > rows
    shape, blocks, lx, rows = geometry(4, (512, 384, 384))
    assert (shape, lx) == ("wide", 4) and blocks == 36864 <= rows


# grids of tests/test_gpu_products_bits.py: the shape that each is there for
GRIDS = {
    (8, "wide"): [(32, 160, 128), (64, 96, 48), (96, 64, 80), (128, 64, 64), (160, 96, 80), (256, 64, 48),
                  (512, 40, 16)],
    (4, "wide"): [(32, 160, 128), (64, 96, 48), (96, 64, 80), (128, 64, 64), (160, 96, 80), (256, 64, 48)],
    (8, "mid"): [(80, 40, 32), (96, 48, 48), (160, 32, 32), (128, 24, 32)],
    (4, "mid"): [(80, 40, 32), (96, 48, 48), (160, 32, 32), (128, 24, 32), (512, 40, 16)],
    (8, "small"): [(40, 10, 1)],
    (4, "small"): [(40, 10, 1)],
}


@pytest.mark.parametrize("elem_bytes, shape", GRIDS)
def test_grids_of_the_products_tests(geometry, elem_bytes, shape):
    for grid in GRIDS[elem_bytes, shape]:
        assert geometry(elem_bytes, grid)[0] == shape, grid


def test_edge_of_the_mid_shape(geometry):
    """Several lines per block; 192 blocks are the fewest."""
    for grid, blocks, lx in [((80, 40, 32), 214, 6), ((96, 48, 48), 461, 5), ((160, 32, 32), 342, 3),
                             ((128, 24, 32), 192, 4)]:
        assert geometry(8, grid)[:3] == ("mid", blocks, lx), grid
    assert geometry(8, (128, 24, 24))[0] == "small"
