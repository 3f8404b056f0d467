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
#include "krylov.h"
using namespace llg;
// The float64 and float32 grids up to kSpeculateMaxNodes nodes whose update
// pass has few enough blocks for its reduction to ride: how many, and how
// many of them run an x-forward pass that cannot carry it.
static int rides() {
  const int nhs[] = {2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256};
  const int ax[] = {1,  4,  6,  8,  10, 12, 16,  20,  24,  32,  40, 48,
                    64, 80, 96, 128, 160, 192, 256, 320, 384, 512};
  int some = 0, lost = 0;
  for (int eb : {4, 8}) for (int nh : nhs) for (int ny : ax) for (int nz : ax) {
    Ctx c;
    c.ny = ny, c.nz = nz, c.geom.nh = nh, c.ng = 2LL * nh * ny * nz;
    if (ny == 1 || c.ng > kSpeculateMaxNodes) continue;
    if (small_update_blocks(c.ng, x_pairs(eb, c)) > kRideMaxBlocks) continue;
    ++some;
    lost += !x_rides(nh, x_shape(eb, nh, (long long)ny * nz));
  }
  printf("%d %d\n", some, lost);
  return 0;
}
int main(int argc, char** argv) {
  if (argc == 1) return rides();
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
    """geometry(elem_bytes, (nx, ny, nz)) -> (shape, blocks, lines per block, partial rows);
    geometry() -> (grids with a riding reduction, those whose x-forward pass cannot carry it)"""
    d = tmp_path_factory.mktemp("geometry")
    src, exe = d / "geometry.hip", d / "geometry"
    src.write_text(PROGRAM)
    subprocess.run([B.hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-I", B.CSRC, "-I",
                    os.path.join(os.path.dirname(B.HERE), "include"), str(src), "-o", str(exe)],
                   check=True, capture_output=True)

    def ask(elem_bytes=None, grid=()):
        if elem_bytes is None:
            return [int(v) for v in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]
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


def test_every_riding_reduction_has_a_carrier(geometry):
    """x_rides leaves the branch out of wide passes only where no reduction rides."""
    some, lost = geometry()
    assert some > 5000 and lost == 0
    assert geometry(8, (4, 160, 128))[0] == geometry(8, (12, 192, 96))[0] == "wide"
