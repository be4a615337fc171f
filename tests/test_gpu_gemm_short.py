"""Small tiles whose K is shorter than their ring of stages, or just longer, so that fewer slabs are requested than there are stages and, with K
groups, one group has a slab less than another: all epilogues against the fp64 oracle."""
import pytest

import test_gpu_gemm_wide as wide_tests

pytestmark = pytest.mark.gpu

# M, N and K in slabs of 128 bytes a row, with the tile; test_wide_rules.py holds the rule to it
SHAPES = [((31, 24, 2), "32x64 k2"), ((33, 136, 4), "32x32 k4"), ((33, 136, 5), "32x32 k4"), ((64, 2560, 3), "32x32 k4"), ((65, 1920, 17), "32x32 k4"),
          ((64, 5760, 2), "32x64 k2"), ((64, 5760, 11), "32x64 k2"), ((31, 24, 1), "64x64"), ((250, 2568, 4), "64x64"), ((250, 2568, 3), "64x64"),
          ((600, 2560, 1), "64x128"), ((577, 2696, 5), "64x128"), ((577, 2696, 6), "64x128")]


@pytest.mark.parametrize("M,N,slabs", [s for s, _ in SHAPES])
def test_linear_with_few_slabs(lvx, M, N, slabs):
    wide_tests.test_linear_on_wide_tiles(lvx, M, N, 64 * slabs, 3)
    wide_tests.test_linear_fp8_on_wide_tiles(lvx, M, N, 128 * slabs)
