"""The rule that chooses tiles of 256 x 256, 192 or 128 (csrc/lvx_launch_rules.h), evaluated on the CPU."""
import ctypes as C
import random
import shutil
import subprocess

import pytest

import test_gpu_gemm_short as short_tests
import test_gpu_gemm_tiles as gemm_tests
import test_gpu_gemm_wide as wide_tests
import test_launch_rules as base

SOURCE = r"""
#include "lvx_launch_rules.h"
extern "C" void linear_choose(int M, int N, int n_slabs, int *tile, int *rows, int *fn, int *large, int *halves) {
    const lvx_gemm_launch_t l = lvx_gemm_choose(nullptr, M, N, n_slabs);
    *tile = l.tile, *rows = l.wide_rows, *fn = l.fn, *large = l.n_large;
    *halves = l.wide_rows > 0 ? (int)lvx_wide_halves(l.wide_rows, (N + 64 * l.fn - 1) / (64 * l.fn), l.n_large) : 0;
}
extern "C" int pair_rows(int M, int N1, int N2, int n_slabs, int *tile) {
    lvx_gemm_segs_t segs = {};
    segs.n = 2, segs.order = LVX_GEMM_ORDER_FIRST, segs.s[0].N = N1, segs.s[1].N = N2;
    const lvx_gemm_launch_t l = lvx_gemm_choose(&segs, M, N1, n_slabs);
    *tile = l.tile;
    return l.wide_rows;
}
extern "C" double wide_us(int M, int N, int fn, int n_large) { return lvx_wide_slab_us(M, (N + 64 * fn - 1) / (64 * fn), n_large, LVX_GEMM_WIDE_US[fn - 2]); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("wide_rules")
    (d / "rules.cpp").write_text(SOURCE)
    r = subprocess.run([cxx, "-O1", "-Wall", "-Werror", "-std=c++17", "-shared", "-fPIC", "-I" + base.CSRC, str(d / "rules.cpp"), "-o", str(d / "librules.so")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lib = C.CDLL(str(d / "librules.so"))
    lib.wide_us.restype = C.c_double
    return lib


def choose(rules, M, N, K, fp8=False):
    out = [C.c_int() for _ in range(5)]
    rules.linear_choose(M, N, K // (128 if fp8 else 64), *(C.byref(o) for o in out))
    return (base.SMALL[out[0].value],) + tuple(o.value for o in out[1:])


def test_gpu_shapes_take_the_tiles_they_name(rules):
    for (M, N, K), tiles in wide_tests.SHAPES + wide_tests.HALF_SHAPES:
        assert choose(rules, M, N, K)[1:] == tiles, (M, N, K)
    for (M, N, K), tiles in wide_tests.FP8_SHAPES:
        assert choose(rules, M, N, K, True)[1:] == tiles, (M, N, K)
    for (M, N, slabs), kernel in short_tests.SHAPES:
        assert choose(rules, M, N, 64 * slabs)[:2] == (kernel, 0) and choose(rules, M, N, 128 * slabs, True)[:2] == (kernel, 0), (M, N, slabs)
    # the shapes of the small tiles stay with them, those of the large ones and the rows that they split off all go to the wide kernel
    for (M, N, K), kernel in gemm_tests.SHAPES:
        assert choose(rules, M, N, K)[:2] == (("128x256", M) if kernel in ("128x256", "128x192") else (kernel, 0)), (M, N, K)
    for (M, N, K), kernel, m1 in gemm_tests.LARGE_SHAPES:
        assert choose(rules, M, N, K)[1] == M, (M, N, K)
    for (M, N, K), kernel, m1 in gemm_tests.FP8_LARGE_SHAPES:
        assert choose(rules, M, N, K, True)[1] == M, (M, N, K)
    # rows that go to a small tile in a second launch
    for shapes, fp8 in ((gemm_tests.SPLIT_SHAPES, False), (gemm_tests.FP8_SPLIT_SHAPES, True)):
        for (M, N, K), kernel, rows in shapes:
            assert 0 < rows < M and choose(rules, M, N, K, fp8)[:2] == (kernel, rows), (M, N, K)
    heads, fh, fw, ffn = gemm_tests.SPLIT_BLOCK
    assert 0 < choose(rules, fh * fw, ffn, 128 * heads, True)[1] < fh * fw
    for (M, N1, N2, K), kernel, rows in gemm_tests.SPLIT_PAIRS:
        tile = C.c_int()
        assert 0 < rows < M and rules.pair_rows(M, N1, N2, K // 64, C.byref(tile)) == rows and base.SMALL[tile.value] == kernel, (M, N1, N2, K)


def test_small_tiles_without_k_groups_stay(rules):
    """Two rounds of 64 x 64 tiles, two to a compute unit, are faster than one of 256 x 128 halves."""
    for M, N, K in ((2110, 936, 3904), (4335, 432, 1280), (1364, 1464, 1792), (6038, 304, 4352)):
        assert choose(rules, M, N, K)[:2] == ("64x64", 0), (M, N, K)


def test_tiles_cover_all_rows_and_whole_tiles_never_cost_more(rules):
    rng = random.Random(5)
    for _ in range(20000):
        M, N = int(60000 ** rng.random()) + 1, 8 * (int(2600 ** rng.random()) + 1)
        kernel, rows, fn, large, halves = choose(rules, M, N, 64 * rng.randint(1, 200))
        if rows == 0:
            continue
        cols, full = -(-N // (64 * fn)), rows // 256 + (rows % 256 > 128)
        assert fn in (2, 3, 4) and 0 <= large <= full * cols and (rows == M) == (kernel == "128x256")
        # 128-row halves: two for each tile that is not whole, one for the last rows that no 256-row tile covers
        assert halves == 2 * (full * cols - large) + (cols if rows > 256 * full else 0)
        assert rules.wide_us(rows, N, fn, large) <= rules.wide_us(rows, N, fn, 0) * (1 + 1e-12)


def test_measured_choices(rules):
    """Whole tiles where they were faster, halves, narrower or other tiles where those were."""
    for (M, N, K), tile in {(4680, 15360, 5120): (4680, 4, 1024), (4680, 13824, 5120): (4680, 4, 972), (4680, 5120, 13824): (4680, 4, 256),
                            (1560, 13824, 5120): (1560, 4, 256), (1886, 7680, 2560): (1886, 4, 210), (1170, 6144, 1536): (1170, 4, 0),
                            (1886, 2560, 2560): (1886, 3, 0), (1731, 5656, 2240): (1731, 3, 210), (1560, 5120, 5120): (1560, 3, 162),
                            (1560, 5120, 13824): (1560, 3, 162), (2449, 7064, 1152): (2449, 3, 256), (427, 6656, 2368): (427, 2, 0),
                            (3227, 2376, 2816): (3227, 3, 169), (1170, 1536, 6144): (0, 0, 0)}.items():
        assert choose(rules, M, N, K)[1:4] == tile, (M, N, K)
