"""The rule that chooses 256 x 256 tiles (csrc/lvx_launch_rules.h), evaluated on the CPU."""
import ctypes as C
import random
import shutil
import subprocess

import pytest

import test_gpu_gemm_tiles as gemm_tests
import test_gpu_gemm_wide as wide_tests
import test_launch_rules as base

SOURCE = r"""
#include "lvx_launch_rules.h"
extern "C" void linear_choose(int M, int N, int n_slabs, int narrow, int resid32, int *tile, int *rows, int *large, int *halves) {
    const lvx_gemm_launch_t l = lvx_gemm_choose(nullptr, M, N, n_slabs, narrow != 0, resid32 != 0);
    *tile = l.tile, *rows = l.wide_rows, *large = l.n_large;
    *halves = l.wide_rows > 0 ? (int)lvx_wide_halves(l.wide_rows, (N + 255) / 256, l.n_large) : 0;
}
extern "C" double wide_us(int M, int N, int n_large) { return lvx_wide_slab_us(M, (N + 255) / 256, n_large); }
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


def choose(rules, M, N, K, fp8=False, resid=False):
    out = [C.c_int() for _ in range(4)]
    rules.linear_choose(M, N, K // (128 if fp8 else 64), int(not fp8), int(resid), *(C.byref(o) for o in out))
    return base.SMALL[out[0].value], out[1].value, out[2].value, out[3].value


def test_gpu_shapes_take_the_tiles_they_name(rules):
    for resid in (False, True):
        for (M, N, K), tiles in wide_tests.SHAPES:
            assert choose(rules, M, N, K, resid=resid) == ("128x256", M) + tiles, (M, N, K)
        for (M, N, K), tiles in wide_tests.FP8_SHAPES:
            assert choose(rules, M, N, K, True, resid) == ("128x256", M) + tiles, (M, N, K)
        # the shapes of the other tiles stay with them
        for (M, N, K), kernel in gemm_tests.SHAPES:
            assert choose(rules, M, N, K, resid=resid)[0] == kernel, (M, N, K)
    # and so do the rows split off with their residual, but for one product that 120 whole tiles serve better
    for (M, N, K), kernel, m1 in gemm_tests.LARGE_SHAPES:
        assert choose(rules, M, N, K, resid=True)[:2] == ((kernel, m1) if (M, N, K) != (1550, 5112, 576) else ("128x256", M)), (M, N, K)
    for (M, N, K), kernel, m1 in gemm_tests.FP8_SPLIT_SHAPES:
        assert choose(rules, M, N, K, True, True)[:2] == (kernel, m1), (M, N, K)


def test_tiles_cover_all_rows_and_whole_tiles_never_cost_more(rules):
    rng = random.Random(5)
    for _ in range(20000):
        M, N = int(60000 ** rng.random()) + 1, 8 * (int(2600 ** rng.random()) + 1)
        kernel, rows, large, halves = choose(rules, M, N, 64 * rng.randint(1, 200), resid=rng.random() < 0.5)
        if rows == 0:
            continue
        cols, full = -(-N // 256), rows // 256 + (rows % 256 > 128)
        assert 0 <= large <= full * cols and (rows == M) == (kernel == "128x256")
        # 128-row halves: two for each tile that is not whole, one for the last rows that no 256-row tile covers
        assert halves == 2 * (full * cols - large) + (cols if rows > 256 * full else 0)
        assert rules.wide_us(rows, N, large) <= rules.wide_us(rows, N, 0) * (1 + 1e-12)


def test_measured_choices(rules):
    """Whole tiles where they were faster, halves or other tiles where those were."""
    for (M, N, K), (tile, large) in {(4680, 15360, 5120): ("128x256", 1024), (4680, 13824, 5120): ("128x256", 972), (4680, 5120, 13824): ("128x256", 256),
                                     (1560, 13824, 5120): ("128x256", 256), (1886, 7680, 2560): ("128x256", 210), (1170, 6144, 1536): ("128x256", 0),
                                     (1170, 4608, 1536): ("128x192", 0), (1886, 2560, 2560): ("128x192", 0), (1731, 5656, 2240): ("128x256", 161),
                                     (2150, 7656, 4224): ("128x256", 0), (3128, 10568, 5376): ("64x64", 504), (2449, 7064, 1152): ("128x256", 256)}.items():
        assert choose(rules, M, N, K)[::2] == (tile, large), (M, N, K)
    assert choose(rules, 1576, 5120, 6208, resid=True)[:2] == ("64x64", 1536) and choose(rules, 4469, 2296, 9664, resid=True)[:2] == ("128x256", 4469)
