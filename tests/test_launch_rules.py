"""The rules that choose a kernel by size (csrc/lvx_launch_rules.h, plain C++), evaluated on the CPU: the GPU tests' shapes take
the kernels that those tests say they take."""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

import test_gpu_attention_split as attention_tests
import test_gpu_conv as conv_tests
import test_gpu_gemm_tiles as gemm_tests
import test_gpu_query_norm as query_norm_tests

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_04677_amd", "csrc")
SOURCE = r"""
#include "lvx_launch_rules.h"
extern "C" {
// widths[n]: the products of one launch (n = 1, order < 0: a plain linear); out: tile, rows of the first launch, time by the rule
void linear_plan(int M, int n, const int *widths, int order, int n_slabs, int narrow, int *tile, int *m1, double *us) {
    lvx_gemm_segs_t segs = {};
    segs.n = n;
    segs.order = order;
    for (int i = 0; i < n; ++i) segs.s[i].N = widths[i];
    const lvx_gemm_plan_t p = lvx_gemm_plan(order < 0 ? nullptr : &segs, M, widths[0], n_slabs, narrow != 0);
    *tile = p.tile, *m1 = p.m1, *us = p.us;
}
void conv_plan(int W, int N, int n_slabs, int M, int max_m, int *kind, int *tile) {
    const lvx_conv_plan_t p = lvx_conv_plan(W, N, n_slabs, M, max_m);
    *kind = p.kind, *tile = p.tile;
}
int sumsq_parts(int M, int N, int n_slabs) { return N / lvx_gemm_part_cols(lvx_gemm_pick_tile(nullptr, M, N, n_slabs)); }
int splits_keys(int n_q, int H, int n_keys, int head_dim) { return lvx_attention_splits_keys(n_q, H, n_keys, head_dim); }
}
"""
SMALL = {0: "64x128", 1: "64x64", 2: "32x64 k2", 3: "32x32 k4", -1: "128x256", -2: "128x192"}
ROWS = {0: "rows 64x64", 1: "rows 128x64", 2: "rows 256x64", 3: "rows 192x128"}


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    lib = str(d / "librules.so")
    r = subprocess.run([cxx, "-O1", "-Wall", "-Werror", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(d / "rules.cpp"), "-o", lib],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return C.CDLL(lib)


ORDER_ALONE, ORDER_FIRST, ORDER_LAUNCH, ORDER_ONE = -1, 0, 1, 2


def linear_plan(rules, M, widths, K, order=ORDER_ALONE, fp8=False, narrow=True):
    """(kernel of the product or of its last rows, rows of the 128 x 256 launch before it, microseconds by the rule)"""
    tile, m1, us = C.c_int(), C.c_int(), C.c_double()
    rules.linear_plan(M, len(widths), (C.c_int * len(widths))(*widths), order, K // (128 if fp8 else 64), int(narrow and not fp8), C.byref(tile), C.byref(m1), C.byref(us))
    return SMALL[tile.value], m1.value, us.value


def conv_plan(rules, H, W, c_in, c_out, max_frames, n_frames):
    kind, tile = C.c_int(), C.c_int()
    rules.conv_plan(W, c_out, 27 * c_in // 64, n_frames * H * W, max_frames * H * W, C.byref(kind), C.byref(tile))
    return ("256x128", ROWS.get(tile.value), SMALL[tile.value])[kind.value]


def test_gpu_gemm_shapes_take_the_kernels_they_name(rules):
    for (M, N, K), kernel in gemm_tests.SHAPES:
        assert linear_plan(rules, M, [N], K)[:2] == (kernel, 0), (M, N, K)
    for (M, N, K), kernel in gemm_tests.FP8_SHAPES:
        assert linear_plan(rules, M, [N], K, fp8=True)[:2] == (kernel, 0), (M, N, K)
    for (M, N, K), kernel, m1 in gemm_tests.LARGE_SHAPES:
        assert linear_plan(rules, M, [N], K)[:2] == (kernel, m1), (M, N, K)
    for (M, N, K), kernel, m1 in gemm_tests.FP8_LARGE_SHAPES:
        assert linear_plan(rules, M, [N], K, fp8=True)[:2] == (kernel, m1), (M, N, K)
    assert {k for _, k in gemm_tests.SHAPES} | {k for _, k, _ in gemm_tests.LARGE_SHAPES} == set(SMALL.values())


def test_gpu_conv_shapes_take_the_kernels_they_name(rules):
    for (H, W, c_in, c_out, frames), kernel in conv_tests.TILE_SHAPES:
        assert conv_plan(rules, H, W, c_in, c_out, frames, frames) == kernel, (H, W, c_in, c_out, frames)
    assert {k for _, k in conv_tests.TILE_SHAPES} == set(ROWS.values()) | {"256x128", "32x32 k4"}
    for (H, W, c_in, c_out, frames), kernels in conv_tests.MIXED_SHAPES:
        assert tuple(conv_plan(rules, H, W, c_in, c_out, frames, n) for n in range(1, frames + 1)) == kernels, (H, W, c_in, c_out, frames)


def test_conv_step_shorter_than_the_longest_takes_its_own_best_kernel(rules):
    """Layers of up to `max_frames` frames whose longest step suits the tiles with shared rows and whose shorter one does not."""
    for H, W, c_in, c_out, max_frames, n in [(109, 80, 448, 496, 4, 3), (42, 127, 448, 248, 8, 5), (84, 98, 384, 224, 4, 3), (21, 339, 64, 376, 4, 3)]:
        assert conv_plan(rules, H, W, c_in, c_out, max_frames, max_frames).startswith("rows")
        assert conv_plan(rules, H, W, c_in, c_out, max_frames, n) == "256x128"
    # K groups sum in another order: a layer takes them for every step or for none
    rng = random.Random(4)
    for _ in range(2000):
        s = (rng.randint(1, 60), rng.randint(1, 60), 64 * rng.randint(1, 4), 8 * rng.randint(1, 40), rng.randint(2, 8))
        assert len({conv_plan(rules, *s, n).startswith("32x32") for n in range(1, s[4] + 1)}) == 1, s


def test_gpu_query_norm_shapes_leave_the_partial_sums_they_name(rules):
    for (H, fh, fw, frames), parts in query_norm_tests.SHAPES:
        assert rules.sumsq_parts(fh * fw * frames, 128 * H, 2 * H) == parts, (H, fh, fw, frames)


def test_gpu_attention_shapes_take_the_forms_they_name(rules):
    for (D, H), split, unsplit, either in attention_tests.GEOMETRIES:
        for n_q in either:
            assert {rules.splits_keys(n_q, H, n_keys, D) for n_keys in attention_tests.KEY_COUNTS} == {0, 1}
        for n_keys in attention_tests.KEY_COUNTS:
            for n_q in split:
                assert rules.splits_keys(n_q, H, n_keys, D) or (n_q <= 128 and n_keys <= 7 * 64), (H, n_q, n_keys)
            for n_q in unsplit:
                assert not rules.splits_keys(n_q, H, n_keys, D), (H, n_q, n_keys)


def test_two_products_in_one_launch_never_cost_more_than_the_large_tiles(rules):
    """Whatever groups the first product would have alone, a wide second product is not pressed into its tiles."""
    rng = random.Random(3)

    def log(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))
    cases = [(1170, 256, 5120, 5120), (4680, 16, 13824, 5120), (256, 512, 5120, 5120), (48, 416, 9712, 384)]
    cases += [(log(1, 5000), 8 * log(1, 1900), 8 * log(1, 1900), 64 * log(1, 216)) for _ in range(5000)]
    kept = 0
    for M, N1, N2, K in cases:
        kernel, _, us = linear_plan(rules, M, [N1, N2], K, ORDER_FIRST)
        tiles = -(-M // 128) * (-(-N1 // 256) + -(-N2 // 256))
        assert us <= -(-tiles // 256) * (K // 64) * 0.8 * 1.0001, (M, N1, N2, K, kernel, us)
        kept += "k" in kernel
    assert kept > 100      # small pairs still run in groups


def test_gpu_product_pairs_tell_the_orders_apart(rules):
    """The pairs whose first product must not depend on its company: some would be summed in other groups if the launch decided."""
    differ = 0
    for M, N1, N2, K in gemm_tests.PAIRS:
        def groups(*a):
            return linear_plan(rules, *a)[0].partition(" ")[2]
        alone = groups(M, [N1], K)
        assert groups(M, [N1, N2], K, ORDER_FIRST) == alone, (M, N1, N2, K)
        differ += groups(M, [N1, N2], K, ORDER_LAUNCH) != alone
    assert differ >= 2
    for M, N1, N2, K in gemm_tests.UNEQUAL_PAIRS:
        assert linear_plan(rules, M, [N1], K)[0].endswith(("k2", "k4"))
        assert "k" not in linear_plan(rules, M, [N1, N2], K, ORDER_FIRST)[0]


def test_near_ties_and_many_rounds_stay_with_one_large_launch(rules):
    """Six rounds of 128 x 192 tiles for five of 128 x 256 (0.99 by the rule) ran slower, and so did rows split off after six or more
    whole rounds; three for three (0.825) and one or two whole rounds gain."""
    for M, N, K in [(5232, 6752, 4672), (2745, 12920, 2688), (3297, 10976, 5248), (5470, 6464, 9216), (3933, 8768, 2368),
                    (4163, 11984, 1472), (4549, 14528, 3648), (4958, 10064, 5760)]:
        assert linear_plan(rules, M, [N], K)[:2] == ("128x256", 0), (M, N, K)
    assert linear_plan(rules, 5812, [14152], 4480, fp8=True)[:2] == ("128x256", 0)
    assert linear_plan(rules, 1731, [5656], 2240)[0] == "128x192"
    assert linear_plan(rules, 1560, [5120], 13824)[:2] == ("64x64", 1536)
    assert linear_plan(rules, 3679, [4560], 7744)[:2] == ("64x64", 3584)


def test_attention_splits_keys_only_where_that_is_faster(rules):
    """(queries, heads, keys, head_dim) measured in both forms."""
    for c in [(2423, 32, 64, 128), (3473, 24, 59, 64), (3728, 18, 128, 128), (2712, 24, 192, 64), (3441, 20, 187, 64), (2127, 32, 256, 128),
              (4324, 18, 256, 128), (2991, 32, 384, 128), (2142, 32, 1851, 128), (4197, 16, 5755, 128), (4118, 24, 3072, 128),
              (1886, 20, 8487, 128), (4680, 40, 24960, 128)]:
        assert not rules.splits_keys(*c), c
    for c in [(291, 2, 64, 128), (394, 12, 320, 128), (2396, 26, 256, 128), (3281, 20, 704, 64), (1170, 12, 6240, 128), (4686, 16, 3480, 128),
              (2823, 22, 2136, 128), (3684, 18, 1920, 64), (3170, 40, 5376, 64), (3622, 18, 6976, 64)]:
        assert rules.splits_keys(*c), c
