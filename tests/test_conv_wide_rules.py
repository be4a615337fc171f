"""The rule that puts convolution steps on wide tiles (csrc/lvx_launch_rules.h), evaluated on the CPU."""
import ctypes as C
import random
import shutil
import subprocess

import pytest

import test_gpu_conv_wide as wide_tests
from test_launch_rules import CSRC, ROWS

SOURCE = r"""
#include "lvx_launch_rules.h"
extern "C" void choose(int W, int N, int n_slabs, int M, int max_m, int *out) {
    const lvx_conv_launch_t l = lvx_conv_choose(W, N, n_slabs, M, max_m);
    out[0] = l.plan.kind, out[1] = l.plan.tile, out[2] = l.fn, out[3] = l.n_large;
    out[4] = l.fn > 0 ? (int)lvx_wide_halves(M, (N + 64 * l.fn - 1) / (64 * l.fn), l.n_large) : 0;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("conv_rules")
    (d / "rules.cpp").write_text(SOURCE)
    r = subprocess.run([cxx, "-O1", "-Wall", "-Werror", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(d / "rules.cpp"), "-o", str(d / "librules.so")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return C.CDLL(str(d / "librules.so"))


def choose(rules, H, W, c_in, c_out, max_frames, n_frames):
    out = (C.c_int * 5)()
    rules.choose(W, c_out, 27 * c_in // 64, n_frames * H * W, max_frames * H * W, out)
    if out[2]:
        return tuple(out[2:])
    return ("256x128", ROWS.get(out[1]), "groups")[out[0]]


def test_gpu_shapes_take_the_kernels_they_name(rules):
    for s, kernel in wide_tests.SHAPES:
        assert choose(rules, *s, s[4]) == kernel, s


def test_measured_choices(rules):
    assert choose(rules, 100, 180, 384, 384, 4, 4)[:2] == (3, 512)
    assert choose(rules, 115, 172, 384, 200, 2, 2)[0] == 4
    # one round of 256 x 128 tiles that leaves compute units idle is faster than half as many tiles of 256 x 192
    assert choose(rules, 71, 59, 320, 384, 4, 4) == "256x128" and choose(rules, 94, 179, 384, 384, 3, 1) == "256x128"
    for s, kernel in {(50, 90, 384, 192, 1): "rows 64x64", (200, 360, 192, 96, 2): "rows 192x128", (240, 400, 64, 64, 4): "rows 256x64"}.items():
        assert choose(rules, *s, s[4]) == kernel, s


def test_a_layer_of_k_groups_keeps_them(rules):
    """They sum in another order than all other kernels: a layer takes them for every step or for none."""
    rng = random.Random(4)
    for _ in range(3000):
        s = (rng.randint(1, 90), rng.randint(1, 90), 64 * rng.randint(1, 6), 8 * rng.randint(1, 64), rng.randint(2, 8))
        assert len({choose(rules, *s, n) == "groups" for n in range(1, s[4] + 1)}) == 1, s
