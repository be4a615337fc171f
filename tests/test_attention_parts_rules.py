"""The rule that splits a block's keys over workgroups (csrc/lvx_launch_rules.h), evaluated on the CPU."""
import ctypes as C
import random
import shutil
import subprocess

import pytest

import test_gpu_attention_parts as parts_tests
from test_launch_rules import CSRC

SOURCE = r"""
#include "lvx_launch_rules.h"
extern "C" int parts(int n_q, int H, int n_keys, int D) { const lvx_attn_split_t s = lvx_attention_parts(n_q, H, n_keys, D); return 2 * s.parts + s.halves; }
extern "C" int few(int n_q, int H, int n_keys, int D) { return lvx_attention_few(n_q, H, n_keys, D); }
extern "C" double few_lds(int n_keys, int D) { return (double)lvx_attention_few_lds(lvx_attention_few_waves(n_keys), D); }
extern "C" double scratch(int n_q, int H, int D) { return (double)lvx_attention_scratch_bytes(n_q, H, D); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("parts_rules")
    (d / "rules.cpp").write_text(SOURCE)
    r = subprocess.run([cxx, "-O1", "-Wall", "-Werror", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(d / "rules.cpp"), "-o", str(d / "librules.so")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lib = C.CDLL(str(d / "librules.so"))
    lib.scratch.restype = lib.few_lds.restype = C.c_double
    return lib


def split(rules, n_q, H, n_keys, D):
    r = rules.parts(n_q, H, n_keys, D)
    return r // 2, bool(r % 2)


def test_gpu_shapes_take_the_ranges_they_name(rules):
    for (D, H, fh, fw, frames, window), form in parts_tests.SHAPES:
        n = fh * fw * frames
        assert split(rules, n, H, fh * fw + (window + 1) * n, D) == form, (D, H, n)
        assert not rules.few(n, H, fh * fw + (window + 1) * n, D), (D, H, n)
    for D, H, fh, fw, frames, window in parts_tests.FEW_SHAPES:
        assert rules.few(fh * fw * frames, H, fh * fw + (window + 1) * fh * fw * frames, D), (D, H)
    for H, D, frame, frames, window, few in parts_tests.LARGE_SCORES:
        assert rules.few(frame * frames, H, frame + (window + 1) * frame * frames, D) == few, (H, D, frame)


def test_where_waves_take_key_tiles_of_their_own(rules):
    """Where that was measured to be faster, and its LDS never more than 128 KB, nor more than a compute unit's for those that share it."""
    for c, few in {(105, 4, 280, 128): 1, (105, 4, 40, 128): 1, (390, 4, 1300, 128): 1, (48, 2, 168, 64): 1, (256, 16, 3072, 128): 1, (250, 16, 6144, 64): 1,
                   (48, 2, 24, 64): 0, (129, 2, 24, 64): 1, (257, 16, 400, 128): 0, (256, 16, 3073, 128): 0, (1024, 16, 64, 128): 1, (1025, 16, 64, 128): 0,
                   (512, 16, 128, 128): 1, (513, 16, 128, 128): 0, (1170, 12, 257, 128): 0, (1170, 12, 6240, 128): 0, (4680, 40, 24960, 128): 0}.items():
        assert rules.few(*c) == few, c
    rng = random.Random(3)
    for _ in range(20000):
        n_q, H, n_keys, D = int(8000 ** rng.random()) + 1, rng.randint(1, 48), int(60000 ** rng.random()) + 1, rng.choice([64, 128])
        lds = rules.few_lds(n_keys, D)
        assert lds <= 128 * 1024
        if rules.few(n_q, H, n_keys, D):
            assert -(-(-(-n_q // 16) * H) // 256) * (lds + 1024) <= 160 * 1024


def test_measured_choices(rules):
    for c, form in {(1170, 12, 6240, 128): (2, True), (1200, 16, 5400, 128): (3, False), (390, 4, 1300, 128): (4, True), (900, 8, 4800, 64): (4, True)}.items():
        assert split(rules, *c) == form, c
    for c in [(105, 4, 560, 128), (48, 2, 168, 64), (1800, 30, 6000, 128), (4680, 40, 24960, 128), (1000, 40, 4000, 128)]:
        assert split(rules, *c)[0] == 1, c


def test_no_range_is_empty_and_the_scratch_holds_all(rules):
    rng = random.Random(8)
    for _ in range(20000):
        n_q, H, n_keys, D = int(8000 ** rng.random()) + 1, rng.randint(1, 48), int(60000 ** rng.random()) + 1, rng.choice([64, 128])
        parts, _ = split(rules, n_q, H, n_keys, D)
        assert 1 <= parts <= -(-n_keys // 64)
        assert parts == 1 or rules.scratch(n_q, H, D) >= parts * n_q * H * (4 * D + 8)


def test_scratch_is_reserved_only_for_rows_that_may_take_ranges(rules):
    """None where no key count splits; up to the longest such chunk all four ranges."""
    for n_q, H in [(1536, 40), (2560, 24), (3072, 20), (1500, 40), (2048, 32), (4680, 40), (1537, 32), (129, 257), (49153, 1)]:
        assert rules.scratch(n_q, H, 128) == 0
        assert all(split(rules, n_q, H, 64 * t, D)[0] == 1 for t in range(1, 600) for D in (64, 128)), (n_q, H)
    for n_q, H in [(1152, 40), (1536, 32), (4096, 12), (1170, 12), (256, 256), (49152, 1)]:
        assert rules.scratch(n_q, H, 128) == 4.0 * n_q * H * (4 * 128 + 8)
