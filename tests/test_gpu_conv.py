"""GPU parity of the streaming causal convolution with a two-frame feature cache (Appendix C) against the fp64 oracle,
through the C ABI: frame-by-frame and chunked streaming must both equal the oracle's whole-sequence convolution."""
import math

import numpy as np
import pytest
import torch

import lvx_synth as S
from oracle import lvx_oracle as O
from test_gpu_parity import DEV, assert_close

pytestmark = pytest.mark.gpu


def conv_inputs(tag, T, H, W, Ci, Co, pad=0):
    x = S.randn_bf16((T, H, W, Ci), S.seed_of(tag, "x"), 1.0, device=DEV)
    w = S.randn_bf16((Co, 27 * Ci + pad), S.seed_of(tag, "w"), 1.0 / math.sqrt(27 * Ci), device=DEV)[:, :27 * Ci]
    b = S.randn_f32((Co,), S.seed_of(tag, "b"), 0.5, device=DEV)
    return x, w, b


@pytest.mark.parametrize("H,W,Ci,Co,chunks,act", [
    (5, 7, 64, 8, [1, 1, 1, 1], 0),          # one frame per step: the overlapping cache shift
    (9, 6, 64, 72, [3, 3, 1, 2], 1),         # ragged column tile, SiLU
    (20, 33, 128, 136, [2, 4, 1], 1),        # 660 pixels per frame: several 256-row tiles with a ragged tail, two column tiles
    (4, 4, 192, 64, [4], 0),                 # whole sequence in one step
])
def test_streaming_conv_equals_whole_sequence_oracle(lvx, H, W, Ci, Co, chunks, act):
    T = sum(chunks)
    x, w, b = conv_inputs("conv_%d_%d_%d_%d" % (H, W, Ci, Co), T, H, W, Ci, Co, pad=64)
    ref = O.causal_conv3d(S.to_f64(x), S.to_f64(w).reshape(Co, 3, 3, 3, Ci), S.to_f64(b))
    if act:
        ref = O.silu(ref)
    conv = lvx.CausalConv(Ci, Co, H, W, max(chunks), DEV)
    y = torch.empty((T, H, W, Co), dtype=torch.bfloat16, device=DEV)
    t = 0
    for n in chunks:
        conv.step(x[t:t + n], w, b, act, y[t:t + n])
        t += n
    torch.cuda.synchronize()
    assert_close(y, ref, "causal conv %dx%d C %d->%d chunks %s" % (H, W, Ci, Co, chunks))
    # causality through the cache: the same frames again after a reset give the same result; without a reset they see the
    # previous sequence's last two frames as history, as the oracle's cache does
    y2 = torch.empty_like(y[:chunks[0]])
    conv.step(x[:chunks[0]], w, b, act, y2)
    torch.cuda.synchronize()
    model = O.CausalConvCache()
    model.frames = S.to_f64(x)[-2:]
    want = model.step(S.to_f64(x[:chunks[0]]), S.to_f64(w).reshape(Co, 3, 3, 3, Ci), S.to_f64(b))
    assert_close(y2, O.silu(want) if act else want, "continuing the stream with the cached two frames")
    conv.reset()
    conv.step(x[:chunks[0]], w, None, 0, y2)
    torch.cuda.synchronize()
    want0 = O.causal_conv3d(S.to_f64(x[:chunks[0]]), S.to_f64(w).reshape(Co, 3, 3, 3, Ci), None)
    assert_close(y2, want0, "after reset, no bias")
    too_long = torch.empty((max(chunks) + 1, H, W, Ci), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(lvx.LvxError) as e:
        conv.step(too_long, w, b, act, torch.empty((max(chunks) + 1, H, W, Co), dtype=torch.bfloat16, device=DEV))
    assert e.value.status == 2
    conv.close()


def test_linear_bias_and_silu_epilogues(lvx):
    M, N, K = 300, 200, 192
    a = S.randn_bf16((M, K), 71, 1.0, device=DEV)
    w = S.randn_bf16((N, K), 72, 1.0 / math.sqrt(K), device=DEV)
    b = S.randn_f32((N,), 73, 0.5, device=DEV)
    ref = O.linear(S.to_f64(a), S.to_f64(w)) + S.to_f64(b)
    c = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear(a, w, c, lvx.EPI_BIAS, gate=b)
    torch.cuda.synchronize()
    assert_close(c, ref, "linear + bias")
    lvx.lvx_linear(a, w, c, lvx.EPI_BIAS_SILU, gate=b)
    torch.cuda.synchronize()
    assert_close(c, O.silu(ref), "linear + bias + silu")


# H, W, C_in, C_out, frames with the kernel the rule picks for a step of all frames; test_launch_rules.py holds the rule to it
TILE_SHAPES = [
    ((7, 5, 64, 24, 3), "32x32 k4"),               # 27 slabs over four K groups
    ((45, 45, 64, 136, 2), "rows 64x64"),          # ragged rows and columns
    ((77, 79, 128, 136, 1), "rows 128x64"),
    ((100, 101, 64, 72, 2), "rows 256x64"),        # 128 x 64 for one frame
    ((150, 151, 64, 136, 1), "rows 192x128"),
    ((2, 2, 64, 600, 160), "rows 64x64"),          # rows of two pixels: tiles across many frames
    ((181, 181, 64, 256, 1), "256x128"),
]


# the same with the kernels of steps of one, two, ... frames: 256 x 128 tiles and tiles with shared rows in one layer
MIXED_SHAPES = [
    ((97, 125, 64, 136, 2), ("rows 256x64", "256x128")),
    ((82, 98, 64, 136, 3), ("rows 128x64", "rows 256x64", "256x128")),
    ((104, 77, 128, 136, 3), ("rows 128x64", "rows 256x64", "256x128")),
]


@pytest.mark.parametrize("H,W,Ci,Co,frames", [s for s, _ in TILE_SHAPES] + [s for s, _ in MIXED_SHAPES])
def test_conv_tiles_and_chunking(lvx, H, W, Ci, Co, frames):
    """Every tile the rule can pick, against the oracle; a frame's bits do not depend on how many frames arrive with it."""
    x, w, b = conv_inputs("ct_%d_%d_%d_%d" % (H, W, Ci, Co), frames, H, W, Ci, Co, pad=8)
    ref = O.causal_conv3d(S.to_f64(x), S.to_f64(w).reshape(Co, 3, 3, 3, Ci), S.to_f64(b))
    conv = lvx.CausalConv(Ci, Co, H, W, frames, DEV)
    y = torch.empty((frames, H, W, Co), dtype=torch.bfloat16, device=DEV)
    conv.step(x, w, b, 0, y)
    torch.cuda.synchronize()
    assert_close(y, ref, "conv %dx%d C %d->%d, %d frames" % (H, W, Ci, Co, frames))
    conv.reset()
    one = torch.empty_like(y)
    for t in range(frames):
        conv.step(x[t:t + 1], w, b, 0, one[t:t + 1])
    torch.cuda.synchronize()
    assert torch.equal(one, y)
    conv.close()


@pytest.mark.parametrize("steps", [(9, 1, 2, 9, 3, 8, 9), (5, 4, 1, 1, 7, 2, 6)])
def test_many_frames_of_few_pixels(lvx, steps):
    """Steps whose frames are shared out over workgroups, after steps of every length: the history is read from where another share's
    frames land."""
    H, W, C = 3, 5, 64
    n = sum(steps)
    x, w, b = conv_inputs("mf_%d" % steps[0], n, H, W, C, 16, pad=8)
    ref = O.causal_conv3d(S.to_f64(x), S.to_f64(w).reshape(16, 3, 3, 3, C), S.to_f64(b))
    conv = lvx.CausalConv(C, 16, H, W, 9, DEV)
    y = torch.empty((n, H, W, 16), dtype=torch.bfloat16, device=DEV)
    at = 0
    for k in steps:
        conv.step(x[at:at + k], w, b, 0, y[at:at + k])
        at += k
    torch.cuda.synchronize()
    assert_close(y, ref, "many frames, steps %s" % (steps,))
    conv.close()
