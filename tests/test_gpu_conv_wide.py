"""The streaming convolution on 256 x 128, 192 and 256 tiles and their halves, and the kernels that keep the steps beside them, against the
oracle; a frame's bits do not depend on how many frames arrive with it."""
import pytest
import torch

import lvx_synth as S
from oracle import lvx_oracle as O
from test_gpu_conv import conv_inputs
from test_gpu_parity import DEV, assert_close

pytestmark = pytest.mark.gpu

# H, W, C_in, C_out, frames with the kernel of a step of all frames ("wide": 64-column groups per tile, whole tiles, halves); test_conv_wide_rules.py
# holds the rule to it
SHAPES = [((95, 115, 64, 72, 3), "rows 192x128"), ((212, 114, 64, 72, 2), "256x128"),
          ((224, 47, 64, 72, 3), (2, 0, 247)), ((191, 84, 64, 72, 3), (2, 188, 1)),
          ((187, 37, 64, 136, 3), (3, 0, 163)), ((149, 110, 64, 264, 1), "256x128"), ((110, 199, 64, 136, 3), (3, 256, 2)),
          ((158, 24, 64, 392, 3), (4, 0, 178)), ((145, 226, 64, 200, 1), (4, 128, 1)), ((84, 98, 128, 248, 3), (4, 0, 193))]


@pytest.mark.parametrize("H,W,Ci,Co,frames", [s for s, _ in SHAPES])
def test_conv_on_wide_tiles(lvx, H, W, Ci, Co, frames):
    act = (H + W) % 2
    x, w, b = conv_inputs("cw_%d_%d_%d_%d" % (H, W, Ci, Co), frames, H, W, Ci, Co, pad=8)
    ref = O.causal_conv3d(S.to_f64(x), S.to_f64(w).reshape(Co, 3, 3, 3, Ci), S.to_f64(b))
    conv = lvx.CausalConv(Ci, Co, H, W, frames, DEV)
    y = torch.full((frames + 1, H, W, Co), 7.0, dtype=torch.bfloat16, device=DEV)
    conv.step(x, w, b, act, y[:frames])
    torch.cuda.synchronize()
    assert_close(y[:frames], O.silu(ref) if act else ref, "conv %dx%d C %d->%d, %d frames" % (H, W, Ci, Co, frames))
    assert bool((y[frames] == 7.0).all())
    conv.reset()
    one = torch.empty_like(y[:frames])
    for t in range(frames):
        conv.step(x[t:t + 1], w, b, act, one[t:t + 1])
    torch.cuda.synchronize()
    assert torch.equal(one, y[:frames])
    conv.close()
