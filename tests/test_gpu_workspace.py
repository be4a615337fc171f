"""The workspace as the calls use it: a block stays inside lvx_workspace_bytes, one of a longer chunk gives the same bits, and calls that never
split their attention over workgroups do not ask for the room of its ranges."""
import math

import pytest
import torch

import lvx_synth as S
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu

H, D, FH, FW, FRAMES, WINDOW = 4, 128, 15, 14, 3, 4     # 630 tokens, whose attention takes four ranges once the ring is full (test_gpu_attention_parts.py)
SINK, CHUNK, CTX = FH * FW, FH * FW * FRAMES, 24
RANGES = lambda n: (4 * n * H * (4 * D + 8) + 255) // 256 * 256


def setup(lvx, fp8):
    d = H * D
    layers = [S.block_weights(d, 256, l, "ws", std=1.0 / math.sqrt(d), device=DEV) for l in range(2)]
    rope = lvx.rope_desc(H, D, (44, 42, 42), 10000.0, FH, FW)
    cache = lvx.KVCache(lvx.cache_desc(2, H, D, FH, FW, FRAMES, WINDOW, 1), DEV)
    cache.attach_sink_source()
    return lvx.StageHandle(layers, rope, 256, fp8=fp8), rope, cache


def canaried(n_bytes):
    """n_bytes of workspace with 4 KB behind them that nobody may touch."""
    buf = torch.full((n_bytes + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    return buf, buf[:n_bytes]


@pytest.mark.parametrize("fp8", [False, True])
def test_rollout_in_a_workspace_of_its_own_size_and_of_a_longer_chunk(lvx, fp8):
    d = H * D
    outs = []
    for tokens in (CHUNK, CHUNK + 1, 20000):            # 20000 tokens of 4 heads take no ranges
        stage, rope, cache = setup(lvx, fp8)
        buf, ws = canaried(lvx.lvx_workspace_bytes(stage, tokens, CTX))
        ctx = S.randn_bf16((CTX, d), S.seed_of("ws_ctx"), device=DEV)
        lvx.lvx_sink_prefill(stage, cache, S.randn_bf16((SINK, d), S.seed_of("ws_sink"), device=DEV), ctx, None, 4, ws)
        for i in range(WINDOW + 2):
            x = S.randn_bf16((CHUNK, d), S.seed_of("ws_x", i), device=DEV)
            lvx.lvx_sink_rope_update(cache, rope, -1, 4 + FRAMES * i)
            lvx.lvx_denoise_stage(stage, cache, x, ctx, None, -0.25, i, 1 + FRAMES * i, ws)
        torch.cuda.synchronize()
        assert bool((buf[-4096:] == 0xA5).all()) and bool(torch.isfinite(x.float()).all())
        outs.append(x)
        with pytest.raises(lvx.LvxError):
            lvx.lvx_denoise_stage(stage, cache, x, ctx, None, -0.25, WINDOW + 2, 1, buf[:lvx.lvx_workspace_bytes(stage, CHUNK, CTX) - 256])
        cache.close()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("fp8", [False, True])
def test_prefill_and_context_ask_for_no_ranges(lvx, fp8):
    d = H * D
    stage, _, cache = setup(lvx, fp8)
    ctx = S.randn_bf16((CTX, d), S.seed_of("ws_ctx"), device=DEV)
    sink = S.randn_bf16((SINK, d), S.seed_of("ws_sink"), device=DEV)
    full = lvx.lvx_workspace_bytes(stage, SINK, CTX)
    out = [torch.empty_like(sink) for _ in range(2)]
    for y, n_bytes in zip(out, (full, full - RANGES(SINK))):
        buf, ws = canaried(n_bytes)
        lvx.lvx_sink_prefill(stage, cache, sink, ctx, None, 4, ws, y)
        torch.cuda.synchronize()
        assert bool((buf[-4096:] == 0xA5).all())
    assert torch.equal(out[0], out[1]) and bool(torch.isfinite(out[0].float()).all())
    with pytest.raises(lvx.LvxError):
        lvx.lvx_sink_prefill(stage, cache, sink, ctx, None, 4, buf[:full - RANGES(SINK) - 256], out[1])
    if not fp8:
        k, v = (torch.empty((2, CTX, d), dtype=torch.bfloat16, device=DEV) for _ in range(2))
        lvx.lvx_context_kv(stage, 0, 2, ctx, k, v, canaried(lvx.lvx_workspace_bytes(stage, 1, CTX) - RANGES(1))[1])
        torch.cuda.synchronize()
        assert bool(torch.isfinite(k.float()).all())
    cache.close()
