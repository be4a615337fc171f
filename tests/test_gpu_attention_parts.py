"""Self-attention of a block with its keys split over workgroups, against fp64 attention over the keys and values that the cache holds: every
form the rule takes, ragged last tiles, ranges whose first tile, or all of whose tiles, hold no finite score for any query.

The block is arranged so that its output minus its input IS the attention's bf16 output: W_o is the identity, the cross-attention and
the feed-forward add zero."""
import math

import numpy as np
import pytest
import torch

import lvx_synth as S
from oracle import lvx_oracle as O
from test_gpu_fp8 import assert_fp8_close, fp8_stage_setup
from test_gpu_parity import DEV, assert_close

pytestmark = pytest.mark.gpu

# head_dim, heads, frame_h, frame_w, chunk_frames, window with the ranges and the form (ranges over workgroups), and those that workgroups of 16
# queries with a range of keys a wave take instead; test_attention_parts_rules.py holds the rules to it
SHAPES = [((128, 4, 15, 14, 3, 4), (4, True)),      # 52.5 tiles: ranges of 13 or 14, one of them the ragged last
          ((128, 8, 4, 107, 3, 2), (4, False)), ((128, 10, 19, 27, 3, 1), (3, False)),
          ((64, 4, 20, 21, 3, 4), (4, True)), ((64, 8, 4, 107, 3, 2), (4, False))]
FEW_SHAPES = [(128, 2, 10, 14, 1, 4), (128, 8, 5, 89, 1, 1), (64, 2, 10, 19, 1, 4)]     # 13.1, 20.9 and 17.8 tiles over eight waves


def axes(D):
    y = D // 6 * 2
    return (D - 2 * y, y, y)


@pytest.mark.parametrize("dead", [False, True])
@pytest.mark.parametrize("shape", [s for s, _ in SHAPES] + FEW_SHAPES)
def test_attention_over_ranges_of_keys(lvx, shape, dead):
    D, H, fh, fw, frames, window = shape
    parts = dict(SHAPES)[shape][0] if shape in dict(SHAPES) else 4
    d, fk, n = H * D, fh * fw, fh * fw * frames
    n_keys = fk + (window + 1) * n
    tag = "ap_%d_%d_%d" % (D, n, int(dead))
    w = S.block_weights(d, 128, 0, tag, std=1.0 / math.sqrt(d), device=DEV)
    w["W_o"] = torch.eye(d, dtype=torch.bfloat16, device=DEV)
    w["Wc_o"], w["W_2"] = torch.zeros_like(w["Wc_o"]), torch.zeros_like(w["W_2"])
    w["W_qkv"] = w["W_qkv"].clone()
    for g in ("g_q", "g_k", "gc_q", "gc_k"):
        w[g] = torch.ones(d, device=DEV)
    mod6 = torch.zeros((6, d), device=DEV)
    mod6[2] = 1.0
    # one channel of every head (the slowest pair of the temporal axis, which hardly rotates) decides a dead key's fate: with a modulation
    # that makes all rows of u one vector, every query is large and positive there, and a key of -3.3e38 gives a score of -inf
    ch = axes(D)[0] - 2
    if dead:
        shift = S.randn_f32((d,), S.seed_of(tag, "shift"), device=DEV).to(torch.bfloat16).float()
        mod6[0], mod6[1] = shift, -1.0
        w["W_qkv"][ch:d:D] = (shift * (12.0 / math.sqrt(d))).to(torch.bfloat16)
    rope = lvx.rope_desc(H, D, axes(D), 10000.0, fh, fw)
    stage = lvx.StageHandle([w], rope, 128)
    cache = lvx.KVCache(lvx.cache_desc(1, H, D, fh, fw, frames, window, 1), DEV)
    past = n_keys - n
    k = S.randn_bf16((past, d), S.seed_of(tag, "k"), 2.0, device=DEV)
    v = S.randn_bf16((past, d), S.seed_of(tag, "v"), device=DEV)
    tiles = -(-n_keys // 64)
    if dead:
        k[:, ch::D] = 0.0
        first = [p * tiles // parts for p in range(parts + 1)]
        gone = {first[0], first[1]} | set(range(first[parts // 2], first[parts // 2 + 1])) | {first[1] + 2}
        for t in gone:
            k[64 * t:64 * t + 64, ch::D] = -3.3e38
    lvx.lvx_kvcache_set_sink(cache, 0, k[:fk], v[:fk])
    for i in range(window):
        lvx.lvx_chunk_append_evict(cache, 0, k[fk + i * n:fk + (i + 1) * n].contiguous(), v[fk + i * n:fk + (i + 1) * n].contiguous(), i)
    x = S.randn_f32((n, d), S.seed_of(tag, "x"), device=DEV)
    ctx = S.randn_bf16((24, d), S.seed_of(tag, "ctx"), device=DEV)
    ws = torch.full((lvx.lvx_workspace_bytes(stage, n, 24),), 255, dtype=torch.uint8, device=DEV)
    y = x.clone()
    t0 = 1 + frames * window
    lvx.lvx_dit_block_f32(stage, 0, cache, y, ctx, mod6, window, t0, ws)
    K, V = torch.empty((n_keys, d), dtype=torch.bfloat16, device=DEV), torch.empty((n_keys, d), dtype=torch.bfloat16, device=DEV)
    lvx.lvx_kvcache_gather(cache, 0, 0, n_keys, K, V)
    torch.cuda.synchronize()
    x64 = S.to_f64(x)
    u = S.to_f64(torch.from_numpy(O.modulate(x64, S.to_f64(mod6[0]), S.to_f64(mod6[1]))).to(torch.bfloat16))
    q = O.rope3d(O.rmsnorm(O.linear(u, S.to_f64(w["W_qkv"][:d])), np.ones(d)).reshape(n, H, D), t0, fh, fw, axes(D))
    got = (S.to_f64(y) - x64).reshape(n, H, D)
    assert np.isfinite(got).all()
    rows = np.unique(np.linspace(0, n - 1, 150).astype(int))
    for h in sorted({0, H // 2, H - 1}):
        c = slice(h * D, (h + 1) * D)
        want = O.attention(q[rows][:, h:h + 1], S.to_f64(K[:n_keys, c])[:, None], S.to_f64(V[:n_keys, c])[:, None], 1.0 / math.sqrt(D))
        assert_close(torch.from_numpy(got[rows, h]), want[:, 0], "%s head %d" % (tag, h))
    cache.close()


@pytest.mark.parametrize("heads,frame,chunk_frames", [(2, (10, 14), 1), (4, (15, 14), 3)])
def test_fp8_block_whose_attention_is_split(lvx, monkeypatch, heads, frame, chunk_frames):
    """The amax of the combined output, not of a range, scales the next linear's codes (outliers in the context and the input as in the
    other FP8 block test)."""
    monkeypatch.setitem(S.PRESETS, "parts", dict(n_heads=heads, head_dim=128, frame_h=frame[0], frame_w=frame[1], chunk_frames=chunk_frames, window=4, sink_frames=1,
                                                 rope_axes=(44, 42, 42), ffn=256, n_ctx=24))
    p, stage, cache, cfg, models, ws, w64, d, n, cfgx, modelsx = fp8_stage_setup(lvx, "parts", 1, "parts8")
    for i in range(p["window"] + (2 if heads == 2 else 0)):
        x = S.randn_bf16((n, d), S.seed_of("parts8_x", i), device=DEV)
        ctx = S.randn_bf16((p["n_ctx"], d), S.seed_of("parts8_ctx", i), device=DEV)
        mod6 = S.randn_f32((6, d), S.seed_of("parts8_mod", i), 0.2, device=DEV)
        mod6[2] += 2.0
        mod6[5] += 1.0
        ref = O.dit_block(S.to_f64(x), w64[0], models[0], S.to_f64(ctx), S.to_f64(mod6), i, 1 + i, cfg)
        exact = O.dit_block(S.to_f64(x), w64[0], modelsx[0], S.to_f64(ctx), S.to_f64(mod6), i, 1 + i, cfgx)
        lvx.lvx_dit_block(stage, 0, cache, x, ctx, mod6, i, 1 + i, ws)
        torch.cuda.synchronize()
        assert_fp8_close(x, ref, exact, "fp8 block step %d" % i)
    cache.close()


# heads, head_dim, tokens a frame, frames a chunk, window: waves with tiles of their own (one and several tiles a wave, K and V^T apart and in one place), and
# the kernel of the longer calls
LARGE_SCORES = [(4, 128, 35, 3, 4, 1), (4, 128, 130, 3, 2, 1), (2, 128, 24, 1, 2, 1), (2, 64, 24, 2, 2, 1), (4, 64, 190, 1, 4, 1), (12, 128, 390, 3, 2, 0)]


@pytest.mark.parametrize("H,D,frame,frames,window,few", LARGE_SCORES)
def test_scores_far_from_zero_keep_their_differences(lvx, H, D, frame, frames, window, few):
    """Scores of 2^22 and a small whole number each, exact in fp32, so that the scaled score, as a number of its own, is 1/8 apart from the next one
    (a rounding there is 2.5 % of a weight, root mean square) while its difference from the reference is not."""
    d, n = H * D, frame * frames
    n_keys = frame + (window + 1) * n
    g = torch.Generator().manual_seed(H * D + n)
    k = torch.zeros((n_keys, H, D))
    k[:, :, 0], k[:, :, 1:17] = 2048.0, torch.randint(-3, 4, (n_keys, H, 16), generator=g).float()
    q = torch.zeros((n, H, D))
    q[:, :, 0], q[:, :, 1:17] = 2048.0, torch.randint(-2, 3, (n, H, 16), generator=g).float()
    k, q = (t.reshape(-1, d).to(torch.bfloat16).to(DEV) for t in (k, q))
    v = S.randn_bf16((n_keys, d), S.seed_of("large_v", n, d), device=DEV)
    cache = lvx.KVCache(lvx.cache_desc(1, H, D, frame, 1, frames, window, 1), DEV)
    lvx.lvx_kvcache_set_sink(cache, 0, k[:frame], v[:frame])
    for i in range(window + 1):
        lvx.lvx_chunk_append_evict(cache, 0, k[frame + i * n:frame + (i + 1) * n].contiguous(), v[frame + i * n:frame + (i + 1) * n].contiguous(), i)
    out = torch.empty((n, d), dtype=torch.bfloat16, device=DEV)
    lvx.lvx_chunk_attention(cache, 0, q, 0.2, out)
    torch.cuda.synchronize()
    q64, k64, v64 = (S.to_f64(t).reshape(-1, H, D) for t in (q, k, v))
    want = O.attention(q64, k64, v64, 0.2)
    e = np.linalg.norm(S.to_f64(out).reshape(n, H, D) - want) / np.linalg.norm(want)
    print("large scores %s: rel %.2e" % ((H, D, n, n_keys), e), flush=True)
    # probabilities and outputs are rounded to bf16 once each, 2^-9 / sqrt(3) = 1.1e-3 root mean square (fewer than one key would have to decide an output
    # for the probabilities' share to be larger), and a row sum of unrounded probabilities adds nothing
    assert e <= 4e-3
    cache.close()
