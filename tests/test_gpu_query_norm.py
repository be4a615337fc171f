"""Blocks of head_dim 128 at widths whose cross-attention query norm is folded into the projection and the attention kernel with partial
sums that do not fill whole vectors, from every kind of GEMM tile, against the oracle; the workspace starts as NaN, so that a
padding float that entered a sum would show."""
import math

import pytest
import torch

import lvx_synth as S
from oracle import lvx_oracle as O
from test_gpu_parity import DEV, assert_close

pytestmark = pytest.mark.gpu

# heads, frame_h, frame_w, chunk_frames with the partial sums that a query row gets; test_launch_rules.py holds the rule to it
SHAPES = [((1, 7, 9, 1), 8), ((3, 5, 11, 1), 24),
          ((5, 9, 11, 2), 40),                        # 16-column sums of K groups
          ((3, 29, 31, 3), 12), ((5, 33, 25, 2), 20), ((9, 31, 31, 1), 36),    # 32-column sums of 64 x 128 tiles, ragged vectors
          ((5, 43, 39, 2), 10), ((9, 31, 31, 2), 18)]                          # 64-column sums of 256-column tiles, the last one half empty


@pytest.mark.parametrize("shape", [s for s, _ in SHAPES])
def test_block_with_folded_query_norm(lvx, shape):
    H, fh, fw, frames = shape
    D, n_ctx, ffn = 128, 33, 256
    d, n, sink_n = H * D, fh * fw * frames, fh * fw
    tag = "qn_%d_%d" % (d, n)
    w = S.block_weights(d, ffn, 0, tag, std=1.0 / math.sqrt(d), device=DEV)
    for g in ("g_q", "g_k", "gc_q", "gc_k"):
        w[g] = S.randn_f32((d,), S.seed_of(tag, g), 0.2, 1.0, device=DEV)
    rope = lvx.rope_desc(H, D, (44, 42, 42), 10000.0, fh, fw)
    stage = lvx.StageHandle([w], rope, ffn)
    cache = lvx.KVCache(lvx.cache_desc(1, H, D, fh, fw, frames, 1, 1), DEV)
    sk, sv = (S.randn_bf16((sink_n, d), S.seed_of(tag, k), device=DEV) for k in ("sk", "sv"))
    lvx.lvx_kvcache_set_sink(cache, 0, sk, sv)
    model = O.RollingKVCache(1)
    model.set_sink(S.to_f64(sk).reshape(sink_n, H, D), S.to_f64(sv).reshape(sink_n, H, D))
    # projected queries of very different sizes: the row's own norm decides
    x = S.randn_f32((n, d), S.seed_of(tag, "x"), device=DEV)
    w["Wc_q"][:, :] = (w["Wc_q"].float() * torch.exp(S.randn_f32((d, 1), S.seed_of(tag, "spread"), 1.0, device=DEV))).to(torch.bfloat16)
    ctx = S.randn_bf16((n_ctx, d), S.seed_of(tag, "ctx"), device=DEV)
    ws = torch.full((lvx.lvx_workspace_bytes(stage, n, n_ctx),), 255, dtype=torch.uint8, device=DEV)
    ref = O.dit_block(S.to_f64(x), S.weights_to_f64(w), model, S.to_f64(ctx), None, 0, 1, O.StageConfig(H, D, fh, fw, frames, 1, 1, (44, 42, 42)))
    lvx.lvx_dit_block_f32(stage, 0, cache, x, ctx, None, 0, 1, ws)
    torch.cuda.synchronize()
    assert_close(x, ref, "block, d %d, %d tokens" % (d, n), relative_to_rms=True)
    cache.close()
