"""Attention with 128 queries per workgroup and the keys split over its halves, and the 256-query form beside it, at the sizes where the
split can go wrong: a single tile (the second half sees no key), odd and even tile counts, ragged last tiles on either half, query
counts around a wave's 32 and a workgroup's 128, and references that differ between the halves."""
import math

import numpy as np
import pytest
import torch

import lvx_synth as S
from test_gpu_parity import DEV, LOG2E

pytestmark = pytest.mark.gpu


# (head_dim, heads), query counts that take the split form (from 8 key tiles on, and above 128 queries from the first), query counts
# that do not, and some that take one or the other by the number of tiles; test_launch_rules.py holds the rule to it
KEY_COUNTS = (1, 63, 64, 65, 128, 129, 192, 200, 1024, 1030, 1090)
GEOMETRIES = [((128, 3), (1, 31, 33, 127, 128, 129, 257), (), ()), ((64, 4), (1, 31, 33, 127, 128, 129, 257), (), ()),
              ((128, 136), (330,), (200, 256), (130,)), ((64, 136), (330,), (130, 200, 256), ())]


@pytest.mark.parametrize("D,H", [g[0] for g in GEOMETRIES])
@pytest.mark.parametrize("prescaled", [False, True])
def test_attention_key_split_edges(lvx, D, H, prescaled):
    d = H * D
    n_qs = next(split + unsplit + either for g, split, unsplit, either in GEOMETRIES if g == (D, H))
    for n_keys in KEY_COUNTS:
        cache = lvx.KVCache(lvx.cache_desc(1, H, D, 1, n_keys, 1, 1, 1), DEV)
        k = S.randn_bf16((n_keys, d), S.seed_of("sp_k", D, H, n_keys), device=DEV)
        v = S.randn_bf16((n_keys, d), S.seed_of("sp_v", D, H, n_keys), device=DEV)
        if n_keys >= 128:
            k[64:128] *= 24.0   # the second tile's logits dwarf the first's: the halves end with far apart references
        lvx.lvx_kvcache_set_sink(cache, 0, k, v)
        for n_q in n_qs:
            q = S.randn_bf16((n_q, d), S.seed_of("sp_q", D, H, n_q), device=DEV)
            out = torch.full((n_q + 1, d), 7.0, dtype=torch.bfloat16, device=DEV)
            scale = 1.0 / math.sqrt(D)
            if prescaled:
                q = (q.float() * (scale * LOG2E)).to(torch.bfloat16)
                lvx.lvx_chunk_attention_prescaled(cache, 0, q, out[:n_q])
                scale = math.log(2.0)
            else:
                lvx.lvx_chunk_attention(cache, 0, q, scale, out[:n_q])
            torch.cuda.synchronize()
            assert bool((out[n_q] == 7.0).all())
            for h in sorted({0, H // 2, H - 1}):
                c = slice(h * D, (h + 1) * D)
                Q, K, V = (S.to_f64(t[:, c]) for t in (q, k, v))
                s = scale * (Q @ K.T)
                p = np.exp(s - s.max(axis=1, keepdims=True))
                p /= p.sum(axis=1, keepdims=True)
                # each probability is rounded to bf16 (8 significant bits: up to 2^-8 of it) and so is the output, whose magnitude
                # is at most sum p |v|; a tenth more for the fp32 scores (up to about 100, each a sum of head_dim products), the
                # exponentials and the sums
                bound = 1.1 * 2.0 ** -7 * (p @ np.abs(V)) + 1e-6
                worst = (np.abs(S.to_f64(out[:n_q, c]) - p @ V) / bound).max()
                assert worst <= 1.0, (D, H, n_keys, n_q, h, worst)
        cache.close()


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("prescaled", [False, True])
def test_later_tiles_without_a_finite_score(lvx, D, prescaled):
    """Key tiles after the first whose scores are all -inf (finite keys and queries whose products overflow) carry no weight, whichever
    half of a workgroup they fall to and whatever follows them."""
    H = 2
    d = H * D
    for n_keys, dead in ((128, (1,)), (100, (1,)), (192, (1,)), (256, (1, 3)), (320, (1, 2)), (320, (1, 2, 3, 4)), (1090, (1, 2, 9, 17))):
        cache = lvx.KVCache(lvx.cache_desc(1, H, D, 1, n_keys, 1, 1, 1), DEV)
        k = S.randn_bf16((n_keys, d), S.seed_of("dt_k", D, n_keys), device=DEV)
        v = S.randn_bf16((n_keys, d), S.seed_of("dt_v", D, n_keys), device=DEV)
        q = S.randn_bf16((150, d), S.seed_of("dt_q", D, n_keys), device=DEV)
        q[:, ::D] = 16.0                      # one channel of every head carries the tiles' fate
        k[:, ::D] = 0.0
        live = torch.ones(n_keys, dtype=torch.bool)
        for t in dead:
            k[64 * t:64 * t + 64, ::D] = -3.0e38
            live[64 * t:64 * t + 64] = False
        lvx.lvx_kvcache_set_sink(cache, 0, k, v)
        scale = 1.0 / math.sqrt(D)
        out = torch.empty((150, d), dtype=torch.bfloat16, device=DEV)
        if prescaled:
            lvx.lvx_chunk_attention_prescaled(cache, 0, q, out)
            scale = math.log(2.0)
        else:
            lvx.lvx_chunk_attention(cache, 0, q, scale, out)
        torch.cuda.synchronize()
        live = live.numpy()
        for h in range(H):
            c = slice(h * D, (h + 1) * D)
            Q, K, V = S.to_f64(q[:, c]), S.to_f64(k[:, c])[live], S.to_f64(v[:, c])[live]
            s = scale * (Q @ K.T)
            p = np.exp(s - s.max(axis=1, keepdims=True))
            p /= p.sum(axis=1, keepdims=True)
            got = S.to_f64(out[:, c])
            assert np.isfinite(got).all(), (D, n_keys, dead, h)
            bound = 1.1 * 2.0 ** -7 * (p @ np.abs(V)) + 1e-6      # as above
            assert (np.abs(got - p @ V) / bound).max() <= 1.0, (D, n_keys, dead, h)
        cache.close()
