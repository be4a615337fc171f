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


@pytest.mark.parametrize("D,H", [(128, 3), (64, 4), (128, 136), (64, 136)])   # 136 heads x 130 queries: 256-query workgroups
@pytest.mark.parametrize("prescaled", [False, True])
def test_attention_key_split_edges(lvx, D, H, prescaled):
    d = H * D
    for n_keys in (1, 63, 64, 65, 128, 129, 192, 200, 1024, 1030, 1090):
        cache = lvx.KVCache(lvx.cache_desc(1, H, D, 1, n_keys, 1, 1, 1), DEV)
        k = S.randn_bf16((n_keys, d), S.seed_of("sp_k", D, H, n_keys), device=DEV)
        v = S.randn_bf16((n_keys, d), S.seed_of("sp_v", D, H, n_keys), device=DEV)
        if n_keys >= 128:
            k[64:128] *= 24.0   # the second tile's logits dwarf the first's: the halves end with far apart references
        lvx.lvx_kvcache_set_sink(cache, 0, k, v)
        for n_q in ((1, 31, 33, 127, 128, 129, 257) if H < 100 else (130, 256)):
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
