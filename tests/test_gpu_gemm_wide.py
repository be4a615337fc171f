"""Products on tiles of 256 x 256, 192 or 128 and their halves against the fp64 oracle: one slab and few, rows and columns past the last tile, rows
that only a half covers, all epilogues, output rows that allow 16-byte stores and rows that do not."""
import math

import numpy as np
import pytest
import torch

import lvx_synth as S
from oracle import lvx_oracle as O
from test_gpu_parity import DEV, assert_close

pytestmark = pytest.mark.gpu

# M, N, K with the rows on wide tiles, their columns / 64, the whole tiles and the halves that the rule takes; test_wide_rules.py holds it to them
SHAPES = [((1567, 13832, 64), (1567, 4, 256, 203)), ((1567, 13832, 320), (1567, 4, 256, 203)), ((1411, 4616, 192), (1411, 4, 0, 228)),
          ((1033, 14432, 3840), (1024, 4, 228, 0)),
          ((1731, 5656, 64), (1731, 3, 210, 0)), ((1731, 5656, 192), (1731, 3, 210, 0)), ((1281, 13272, 128), (1281, 3, 350, 70)),
          ((4353, 4616, 128), (4353, 3, 425, 25)), ((1901, 2568, 192), (1901, 3, 0, 210)),
          ((515, 9832, 64), (515, 2, 154, 77)), ((515, 9832, 192), (515, 2, 154, 77)), ((129, 10904, 128), (129, 2, 0, 172))]
# halves only, the last rows (a few of 128) beside those of the same columns: three rows of halves, and eight and one
HALF_SHAPES = [((267, 6632, 192), (267, 2, 0, 156)), ((267, 10920, 128), (267, 3, 0, 171)), ((1129, 3752, 192), (1129, 3, 0, 180)),
               ((1129, 5544, 128), (1129, 4, 0, 198))]
FP8_SHAPES = [((1567, 13832, 256), (1567, 4, 256, 203)), ((1411, 4616, 1920), (1411, 4, 0, 228)),
              ((1731, 5656, 128), (1731, 3, 210, 0)), ((1731, 5656, 384), (1731, 3, 210, 0)), ((1901, 2568, 256), (1901, 3, 0, 210)),
              ((515, 9832, 128), (515, 2, 154, 77)), ((129, 10904, 1920), (129, 2, 0, 172))]


def padded(M, N, pad, dtype, fill=7.0):
    return torch.full((M + 1, N + pad), fill, dtype=dtype, device=DEV)


@pytest.mark.parametrize("pad", [8, 3])
@pytest.mark.parametrize("M,N,K", [s for s, _ in SHAPES])
def test_linear_on_wide_tiles(lvx, M, N, K, pad):
    a = S.randn_bf16((M, K + 8), S.seed_of("wt_a", M, K), device=DEV)[:, :K]
    w = S.randn_bf16((N, K + 64), S.seed_of("wt_w", N, K), 1.0 / math.sqrt(K), device=DEV)[:, :K]
    g = S.randn_f32((N + 1,), 7, 0.5, 1.0, device=DEV)[1:]          # a gate vector at a 4-byte boundary
    r = S.randn_f32((M, N + pad), S.seed_of("wt_r", M, N), device=DEV)
    rb = r.to(torch.bfloat16)
    ref = torch.from_numpy(O.linear(S.to_f64(a), S.to_f64(w)))
    g64, r64, rb64 = (torch.from_numpy(S.to_f64(t)) for t in (g, r[:, :N], rb[:, :N]))
    bound = 4.0 * K * 2.0 ** -24 + 1e-6      # fp32 sums of K products of size 1 / sqrt(K), as in test_gpu_gemm_tiles.py

    def run(epi, dtype, resid=None, gate=None):
        out = padded(M, N, pad, dtype)
        lvx.lvx_linear(a, w, out[:M, :N], epi, resid=resid, gate=gate)
        torch.cuda.synchronize()
        assert bool((out[M] == 7.0).all()) and bool((out[:, N:] == 7.0).all()), epi
        return out[:M, :N]
    assert_close(run(lvx.EPI_STORE, torch.bfloat16), ref.numpy(), "store %dx%dx%d" % (M, N, K))
    assert_close(run(lvx.EPI_GELU_TANH, torch.bfloat16), O.gelu_tanh(ref.numpy()), "gelu")
    assert_close(run(lvx.EPI_BIAS, torch.bfloat16, gate=g), (ref + g64).numpy(), "bias")
    assert_close(run(lvx.EPI_BIAS_SILU, torch.bfloat16, gate=g), O.silu((ref + g64).numpy()), "bias + silu")
    assert_close(run(lvx.EPI_RESID_GATE, torch.bfloat16, resid=rb[:, :N], gate=g), (rb64 + g64 * ref).numpy(), "bf16 residual")
    assert np.abs(S.to_f64(run(lvx.EPI_STORE_F32, torch.float32)) - ref.numpy()).max() <= bound
    x = r.clone()
    lvx.lvx_linear(a, w, x[:, :N], lvx.EPI_RESID_GATE_F32, resid=x[:, :N], gate=g)       # in place
    torch.cuda.synchronize()
    assert np.abs(S.to_f64(x[:, :N]) - (r64 + g64 * ref).numpy()).max() <= 4.0 * bound
    assert torch.equal(x[:, N:], r[:, N:])


@pytest.mark.parametrize("M,N,K", [s for s, _ in SHAPES])
def test_fp32_outputs_are_the_sums_that_bf16_outputs_round(lvx, M, N, K):
    """Plain fp32 outputs leave the matrix core with rows and columns exchanged; their sums are the same, bit for bit."""
    a = S.randn_bf16((M, K), S.seed_of("wf_a", M, K), device=DEV)
    w = S.randn_bf16((N, K), S.seed_of("wf_w", N, K), 1.0 / math.sqrt(K), device=DEV)
    out, out32 = padded(M, N, 8, torch.bfloat16), padded(M, N, 5, torch.float32)
    lvx.lvx_linear(a, w, out[:M, :N], lvx.EPI_STORE)
    lvx.lvx_linear(a, w, out32[:M, :N], lvx.EPI_STORE_F32)
    torch.cuda.synchronize()
    assert torch.equal(out32[:M, :N].to(torch.bfloat16), out[:M, :N])
    assert bool((out32[M] == 7.0).all()) and bool((out32[:, N:] == 7.0).all())


@pytest.mark.parametrize("M,N,K", [s for s, _ in HALF_SHAPES])
def test_halves_alone_cover_the_output(lvx, M, N, K):
    a = S.randn_bf16((M, K), S.seed_of("wh_a", M, K), device=DEV)
    w = S.randn_bf16((N, K), S.seed_of("wh_w", N, K), 1.0 / math.sqrt(K), device=DEV)
    out = padded(M, N, 8, torch.bfloat16)
    lvx.lvx_linear(a, w, out[:M, :N], lvx.EPI_STORE)
    torch.cuda.synchronize()
    assert_close(out[:M, :N], O.linear(S.to_f64(a), S.to_f64(w)), "halves %dx%dx%d" % (M, N, K))
    assert bool((out[M] == 7.0).all()) and bool((out[:, N:] == 7.0).all())


@pytest.mark.parametrize("M,N,K", [s for s, _ in FP8_SHAPES])
def test_linear_fp8_on_wide_tiles(lvx, M, N, K):
    aq, sa = lvx.lvx_fp8_quantize(S.randn_bf16((M, K), S.seed_of("w8_a", M, K), device=DEV), row_pad=16)
    wq, sw = lvx.lvx_fp8_quantize(S.randn_bf16((N, K), S.seed_of("w8_w", N, K), 1.0 / math.sqrt(K), device=DEV), row_pad=128)
    dec = [S.to_f64(q.contiguous().view(torch.float8_e4m3fn).float()) * float(s.item()) for q, s in ((aq, sa), (wq, sw))]
    ref = O.linear(dec[0], dec[1])
    g = S.randn_f32((N,), 7, 0.5, 1.0, device=DEV)
    out = padded(M, N, 8, torch.bfloat16)
    lvx.lvx_linear_fp8(aq, sa, wq, sw, out[:M, :N], lvx.EPI_STORE)
    x = S.randn_f32((M, N + 3), S.seed_of("w8_r", M, N), device=DEV)
    r = x.clone()
    lvx.lvx_linear_fp8(aq, sa, wq, sw, x[:, :N], lvx.EPI_RESID_GATE_F32, resid=x[:, :N], gate=g)
    torch.cuda.synchronize()
    assert_close(out[:M, :N], ref, "fp8 store %dx%dx%d" % (M, N, K))
    assert bool((out[M] == 7.0).all()) and bool((out[:, N:] == 7.0).all()) and torch.equal(x[:, N:], r[:, N:])
    # the FP8 products' alignment in the matrix core: see test_gpu_gemm_tiles.py
    assert np.abs(S.to_f64(x[:, :N]) - (S.to_f64(r[:, :N]) + S.to_f64(g) * ref)).max() <= 1e-4 * math.sqrt(K)


@pytest.mark.parametrize("M,N1,N2", [(4353, 2328, 2296), (1567, 6920, 6912), (515, 4936, 4896)])
def test_segments_on_wide_tiles(lvx, M, N1, N2):
    """Two products of one launch whose widths end inside a tile, the first stored fp32."""
    K = 128
    a = S.randn_bf16((M, K), S.seed_of("ws_a"), device=DEV)
    w = S.randn_bf16((N1 + N2, K), S.seed_of("ws_w"), 1.0 / math.sqrt(K), device=DEV)
    ref = O.linear(S.to_f64(a), S.to_f64(w))
    for pad in (8, 2):
        c1, c2 = padded(M, N1, pad, torch.float32), padded(M, N2, pad, torch.bfloat16)
        lvx.lvx_linear_dual(a, w[:N1], w[N1:], c1[:M, :N1], c2[:M, :N2])
        torch.cuda.synchronize()
        assert np.abs(S.to_f64(c1[:M, :N1]) - ref[:, :N1]).max() <= 4.0 * K * 2.0 ** -24 + 1e-6
        assert_close(c2[:M, :N2], ref[:, N1:], "second product")
        for c, n in ((c1, N1), (c2, N2)):
            assert bool((c[M] == 7.0).all()) and bool((c[:, n:] == 7.0).all())
