"""The GEMM's tile shapes against the fp64 oracle at the sizes where each can go wrong: one row / column less and more than a
tile, a contraction of a single slab, slab counts that do not divide over the K groups or the stages in flight."""
import math

import numpy as np
import pytest
import torch

import lvx_synth as S
from oracle import lvx_oracle as O
from test_gpu_parity import DEV, assert_close

pytestmark = pytest.mark.gpu

# M x N x K with the tile the launcher's rule picks for it (rows x columns, k: K groups; 128x192 and 128x256: the wide kernel, whole tiles or halves);
# test_launch_rules.py and test_wide_rules.py hold the rule to it
SHAPES = [((31, 24, 192), "32x32 k4"), ((33, 136, 320), "32x32 k4"), ((65, 1920, 448), "32x32 k4"),
          ((64, 5760, 128), "32x64 k2"), ((63, 7000, 320), "32x64 k2"), ((95, 5000, 1088), "32x64 k2"),
          ((1, 8, 64), "64x64"), ((64, 2560, 64), "64x64"), ((250, 2568, 192), "64x64"), ((257, 2560, 704), "64x64"),
          ((600, 2560, 64), "64x128"), ((577, 2696, 576), "64x128"), ((1151, 1544, 832), "64x128"),
          ((1170, 4616, 192), "128x192"), ((1901, 2568, 128), "128x192"),
          ((1300, 5120, 128), "128x256"), ((1411, 4616, 192), "128x256")]
FP8_SHAPES = [((1, 8, 128), "64x64"), ((33, 136, 640), "32x32 k4"), ((65, 1920, 896), "32x32 k4"), ((64, 5760, 256), "32x64 k2"),
              ((95, 5000, 1152), "32x64 k2"), ((257, 2560, 1408), "64x64"), ((600, 2560, 128), "64x128"), ((1151, 1544, 1664), "64x128"),
              ((1901, 2568, 256), "128x256"),
              ((1411, 4616, 1920), "128x256"), ((1411, 4616, 2048), "128x256")]
# products that 128-row tiles alone would take as named (tile and the rows before it, 0: one launch; see lvx_gemm_plan); all their rows go to the wide kernel
LARGE_SHAPES = [((1550, 5120, 1152), "64x64", 1536), ((1567, 5112, 1408), "64x64", 1536),
                ((1550, 5112, 576), "128x192", 0), ((1886, 2568, 192), "128x192", 0), ((2048, 3072, 64), "128x192", 0)]
FP8_LARGE_SHAPES = [((1550, 5120, 1152), "64x64", 1536), ((1567, 5112, 1408), "64x64", 1536)]
# products whose first rows go to the wide kernel in whole rounds and the rest, at the tile's row edges and between them, to a small tile in a second launch
SPLIT_SHAPES = [((1665, 10536, 1088), "64x128", 1536), ((1728, 10448, 640), "64x128", 1536)]
FP8_SPLIT_SHAPES = [((1665, 10552, 1408), "64x128", 1536), ((2181, 8136, 1280), "64x128", 2048), ((1728, 10688, 1536), "64x128", 1536)]
SPLIT_PAIRS = [((1699, 5320, 5136, 1280), "64x128", 1536), ((2241, 3224, 4840, 512), "64x128", 2048)]


@pytest.mark.parametrize("M,N,K", [s for s, _ in SHAPES])
def test_linear_tile_edges(lvx, M, N, K):
    a = S.randn_bf16((M, K + 8), S.seed_of("gt_a", M, K), device=DEV)[:, :K]
    w = S.randn_bf16((N, K + 64), S.seed_of("gt_w", N, K), 1.0 / math.sqrt(K), device=DEV)[:, :K]
    g = S.randn_f32((N,), 7, 0.5, 1.0, device=DEV)
    r = S.randn_f32((M, N), S.seed_of("gt_r", M, N), device=DEV)
    ref = O.linear(S.to_f64(a), S.to_f64(w))
    out = torch.full((M, N + 8), 7.0, dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear(a, w, out[:, :N], lvx.EPI_STORE)
    gelu = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear(a, w, gelu, lvx.EPI_GELU_TANH)
    x = r.clone()
    lvx.lvx_linear(a, w, x, lvx.EPI_RESID_GATE_F32, resid=x, gate=g)       # in place on the fp32 stream
    f32 = torch.full((M, N + 8), 7.0, dtype=torch.float32, device=DEV)
    lvx.lvx_linear(a, w, f32[:, :N], lvx.EPI_STORE_F32)
    torch.cuda.synchronize()
    assert_close(out[:, :N], ref, "store %dx%dx%d" % (M, N, K))
    assert_close(gelu, O.gelu_tanh(ref), "gelu")
    assert bool((out[:, N:] == 7.0).all()) and bool((f32[:, N:] == 7.0).all())
    # fp32 accumulation of K products of size 1/sqrt(K): at most K roundings of 2^-24 of a partial sum of size about 1 each
    bound = 4.0 * K * 2.0 ** -24 + 1e-6
    assert np.abs(S.to_f64(f32[:, :N]) - ref).max() <= bound
    assert np.abs(S.to_f64(x) - (S.to_f64(r) + S.to_f64(g) * ref)).max() <= 4.0 * bound


# two products of one input: the first summed as alone (the launch as a whole would take other K groups for the last two), and
# pairs of which the second is too wide for the groups that the first has alone
PAIRS = [(40, 512, 512, 512), (33, 520, 264, 320), (390, 1536, 512, 512), (96, 1024, 2048, 512), (200, 2048, 2048, 512)]
UNEQUAL_PAIRS = [(633, 32, 7000, 576), (1170, 256, 5120, 320)]


@pytest.mark.parametrize("M,N1,N2,K", PAIRS)
def test_product_bits_do_not_depend_on_its_company(lvx, M, N1, N2, K):
    """A projection launched with another one that is not far wider sums in the same order as alone."""
    a = S.randn_bf16((M, K), S.seed_of("co_a", M, K), device=DEV)
    w = S.randn_bf16((N1 + N2, K), S.seed_of("co_w", N1, N2, K), 1.0 / math.sqrt(K), device=DEV)
    c1 = torch.empty((M, N1), dtype=torch.float32, device=DEV)
    c2 = torch.empty((M, N2), dtype=torch.bfloat16, device=DEV)
    alone = torch.empty_like(c1)
    lvx.lvx_linear_dual(a, w[:N1], w[N1:], c1, c2)
    lvx.lvx_linear(a, w[:N1], alone, lvx.EPI_STORE_F32)
    torch.cuda.synchronize()
    assert torch.equal(c1, alone)


@pytest.mark.parametrize("M,N1,N2,K", UNEQUAL_PAIRS)
def test_narrow_product_beside_a_wide_one(lvx, M, N1, N2, K):
    a = S.randn_bf16((M, K), S.seed_of("up_a", M, K), device=DEV)
    w = S.randn_bf16((N1 + N2, K), S.seed_of("up_w", N1, N2, K), 1.0 / math.sqrt(K), device=DEV)
    c1 = torch.full((M, N1 + 8), 7.0, dtype=torch.float32, device=DEV)
    c2 = torch.full((M, N2 + 8), 7.0, dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear_dual(a, w[:N1], w[N1:], c1[:, :N1], c2[:, :N2])
    torch.cuda.synchronize()
    ref = O.linear(S.to_f64(a), S.to_f64(w))
    assert np.abs(S.to_f64(c1[:, :N1]) - ref[:, :N1]).max() <= 4.0 * K * 2.0 ** -24 + 1e-6     # as in test_linear_tile_edges
    assert_close(c2[:, :N2], ref[:, N1:], "wide product")
    assert bool((c1[:, N1:] == 7.0).all()) and bool((c2[:, N2:] == 7.0).all())


@pytest.mark.parametrize("M,N,K", [s for s, _ in FP8_SHAPES])
def test_linear_fp8_tile_edges(lvx, M, N, K):
    """FP8 codes are exact inputs: the product of the decoded values, scaled, is what every tile has to give."""
    aq, sa = lvx.lvx_fp8_quantize(S.randn_bf16((M, K), S.seed_of("g8_a", M, K), device=DEV), row_pad=16)
    wq, sw = lvx.lvx_fp8_quantize(S.randn_bf16((N, K), S.seed_of("g8_w", N, K), 1.0 / math.sqrt(K), device=DEV), row_pad=128)
    g = S.randn_f32((N,), 7, 0.5, 1.0, device=DEV)
    r = S.randn_f32((M, N), S.seed_of("g8_r", M, N), device=DEV)
    dec = [S.to_f64(q.contiguous().view(torch.float8_e4m3fn).float()) * float(s.item()) for q, s in ((aq, sa), (wq, sw))]
    ref = O.linear(dec[0], dec[1])
    out = torch.full((M, N + 8), 7.0, dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear_fp8(aq, sa, wq, sw, out[:, :N], lvx.EPI_STORE)
    gelu = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear_fp8(aq, sa, wq, sw, gelu, lvx.EPI_GELU_TANH)
    x = r.clone()
    lvx.lvx_linear_fp8(aq, sa, wq, sw, x, lvx.EPI_RESID_GATE_F32, resid=x, gate=g)
    torch.cuda.synchronize()
    assert_close(out[:, :N], ref, "fp8 store %dx%dx%d" % (M, N, K))
    assert_close(gelu, O.gelu_tanh(ref), "fp8 gelu")
    assert bool((out[:, N:] == 7.0).all())
    # the matrix core aligns the FP8 products it adds up to the largest of them, so a sum of products of size 1 / sqrt(K) each,
    # up to 448 * 448 quantisation steps wide, carries errors up to about 1e-4 (measured 6e-5 .. 1.9e-4 at a gate of 1, the same
    # for both shapes of the instruction); bound as for the FP8 linear of test_gpu_fp8.py
    assert np.abs(S.to_f64(x) - (S.to_f64(r) + S.to_f64(g) * ref)).max() <= 1e-4 * math.sqrt(K)


@pytest.mark.parametrize("M,N,K", [s for s, k in SHAPES if k in ("32x32 k4", "64x64", "64x128")])
def test_bf16_residual_in_place_at_tile_edges(lvx, M, N, K):
    """Small tiles read the bf16 residual of several blocks before they store the first: rows and columns past the edge, output in its place."""
    a = S.randn_bf16((M, K), S.seed_of("ri_a", M, K), device=DEV)
    w = S.randn_bf16((N, K), S.seed_of("ri_w", N, K), 1.0 / math.sqrt(K), device=DEV)
    g = S.randn_f32((N,), 7, 0.5, 1.0, device=DEV)
    x = S.randn_f32((M + 1, N + 8), S.seed_of("ri_r", M, N), device=DEV).to(torch.bfloat16)
    r = x.clone()
    lvx.lvx_linear(a, w, x[:M, :N], lvx.EPI_RESID_GATE, resid=x[:M, :N], gate=g)
    torch.cuda.synchronize()
    ref = S.to_f64(r[:M, :N]) + S.to_f64(g) * O.linear(S.to_f64(a), S.to_f64(w))
    # one rounding to bf16 (half a unit in the last place) of an fp32 sum of K products of size 1 / sqrt(K), times a gate of about 1
    assert (np.abs(S.to_f64(x[:M, :N]) - ref) <= 2.0 ** -8 * np.abs(ref) + 4.0 * (4.0 * K * 2.0 ** -24 + 1e-6)).all()
    assert torch.equal(x[M], r[M]) and torch.equal(x[:, N:], r[:, N:])


@pytest.mark.parametrize("M,N,K", [s for s, _, _ in LARGE_SHAPES + SPLIT_SHAPES])
def test_rows_split_over_two_launches_and_narrow_tiles(lvx, M, N, K):
    a = S.randn_bf16((M, K + 8), S.seed_of("rs_a", M, K), device=DEV)[:, :K]
    w = S.randn_bf16((N, K + 64), S.seed_of("rs_w", N, K), 1.0 / math.sqrt(K), device=DEV)[:, :K]
    g = S.randn_f32((N,), 7, 0.5, 1.0, device=DEV)
    r = S.randn_f32((M, N + 8), S.seed_of("rs_r", M, N), device=DEV)
    ref = O.linear(S.to_f64(a), S.to_f64(w))
    out = torch.full((M + 1, N + 8), 7.0, dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear(a, w, out[:M, :N], lvx.EPI_STORE)
    x = r.clone()
    lvx.lvx_linear(a, w, x[:, :N], lvx.EPI_RESID_GATE_F32, resid=x[:, :N], gate=g)
    rb = r.to(torch.bfloat16)
    xb = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear(a, w, xb, lvx.EPI_RESID_GATE, resid=rb[:, :N], gate=g)
    c1 = torch.empty((M, N), dtype=torch.float32, device=DEV)
    c2 = torch.empty((M, 8), dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear_dual(a, w, w[:8], c1, c2)
    torch.cuda.synchronize()
    assert_close(out[:M, :N], ref, "store %dx%dx%d" % (M, N, K))
    assert bool((out[M] == 7.0).all()) and bool((out[:, N:] == 7.0).all())
    bound = 4.0 * K * 2.0 ** -24 + 1e-6
    assert np.abs(S.to_f64(x[:, :N]) - (S.to_f64(r[:, :N]) + S.to_f64(g) * ref)).max() <= 4.0 * bound
    assert torch.equal(x[:, N:], r[:, N:])
    assert_close(xb, S.to_f64(rb[:, :N]) + S.to_f64(g) * ref, "bf16 residual")
    assert np.abs(S.to_f64(c1) - ref).max() <= bound
    assert_close(c2, ref[:, :8], "second product")
    # the last rows, in front of the others: a row's bits are the same wherever it stands
    turned = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear(torch.roll(a, 200, 0), w, turned, lvx.EPI_STORE)
    torch.cuda.synchronize()
    assert torch.equal(torch.roll(turned, -200, 0), out[:M, :N])


@pytest.mark.parametrize("M,N1,N2,K", [s for s, _, _ in SPLIT_PAIRS])
def test_rows_of_two_products_split_over_two_launches(lvx, M, N1, N2, K):
    """Each product's output moves by its own row stride and element size."""
    a = S.randn_bf16((M, K + 8), S.seed_of("sp_a", M, K), device=DEV)[:, :K]
    w = S.randn_bf16((N1 + N2, K), S.seed_of("sp_w", N1, N2, K), 1.0 / math.sqrt(K), device=DEV)
    ref = O.linear(S.to_f64(a), S.to_f64(w))
    bound = 4.0 * K * 2.0 ** -24 + 1e-6
    for dtype in (torch.float32, torch.bfloat16):
        c1 = torch.full((M + 1, N1 + 8), 7.0, dtype=dtype, device=DEV)
        c2 = torch.full((M + 1, N2 + 24), 7.0, dtype=torch.bfloat16, device=DEV)
        lvx.lvx_linear_dual(a, w[:N1], w[N1:], c1[:M, :N1], c2[:M, :N2])
        torch.cuda.synchronize()
        if dtype == torch.float32:
            assert np.abs(S.to_f64(c1[:M, :N1]) - ref[:, :N1]).max() <= bound
        else:
            assert_close(c1[:M, :N1], ref[:, :N1], "first product")
        assert_close(c2[:M, :N2], ref[:, N1:], "second product")
        for c, n in ((c1, N1), (c2, N2)):
            assert bool((c[M] == 7.0).all()) and bool((c[:, n:] == 7.0).all())


@pytest.mark.parametrize("M,N,K", [s for s, _, _ in FP8_LARGE_SHAPES + FP8_SPLIT_SHAPES])
def test_fp8_rows_split_over_two_launches(lvx, M, N, K):
    aq, sa = lvx.lvx_fp8_quantize(S.randn_bf16((M, K), S.seed_of("r8_a", M, K), device=DEV), row_pad=16)
    wq, sw = lvx.lvx_fp8_quantize(S.randn_bf16((N, K), S.seed_of("r8_w", N, K), 1.0 / math.sqrt(K), device=DEV), row_pad=128)
    dec = [S.to_f64(q.contiguous().view(torch.float8_e4m3fn).float()) * float(s.item()) for q, s in ((aq, sa), (wq, sw))]
    ref = O.linear(dec[0], dec[1])
    r = S.randn_f32((M, N), S.seed_of("r8_r", M, N), device=DEV)
    out = torch.full((M + 1, N + 8), 7.0, dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear_fp8(aq, sa, wq, sw, out[:M, :N], lvx.EPI_STORE)
    x = r.clone()
    lvx.lvx_linear_fp8(aq, sa, wq, sw, x, lvx.EPI_RESID_GATE_F32, resid=x)
    torch.cuda.synchronize()
    assert_close(out[:M, :N], ref, "fp8 store %dx%dx%d" % (M, N, K))
    assert bool((out[M] == 7.0).all()) and bool((out[:, N:] == 7.0).all())
    # the FP8 products' alignment in the matrix core: see test_linear_fp8_tile_edges
    assert np.abs(S.to_f64(x) - (S.to_f64(r) + ref)).max() <= 1e-4 * math.sqrt(K)
    g = S.randn_f32((N,), 7, 0.5, 1.0, device=DEV)
    rb = r.to(torch.bfloat16)
    xb = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    lvx.lvx_linear_fp8(aq, sa, wq, sw, xb, lvx.EPI_RESID_GATE, resid=rb, gate=g)
    # the last rows, in front of the others: a row's bits are the same wherever it stands
    turned = torch.empty((M, N), dtype=torch.float32, device=DEV)
    lvx.lvx_linear_fp8(torch.roll(aq, 200, 0), sa, wq, sw, turned, lvx.EPI_RESID_GATE_F32, resid=torch.roll(r, 200, 0))
    torch.cuda.synchronize()
    assert_close(xb, S.to_f64(rb) + S.to_f64(g) * ref, "fp8 bf16 residual")
    assert torch.equal(torch.roll(turned, -200, 0), x)


# heads of 128, frame, FFN width of a block of one-frame chunks whose first FFN product has the rows of its output's largest value in the second launch
SPLIT_BLOCK = (11, 45, 37, 10496)


def test_largest_value_of_an_fp8_output_may_lie_behind_the_split(lvx):
    """A block's FFN bit for bit as its public parts: the attentions add zero, so what the block adds is the FFN of its input, and the scale of the hidden
    tensor's codes comes from the last row, whose values only the second launch sees."""
    H, fh, fw, ffn = SPLIT_BLOCK
    d, n = 128 * H, fh * fw
    w = S.block_weights(d, ffn, 0, "sb", std=1.0 / math.sqrt(d), device=DEV)
    w["W_o"], w["Wc_o"] = torch.zeros_like(w["W_o"]), torch.zeros_like(w["Wc_o"])
    w["W_1"][:, 5] *= 8.0
    stage = lvx.StageHandle([w], lvx.rope_desc(H, 128, (44, 42, 42), 10000.0, fh, fw), ffn, fp8=True)
    cache = lvx.KVCache(lvx.cache_desc(1, H, 128, fh, fw, 1, 1, 1), DEV)
    lvx.lvx_kvcache_set_sink(cache, 0, *(S.randn_bf16((n, d), S.seed_of("sb", s), device=DEV) for s in "kv"))
    x = S.randn_bf16((n, d), S.seed_of("sb_x"), device=DEV)
    x[n - 1, 5] = 300.0          # after the norm this row is little else than its channel 5
    u, hidden, y = torch.empty_like(x), torch.empty((n, ffn), dtype=torch.bfloat16, device=DEV), x.float()
    lvx.lvx_layernorm_modulate(x, None, None, 1e-6, u)
    (uq, su), (q1, s1), (q2, s2) = (lvx.lvx_fp8_quantize(t) for t in (u, w["W_1"], w["W_2"]))
    lvx.lvx_linear_fp8(uq, su, q1, s1, hidden, lvx.EPI_GELU_TANH)
    hq, sh = lvx.lvx_fp8_quantize(hidden)
    lvx.lvx_linear_fp8(hq, sh, q2, s2, y, lvx.EPI_RESID_GATE_F32, resid=y)
    ctx = S.randn_bf16((24, d), S.seed_of("sb_ctx"), device=DEV)
    ws = torch.empty(lvx.lvx_workspace_bytes(stage, n, 24), dtype=torch.uint8, device=DEV)
    got = x.float()
    lvx.lvx_dit_block_f32(stage, 0, cache, got, ctx, None, 0, 1, ws)
    torch.cuda.synchronize()
    top = hidden.float().abs().amax(1)
    assert int(top.argmax()) == n - 1 and float(top[n - 1]) > 1.5 * float(top[:n - 1].max())
    assert torch.equal(got, y)
    cache.close()
