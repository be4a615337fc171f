// bf16 linears of the DiT blocks (C[M][N] = epilogue(A[M][K] * W[N][K]^T), fp32 accumulate; Appendix C, shapes are the workload's) and the
// decoder's 3x3x3 convolution as an implicit GEMM: entry points, dispatch, and the convolution's kernel of 256 x 128 tiles.
//
// Both operands have the contraction index contiguous in memory (activations [token][in], weights [out][in]), so both
// stream global -> LDS as 16-byte chunks and are read back as direct v_mfma_f32_16x16x32_bf16 operands with 16-byte ds_reads (the 16 x 16 x 32
// form moves a fifth less through the register file per flop than 32 x 32 x 16 and runs 1-5 % faster here, the chip being power-limited).
// The large products run on lvx_gemm_wide.h, the small ones on lvx_gemm_core.h; lvx_gemm_choose and lvx_conv_choose say which.
#include "lvx_conv_gemm.h"
#include "lvx_gemm_wide.h"

namespace {

constexpr int BK = 64;
constexpr int GROUP_M = 8;

// Convolution, 256 x 128 tiles: rows gathered from the zero-padded volume, a tap being a constant shift of the row addresses.
// gfx950's global_load_lds_dwordx4 moves 16 bytes per lane from global memory straight into LDS (LDS byte address = M0 + 16*lane), so a slab
// needs no staging registers, no ds_write and no trip through the register file; three 48 KB stages.  A wave instruction fills 1024
// contiguous LDS bytes = 8 rows of 64 bf16, so rows cannot be padded; bank conflicts are avoided by an XOR swizzle instead: the 16-byte
// chunk c of LDS row r holds global chunk c ^ ((r >> 1) & 7) (the lane simply fetches that chunk): 16 consecutive rows read at one k-chunk then
// cover 16 distinct 16-byte units of the 256-byte bank row.  The loads are issued through inline asm with explicit s_waitcnt vmcnt(n): the
// compiler would otherwise wait for ALL outstanding loads before any LDS read that might alias.
// It keeps the steps whose last round of such tiles is well filled: four 50 x 90 frames 384 -> 384 channels 139 us, on wide tiles 141 to 145.
template <int EPI>
__global__ void __launch_bounds__(512)
    lvx_conv_large_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W, int64_t ldw, bf16_t *C, int64_t ldc, int M, int N, int K,
                          const float *__restrict__ bias, int tiles_m, int tiles_n, int per_xcd, lvx_conv_map_t cm) {
    constexpr int BM = 256, BN = 128, WAVES_N = 2, NW = 8;
    constexpr int FM = 4, FN = 4;  // 16 x 16 accumulator blocks per wave: 64 x 64
    constexpr int ROW_B = BK * 2;  // bytes per LDS row (unpadded)
    constexpr int A_B = BM * ROW_B, STAGE_B = (BM + BN) * ROW_B;
    constexpr int NSTAGE = 3;
    constexpr int QPW = (BM + BN) / 8 / NW;  // loads per wave and slab (8 rows each)
    constexpr int A_Q = BM / 8 / NW;         // of which the first A_Q fetch A rows

    __shared__ __attribute__((aligned(1024))) char lds[NSTAGE * STAGE_B];

    int tm, tn;
    if (!lvx_gemm_tile_of(tiles_m, tiles_n, per_xcd, GROUP_M, tm, tn)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, q4 = lane >> 4;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;

    // load q of this wave covers stage rows 8*(wave + NW*q) .. +7 (A rows first, then W rows); lane -> (row, position)
    uint32_t doff[QPW];
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
        const int row_s = 8 * (wave + NW * q) + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row_s >> 1) & 7);
        if (q < A_Q) {
            int r = tm * BM + row_s;
            if (r > M - 1) r = M - 1;
            doff[q] = (uint32_t)(lvx_conv_pixel_offset(cm, r) + chunk * 16);
        } else {
            int r = tn * BN + (row_s - BM);
            if (r > N - 1) r = N - 1;
            doff[q] = (uint32_t)(((size_t)r * ldw + chunk * 8) * sizeof(bf16_t));
        }
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds_base + wave * 1024);
    lvx_conv_walk_t walk;  // the slab to load: its byte offset in the rows of the volume and of W
#define LVX_DMA_ISSUE(stage_, q_)                                                                                           \
    lvx_dma16((q_) < A_Q ? reinterpret_cast<const char *>(A) + walk.a : reinterpret_cast<const char *>(W) + walk.w, doff[q_], \
              lds_wave + (uint32_t)((stage_) * STAGE_B + (q_) * NW * 1024))

    // fragment reads for v_mfma_f32_16x16x32_bf16: lane (l16, q4) reads row l16 of a 16-row block, k-chunk 4*ks + q4 of the
    // slab's 8, at its swizzled position
    const int swz = (l16 >> 1) & 7;
    const char *a_rd = lds + (wm * 64 + l16) * ROW_B;
    const char *w_rd = lds + A_B + (wn * 64 + l16) * ROW_B;
    bf16x8_t af[2][FM], wf[2][FN];
#define LVX_DMA_READ_A(stage_, ks_, i0_, i1_)                                                                               \
    {                                                                                                                       \
        const int co_ = (((ks_) * 4 + q4) ^ swz) * 16 + (stage_) * STAGE_B;                                                 \
        _Pragma("unroll") for (int i = i0_; i < i1_; ++i) af[(ks_) & 1][i] = *reinterpret_cast<const bf16x8_t *>(a_rd + i * 16 * ROW_B + co_); \
    }
#define LVX_DMA_READ_W(stage_, ks_, j0_, j1_)                                                                               \
    {                                                                                                                       \
        const int co_ = (((ks_) * 4 + q4) ^ swz) * 16 + (stage_) * STAGE_B;                                                 \
        _Pragma("unroll") for (int j = j0_; j < j1_; ++j) wf[(ks_) & 1][j] = *reinterpret_cast<const bf16x8_t *>(w_rd + j * 16 * ROW_B + co_); \
    }
    // MFMAs of k-step ks_ for accumulator rows [i0_, i1_)
#define LVX_DMA_MFMAS(ks_, i0_, i1_)                                                                         \
    _Pragma("unroll") for (int i = i0_; i < i1_; ++i) _Pragma("unroll") for (int j = 0; j < FN; ++j)         \
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[(ks_) & 1][i], wf[(ks_) & 1][j], acc[i][j], 0, 0, 0);

    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int n_k = K / BK;  // at least 27 slabs
    const int last = n_k - 1;
#pragma unroll
    for (int q = 0; q < QPW; ++q) LVX_DMA_ISSUE(0, q);
    walk.next(cm);
#pragma unroll
    for (int q = 0; q < QPW; ++q) LVX_DMA_ISSUE(1, q);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(QPW) : "memory");
    __syncthreads();
    LVX_DMA_READ_A(0, 0, 0, FM);
    LVX_DMA_READ_W(0, 0, 0, FN);

    // Slab t is in stage t % 3.  Per slab four MFMA groups (each k-step as two halves of the accumulator rows): the first three
    // read the fragments still missing for what follows and issue a third of the DMA for slab t+2 each (into the stage that
    // was read during slab t-1); then wait until this wave's DMA for slab t+1 has landed, one workgroup barrier, and the
    // fourth group, which already reads k-step 0 of slab t+1.
    int cur = 0, nxt = 1, nx2 = 2;
    for (int t = 0; t < n_k; ++t) {
        if (t + 2 <= last) walk.next(cm);  // past the end: a harmless reload of the last slab
        LVX_DMA_READ_W(cur, 1, 0, FN);
        __builtin_amdgcn_sched_barrier(0);
        LVX_DMA_MFMAS(0, 0, FM / 2);
#pragma unroll
        for (int q = 0; q < QPW; ++q)
            if ((q * 3) / QPW == 0) LVX_DMA_ISSUE(nx2, q);
        __builtin_amdgcn_sched_barrier(0);
        LVX_DMA_READ_A(cur, 1, 0, FM / 2);
        __builtin_amdgcn_sched_barrier(0);
        LVX_DMA_MFMAS(0, FM / 2, FM);
#pragma unroll
        for (int q = 0; q < QPW; ++q)
            if ((q * 3) / QPW == 1) LVX_DMA_ISSUE(nx2, q);
        __builtin_amdgcn_sched_barrier(0);
        LVX_DMA_READ_A(cur, 1, FM / 2, FM);
        __builtin_amdgcn_sched_barrier(0);
        LVX_DMA_MFMAS(1, 0, FM / 2);
#pragma unroll
        for (int q = 0; q < QPW; ++q)
            if ((q * 3) / QPW == 2) LVX_DMA_ISSUE(nx2, q);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(QPW) : "memory");
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        LVX_DMA_READ_A(nxt, 0, 0, FM);
        LVX_DMA_READ_W(nxt, 0, 0, FN);
        __builtin_amdgcn_sched_barrier(0);
        LVX_DMA_MFMAS(1, FM / 2, FM);
        __builtin_amdgcn_sched_barrier(0);
        const int tmp = cur;
        cur = nxt;
        nxt = nx2;
        nx2 = tmp;
    }
    // no load may still be in flight when the workgroup releases its LDS
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    float gt[FN];
    lvx_gemm_gates<FN>(gt, EPI, bias, N, tn * BN + wn * 64 + l16);
    lvx_gemm_epilogue<FM, FN, EPI, false>(acc, acc, C, ldc, nullptr, 0, gt, M, N, tm * BM + wm * 64 + 4 * q4, tn * BN + wn * 64 + l16, 1.f);
#undef LVX_DMA_ISSUE
#undef LVX_DMA_READ_A
#undef LVX_DMA_READ_W
#undef LVX_DMA_MFMAS
}

// The linears: see lvx_gemm_choose.
lvx_status_t launch_linear(const bf16_t *A, int64_t lda, const bf16_t *W, int64_t ldw, bf16_t *C, int64_t ldc, int M, int N, int K, int epi,
                           const bf16_t *R, int64_t ldr, const float *gate, hipStream_t stream, const lvx_gemm_segs_t *segs = nullptr) {
    const lvx_gemm_launch_t plan = lvx_gemm_choose(segs, M, N, K / BK);
    lvx_gemm_args_t p = {};
    p.A = (const char *)A, p.lda = lda * 2;
    p.W = (const char *)W, p.ldw = ldw * 2;
    p.C = C, p.ldc = ldc;
    p.R = R, p.ldr = ldr;
    p.gate = gate;
    p.N = N, p.n_slabs = K / BK;
    p.epi = epi;
    if (segs != nullptr) p.segs = *segs;
    if (plan.wide_rows > 0) {
        p.M = plan.wide_rows;
        lvx_status_t st;
        switch (epi) {
#define LVX_WIDE_CASE(E_) \
    case E_: st = plan.fn == 2 ? lvx_gemm_wide_launch<E_, false, 2>(p, plan.n_large, stream) : plan.fn == 3 ? lvx_gemm_wide_launch<E_, false, 3>(p, plan.n_large, stream) : lvx_gemm_wide_launch<E_, false, 4>(p, plan.n_large, stream); break;
            LVX_WIDE_CASE(LVX_EPI_STORE)
            LVX_WIDE_CASE(LVX_EPI_GELU_TANH)
            LVX_WIDE_CASE(LVX_EPI_RESID_GATE)
            LVX_WIDE_CASE(LVX_EPI_RESID_GATE_F32)
            LVX_WIDE_CASE(LVX_EPI_BIAS)
            LVX_WIDE_CASE(LVX_EPI_BIAS_SILU)
            LVX_WIDE_CASE(LVX_EPI_STORE_F32)
            LVX_WIDE_CASE(LVX_EPI_SEGMENTS)
#undef LVX_WIDE_CASE
            default: return lvx_fail(LVX_ERR_INVALID_ARG, "unknown epilogue %d", epi);
        }
        LVX_TRY(st);
        if (plan.wide_rows == M) return LVX_OK;
    }
    // the rows behind, or all, on a small tile
    const int m1 = plan.wide_rows;
    const bool c_f32 = epi == LVX_EPI_RESID_GATE_F32 || epi == LVX_EPI_STORE_F32;
    p.A += (size_t)m1 * p.lda;
    p.C = (char *)C + (size_t)m1 * ldc * (c_f32 ? 4 : 2);
    if (R != nullptr) p.R = (const char *)R + (size_t)m1 * ldr * (epi == LVX_EPI_RESID_GATE_F32 ? 4 : 2);
    p.M = M - m1;
    for (int i = 0; i < p.segs.n; ++i) p.segs.s[i].C = (char *)p.segs.s[i].C + (size_t)m1 * p.segs.s[i].ldc * (p.segs.s[i].f32 ? 4 : 2);
    return lvx_gemm_launch_small<false>(plan.tile, p, stream);
}

}  // namespace

// C1 = A W1^T ([M][N1]) and C2 = A W2^T ([M][N2]) in one launch (same K and weight row stride).  Two uses: two small-M
// projections of the same input fill the chip together where each alone leaves most of it idle (the context's K and V
// projections: 100 tiles each on 256 CUs); and the fused QKV projection with its q | k columns stored in fp32 (they go on to
// the RMSNorm + RoPE kernel, which rounds to bf16 once, after the rotation) and its v columns in bf16.
static lvx_status_t check_dual(const void *A, int64_t lda, const void *W1, const void *W2, int64_t ldw, const void *C1, int64_t ldc1,
                               const void *C2, int64_t ldc2, int M, int N1, int N2, int K) {
    LVX_REQUIRE(A && W1 && W2 && C1 && C2, LVX_ERR_INVALID_ARG, "linear dual: NULL pointer");
    LVX_REQUIRE(lvx_aligned16(A) && lvx_aligned16(W1) && lvx_aligned16(W2) && lvx_aligned16(C1) && lvx_aligned16(C2), LVX_ERR_INVALID_ARG,
                "pointers must be 16-byte aligned");
    LVX_REQUIRE(M >= 0 && N1 > 0 && N2 > 0 && K > 0 && K % BK == 0 && N1 % 8 == 0 && N2 % 8 == 0, LVX_ERR_SHAPE,
                "linear dual: M %d, N1 %d, N2 %d, K %d (K %% 64 == 0, N %% 8 == 0)", M, N1, N2, K);
    LVX_REQUIRE(lda >= K && lda % 8 == 0 && ldw >= K && ldw % 8 == 0 && ldc1 >= N1 && ldc2 >= N2, LVX_ERR_SHAPE, "bad leading dimension");
    const uint64_t n_max = (uint64_t)(N1 > N2 ? N1 : N2);
    LVX_REQUIRE((uint64_t)M * (uint64_t)lda * 2 < (1ull << 32) && n_max * (uint64_t)ldw * 2 < (1ull << 32), LVX_ERR_SHAPE,
                "operand larger than 4 GiB (32-bit byte offsets inside the kernel)");
    return LVX_OK;
}

lvx_status_t lvx_launch_linear_dual(const bf16_t *A, int64_t lda, const bf16_t *W1, const bf16_t *W2, int64_t ldw, void *C1, int64_t ldc1,
                                    int c1_is_f32, bf16_t *C2, int64_t ldc2, int M, int N1, int N2, int K, hipStream_t stream) {
    LVX_TRY(check_dual(A, lda, W1, W2, ldw, C1, ldc1, C2, ldc2, M, N1, N2, K));
    if (M == 0) return LVX_OK;
    lvx_gemm_segs_t segs;
    segs.n = 2;
    segs.order = LVX_GEMM_ORDER_FIRST;
    segs.s[0] = {W1, C1, ldc1, N1, 0, c1_is_f32 ? 1 : 0, 0};
    segs.s[1] = {W2, C2, ldc2, N2, 0, 0, 0};
    return launch_linear(A, lda, W1, ldw, (bf16_t *)C1, ldc1, M, N1, K, (int)LVX_EPI_SEGMENTS, nullptr, 0, nullptr, stream, &segs);
}

// Up to LVX_GEMM_MAX_SEGS projections of the same activations in one launch (same K, same weight row stride; each with its own
// weight matrix, output, width and row stride; bf16 or fp32 plain store): the context's K and V projections of several layers.
lvx_status_t lvx_launch_linear_segments(const bf16_t *A, int64_t lda, int64_t ldw, const lvx_gemm_segs_t &segs, int M, int K, hipStream_t stream) {
    LVX_REQUIRE(segs.n >= 1 && segs.n <= LVX_GEMM_MAX_SEGS, LVX_ERR_INVALID_ARG, "linear segments: %d segments (1..%d)", segs.n, LVX_GEMM_MAX_SEGS);
    for (int i = 0; i < segs.n; ++i)
        LVX_TRY(check_dual(A, lda, segs.s[i].W, segs.s[i].W, ldw, segs.s[i].C, segs.s[i].ldc, segs.s[i].C, segs.s[i].ldc, M, segs.s[i].N, segs.s[i].N, K));
    for (int i = 0; i < segs.n; ++i)
        LVX_REQUIRE(segs.s[i].sumsq == nullptr || (segs.s[i].N % 64 == 0 && !segs.s[i].f32 && segs.n == 1 &&
                                                   segs.s[i].ld_sumsq >= lvx_gemm_sumsq_parts(M, segs.s[i].N, K)),
                    LVX_ERR_SHAPE, "linear segments: row sums of squares need one bf16 segment of N %% 64 == 0 and room for its partial sums");
    if (M == 0) return LVX_OK;
    return launch_linear(A, lda, segs.s[0].W, ldw, (bf16_t *)segs.s[0].C, segs.s[0].ldc, M, segs.s[0].N, K, (int)LVX_EPI_SEGMENTS, nullptr, 0,
                                  nullptr, stream, &segs);
}

int lvx_gemm_sumsq_parts(int M, int N, int K) { return N / lvx_gemm_part_cols(lvx_gemm_pick_tile(nullptr, M, N, K / BK)); }

extern "C" lvx_status_t lvx_linear_dual(const void *dev_a, int64_t lda, const void *dev_w1, const void *dev_w2, int64_t ldw, void *dev_c1,
                                        int64_t ldc1, int32_t c1_is_f32, void *dev_c2, int64_t ldc2, int32_t M, int32_t N1, int32_t N2,
                                        int32_t K, lvx_stream_t stream) {
    return lvx_launch_linear_dual((const bf16_t *)dev_a, lda, (const bf16_t *)dev_w1, (const bf16_t *)dev_w2, ldw, dev_c1, ldc1, c1_is_f32,
                                  (bf16_t *)dev_c2, ldc2, M, N1, N2, K, (hipStream_t)stream);
}

// Implicit-GEMM 3x3x3 convolution: rows = output pixels, K = 27 taps x C channels gathered from the padded volume P; lvx_conv_choose
// says which kernel.
lvx_status_t lvx_launch_conv_gemm(const bf16_t *P, const lvx_conv_map_t &cm, const bf16_t *Wt, int64_t ldw, const float *bias, int act,
                                  bf16_t *Y, int64_t ldy, int M, int max_m, int N, hipStream_t stream) {
    const int K = 27 * cm.C, n_slabs = K / BK, epi = act ? (int)LVX_EPI_BIAS_SILU : (int)LVX_EPI_BIAS;
    const lvx_conv_launch_t c = lvx_conv_choose(cm.W, N, n_slabs, M, max_m);
    const lvx_conv_plan_t &plan = c.plan;
    if (c.fn == 0 && plan.kind == LVX_CONV_LARGE) {
        const int tiles_m = (M + 255) / 256, tiles_n = (N + 127) / 128, per_xcd = (tiles_m * tiles_n + 7) / 8;
        hipLaunchKernelGGL((act ? lvx_conv_large_kernel<LVX_EPI_BIAS_SILU> : lvx_conv_large_kernel<LVX_EPI_BIAS>), dim3(per_xcd * 8), dim3(512), 0, stream, P, Wt, ldw, Y, ldy,
                           M, N, K, bias, tiles_m, tiles_n, per_xcd, cm);
        LVX_CHECK_HIP(hipGetLastError());
        return LVX_OK;
    }
    if (c.fn == 0 && plan.kind == LVX_CONV_ROWS) {
        lvx_conv_args_t r = {(const char *)P, (const char *)Wt, ldw * 2, Y, ldy, bias, M / cm.W * (cm.W + 2), N, n_slabs / 3, act, 0, 0, 0, 0, cm};
#define LVX_TILE_LAUNCH(ID_, BM_, BN_, WM_, WN_, NST_, US_) \
    if (plan.tile == ID_) return lvx_conv_rows_launch<BM_, BN_, WM_, WN_, NST_>(r, stream);
        LVX_CONV_ROW_TILES(LVX_TILE_LAUNCH)
#undef LVX_TILE_LAUNCH
    }
    lvx_gemm_args_t p = {};
    p.A = (const char *)P;
    p.W = (const char *)Wt, p.ldw = ldw * 2;
    p.C = Y, p.ldc = ldy;
    p.gate = bias;
    p.M = M, p.N = N, p.n_slabs = n_slabs;
    p.epi = epi;
    p.conv = cm;
#define LVX_CONV_WIDE(FN_) \
    if (c.fn == FN_)       \
        return act ? lvx_gemm_wide_launch<LVX_EPI_BIAS_SILU, false, FN_, true>(p, c.n_large, stream) : lvx_gemm_wide_launch<LVX_EPI_BIAS, false, FN_, true>(p, c.n_large, stream);
    LVX_CONV_WIDE(2)
    LVX_CONV_WIDE(3)
    LVX_CONV_WIDE(4)
#undef LVX_CONV_WIDE
    return lvx_gemm_launch_small<false, true>(plan.tile, p, stream);
}

extern "C" lvx_status_t lvx_linear(const void *dev_a, int64_t lda, const void *dev_w, int64_t ldw, void *dev_c, int64_t ldc, int32_t M,
                                   int32_t N, int32_t K, lvx_epilogue_t epi, const void *dev_resid, int64_t ldr, const float *dev_gate,
                                   lvx_stream_t stream) {
    LVX_REQUIRE(dev_a != nullptr && dev_w != nullptr && dev_c != nullptr, LVX_ERR_INVALID_ARG, "A, W or C is NULL");
    LVX_REQUIRE(lvx_aligned16(dev_a) && lvx_aligned16(dev_w) && lvx_aligned16(dev_c) && lvx_aligned16(dev_resid), LVX_ERR_INVALID_ARG,
                "pointers must be 16-byte aligned");
    LVX_REQUIRE(M >= 0 && N > 0 && K > 0, LVX_ERR_SHAPE, "M %d, N %d, K %d", M, N, K);
    LVX_REQUIRE(K % BK == 0, LVX_ERR_SHAPE, "K %d must be a multiple of %d", K, BK);
    LVX_REQUIRE(N % 8 == 0, LVX_ERR_SHAPE, "N %d must be a multiple of 8", N);
    LVX_REQUIRE(lda >= K && lda % 8 == 0 && ldw >= K && ldw % 8 == 0 && ldc >= N, LVX_ERR_SHAPE, "bad leading dimension");
    LVX_REQUIRE((uint64_t)M * (uint64_t)lda * 2 < (1ull << 32) && (uint64_t)N * (uint64_t)ldw * 2 < (1ull << 32), LVX_ERR_SHAPE,
                "operand larger than 4 GiB (32-bit byte offsets inside the kernel)");
    LVX_REQUIRE((int)epi >= (int)LVX_EPI_STORE && (int)epi <= (int)LVX_EPI_STORE_F32, LVX_ERR_INVALID_ARG, "unknown epilogue %d", (int)epi);
    if (epi == LVX_EPI_RESID_GATE || epi == LVX_EPI_RESID_GATE_F32) {
        LVX_REQUIRE(dev_resid != nullptr, LVX_ERR_INVALID_ARG, "residual epilogue needs a residual pointer");
        LVX_REQUIRE(ldr >= N, LVX_ERR_SHAPE, "bad residual leading dimension");
    }
    if (M == 0) return LVX_OK;
    return launch_linear((const bf16_t *)dev_a, lda, (const bf16_t *)dev_w, ldw, (bf16_t *)dev_c, ldc, M, N, K, (int)epi,
                                  (const bf16_t *)dev_resid, ldr, dev_gate, (hipStream_t)stream);
}
