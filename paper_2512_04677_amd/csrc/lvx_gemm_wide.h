// Matrix products on tiles of 256 x 256, 192 or 128 and their halves of 128 rows in one launch (bf16 and FP8 operands).
//
// What bounds a large product is the power that its matrix instructions draw, if the loads keep up: 128 x 256 tiles bring 48 KB into LDS per 4.2
// MFLOP, 256 x 256 tiles 64 KB per 8.4.  Eight waves in two groups of four (the two waves of a SIMD belong to different groups) take 128 x 64
// of a tile each.  A group alternates between a memory phase (fragments LDS -> registers, direct-to-LDS loads of later slabs) and a matrix phase
// (32 instructions back to back), the groups half a period apart, with a barrier after each phase: the matrix pipe of a SIMD is fed by one wave
// while the other one reads.  A tile that remains after whole rounds of the chip, or has at most 128 rows, is worked as 128 x 256 halves by
// the same launch, so that the last round costs half as much.
// Microseconds in bf16, before (one kernel of 128 x 256 tiles, four MFMA groups a slab in step with its loads) -> now: 4680 x 15360 x 5120 612 -> 509,
// 4680 x 13824 x 5120 with GELU 557 -> 469, 4680 x 5120 x 5120 196 -> 174, with the fp32 residual 224 -> 192, 4680 x 5120 x 13824 with it 583 -> 489,
// 8192 x 8192 x 8192 868 -> 696 (1.58 PFLOP/s), 1886 x 7680 x 2560 68 -> 58.  FP8 (before: 32x32x64 instructions): 4680 x 15360 x 5120 325 -> 269,
// 4680 x 13824 x 5120 with GELU 304 -> 245, 4680 x 5120 x 13824 with the residual 290 -> 245, 4096 x 8192 x 13824 379 -> 292 (3.2 PFLOP/s).
// Without its stores the bf16 kernel runs at 1.60 PFLOP/s, the rate at which the chip's power holds a library's product as well.  The last slabs
// stand in a loop of their own: with their conditions in the main one it ran 1 to 8 % slower.  Four phases of 16 instructions instead of two cost
// 2 %, raised wave priorities change nothing, halves with a third of a slab's loads in each of two phases neither.
// Tiles of 192 or 128 columns (FN = 3, 2) serve the products whose last round 256 columns leave half empty: 1560 x 5120 x 13824 with the residual 232
// (rows split off to 64 x 64 tiles) -> 190, 1886 x 2560 x 2560 with it 32.9 (a kernel of 128 x 192 tiles) -> 31.4; which: lvx_gemm_choose.
// The decoder's convolution runs on the same kernel (CONV); see lvx_conv_choose.
#pragma once
#include "lvx_gemm_core.h"

constexpr int LVX_WIDE_HALF_B = 128 * 128;  // bytes of 128 rows of a slab

template <bool V>
struct lvx_bool_t {
    static constexpr bool value = V;
};

// Workgroup -> tile.  n_large 256 x 256 tiles, the first of the walk (bands of group_m row tiles, column-major inside a band), are taken
// whole; the rest of them in halves of 128 rows, after these the last 128 rows at most that no 256-row tile covers.  Workgroup ids are
// dealt to the XCDs round-robin by hardware; each XCD gets a contiguous range of either kind, whole tiles first.  Where they do not divide by
// 8 the first XCDs get one whole tile more and the last ones one half more, and an XCD's halves follow its whole tiles without a gap: a workgroup
// that has nothing to do still takes its turn at a shader engine, and the next one then waits for a busy engine while another one
// has an idle compute unit (6953 x 2120 x 2496, 243 whole tiles and 9 halves: 83 us with such gaps).  Of halves alone the last rows' stand beside the
// others of their columns (283 x 13048 x 5824, behind all others: 60 us, they stream W once more; so 52).
struct lvx_wide_grid_t {
    int32_t full_m, tiles_n, n_large, n_half, group_m;
};
__device__ __forceinline__ bool lvx_wide_tile_of(const lvx_wide_grid_t &g, bool &half, int &row0, int &tn) {
    const int total = g.full_m * g.tiles_n, x = (int)blockIdx.x & 7, y = 7 - x, i = (int)blockIdx.x >> 3;
    const int each_l = g.n_large >> 3, more_l = g.n_large & 7, each_h = g.n_half >> 3, more_h = g.n_half & 7;
    const int mine_l = each_l + (x < more_l ? 1 : 0), mine_h = each_h + (y < more_h ? 1 : 0);
    if (i >= mine_l + mine_h) return false;
    half = i >= mine_l;
    int idx, sel = 0;
    if (!half) {
        idx = x * each_l + (x < more_l ? x : more_l) + i;
    } else {
        const int u = y * each_h + (y < more_h ? y : more_h) + i - mine_l, split = 2 * (total - g.n_large);
        if (g.n_large == 0) {  // halves only: rows of 128 in bands of as many rows, the last ones among them, so that they find their columns of W in L2
            const int rows = g.n_half / g.tiles_n, first = u / (2 * g.group_m * g.tiles_n) * 2 * g.group_m, at = u - first * g.tiles_n;
            const int band = rows - first < 2 * g.group_m ? rows - first : 2 * g.group_m;
            row0 = (first + at % band) * 128;
            tn = at / band;
            return true;
        }
        idx = u < split ? g.n_large + (u >> 1) : total + u - split;
        sel = u < split ? u & 1 : 0;
    }
    if (idx >= total) {
        row0 = g.full_m * 256, tn = idx - total;
        return true;
    }
    const int band = idx / (g.group_m * g.tiles_n), first_m = band * g.group_m;
    const int band_m = g.full_m - first_m < g.group_m ? g.full_m - first_m : g.group_m;
    const int in_band = idx - band * g.group_m * g.tiles_n;
    row0 = (first_m + in_band % band_m) * 256 + sel * 128;
    tn = in_band / band_m;
    return true;
}

// Column of a wave's 16 * FN that row r of its rows of the W tile stands for: a lane's accumulators of two neighbouring 16-column blocks are then
// eight consecutive columns, so outputs and residuals move in 16-byte pieces, four lanes to a 64-byte (fp32: 128-byte) run.  (Three
// blocks: the last one stands alone, four columns a lane.)  Plain fp32 outputs (`by_col`) keep their order: see lvx_gemm_wide_kernel.
template <int FN>
__device__ __forceinline__ int lvx_wide_col(int r, bool by_col) {
    if (by_col || (FN % 2 == 1 && r >= 16 * (FN - 1))) return r;
    return (r >> 5) * 32 + ((r >> 2) & 3) * 8 + ((r >> 4) & 1) * 4 + (r & 3);
}

// Epilogue of 64 rows x 16 * FN columns of a wave.  acc[i][2 h + j][e]: row m0 + 16 i, column n0 + 32 h + 4 j + e (m0, n0 include the lane's l16
// and 8 * q4; an unpaired last block: column n0 - 4 * q4 + 32 h + e).  N is a multiple of 8: eight columns are inside or outside together.
// vec: rows and bases allow 16-byte accesses.  Returns the largest magnitude among the bf16 values that this lane stores (FP8).
template <int EPI, bool FP8, int FN>
__device__ __forceinline__ uint32_t lvx_wide_epilogue(const f32x4_t (&acc)[4][FN], void *Cv, int64_t ldc, const void *Rv, int64_t ldr, const float *__restrict__ gate,
                                                      int M, int N, int m0, int n0, int q4, float alpha, bool vec) {
    constexpr bool RES32 = EPI == LVX_EPI_RESID_GATE_F32, RES16 = EPI == LVX_EPI_RESID_GATE;
    constexpr bool BIAS = EPI == LVX_EPI_BIAS || EPI == LVX_EPI_BIAS_SILU;
    constexpr int NH = (FN + 1) / 2;
    float gt[NH][8];  // gate (residual epilogues) or bias of the lane's columns
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const int nb = n0 + 32 * h - (2 * h + 1 == FN ? 4 * q4 : 0);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int n = nb + e < N ? nb + e : N - 1;
            gt[h][e] = RES32 || RES16 || BIAS ? (gate != nullptr ? gate[n] : BIAS ? 0.f : 1.f) : 0.f;
        }
    }
    uint32_t amax_b = 0;
    float res[2][NH][8];  // residuals of two rows, the next ones on their way while these are used
    auto fetch = [&](int i) {
        if (!RES32 && !RES16) return;
        const int m = m0 + 16 * i < M ? m0 + 16 * i : M - 1;
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const bool four = 2 * h + 1 == FN;
            const int nb = n0 + 32 * h - (four ? 4 * q4 : 0), n = nb < N ? nb : 0;
            if (RES32) {
                const float *r = reinterpret_cast<const float *>(Rv) + (size_t)m * ldr + n;
                if (vec) {
#pragma unroll
                    for (int c = 0; c < (four ? 1 : 2); ++c) {
                        const f32x4_t a = *reinterpret_cast<const f32x4_t *>(r + 4 * c);
#pragma unroll
                        for (int e = 0; e < 4; ++e) res[i & 1][h][4 * c + e] = a[e];
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < (four ? 4 : 8); ++e) res[i & 1][h][e] = r[e];
                }
            } else {
                const bf16_t *r = reinterpret_cast<const bf16_t *>(Rv) + (size_t)m * ldr + n;
                if (vec) {
#pragma unroll
                    for (int c = 0; c < (four ? 1 : 2); ++c) {
                        const uint2 a = *reinterpret_cast<const uint2 *>(r + 4 * c);
                        res[i & 1][h][4 * c] = bf16_lo(a.x), res[i & 1][h][4 * c + 1] = bf16_hi(a.x);
                        res[i & 1][h][4 * c + 2] = bf16_lo(a.y), res[i & 1][h][4 * c + 3] = bf16_hi(a.y);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < (four ? 4 : 8); ++e) res[i & 1][h][e] = bf16_bits_to_f32(r[e]);
                }
            }
        }
    };
    fetch(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i < 3) fetch(i + 1);  // (the rows of one lane do not overlap: reading ahead of the stores below is sound also where C is R)
        const int m = m0 + 16 * i;
        if (m >= M) continue;
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const bool four = 2 * h + 1 == FN;  // the unpaired last block
            const int n = n0 + 32 * h - (four ? 4 * q4 : 0);
            if (n >= N) continue;
            float v[8];
#pragma unroll
            for (int e = 0; e < (four ? 4 : 8); ++e) {
                float x = acc[i][2 * h + (e >> 2)][e & 3];
                if (FP8) x *= alpha;
                if (EPI == LVX_EPI_GELU_TANH) x = gelu_tanh_f32(x);
                if (BIAS) x += gt[h][e];
                if (EPI == LVX_EPI_BIAS_SILU) x = x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
                if (RES32 || RES16) x = res[i & 1][h][e] + gt[h][e] * x;
                v[e] = x;
            }
            if (RES32) {
                float *c = reinterpret_cast<float *>(Cv) + (size_t)m * ldc + n;
                if (vec) {
                    *reinterpret_cast<f32x4_t *>(c) = f32x4_t{v[0], v[1], v[2], v[3]};
                    if (!four) *reinterpret_cast<f32x4_t *>(c + 4) = f32x4_t{v[4], v[5], v[6], v[7]};
                } else {
#pragma unroll
                    for (int e = 0; e < (four ? 4 : 8); ++e) c[e] = v[e];
                }
            } else {
                bf16_t *c = reinterpret_cast<bf16_t *>(Cv) + (size_t)m * ldc + n;
                uint32_t w[4];
#pragma unroll
                for (int e = 0; e < (four ? 2 : 4); ++e) {
                    w[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
                    if (FP8) {
                        const uint32_t lo = w[e] & 0x7fffu, hi = (w[e] >> 16) & 0x7fffu;
                        amax_b = amax_b > lo ? amax_b : lo;
                        amax_b = amax_b > hi ? amax_b : hi;
                    }
                }
                if (vec && four) {
                    *reinterpret_cast<uint2 *>(c) = make_uint2(w[0], w[1]);
                } else if (vec) {
                    *reinterpret_cast<u32x4_t *>(c) = u32x4_t{w[0], w[1], w[2], w[3]};
                } else {
#pragma unroll
                    for (int e = 0; e < (four ? 4 : 8); ++e) c[e] = (bf16_t)(e & 1 ? w[e >> 1] >> 16 : w[e >> 1] & 0xffffu);
                }
            }
        }
    }
    return amax_b;
}

// Sum of squares of the wave's 64 columns of each of its rows (fp32 accumulators), see lvx_gemm_seg_t::sumsq.
__device__ __forceinline__ void lvx_wide_row_sumsq(const f32x4_t (&acc)[4][4], float *out, int64_t ld, int part, int M, int m0, int q4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) ss += acc[i][j][e] * acc[i][j][e];
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        const int m = m0 + 16 * i;
        if (q4 == 0 && m < M) out[(size_t)m * ld + part] = ss;
    }
}

// FN: 16-column blocks per wave, so tiles are 256 x 64 FN (linears: 4).  CONV: the rows of A are gathered from the padded volume.
// By which operand the matrix instruction takes first, a lane's accumulators are four columns of one row, or four rows of one column (by_col): so
// plain fp32 outputs (bf16 products only), which nothing else is read or written beside, leave as 64-byte runs of 16 neighbouring lanes.  As 16-byte
// pieces, 16 rows to a quarter of a wave, they held up short products: 5145 x 1280 x 320 12.5 -> 10.7 us, 1511 x 5920 x 256 15.1 -> 13.0, 234 products
// 0.85 to 1.02 of the time, mean 0.95.
template <int EPI, bool FP8, int FN = 4, bool CONV = false>
__global__ void __launch_bounds__(512) lvx_gemm_wide_kernel(const lvx_gemm_args_t p, const lvx_wide_grid_t g) {
    constexpr int BN = 64 * FN, W_B = BN * 128;           // bytes of a slab's W rows
    constexpr int STAGE_B = 2 * LVX_WIDE_HALF_B + W_B;    // 256 rows: two stages of {A rows 0 .. 127, A rows 128 .. 255, W rows}
    constexpr int STAGE3_B = LVX_WIDE_HALF_B + W_B;       // 128 rows: three stages of {A rows, W rows}
    __shared__ __attribute__((aligned(1024))) char lds[2 * STAGE_B > 3 * STAGE3_B ? 2 * STAGE_B : 3 * STAGE3_B];
    bool half;
    int row0, tn;
    if (!lvx_wide_tile_of(g, half, row0, tn)) return;
    lvx_gemm_out_t o = {p.W, p.C, p.ldc, p.N, EPI, nullptr, 0};
    if (EPI == LVX_EPI_SEGMENTS) o = lvx_gemm_select(p, tn);
    const int M = p.M, N = o.N, col0 = tn * BN;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, q4 = lane >> 4;
    const int wm = wave >> 2, wn = wave & 3;

    // A wave brings two pieces of eight rows of each half of A and FN of W: rows 8 * (wave + 8 q) .. + 7.  The 16-byte chunk c of LDS row r
    // sits at position c ^ ((r >> 1) & 7), as in the other kernels.  Rows and columns past the edge are clamped (never stored).
    uint32_t da[2][2], dw[FN];
#pragma unroll
    for (int q = 0; q < FN; ++q) {
        const int r = 8 * (wave + 8 * q) + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int ra = row0 + h * 128 + r;
            if (ra > M - 1) ra = M - 1;
            if (q < 2) da[h][q] = (uint32_t)((CONV ? lvx_conv_pixel_offset(p.conv, ra) : (size_t)ra * p.lda) + chunk * 16);
        }
        int rw = col0 + r / (16 * FN) * (16 * FN) + lvx_wide_col<FN>(r % (16 * FN), o.epi == LVX_EPI_STORE_F32);
        if (rw > N - 1) rw = N - 1;
        dw[q] = (uint32_t)((size_t)rw * p.ldw + chunk * 16);
    }
    const uint32_t ring_wave = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds + wave * 1024;
    const int last = p.n_slabs - 1, second = last < 1 ? last : 1;  // (a single slab is requested twice: nobody reads the second copy)
    // `off` bytes into the rows of A half h / of W, to LDS offset `at`
    auto load_a = [&](int h, size_t off, int at) {
#pragma unroll
        for (int q = 0; q < 2; ++q) lvx_dma16(p.A + off, da[h][q], ring_wave + (uint32_t)(at + q * 8192));
    };
    auto load_w = [&](size_t off, int at) {
#pragma unroll
        for (int q = 0; q < FN; ++q) lvx_dma16(o.W + off, dw[q], ring_wave + (uint32_t)(at + q * 8192));
    };
    const int swz = (l16 >> 1) & 7;
    const int ch[2] = {(q4 ^ swz) * 16, ((4 + q4) ^ swz) * 16};
    const char *a_rd = lds + (wm * 64 + l16) * 128, *w_rd = lds + (wn * 16 * FN + l16) * 128;
    lvx_frag_t<FP8> a[4], w[FN];
#define LVX_WIDE_READ_A(at_) \
    _Pragma("unroll") for (int k = 0; k < 2; ++k) _Pragma("unroll") for (int i = 0; i < 4; ++i) lvx_frag_read(a[i], k, a_rd + (at_) + i * 2048 + ch[k]);
#define LVX_WIDE_READ_W(at_) \
    _Pragma("unroll") for (int j = 0; j < FN; ++j) _Pragma("unroll") for (int k = 0; k < 2; ++k) lvx_frag_read(w[j], k, w_rd + (at_) + j * 2048 + ch[k]);
    // The matrix phase: the fragments of the memory phase are there before the barrier that hands the partner the LDS ports, so that what
    // the partner loads next may land where they were read from.
#define LVX_WIDE_MATRIX_PHASE(acc_)                                                                                                    \
    {                                                                                                                                  \
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                                                                             \
        asm volatile("s_barrier" ::: "memory");                                                                                        \
        LVX_SCHED_FENCE();                                                                                                             \
        _Pragma("unroll") for (int h = 0; h < FN; h += 2) {                                                                            \
            if constexpr (FP8) {                                                                                                       \
                _Pragma("unroll") for (int i = 0; i < 4; ++i) _Pragma("unroll") for (int j = h; j < h + 2 && j < FN; ++j)              \
                    acc_[i][j] = lvx_mfma_fp8(w[j].v, a[i].v, acc_[i][j]);                                                             \
            } else {                                                                                                                   \
                _Pragma("unroll") for (int k = 0; k < 2; ++k) _Pragma("unroll") for (int i = 0; i < 4; ++i) _Pragma("unroll") for (int j = h; j < h + 2 && j < FN; ++j) \
                    acc_[i][j] = BY_COL ? lvx_mfma_bf16(a[i].h[k], w[j].h[k], acc_[i][j]) : lvx_mfma_bf16(w[j].h[k], a[i].h[k], acc_[i][j]); \
            }                                                                                                                          \
        }                                                                                                                              \
        LVX_SCHED_FENCE();                                                                                                             \
        asm volatile("s_barrier" ::: "memory");                                                                                        \
        LVX_SCHED_FENCE();                                                                                                             \
    }
#define LVX_WIDE_WAIT(n_) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n_) : "memory")
#define LVX_WIDE_ZERO(acc_) \
    _Pragma("unroll") for (int i = 0; i < 4; ++i) _Pragma("unroll") for (int j = 0; j < FN; ++j) acc_[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int m0 = row0 + wm * 64, n0 = col0 + wn * 16 * FN + 8 * q4;
    const float alpha = FP8 ? p.scale_a[0] * p.scale_w[0] : 1.f;
    const bool f32 = EPI == LVX_EPI_RESID_GATE_F32;
    const bool resid = EPI == LVX_EPI_RESID_GATE_F32 || EPI == LVX_EPI_RESID_GATE;
    const bool vec = ((o.ldc | (resid ? p.ldr : 0)) & (f32 ? 3 : 7)) == 0;  // (bases are 16-byte aligned)
    uint32_t amax_b = 0;
    auto finish = [&](auto by_col, const f32x4_t(&acc)[4][FN], int m) {  // m: the first row
        if constexpr (decltype(by_col)::value) {
            const float none[FN] = {};
            lvx_gemm_epilogue<4, FN, LVX_EPI_STORE_F32, FP8>(acc, acc, o.C, o.ldc, nullptr, 0, none, M, N, m + 4 * q4, n0 - 8 * q4 + l16, alpha);
        } else {
            constexpr int E = EPI == LVX_EPI_SEGMENTS ? (int)LVX_EPI_STORE : EPI;
            const uint32_t b = lvx_wide_epilogue<E, FP8, FN>(acc, o.C, o.ldc, p.R, p.ldr, p.gate, M, N, m + l16, n0, q4, alpha, vec);
            amax_b = amax_b > b ? amax_b : b;
            if constexpr (EPI == LVX_EPI_SEGMENTS && FN == 4)
                if (o.sumsq != nullptr && n0 - 8 * q4 < N) lvx_wide_row_sumsq(acc, o.sumsq, o.ld_sumsq, tn * 4 + wn, M, m + l16, q4);
        }
    };
    // where the loop's next slabs lie in the rows of A and W: `near` the next but one of the last requested, `far` the one after it
    lvx_conv_walk_t near, far;
    auto advance = [&]() {
        near = far;
        if (CONV)
            far.next(p.conv);
        else
            far.a += 128, far.w += 128;
    };

    auto work = [&](auto by_col) {
        constexpr bool BY_COL = decltype(by_col)::value;
        if (!half) {
            // Slab t is in stage t % 2.  Two phases a slab: rows 0 .. 127 with W, then rows 128 .. 255.  A place is free once both groups have
            // read it, half a period after its memory phase: the second A half of slab t + 1 is requested in the first memory phase of slab t
            // (its place was last read in the second one of slab t - 1), the rest of slab t + 2 in the second.  So a load has one and a half
            // slabs' time to land.  The last two slabs request nothing and wait for all.
            f32x4_t acc[2][4][FN];
            LVX_WIDE_ZERO(acc[0]);
            LVX_WIDE_ZERO(acc[1]);
            constexpr int A0 = 0, A1 = LVX_WIDE_HALF_B, W0 = 2 * LVX_WIDE_HALF_B;
            load_a(0, near.a, A0), load_w(near.w, W0), load_a(1, near.a, A1);
            if (second > 0) advance();
            load_a(0, far.a, STAGE_B + A0), load_w(far.w, STAGE_B + W0);
            advance();
            LVX_WIDE_WAIT(FN + 4);
            asm volatile("s_barrier" ::: "memory");
            if (wm == 1) asm volatile("s_barrier" ::: "memory");  // this group runs half a period behind
            int st = 0, t = 0;
            auto slab = [&](bool load_first, bool load_second) {
                LVX_WIDE_READ_A(st + A0);
                LVX_WIDE_READ_W(st + W0);
                LVX_SCHED_FENCE();
                if (load_first) {
                    load_a(1, near.a, STAGE_B - st + A1);
                    LVX_WIDE_WAIT(FN + 4);
                } else
                    LVX_WIDE_WAIT(0);
                LVX_WIDE_MATRIX_PHASE(acc[0]);
                LVX_WIDE_READ_A(st + A1);
                LVX_SCHED_FENCE();
                if (load_second) {
                    load_a(0, far.a, st + A0), load_w(far.w, st + W0);
                    LVX_WIDE_WAIT(FN + 4);
                    advance();
                } else
                    LVX_WIDE_WAIT(0);
                LVX_WIDE_MATRIX_PHASE(acc[1]);
                st = STAGE_B - st;
            };
            for (; t + 1 < last; ++t) slab(true, true);
            for (; t <= last; ++t) slab(t < last, false);
            if (wm == 0) asm volatile("s_barrier" ::: "memory");
            finish(by_col, acc[0], m0);
            finish(by_col, acc[1], m0 + 128);
        } else {
            // Slab t is in stage t % 3, one phase a slab; slab t + 2 is requested where slab t - 1 was read a phase ago.
            f32x4_t acc[4][FN];
            LVX_WIDE_ZERO(acc);
            constexpr int A = 0, W0 = LVX_WIDE_HALF_B;
            int cur = 0, nxt = STAGE3_B, nx2 = 2 * STAGE3_B;
            load_a(0, far.a, A), load_w(far.w, W0);
            if (second > 0) advance();
            load_a(0, far.a, nxt + A), load_w(far.w, nxt + W0);
            advance();
            LVX_WIDE_WAIT(FN + 2);
            asm volatile("s_barrier" ::: "memory");
            if (wm == 1) asm volatile("s_barrier" ::: "memory");
            int t = 0;
            auto slab = [&](bool load) {
                LVX_WIDE_READ_A(cur + A);
                LVX_WIDE_READ_W(cur + W0);
                LVX_SCHED_FENCE();
                if (load) {
                    load_a(0, far.a, nx2 + A), load_w(far.w, nx2 + W0);
                    LVX_WIDE_WAIT(FN + 2);
                    advance();
                } else
                    LVX_WIDE_WAIT(0);
                LVX_WIDE_MATRIX_PHASE(acc);
                const int tmp = cur;
                cur = nxt, nxt = nx2, nx2 = tmp;
            };
            for (; t + 1 < last; ++t) slab(true);
            for (; t <= last; ++t) slab(false);
            if (wm == 0) asm volatile("s_barrier" ::: "memory");
            finish(by_col, acc, m0);
        }
    };
    if constexpr (EPI == LVX_EPI_SEGMENTS) {
        if (o.epi == LVX_EPI_STORE_F32)
            work(lvx_bool_t<true>());
        else
            work(lvx_bool_t<false>());
    } else
        work(lvx_bool_t<EPI == LVX_EPI_STORE_F32>());
    if (FP8 && p.amax != nullptr) lvx_amax_publish(amax_b, p.amax, (int)blockIdx.x * 8 + wave, lane);
}

// Launch with n_large whole tiles (arguments checked, p.M > 0, p.segs filled but for tn_begin).
template <int EPI, bool FP8, int FN = 4, bool CONV = false>
static lvx_status_t lvx_gemm_wide_launch(lvx_gemm_args_t &p, int n_large, hipStream_t stream) {
    lvx_wide_grid_t g;
    g.tiles_n = (int)lvx_gemm_col_tiles(&p.segs, p.N, 64 * FN);
    for (int i = 0, t = 0; i < p.segs.n; ++i) p.segs.s[i].tn_begin = t, t += (p.segs.s[i].N + 64 * FN - 1) / (64 * FN);
    g.full_m = lvx_wide_full_rows(p.M);
    g.n_large = n_large;
    g.n_half = (int)lvx_wide_halves(p.M, g.tiles_n, n_large);
    g.group_m = 4;
    const int surplus = n_large % 8 + g.n_half % 8;  // an XCD has both surpluses only if there are more than 8
    const int most = n_large / 8 + g.n_half / 8 + (surplus > 8 ? 2 : surplus > 0 ? 1 : 0);
    hipLaunchKernelGGL((lvx_gemm_wide_kernel<EPI, FP8, FN, CONV>), dim3(8 * most), dim3(512), 0, stream, p, g);
    LVX_CHECK_HIP(hipGetLastError());
    return LVX_OK;
}
