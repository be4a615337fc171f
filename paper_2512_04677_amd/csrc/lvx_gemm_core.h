// Pieces shared by the GEMM kernels (bf16 and FP8 operands): kernel arguments, epilogue, and the kernel for products that the tiles of
// lvx_gemm_wide.h would leave most of the chip idle with.
//
// A 128-byte piece of a row (64 bf16 or 128 FP8 elements of the contraction) is the unit of everything here: a K slab is one
// such piece of every row of the A and W tiles, an LDS row holds one, a direct-to-LDS wave instruction moves eight.  A lane of
// a 16-row MFMA operand takes the 16-byte chunks q4 and 4 + q4 of its row (q4 = lane / 16).  For bf16 these are the operands of
// two v_mfma_f32_16x16x32_bf16; for FP8 the two together are the 32-byte operand of one v_mfma_f32_16x16x128_f8f6f4 (which
// elements of the contraction a lane holds does not matter as long as A and W agree).  So one data path serves both types.
#pragma once
#include "lvx_internal.h"

typedef __attribute__((__vector_size__(8 * sizeof(int)))) int i32x8_t;

#define LVX_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// One product C[M][N] = epilogue(A W^T), or up to LVX_GEMM_MAX_SEGS of the same A (segs.n > 0: then W, C, ldc and N come from
// the segment table).  lda, ldw in BYTES; ldc, ldr in elements of C / R.
struct lvx_gemm_args_t {
    const char *A, *W;
    int64_t lda, ldw;
    void *C;
    int64_t ldc;
    const void *R;
    int64_t ldr;
    const float *gate;                // gate (residual epilogues) or bias
    const float *scale_a, *scale_w;   // FP8: dequantisation scales (device)
    uint32_t *amax;                   // FP8: where the amax of a bf16 output goes, or NULL
    int32_t M, N, n_slabs, epi;
    int32_t tiles_m, tiles_n, per_xcd, group_m;
    lvx_gemm_segs_t segs;
    lvx_conv_map_t conv;
};

// Convolution: byte offset in the padded volume of output pixel r's tap (0,0,0); and of K slab kt relative to it for the small tiles, which
// walk K tap by tap (the tap's shift plus the slab's channel offset inside the tap: wave-uniform scalar arithmetic).
__device__ __forceinline__ size_t lvx_conv_pixel_offset(const lvx_conv_map_t &cm, int r) {
    const int hw = cm.H * cm.W;
    const int t = r / hw, rem = r - t * hw;
    const int y = rem / cm.W, x = rem - y * cm.W;
    return ((size_t)t * cm.frame_pitch + (size_t)y * cm.row_pitch + (size_t)x * cm.C) * sizeof(bf16_t);
}
__device__ __forceinline__ size_t lvx_conv_slab_offset(const lvx_conv_map_t &cm, int kt) {
    const int tap = kt / cm.slabs_per_tap, kc = kt - tap * cm.slabs_per_tap;
    const int dt = tap / 9, dy = (tap - dt * 9) / 3, dx = tap - dt * 9 - dy * 3;
    return ((size_t)dt * cm.frame_pitch + (size_t)dy * cm.row_pitch + (size_t)dx * cm.C) * sizeof(bf16_t) + (size_t)kc * 128;
}

// The walk of the 256 x 128 tiles, slab after slab: K runs (dt, dy, 64 channels, dx), the order of the tiles with shared input rows, so
// that the steps of one layer may take either.  a: byte offset in the volume, as above; w: in a row of the weights.
struct lvx_conv_walk_t {
    size_t a = 0, w = 0;
    int dx = 0, kc = 0, dy = 0;
    __device__ __forceinline__ void next(const lvx_conv_map_t &cm) {
        const int64_t tap = (int64_t)cm.C * (int)sizeof(bf16_t), row = (int64_t)cm.row_pitch * (int)sizeof(bf16_t), frame = (int64_t)cm.frame_pitch * (int)sizeof(bf16_t);
        if (++dx < 3) {
            a += tap, w += tap;
        } else if (dx = 0, ++kc < cm.slabs_per_tap) {
            a += 128 - 2 * tap, w += 128 - 2 * tap;
        } else {  // from the last 64 channels of tap dx = 2 to the first of the next line's dx = 0
            kc = 0;
            a += 128 - 3 * tap + row, w += 128;
            if (++dy == 3) dy = 0, a += frame - 3 * row;
        }
    }
};

// One MFMA operand fragment: the two 16-byte chunks of a lane's row.
template <bool FP8>
struct lvx_frag_t;
template <>
struct lvx_frag_t<false> {
    u32x4_t h[2];
};
template <>
struct lvx_frag_t<true> {
    i32x8_t v;
};
__device__ __forceinline__ void lvx_frag_read(lvx_frag_t<false> &f, int half, const char *p) { f.h[half] = *reinterpret_cast<const u32x4_t *>(p); }
__device__ __forceinline__ void lvx_frag_read(lvx_frag_t<true> &f, int half, const char *p) {
    const u32x4_t v = *reinterpret_cast<const u32x4_t *>(p);
#pragma unroll
    for (int e = 0; e < 4; ++e) f.v[4 * half + e] = (int)v[e];
}
__device__ __forceinline__ f32x4_t lvx_mfma_bf16(u32x4_t a, u32x4_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4_t lvx_mfma_fp8(i32x8_t a, i32x8_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
}

// Workgroup -> tile.  Workgroup ids are dealt to the XCDs round-robin by hardware; each XCD gets a contiguous range of tiles,
// walked column-major inside bands of group_m row tiles, so the workgroups running together on one XCD share A and W slabs in
// that XCD's L2.  False: no tile for this workgroup (the grid is rounded up to whole XCD rows).
__device__ __forceinline__ bool lvx_gemm_tile_of(int tiles_m, int tiles_n, int per_xcd, int group_m, int &tm, int &tn) {
    const int widx = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (widx >= tiles_m * tiles_n) return false;
    const int band = widx / (group_m * tiles_n);
    const int first_m = band * group_m;
    const int band_m = tiles_m - first_m < group_m ? tiles_m - first_m : group_m;
    const int in_band = widx - band * group_m * tiles_n;
    tm = first_m + in_band % band_m;
    tn = in_band / band_m;
    return true;
}

// The workgroup's product: the plain one, or the segment its column tile lies in (workgroup-uniform).
struct lvx_gemm_out_t {
    const char *W;
    void *C;
    int64_t ldc;
    int N, epi;
    float *sumsq;
    int ld_sumsq;
};
__device__ __forceinline__ lvx_gemm_out_t lvx_gemm_select(const lvx_gemm_args_t &p, int &tn) {
    lvx_gemm_out_t o = {p.W, p.C, p.ldc, p.N, p.epi, nullptr, 0};
    if (p.segs.n > 0) {
        int sg = 0;
        for (int i = 1; i < p.segs.n; ++i)
            if (tn >= p.segs.s[i].tn_begin) sg = i;
        tn -= p.segs.s[sg].tn_begin;
        o.W = reinterpret_cast<const char *>(p.segs.s[sg].W);
        o.C = p.segs.s[sg].C;
        o.ldc = p.segs.s[sg].ldc;
        o.N = p.segs.s[sg].N;
        o.epi = p.segs.s[sg].f32 != 0 ? LVX_EPI_STORE_F32 : LVX_EPI_STORE;
        o.sumsq = p.segs.s[sg].sumsq;
        o.ld_sumsq = p.segs.s[sg].ld_sumsq;
    }
    return o;
}

// Per column block the gate (residual epilogues; 1 without one) or the bias (0) of this lane's column.
template <int FN>
__device__ __forceinline__ void lvx_gemm_gates(float (&gt)[FN], int epi, const float *__restrict__ gate, int N, int n0) {
    const bool resid = epi == LVX_EPI_RESID_GATE || epi == LVX_EPI_RESID_GATE_F32, bias = epi == LVX_EPI_BIAS || epi == LVX_EPI_BIAS_SILU;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int n = n0 + j * 16 < N ? n0 + j * 16 : N - 1;
        gt[j] = resid ? 1.f : 0.f;
        if ((resid || bias) && gate != nullptr) gt[j] = gate[n];
    }
}

// Epilogue.  Accumulator register e of 16 x 16 block (i,j) holds row m0 + 16i + e and column n0 + 16j of C (m0, n0 already
// include the lane's 4*q4 / l16 offsets): for a fixed register, each group of 16 lanes writes 16 consecutive columns of one
// row.  Rows outermost, column blocks innermost, so neighbouring 32-byte (fp32: 64-byte) runs of a cache line reach L2
// together.  Interior tiles take the branch-free path; only tiles on the M or N edge check every element.
// rres: the fp32 residual, fetched before the main loop; a bf16 one is read here, that of several blocks before the first store, which
// the compiler would not read past (64 x 64 tiles, 1663 x 376 x 2944 15.8 -> 13.0 us; 64 x 128, 651 x 1624 x 1792 10.9 -> 9.5); gt: lvx_gemm_gates.
// Returns the largest magnitude (bit pattern without sign) among the bf16 values this lane stores, for FP8 products that feed another one.
template <int FM, int FN, int EPI, bool FP8>
__device__ __forceinline__ uint32_t lvx_gemm_epilogue(const f32x4_t (&acc)[FM][FN], const f32x4_t (&rres)[FM][FN], void *Cv, int64_t ldc, const void *Rv,
                                                      int64_t ldr, const float (&gt)[FN], int M, int N, int m0, int n0, float alpha) {
    const bool interior = (m0 - (m0 & 12) + FM * 16 <= M) && (n0 - (n0 & 15) + FN * 16 <= N);
    uint32_t amax_b = 0;
    constexpr bool RES16 = EPI == LVX_EPI_RESID_GATE, BATCH = RES16 && FM * FN > 1;
    float res16[FM][FN][4];
    if (BATCH) {
        int mr = m0, nr = n0;
        asm volatile("" : "+v"(mr), "+v"(nr));  // addresses of their own: shared with the fp32 residual's they are formed ahead of every product's first loads
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = mr + i * 16 + e < M ? mr + i * 16 + e : M - 1;
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    res16[i][j][e] = bf16_bits_to_f32(reinterpret_cast<const bf16_t *>(Rv)[(size_t)m * ldr + (nr + j * 16 < N ? nr + j * 16 : N - 1)]);
            }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + i * 16 + e;
            if (!interior && m >= M) continue;
            bf16_t *cp = reinterpret_cast<bf16_t *>(Cv) + (size_t)m * ldc + n0;
            float *cpf = reinterpret_cast<float *>(Cv) + (size_t)m * ldc + n0;
            const bf16_t *rp = reinterpret_cast<const bf16_t *>(Rv) + (size_t)m * ldr + n0;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if (!interior && n0 + j * 16 >= N) continue;
                float v = acc[i][j][e];
                if (FP8) v *= alpha;
                if (EPI == LVX_EPI_GELU_TANH) v = gelu_tanh_f32(v);
                if (EPI == LVX_EPI_BIAS || EPI == LVX_EPI_BIAS_SILU) v += gt[j];
                if (EPI == LVX_EPI_BIAS_SILU) v = v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * v));
                if (RES16) v = (BATCH ? res16[i][j][e] : bf16_bits_to_f32(rp[j * 16])) + gt[j] * v;
                if (EPI == LVX_EPI_RESID_GATE_F32)
                    cpf[j * 16] = rres[i][j][e] + gt[j] * v;
                else if (EPI == LVX_EPI_STORE_F32)
                    cpf[j * 16] = v;
                else {
                    const uint32_t b = pack_bf16x2(v, 0.f) & 0xffffu;
                    cp[j * 16] = (bf16_t)b;
                    if (FP8) amax_b = amax_b > (b & 0x7fffu) ? amax_b : (b & 0x7fffu);
                }
            }
        }
    }
    return amax_b;
}

// The same with the epilogue chosen at run time (one uniform branch after the main loop: one kernel per tile and type instead of
// one per epilogue as well).
template <int FM, int FN, bool FP8>
__device__ __forceinline__ uint32_t lvx_gemm_epilogue_any(int epi, const f32x4_t (&acc)[FM][FN], const f32x4_t (&rres)[FM][FN], void *C, int64_t ldc,
                                                          const void *R, int64_t ldr, const float (&gt)[FN], int M, int N, int m0, int n0, float alpha) {
#define LVX_EPI_CASE(E_) \
    case E_: return lvx_gemm_epilogue<FM, FN, E_, FP8>(acc, rres, C, ldc, R, ldr, gt, M, N, m0, n0, alpha);
    switch (epi) {
        LVX_EPI_CASE(LVX_EPI_GELU_TANH)
        LVX_EPI_CASE(LVX_EPI_RESID_GATE)
        LVX_EPI_CASE(LVX_EPI_RESID_GATE_F32)
        LVX_EPI_CASE(LVX_EPI_BIAS)
        LVX_EPI_CASE(LVX_EPI_BIAS_SILU)
        LVX_EPI_CASE(LVX_EPI_STORE_F32)
        default: return lvx_gemm_epilogue<FM, FN, LVX_EPI_STORE, FP8>(acc, rres, C, ldc, R, ldr, gt, M, N, m0, n0, alpha);
    }
#undef LVX_EPI_CASE
}

// Sum of squares of FN * 16 columns for each of a wave's rows (fp32 accumulators), one float per row at out[m * ld + part].
template <int FM, int FN>
__device__ __forceinline__ void lvx_gemm_row_sumsq(const f32x4_t (&acc)[FM][FN], float *out, int64_t ld, int part, int M, int m0, int l16) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float ss = 0.f;
#pragma unroll
            for (int j = 0; j < FN; ++j) ss += acc[i][j][e] * acc[i][j][e];
            ss += __shfl_xor(ss, 1);
            ss += __shfl_xor(ss, 2);
            ss += __shfl_xor(ss, 4);
            ss += __shfl_xor(ss, 8);
            const int m = m0 + i * 16 + e;
            if (l16 == 0 && m < M) out[(size_t)m * ld + part] = ss;
        }
}

// FP8: one atomic per wave hands the largest magnitude it stored to the next linear's quantisation.
__device__ __forceinline__ void lvx_amax_publish(uint32_t amax_b, uint32_t *slots, int slot, int lane) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)amax_b, s);
        amax_b = amax_b > o ? amax_b : o;
    }
    if (lane == 0 && amax_b != 0) atomicMax(slots + (slot & (LVX_AMAX_SLOTS - 1)), amax_b << 16);
}

// Waits until the loads of a wave's current slab have landed: QPW of each of the `ahead` slabs requested behind it, at most MAX, may be in flight.
template <int MAX, int QPW>
__device__ __forceinline__ void lvx_wait_slab(int ahead) {
    if constexpr (MAX > 0) {
        if (ahead < MAX) return lvx_wait_slab<MAX - 1, QPW>(ahead);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAX * QPW) : "memory");
}

// ---- small tiles ---------------------------------------------------------------------------------------------------------------
// What bounds a product with few rows is how fast a compute unit can pull slabs out of L2 and HBM (about 50 bytes a nanosecond
// with its LDS full of loads in flight, whatever the tile), so the tile is chosen to have as many compute units pull as there
// are, each as few bytes as possible: NST stages of one slab each keep NST - 1 slabs in flight, KG groups of WM x WN waves work
// on different slabs of the same tile (slab t belongs to group t % KG, each group has a ring of its own; the accumulators meet in LDS at
// the end, in a fixed order), which is how a 32 x 32 tile still has four slabs' loads and four MFMA chains going at once.
// Per slab and group: wait for its slab, one barrier, issue the load NST - 1 slabs ahead into the stage just released, multiply.
// Measured (microseconds, weights read from HBM; before: a kernel of 128 x 256 tiles): 64 x 1920 x 6144 77 -> 16.5 (32 x 32, four
// groups), 64 x 5760 x 1920 28 -> 10 (32 x 64, two groups), 256 x 2560 x 6912 95 -> 32 (64 x 64), 1170 x 1536 x 6144 69 -> 38
// (64 x 128), the same shapes in FP8 40 -> 9.7, 16 -> 6.8, 50 -> 18, 38 -> 20.
// Only slabs that exist are requested, and the residual and the gate or bias before the first of them: a short K is a chain of latencies, and
// re-requests of the last slab (up to 5 loads for 2 slabs) and reads at its end were half a microsecond of each product of a 105-token stage
// (the stage 255 -> 246 us); 1170 x 1536 x 6144 with the residual 33.4 -> 32.5.
template <int BM, int BN, int WM, int WN, int NST, int KG, bool FP8, bool CONV>
__global__ void __launch_bounds__(64 * WM * WN * KG) lvx_gemm_tile_kernel(const lvx_gemm_args_t p) {
    constexpr int NW = WM * WN, WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
    constexpr int STAGE_B = (BM + BN) * 128;
    constexpr int QPW = (BM + BN) / 8 / NW, A_Q = BM / 8 / NW;  // direct-to-LDS loads per wave and slab, the first A_Q of them A rows
    static_assert((BM + BN) / 8 % NW == 0 && BM / 8 % NW == 0, "the loads must divide over the waves, A and W separately");
    static_assert(KG == 1 || BM * BN * 4 <= NST * STAGE_B, "the groups' accumulators meet in the stages' LDS");
    __shared__ __attribute__((aligned(1024))) char lds[KG * NST * STAGE_B];

    int tm, tn;
    if (!lvx_gemm_tile_of(p.tiles_m, p.tiles_n, p.per_xcd, p.group_m, tm, tn)) return;
    const lvx_gemm_out_t o = lvx_gemm_select(p, tn);
    const int M = p.M, N = o.N, n_slabs = p.n_slabs;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, l16 = lane & 15, q4 = lane >> 4;
    const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(wv / NW), wave = wv % NW;
    const int wm = wave / WN, wn = wave % WN;
    char *ring = lds + kg * NST * STAGE_B;

    // load q of this wave covers stage rows 8 * (wave + NW q) .. + 7, A rows first; 16-byte chunk c of row r sits at position
    // c ^ ((r >> 1) & 7), so that 16 consecutive rows read at one chunk hit 16 distinct 16-byte units of the bank row
    uint32_t doff[QPW];
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
        const int row_s = 8 * (wave + NW * q) + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row_s >> 1) & 7);
        if (q < A_Q) {
            int r = tm * BM + row_s;
            if (r > M - 1) r = M - 1;
            doff[q] = (uint32_t)((CONV ? lvx_conv_pixel_offset(p.conv, r) : (size_t)r * p.lda) + chunk * 16);
        } else {
            int r = tn * BN + row_s - BM;
            if (r > N - 1) r = N - 1;
            doff[q] = (uint32_t)((size_t)r * p.ldw + chunk * 16);
        }
    }
    const uint32_t ring_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)ring + wave * 1024);
    auto issue = [&](int stage, int it) {  // the group's it-th slab
        const int kt = it * KG + kg;
        const size_t a_off = CONV ? lvx_conv_slab_offset(p.conv, kt) : (size_t)kt * 128;
#pragma unroll
        for (int q = 0; q < QPW; ++q)
            lvx_dma16(q < A_Q ? p.A + a_off : o.W + (size_t)kt * 128, doff[q], ring_wave + (uint32_t)(stage * STAGE_B + q * NW * 1024));
    };
    const int swz = (l16 >> 1) & 7;
    const char *a_rd = ring + (wm * WTM + l16) * 128, *w_rd = ring + BM * 128 + (wn * WTN + l16) * 128;
    const int ch[2] = {(q4 ^ swz) * 16, ((4 + q4) ^ swz) * 16};

    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int m0 = tm * BM + wm * WTM + 4 * q4, n0 = tn * BN + wn * WTN + l16;
    // what the end needs besides the product is on its way before the first slab: the blocks that this wave stores (all of its own, with K
    // groups block kg of its wave position)
    constexpr int SM = KG == 1 ? FM : 1, SN = KG == 1 ? FN : 1;
    static_assert(KG == 1 || FM * FN <= KG, "a wave stores one block at most");
    const int sm0 = KG == 1 ? m0 : m0 + kg / FN * 16, sn0 = KG == 1 ? n0 : n0 + kg % FN * 16;
    const bool stores = KG == 1 || kg < FM * FN;
    f32x4_t rres[SM][SN];
    float gt[SN];
    if (stores) {
        lvx_gemm_gates<SN>(gt, o.epi, p.gate, N, sn0);
        if (o.epi == LVX_EPI_RESID_GATE_F32) {
            const float *R = reinterpret_cast<const float *>(p.R);
#pragma unroll
            for (int i = 0; i < SM; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = sm0 + i * 16 + e < M ? sm0 + i * 16 + e : M - 1;
#pragma unroll
                    for (int j = 0; j < SN; ++j) rres[i][j][e] = R[(size_t)row * p.ldr + (sn0 + j * 16 < N ? sn0 + j * 16 : N - 1)];
                }
        }
    }
    const float scale_a = FP8 ? p.scale_a[0] : 1.f, scale_w = FP8 ? p.scale_w[0] : 1.f;
    const int n_mine = KG == 1 ? n_slabs : (n_slabs - kg + KG - 1) / KG;  // the group's slabs
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
        if (s < n_mine) issue(s, s);
    int cur = 0, prv = NST - 1, t = 0;
    auto multiply = [&]() {
        lvx_frag_t<FP8> a[FM], b[FN];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < FN; ++j) lvx_frag_read(b[j], h, w_rd + cur * STAGE_B + j * 2048 + ch[h]);
#pragma unroll
            for (int i = 0; i < FM; ++i) lvx_frag_read(a[i], h, a_rd + cur * STAGE_B + i * 2048 + ch[h]);
        }
        if constexpr (FP8) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = lvx_mfma_fp8(a[i].v, b[j].v, acc[i][j]);
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) acc[i][j] = lvx_mfma_bf16(a[i].h[h], b[j].h[h], acc[i][j]);
        }
        prv = cur;
        cur = cur + 1 == NST ? 0 : cur + 1;
    };
    for (; t + NST - 1 < n_mine; ++t) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * QPW) : "memory");
        __syncthreads();
        LVX_SCHED_FENCE();
        issue(prv, t + NST - 1);
        multiply();
    }
    // the last slabs, all requested by now, in a loop of their own (in the one above its conditions cost long products 5 to 10 %); every group
    // passes the same number of barriers
    const int n_it = (n_slabs + KG - 1) / KG;
    for (; t < n_it; ++t) {
        lvx_wait_slab<NST - 2, QPW>(n_mine - 1 - t);
        __syncthreads();
        LVX_SCHED_FENCE();
        if (KG == 1 || t < n_mine) multiply();
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load may still be in flight when the LDS is reused or released

    const float alpha = scale_a * scale_w;
    uint32_t amax_b = 0;
    if constexpr (KG == 1) {
        amax_b = lvx_gemm_epilogue_any<FM, FN, FP8>(o.epi, acc, rres, o.C, o.ldc, p.R, p.ldr, gt, M, N, m0, n0, alpha);
        if (o.sumsq != nullptr && n0 - l16 < N) lvx_gemm_row_sumsq<FM, FN>(acc, o.sumsq, o.ld_sumsq, (tn * BN + wn * WTN) / WTN, M, m0, l16);
    } else {
        // the groups' partial sums, added in the order of the groups; the 16 x 16 blocks of a wave position are dealt to its KG waves
        constexpr int PER = FM * FN;
        float *red = reinterpret_cast<float *>(lds);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) *reinterpret_cast<f32x4_t *>(red + ((((kg * NW + wave) * FM + i) * FN + j) * 64 + lane) * 4) = acc[i][j];
        __syncthreads();
        if (stores) {
            f32x4_t v[1][1];
            v[0][0] = *reinterpret_cast<const f32x4_t *>(red + ((wave * PER + kg) * 64 + lane) * 4);
#pragma unroll
            for (int g = 1; g < KG; ++g) v[0][0] += *reinterpret_cast<const f32x4_t *>(red + (((g * NW + wave) * PER + kg) * 64 + lane) * 4);
            amax_b = lvx_gemm_epilogue_any<1, 1, FP8>(o.epi, v, rres, o.C, o.ldc, p.R, p.ldr, gt, M, N, sm0, sn0, alpha);
            if (o.sumsq != nullptr && sn0 - l16 < N) lvx_gemm_row_sumsq<1, 1>(v, o.sumsq, o.ld_sumsq, (sn0 - l16) / 16, M, sm0, l16);
        }
    }
    if (FP8 && p.amax != nullptr) lvx_amax_publish(amax_b, p.amax, (int)blockIdx.x * NW * KG + wv, lane);
}

// Launch of small tile `tile` (arguments checked, p.M > 0, p.segs filled but for tn_begin).
template <bool FP8, bool CONV = false>
static lvx_status_t lvx_gemm_launch_small(int tile, lvx_gemm_args_t &p, hipStream_t stream) {
#define LVX_TILE_LAUNCH(ID_, BM_, BN_, WM_, WN_, NST_, KG_, PC_, US_)                                                                  \
    case ID_: {                                                                                                                         \
        p.tiles_m = (p.M + BM_ - 1) / BM_;                                                                                              \
        p.tiles_n = (int)lvx_gemm_col_tiles(&p.segs, p.N, BN_);                                                                         \
        for (int i = 0, t = 0; i < p.segs.n; ++i) p.segs.s[i].tn_begin = t, t += (p.segs.s[i].N + BN_ - 1) / BN_;                       \
        p.per_xcd = (p.tiles_m * p.tiles_n + 7) / 8;                                                                                    \
        p.group_m = 8;                                                                                                                  \
        if constexpr (!CONV || KG_ > 2)  /* convolutions have tiles of their own above the smallest */                                 \
            hipLaunchKernelGGL((lvx_gemm_tile_kernel<BM_, BN_, WM_, WN_, NST_, KG_, FP8, CONV>), dim3(p.per_xcd * 8), dim3(64 * WM_ * WN_ * KG_), 0, stream, p); \
        break;                                                                                                                          \
    }
    switch (tile) { LVX_GEMM_SMALL_TILES(LVX_TILE_LAUNCH) }
#undef LVX_TILE_LAUNCH
    LVX_CHECK_HIP(hipGetLastError());
    return LVX_OK;
}
