// Implicit GEMM of the 3x3x3 convolution with the three horizontal taps of a slab sharing one set of input rows.
//
// What bounds a convolution tile is how fast its slabs reach LDS, and the rows of tap dx + 1 are the rows of tap dx moved by one
// pixel.  Rows are therefore counted over padded pixels (x runs to W + 1; the two border columns are computed and dropped: 2 / W more
// work), which makes the rows of all three taps BM + 2 consecutive rows: a stage holds those once, and the three taps' weights.  64 x 64:
// 33 KB instead of 48 per three slabs; 192 x 128: 73 KB where 256 x 128 tiles took 108 for the same products.
// K runs (dt, dy, 64 channels, dx); the order of summation is the same for every tile, the 256 x 128 one of lvx_gemm.hip included.
#pragma once
#include "lvx_gemm_core.h"

struct lvx_conv_args_t {
    const char *P, *Wt;
    int64_t ldw;  // bytes
    bf16_t *Y;
    int64_t ldy;
    const float *bias;
    int32_t M, N, n_it, silu;  // M: padded pixels, frames * H * (W + 2); n_it: 9 * slabs_per_tap stages
    int32_t tiles_m, tiles_n, per_xcd, group_m;
    lvx_conv_map_t cm;
};

template <int BM, int BN, int WM, int WN, int NST>
__global__ void __launch_bounds__(64 * WM * WN) lvx_conv_rows_kernel(const lvx_conv_args_t p) {
    constexpr int NW = WM * WN, WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
    constexpr int A_ROWS = BM + 8, STAGE_B = (A_ROWS + 3 * BN) * 128;
    constexpr int A_Q = BM / 8 / NW, W_Q = 3 * BN / 8 / NW, QPW = A_Q + 1 + W_Q;  // direct-to-LDS loads per wave and stage
    static_assert(BM / 8 % NW == 0 && 3 * BN / 8 % NW == 0 && NW == 8, "the loads must divide over the waves");
    __shared__ __attribute__((aligned(1024))) char lds[NST * STAGE_B];

    int tm, tn;
    if (!lvx_gemm_tile_of(p.tiles_m, p.tiles_n, p.per_xcd, p.group_m, tm, tn)) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, q4 = lane >> 4;
    const int wm = wave / WN, wn = wave % WN;
    const int row_px = p.cm.W + 2, frame_px = p.cm.H * row_px;

    // load q of this wave: eight A rows; then one row of the last eight (BM + wave: two of them are read, each wave brings one so that all
    // have the same number of loads in flight); then eight rows of the weights, tap by tap.  Chunk c of row r sits at c ^ ((r >> 1) & 7).
    uint32_t doff[QPW];
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
        const int r8 = q < A_Q ? 8 * (wave + NW * q) : q == A_Q ? BM : 8 * (wave + NW * (q - A_Q - 1));
        const int row_s = r8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row_s >> 1) & 7);
        if (q <= A_Q) {
            int r = tm * BM + row_s;
            if (r > p.M - 1) r = p.M - 1;
            const int t = r / frame_px, rem = r - t * frame_px;
            const int y = rem / row_px, x = rem - y * row_px;
            doff[q] = (uint32_t)(((size_t)t * p.cm.frame_pitch + (size_t)y * p.cm.row_pitch + (size_t)x * p.cm.C) * sizeof(bf16_t)) + chunk * 16;
        } else {
            const int dx = row_s / BN;
            int r = tn * BN + row_s - dx * BN;
            if (r > p.N - 1) r = p.N - 1;
            doff[q] = (uint32_t)((size_t)r * p.ldw + (size_t)dx * p.cm.C * sizeof(bf16_t)) + chunk * 16;
        }
    }
    const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds);
    const bool mine = (lane >> 3) == wave;
    auto issue = [&](int stage, int it) {  // past the end: a harmless reload of the last stage
        it = it < p.n_it - 1 ? it : p.n_it - 1;
        const int tap = it / p.cm.slabs_per_tap, kc = it - tap * p.cm.slabs_per_tap;
        const int dt = tap / 3, dy = tap - dt * 3;
        const char *a = p.P + ((size_t)dt * p.cm.frame_pitch + (size_t)dy * p.cm.row_pitch) * sizeof(bf16_t) + (size_t)kc * 128;
        const char *w = p.Wt + (size_t)tap * 3 * p.cm.C * sizeof(bf16_t) + (size_t)kc * 128;
        const uint32_t at = base + (uint32_t)(stage * STAGE_B);
#pragma unroll
        for (int q = 0; q < A_Q; ++q) lvx_dma16(a, doff[q], at + (uint32_t)((wave + NW * q) * 1024));
        if (mine) lvx_dma16(a, doff[A_Q], at + BM * 128);
#pragma unroll
        for (int q = 0; q < W_Q; ++q) lvx_dma16(w, doff[A_Q + 1 + q], at + (uint32_t)(A_ROWS * 128 + (wave + NW * q) * 1024));
    };
    int a_rd[3][2], w_rd[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) a_rd[dx][h] = (wm * WTM + l16 + dx) * 128 + (((4 * h + q4) ^ (((l16 + dx) >> 1) & 7)) * 16);
        w_rd[h] = A_ROWS * 128 + (wn * WTN + l16) * 128 + (((4 * h + q4) ^ ((l16 >> 1) & 7)) * 16);
    }

    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) issue(s, s);
    int cur = 0, prv = NST - 1;
    for (int t = 0; t < p.n_it; ++t) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * QPW) : "memory");
        __syncthreads();
        LVX_SCHED_FENCE();
        issue(prv, t + NST - 1);
        const char *st = lds + cur * STAGE_B;
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4_t a[FM], b[FN];
#pragma unroll
                for (int j = 0; j < FN; ++j) b[j] = *reinterpret_cast<const u32x4_t *>(st + w_rd[h] + (dx * BN + j * 16) * 128);
#pragma unroll
                for (int i = 0; i < FM; ++i) a[i] = *reinterpret_cast<const u32x4_t *>(st + a_rd[dx][h] + i * 2048);
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) acc[i][j] = lvx_mfma_bf16(a[i], b[j], acc[i][j]);
            }
        }
        prv = cur;
        cur = cur + 1 == NST ? 0 : cur + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load may still be in flight when the LDS is released

    const int m0 = tm * BM + wm * WTM + 4 * q4, n0 = tn * BN + wn * WTN + l16;
    float bias[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) bias[j] = p.bias != nullptr && n0 + j * 16 < p.N ? p.bias[n0 + j * 16] : 0.f;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + i * 16 + e;
            const int row = m / row_px, x = m - row * row_px;
            if (m >= p.M || x >= p.cm.W) continue;
            bf16_t *yp = p.Y + ((size_t)row * p.cm.W + x) * p.ldy + n0;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if (n0 + j * 16 >= p.N) continue;
                float v = acc[i][j][e] + bias[j];
                if (p.silu) v = v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * v));
                yp[j * 16] = (bf16_t)(pack_bf16x2(v, 0.f) & 0xffffu);
            }
        }
}

template <int BM, int BN, int WM, int WN, int NST>
static lvx_status_t lvx_conv_rows_launch(lvx_conv_args_t &p, hipStream_t stream) {
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    p.per_xcd = (p.tiles_m * p.tiles_n + 7) / 8;
    p.group_m = 8;
    hipLaunchKernelGGL((lvx_conv_rows_kernel<BM, BN, WM, WN, NST>), dim3(p.per_xcd * 8), dim3(64 * WM * WN), 0, stream, p);
    LVX_CHECK_HIP(hipGetLastError());
    return LVX_OK;
}
