// Token-major keys and values -> the cache's packed form (see lvx_cache.hip), one tile per workgroup.
#pragma once
#include "lvx_internal.h"

// 256 threads = one head x one 64-key tile of the destination.  Copies the rows of K that fall into the tile (k NULL: values only)
// and writes the matching part of the transposed V tile (through LDS).  Only keys in [key0, key0+n) are touched: a tile
// shared with a neighbouring slot keeps the neighbour's keys.
template <int D>
__device__ __forceinline__ void lvx_pack_tile(const bf16_t *__restrict__ k, const bf16_t *__restrict__ v, int64_t ld, int n, int cap, int key0, int tile,
                                              int h, bf16_t *__restrict__ kp, bf16_t *__restrict__ vtp) {
    constexpr int KT = LVX_KEY_TILE;
    constexpr int CPR = D / 8;        // 16-byte chunks per row
    constexpr int LDS_LD = D + 8;     // padded row, keeps 16-byte alignment
    __shared__ __attribute__((aligned(16))) bf16_t vs[KT * LDS_LD];

    const int tid = threadIdx.x;
    const int key_lo = tile * KT;
    const int n_tiles = cap / KT;

    for (int g = tid; g < KT * CPR; g += 256) {
        const int r = g / CPR, c = g % CPR;
        const int key = key_lo + r;
        const int src = key - key0;
        uint4 val = make_uint4(0, 0, 0, 0);
        if (src >= 0 && src < n) {
            const size_t so = (size_t)src * ld + (size_t)h * D + c * 8;
            if (k != nullptr) *reinterpret_cast<uint4 *>(kp + ((size_t)h * cap + key) * D + c * 8) = *reinterpret_cast<const uint4 *>(k + so);
            val = *reinterpret_cast<const uint4 *>(v + so);
        }
        *reinterpret_cast<uint4 *>(&vs[r * LDS_LD + c * 8]) = val;
    }
    __syncthreads();
    bf16_t *vt_tile = vtp + ((size_t)h * n_tiles + tile) * (size_t)D * KT;
    for (int g = tid; g < D * (KT / 8); g += 256) {
        const int d = g / (KT / 8), kc = g % (KT / 8);
        const int lo = key_lo + kc * 8 - key0;  // source index of the first of 8 keys
        if (lo + 7 < 0 || lo >= n) continue;
        bf16_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = vs[(kc * 8 + j) * LDS_LD + d];
        bf16_t *dst = vt_tile + (size_t)d * KT + kc * 8;
        if (lo >= 0 && lo + 7 < n) {
            uint4 o;
            o.x = e[0] | ((uint32_t)e[1] << 16);
            o.y = e[2] | ((uint32_t)e[3] << 16);
            o.z = e[4] | ((uint32_t)e[5] << 16);
            o.w = e[6] | ((uint32_t)e[7] << 16);
            *reinterpret_cast<uint4 *>(dst) = o;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (lo + j >= 0 && lo + j < n) dst[j] = e[j];
        }
    }
}

// Values to transpose beside another kernel's work (K goes elsewhere): the workgroups of a launch that do it, tile by tile, head by
// head, row set by row set.
struct lvx_pack_job_t {
    const bf16_t *v;
    bf16_t *vtp;
    int64_t ld, batch_stride_src, batch_stride_dst;
    int32_t n, cap, key0, tile0, n_tiles, H, n_batch;
};
static inline lvx_pack_job_t lvx_pack_job(const bf16_t *v, int64_t ld, int n, int H, int cap, int key0, bf16_t *vt_packed, int n_batch = 1,
                                          int64_t batch_stride_src = 0, int64_t batch_stride_dst = 0) {
    const int tile0 = key0 / LVX_KEY_TILE, tile1 = (key0 + n - 1) / LVX_KEY_TILE;
    return {v, vt_packed, ld, batch_stride_src, batch_stride_dst, n, cap, key0, tile0, tile1 - tile0 + 1, H, n_batch};
}
template <int D>
__device__ __forceinline__ void lvx_pack_job_tile(const lvx_pack_job_t &p, int idx) {
    if (idx >= p.n_tiles * p.H * p.n_batch) return;
    const int t = idx % p.n_tiles, h = idx / p.n_tiles % p.H, b = idx / (p.n_tiles * p.H);
    lvx_pack_tile<D>(nullptr, p.v + (size_t)b * p.batch_stride_src, p.ld, p.n, p.cap, p.key0, p.tile0 + t, h, nullptr, p.vtp + (size_t)b * p.batch_stride_dst);
}
