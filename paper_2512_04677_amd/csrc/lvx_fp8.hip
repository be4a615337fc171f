// FP8 (E4M3) linears with per-tensor dynamic scaling (paper Appendix C, "FP8 Quantization": every linear projection of the
// DiT takes FP8 operands; embeddings and heads, which are outside the stage, do not).
//
//   amax   = max |x| over the whole tensor                                   (lvx_fp8_amax_kernel, atomic max on the bit pattern)
//   code   = E4M3(x * (448 / amax)), round to nearest even, saturating       (lvx_fp8_quant_kernel, v_cvt_pk_fp8_f32)
//   C      = (amax_a / 448) * (amax_w / 448) * (code_a . code_w)             (lvx_gemm_wide_kernel and lvx_gemm_tile_kernel, fp32 accumulate)
//
// The two scale factors and the product x * (448/amax) are formed in fp32: that product is what decides the 8-bit code.
// gfx950 converts to and multiplies the OCP form of E4M3 (bias 7, largest finite value 448, no infinities).
//
// The products run on the kernels of the bf16 linears with one-byte elements: a slab of the contraction is again 128 bytes of a row, 128 elements,
// and v_mfma_f32_16x16x128_f8f6f4 multiplies them at twice the bf16 rate (the older 32x32x16 fp8 form runs at the bf16 rate on this chip).
#include "lvx_gemm_wide.h"

#include <mutex>

// Scratch of lvx_fp8_quantize_static: the amax slot array that lvx_fp8_quantize takes from its caller, here owned by the
// library.  One copy per GPU the library runs on, resident until the process ends.  In host code this name only stands for
// the symbol: the device address is resolved per device with hipGetSymbolAddress (static_scratch() below) and only that
// pointer is ever handed to a kernel.
static __device__ __align__(256) uint32_t scratch[LVX_AMAX_SLOTS];

namespace {

constexpr float E4M3_MAX = 448.0f;

constexpr int MAX_DEVICES = 64;
uint32_t *g_scratch_ptr[MAX_DEVICES];  // device address of `scratch` on each device, resolved on first use
std::mutex g_scratch_mutex;

// Device address of this device's copy of `scratch`.  No allocation: the array is part of the code object's data.
lvx_status_t static_scratch(uint32_t **out) {
    int dev = -1;
    LVX_CHECK_HIP(hipGetDevice(&dev));
    LVX_REQUIRE(dev >= 0 && dev < MAX_DEVICES, LVX_ERR_UNSUPPORTED, "device ordinal %d outside [0,%d)", dev, MAX_DEVICES);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void *p = nullptr;
        LVX_CHECK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        LVX_REQUIRE(p != nullptr && (((uintptr_t)p) & 255u) == 0, LVX_ERR_HIP, "address of the static scratch array is NULL or misaligned");
        g_scratch_ptr[dev] = (uint32_t *)p;
    }
    *out = g_scratch_ptr[dev];
    return LVX_OK;
}

// ---- quantisation ---------------------------------------------------------------------------------------------------
// amax_slots: LVX_AMAX_SLOTS fp32 bit patterns whose maximum is max|x| (non-negative floats order like their bit patterns),
// zeroed before the producers run.  Producers spread their atomic maxima over the slots (thousands of atomics on ONE address
// would serialise in L2 and cost more than the pass itself); the quantisation kernel reduces the slots.
__global__ void __launch_bounds__(256) lvx_fp8_amax_kernel(const bf16_t *__restrict__ x, int64_t ld, int rows, int chunks_per_row,
                                                           uint32_t *amax_slots) {
    const size_t total = (size_t)rows * chunks_per_row;
    uint32_t m = 0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        const size_t r = i / chunks_per_row, c = i % chunks_per_row;
        const uint4 v = reinterpret_cast<const uint4 *>(x + r * ld)[c];
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t lo = w[e] & 0x7fffu, hi = (w[e] >> 16) & 0x7fffu;
            m = m > lo ? m : lo;
            m = m > hi ? m : hi;
        }
    }
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)m, s);
        m = m > o ? m : o;
    }
    __shared__ uint32_t wave_max[4];
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        m = wave_max[0];
#pragma unroll
        for (int w = 1; w < 4; ++w) m = m > wave_max[w] ? m : wave_max[w];
        if (m != 0) atomicMax(amax_slots + (blockIdx.x & (LVX_AMAX_SLOTS - 1)), m << 16);
    }
}

// 16 bf16 -> 16 codes per thread; also publishes the dequantisation scale amax/448 (1 for an all-zero tensor)
// zero_slots (may be NULL): another slot array, not in use by any kernel in flight, that this kernel clears for the next
// producer (the arrays alternate, so no separate clearing launch is needed between quantisations).
__global__ void __launch_bounds__(256) lvx_fp8_quant_kernel(const bf16_t *__restrict__ x, int64_t ld, int rows, int chunks_per_row,
                                                            const uint32_t *__restrict__ amax_slots, uint32_t *__restrict__ zero_slots,
                                                            uint8_t *__restrict__ q, int64_t ldq, float *__restrict__ scale_out) {
    uint32_t mb = amax_slots[threadIdx.x & (LVX_AMAX_SLOTS - 1)];
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)mb, s);
        mb = mb > o ? mb : o;
    }
    if (zero_slots != nullptr && blockIdx.x == 0 && threadIdx.x < LVX_AMAX_SLOTS) zero_slots[threadIdx.x] = 0;
    const float amax = __uint_as_float(mb);
    const float inv = amax > 0.f ? E4M3_MAX / amax : 0.f;
    if (blockIdx.x == 0 && threadIdx.x == 0) *scale_out = amax > 0.f ? amax / E4M3_MAX : 1.0f;
    const size_t total = (size_t)rows * chunks_per_row;  // chunks of 16 elements
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        const size_t r = i / chunks_per_row, c = i % chunks_per_row;
        const uint4 *src = reinterpret_cast<const uint4 *>(x + r * ld) + 2 * c;
        const uint4 v0 = src[0], v1 = src[1];
        const uint32_t w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // |x * inv| <= 448 (1 + 2^-23): far below the midpoint to the next (non-existent) grid value, the clamp only
            // guards the conversion's out-of-range behaviour
            float a = fminf(fmaxf(bf16_lo(w[2 * e]) * inv, -E4M3_MAX), E4M3_MAX);
            float b = fminf(fmaxf(bf16_hi(w[2 * e]) * inv, -E4M3_MAX), E4M3_MAX);
            float c2 = fminf(fmaxf(bf16_lo(w[2 * e + 1]) * inv, -E4M3_MAX), E4M3_MAX);
            float d = fminf(fmaxf(bf16_hi(w[2 * e + 1]) * inv, -E4M3_MAX), E4M3_MAX);
            int p = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
            p = __builtin_amdgcn_cvt_pk_fp8_f32(c2, d, p, true);
            o[e] = (uint32_t)p;
        }
        *reinterpret_cast<uint4 *>(q + r * ldq + 16 * c) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

int grid_for(size_t n_items) {
    size_t g = (n_items + 255) / 256;
    if (g > 256 * 16) g = 256 * 16;
    return (int)(g ? g : 1);
}

}  // namespace

lvx_status_t lvx_launch_fp8_amax(const bf16_t *x, int64_t ld, int rows, int cols, uint32_t *amax_slots, hipStream_t stream) {
    if (rows == 0) return LVX_OK;
    int amax_grid = grid_for((size_t)rows * (cols / 8));
    if (amax_grid > 1024) amax_grid = 1024;  // 4 workgroups per CU, one atomic each
    hipLaunchKernelGGL(lvx_fp8_amax_kernel, dim3(amax_grid), dim3(256), 0, stream, x, ld, rows, cols / 8, amax_slots);
    LVX_CHECK_HIP(hipGetLastError());
    return LVX_OK;
}

lvx_status_t lvx_launch_fp8_quant(const bf16_t *x, int64_t ld, int rows, int cols, uint8_t *q, int64_t ldq, const uint32_t *amax_slots,
                                  uint32_t *zero_slots, float *scale, hipStream_t stream) {
    if (rows == 0) return LVX_OK;
    hipLaunchKernelGGL(lvx_fp8_quant_kernel, dim3(grid_for((size_t)rows * (cols / 16))), dim3(256), 0, stream, x, ld, rows, cols / 16,
                       amax_slots, zero_slots, q, ldq, scale);
    LVX_CHECK_HIP(hipGetLastError());
    return LVX_OK;
}

lvx_status_t lvx_launch_fp8_quantize(const bf16_t *x, int64_t ld, int rows, int cols, uint8_t *q, int64_t ldq, uint32_t *amax_slots,
                                     float *scale, hipStream_t stream) {
    if (rows == 0) return LVX_OK;
    LVX_TRY(lvx_launch_fill_zero(amax_slots, LVX_AMAX_SLOTS * sizeof(uint32_t), stream));
    LVX_TRY(lvx_launch_fp8_amax(x, ld, rows, cols, amax_slots, stream));
    return lvx_launch_fp8_quant(x, ld, rows, cols, q, ldq, amax_slots, nullptr, scale, stream);
}

extern "C" lvx_status_t lvx_fp8_quantize(const void *dev_x, int64_t ld, int32_t rows, int32_t cols, void *dev_q, int64_t ldq,
                                         void *dev_scratch256, float *dev_scale, lvx_stream_t stream) {
    LVX_REQUIRE(dev_x != nullptr && dev_q != nullptr && dev_scratch256 != nullptr && dev_scale != nullptr, LVX_ERR_INVALID_ARG,
                "x, q, scratch or scale is NULL");
    LVX_REQUIRE(lvx_aligned16(dev_x) && lvx_aligned16(dev_q) && lvx_aligned16(dev_scratch256) && (((uintptr_t)dev_scale) & 3u) == 0,
                LVX_ERR_INVALID_ARG, "x, q and scratch must be 16-byte aligned, scale 4-byte aligned");
    LVX_REQUIRE(rows >= 0 && cols > 0 && cols % 16 == 0, LVX_ERR_SHAPE, "rows %d, cols %d (cols must be a positive multiple of 16)", rows, cols);
    LVX_REQUIRE(ld >= cols && ld % 8 == 0 && ldq >= cols && ldq % 16 == 0, LVX_ERR_SHAPE,
                "row strides: ld a multiple of 8 and ldq a multiple of 16, both >= cols");
    return lvx_launch_fp8_quantize((const bf16_t *)dev_x, ld, rows, cols, (uint8_t *)dev_q, ldq, (uint32_t *)dev_scratch256, dev_scale,
                                   (hipStream_t)stream);
}

extern "C" lvx_status_t lvx_fp8_quantize_static(const void *dev_x, int64_t ld, int32_t rows, int32_t cols, void *dev_q, int64_t ldq,
                                                float *dev_scale, lvx_stream_t stream) {
    LVX_REQUIRE(dev_x != nullptr && dev_q != nullptr && dev_scale != nullptr, LVX_ERR_INVALID_ARG, "x, q or scale is NULL");
    LVX_REQUIRE(lvx_aligned16(dev_x) && lvx_aligned16(dev_q) && (((uintptr_t)dev_scale) & 3u) == 0, LVX_ERR_INVALID_ARG,
                "x and q must be 16-byte aligned, scale 4-byte aligned");
    LVX_REQUIRE(rows >= 0 && cols > 0 && cols % 16 == 0, LVX_ERR_SHAPE, "rows %d, cols %d (cols must be a positive multiple of 16)", rows, cols);
    LVX_REQUIRE(ld >= cols && ld % 8 == 0 && ldq >= cols && ldq % 16 == 0, LVX_ERR_SHAPE,
                "row strides: ld a multiple of 8 and ldq a multiple of 16, both >= cols");
    LVX_REQUIRE((uint64_t)rows * (uint64_t)cols <= (uint64_t)LVX_FP8_QUANTIZE_STATIC_MAX_ELEMS, LVX_ERR_SHAPE,
                "tensor of %d x %d elements exceeds the %lld elements lvx_fp8_quantize_static accepts (use lvx_fp8_quantize)", rows, cols,
                (long long)LVX_FP8_QUANTIZE_STATIC_MAX_ELEMS);
    uint32_t *slots = nullptr;
    LVX_TRY(static_scratch(&slots));
    // the array keeps the previous call's maxima: lvx_launch_fp8_quantize clears it (by kernel) before collecting
    return lvx_launch_fp8_quantize((const bf16_t *)dev_x, ld, rows, cols, (uint8_t *)dev_q, ldq, slots, dev_scale, (hipStream_t)stream);
}

lvx_status_t lvx_launch_linear_fp8(const void *dev_aq, int64_t lda, const float *dev_scale_a, const void *dev_wq, int64_t ldw,
                                   const float *dev_scale_w, void *dev_c, int64_t ldc, int32_t M, int32_t N, int32_t K, lvx_epilogue_t epi,
                                   const void *dev_resid, int64_t ldr, const float *dev_gate, uint32_t *amax_slots, hipStream_t stream) {
    LVX_REQUIRE(dev_aq != nullptr && dev_wq != nullptr && dev_c != nullptr && dev_scale_a != nullptr && dev_scale_w != nullptr,
                LVX_ERR_INVALID_ARG, "A, W, C or a scale pointer is NULL");
    LVX_REQUIRE(lvx_aligned16(dev_aq) && lvx_aligned16(dev_wq) && lvx_aligned16(dev_c) && lvx_aligned16(dev_resid), LVX_ERR_INVALID_ARG,
                "pointers must be 16-byte aligned");
    LVX_REQUIRE(M >= 0 && N > 0 && K > 0, LVX_ERR_SHAPE, "M %d, N %d, K %d", M, N, K);
    LVX_REQUIRE(K % 128 == 0, LVX_ERR_SHAPE, "K %d must be a multiple of 128", K);
    LVX_REQUIRE(N % 8 == 0, LVX_ERR_SHAPE, "N %d must be a multiple of 8", N);
    LVX_REQUIRE(lda >= K && lda % 16 == 0 && ldw >= K && ldw % 16 == 0 && ldc >= N, LVX_ERR_SHAPE, "bad leading dimension");
    LVX_REQUIRE((uint64_t)M * (uint64_t)lda < (1ull << 32) && (uint64_t)N * (uint64_t)ldw < (1ull << 32), LVX_ERR_SHAPE,
                "operand larger than 4 GiB (32-bit byte offsets inside the kernel)");
    LVX_REQUIRE(epi == LVX_EPI_STORE || epi == LVX_EPI_GELU_TANH || epi == LVX_EPI_RESID_GATE || epi == LVX_EPI_RESID_GATE_F32,
                LVX_ERR_INVALID_ARG, "unknown epilogue %d", (int)epi);
    if (epi == LVX_EPI_RESID_GATE || epi == LVX_EPI_RESID_GATE_F32) {
        LVX_REQUIRE(dev_resid != nullptr, LVX_ERR_INVALID_ARG, "residual epilogue needs a residual pointer");
        LVX_REQUIRE(ldr >= N, LVX_ERR_SHAPE, "bad residual leading dimension");
    }
    if (M == 0) return LVX_OK;
    const lvx_gemm_launch_t plan = lvx_gemm_choose(nullptr, M, N, K / 128);
    lvx_gemm_args_t p = {};
    p.A = (const char *)dev_aq, p.lda = lda;
    p.W = (const char *)dev_wq, p.ldw = ldw;
    p.C = dev_c, p.ldc = ldc;
    p.R = dev_resid, p.ldr = ldr;
    p.gate = dev_gate;
    p.scale_a = dev_scale_a, p.scale_w = dev_scale_w;
    p.amax = amax_slots;
    p.N = N, p.n_slabs = K / 128;
    p.epi = (int)epi;
    if (plan.wide_rows > 0) {
        p.M = plan.wide_rows;
#define LVX8_WIDE(E_)                                                                                        \
        if (epi == E_)                                                                                       \
            LVX_TRY((plan.fn == 2   ? lvx_gemm_wide_launch<E_, true, 2>(p, plan.n_large, (hipStream_t)stream) \
                     : plan.fn == 3 ? lvx_gemm_wide_launch<E_, true, 3>(p, plan.n_large, (hipStream_t)stream) \
                                    : lvx_gemm_wide_launch<E_, true, 4>(p, plan.n_large, (hipStream_t)stream)));
        LVX8_WIDE(LVX_EPI_STORE)
        LVX8_WIDE(LVX_EPI_GELU_TANH)
        LVX8_WIDE(LVX_EPI_RESID_GATE)
        LVX8_WIDE(LVX_EPI_RESID_GATE_F32)
#undef LVX8_WIDE
        if (plan.wide_rows == M) return LVX_OK;
    }
    // the rows behind, or all, on a small tile
    const int m1 = plan.wide_rows;
    const int64_t c_bytes = epi == LVX_EPI_RESID_GATE_F32 ? 4 : 2;
    p.A += (size_t)m1 * lda;
    p.C = (char *)dev_c + (size_t)m1 * ldc * c_bytes;
    if (dev_resid != nullptr) p.R = (const char *)dev_resid + (size_t)m1 * ldr * c_bytes;
    p.M = M - m1;
    return lvx_gemm_launch_small<true>(plan.tile, p, stream);
}

extern "C" lvx_status_t lvx_linear_fp8(const void *dev_aq, int64_t lda, const float *dev_scale_a, const void *dev_wq, int64_t ldw,
                                       const float *dev_scale_w, void *dev_c, int64_t ldc, int32_t M, int32_t N, int32_t K,
                                       lvx_epilogue_t epi, const void *dev_resid, int64_t ldr, const float *dev_gate, lvx_stream_t stream) {
    return lvx_launch_linear_fp8(dev_aq, lda, dev_scale_a, dev_wq, ldw, dev_scale_w, dev_c, ldc, M, N, K, epi, dev_resid, ldr, dev_gate, nullptr,
                                 (hipStream_t)stream);
}
