// What the projection kernels share: epilogue arithmetic, the wait for loads in flight, the epilogues' extra arguments.
#pragma once

#include "pc_internal.h"

namespace pc {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// silu(g) * u of the matrix-core epilogues, whose results are rounded to 16 bits: exp2 and reciprocal are the hardware's
// (the fp32 value is off by 5.3e-8 of its size instead of 4.7e-8; rounded to half or bfloat16 both forms are equally far from
// 64-bit values in all of seven digits, gates and ups of deviation 0.3 to 40).  The epilogue is
// vector-ALU work that nothing overlaps, one block per CU: with expf, an IEEE division and a range test per value it took
// a tenth of the kernel (gate/up of the 1.5B shape: 1020 -> 935 us at 16384 rows, 28.3 -> 25.7 us at 256 rows).
__device__ inline float silu_mul(float g, float u) {
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.4426950408889634f)) * u;
}

// exp(d) for d <= 0 to about one unit in the last place: d log2(e) in two pieces, the small one added to first order
__device__ inline float exp_neg(float d) {
    const float p = d * 1.44269502f;
    const float r = __builtin_amdgcn_exp2f(p);
    const float e = fmaf(d, 1.92596299e-8f, fmaf(d, 1.44269502f, -p));
    return p < -126.f ? 0.f : fmaf(r, e * 0.693147181f, r);
}

// Four values packed into two words.  Values beyond the half range are clamped and counted on a path of their own; one
// test covers the four (their absolute sum is at most 65504 only if none is beyond it, infinite or not a number).
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
template <typename T> __device__ inline u32x2 pack4_sat(float a, float b, float c, float d, uint32_t *sat) {
    return (u32x2){pack2_sat<T>(a, b, sat), pack2_sat<T>(c, d, sat)};
}
template <> __device__ inline u32x2 pack4_sat<f16_t>(float a, float b, float c, float d, uint32_t *sat) {
    typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
    if (fabsf(a) + fabsf(b) + fabsf(c) + fabsf(d) <= 65504.f)
        return __builtin_bit_cast(u32x2, (f16x4){(_Float16)a, (_Float16)b, (_Float16)c, (_Float16)d});
    return (u32x2){pack2_sat<f16_t>(a, b, sat), pack2_sat<f16_t>(c, d, sat)};
}

// A rotary pair (x1, x2) turned by the angle of cosine c and sine s.  Which product is rounded is written out: left to the compiler,
// it differs from kernel to kernel, and a row's q and k would depend on the tile (in 8 of 100000 values of half).
__device__ inline float rotated_first(float x1, float x2, float c, float s) { return fmaf(x1, c, -(x2 * s)); }
__device__ inline float rotated_second(float x1, float x2, float c, float s) { return fmaf(x1, s, x2 * c); }

template <int N> __device__ inline void wait_vmcnt_le() {
    // s_waitcnt with only the vector-memory counter set (gfx9 encoding: vmcnt = bits 15:14 | 3:0)
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// What an epilogue needs besides the common arguments.
struct NoExtra {};
template <int EPI> struct GemmExtra { typedef NoExtra type; };
template <> struct GemmExtra<EPI_SWIGLU_RS> { typedef GemmRowScale type; };
template <> struct GemmExtra<EPI_LOGPROB> { typedef GemmLogprob type; };
template <> struct GemmExtra<EPI_QKV> { typedef GemmQkv type; };
template <> struct GemmExtra<EPI_RESID_SLICES> { typedef GemmSlices type; };

// gemm_large.hip: large batches.  Each launches nothing and says so (0, false) if it does not take the call, or if the 256 x 128
// tile of gemm.hip is the faster one for it.
void gemm_large_init();   // once per device, like gemm_init
int launch_gemm_large(int dtype, const void *A, WeightRef W, void *C, int M, int N, int K, int epi, float *slices, size_t slice_cap,
                      uint32_t *sat, hipStream_t s, const GemmRowScale *row_scale);   // the number of K slices, as launch_gemm
int gemm_large_resid_slices(int M, int N, int K, const float *slices, size_t slice_cap);   // how many it would cut such a launch into
bool launch_gemm_large_qkv(int dtype, const void *A, WeightRef W, int M, int N, int K, const GemmQkv &q, uint32_t *sat, hipStream_t s);
int launch_gemm_large_logprob(int dtype, const void *A, WeightRef W, int M, int N, int K, const GemmLogprob &lp,
                              hipStream_t s);          // the number of column strips

}   // namespace pc
