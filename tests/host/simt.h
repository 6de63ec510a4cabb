// Runs a kernel's source on the CPU, a workgroup at a time: what csrc/sampler.hip uses of the device language, for g++.  Each thread
// is a fiber.  A wave's lanes meet at lane operations, the waves at barriers only; between two barriers one wave runs after the other, in an
// order that the caller picks, so what no barrier orders happens as far out of order as it can.
//
// The file with the kernels is compiled with -fsanitize=thread, which makes the compiler report every load and store to the functions
// __tsan_*; those are defined in simt.cpp, not by the sanitizer's library.  Two waves' accesses to one word of LDS without a barrier in
// between are recorded there as a race unless both only read or both are atomic.
#pragma once

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

struct simt_dim { int x; };
extern simt_dim threadIdx, blockIdx, blockDim;

void simt_barrier(int line);
const uint64_t *simt_exchange(uint64_t mine, uint64_t *live);   // every live lane's value, 64 of them
enum { SIMT_READ = 0, SIMT_WRITE = 1, SIMT_ATOMIC = 2 };
void simt_access(const void *p, int bytes, int kind);
extern long simt_word_adds;   // atomic adds to 64-bit integers

#define __global__
#define __device__
#define __launch_bounds__(...)
#define __shared__ static
#define __syncthreads() simt_barrier(__LINE__)
#define __builtin_amdgcn_sched_barrier(x)
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define SIMT_UNSEEN __attribute__((noinline, no_sanitize("thread")))

using std::max;
using std::min;
struct float4 { float x, y, z, w; };
struct uint2 { uint32_t x, y; };

inline uint32_t __float_as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
inline int __float_as_int(float f) { return (int)__float_as_uint(f); }
inline float __int_as_float(int i) { return __uint_as_float((uint32_t)i); }
inline unsigned long long __double_as_longlong(double d) { unsigned long long u; memcpy(&u, &d, 8); return u; }
inline double __longlong_as_double(long long i) { double d; memcpy(&d, &i, 8); return d; }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
inline int __clz(int v) { return v ? __builtin_clz((unsigned)v) : 32; }
inline int __popc(uint32_t v) { return __builtin_popcount(v); }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __ffsll(long long v) { return __builtin_ffsll(v); }
inline float __builtin_amdgcn_exp2f(float x) { return exp2f(x); }

template <typename T> SIMT_UNSEEN T atomicAdd(T *p, T v) { simt_access(p, sizeof(T), SIMT_ATOMIC); simt_word_adds += sizeof(T) == 8 && std::is_integral<T>::value; const T old = *p; *p = old + v; return old; }
template <typename T> SIMT_UNSEEN T atomicMax(T *p, T v) { simt_access(p, sizeof(T), SIMT_ATOMIC); const T old = *p; *p = old < v ? v : old; return old; }
template <typename T> SIMT_UNSEEN T atomicMin(T *p, T v) { simt_access(p, sizeof(T), SIMT_ATOMIC); const T old = *p; *p = v < old ? v : old; return old; }
template <typename T> SIMT_UNSEEN T __hip_atomic_load(const T *p, int, int) { simt_access(p, sizeof(T), SIMT_ATOMIC); return *p; }

template <typename T> SIMT_UNSEEN T simt_from(T v, int lane) {
    uint64_t u = 0, live;
    memcpy(&u, &v, sizeof(T));
    const uint64_t w = simt_exchange(u, &live)[lane & 63];
    T r;
    memcpy(&r, &w, sizeof(T));
    return r;
}
template <typename T> T __shfl(T v, int lane, int) { return simt_from(v, lane); }
template <typename T> T __shfl_xor(T v, int mask, int) { return simt_from(v, (threadIdx.x & 63) ^ mask); }
template <typename T> T __shfl_up(T v, int by, int) { const int lane = threadIdx.x & 63; return simt_from(v, lane < by ? lane : lane - by); }
inline int __builtin_amdgcn_readlane(int v, int lane) { return simt_from(v, lane); }
SIMT_UNSEEN inline unsigned long long __ballot(int p) {
    uint64_t live, r = 0;
    const uint64_t *v = simt_exchange((uint64_t)(p != 0), &live);
    for (int i = 0; i < 64; ++i) r |= (live >> i & 1) && v[i] ? 1ull << i : 0;
    return r;
}
// row_shr:1..15 and row_bcast:15/31 of the lane-move (DPP) operand forms; a lane without a source, or in a row left out, keeps `old`
SIMT_UNSEEN inline int __builtin_amdgcn_update_dpp(int old, int src, int ctrl, int rows, int, bool) {
    const int lane = threadIdx.x & 63, row = lane / 16;
    int from = -1;
    if (ctrl > 0x110 && ctrl <= 0x11f) from = lane % 16 >= ctrl - 0x110 ? lane - (ctrl - 0x110) : -1;
    else if (ctrl == 0x142) from = row >= 1 ? 16 * row - 1 : -1;
    else if (ctrl == 0x143) from = row >= 2 ? 31 : -1;
    else __builtin_trap();
    const int got = simt_from(src, from < 0 ? lane : from);
    return from >= 0 && (rows >> row & 1) ? got : old;
}
