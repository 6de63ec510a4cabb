// Row-wise kernels of the decoder forward (Section 3.1 policy pi_theta):
// embedding gather, RMSNorm, rotary positions + KV append, and the small
// bookkeeping kernels of the paged cache.  All are HBM/latency bound.
#include <algorithm>

#include "pc_internal.h"

namespace pc {

static constexpr int WAVE = 64;

__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    return v;
}

// ------------------------------------------------------------------ embed
template <typename T, bool VEC>
__global__ void embed_kernel(const T *__restrict__ table, const int32_t *__restrict__ tokens, int d, int vocab,
                             float *__restrict__ h) {
    int r = blockIdx.x;
    int tok = tokens[r];
    if (tok < 0 || tok >= vocab) tok = 0;
    const T *src = table + (int64_t)tok * d;
    float *dst = h + (int64_t)r * d;
    if (VEC) {   // four elements per access (16384 rows of 1536: 48 us one by one, 28 us)
        for (int i = 4 * threadIdx.x; i < d; i += 4 * blockDim.x) {
            struct alignas(4 * sizeof(T)) Four { T e[4]; };
            const Four f = *(const Four *)(src + i);
            *(float4 *)(dst + i) = make_float4(to_f32(f.e[0]), to_f32(f.e[1]), to_f32(f.e[2]), to_f32(f.e[3]));
        }
    } else {
        for (int i = threadIdx.x; i < d; i += blockDim.x) dst[i] = to_f32(src[i]);
    }
}

void launch_embed(int dtype, const void *table, const int32_t *tokens, int rows, int d, int vocab, float *h,
                  hipStream_t s) {
    if (rows <= 0) return;
    // the table is the caller's (fp32, or bf16 for both 16-bit kernel dtypes) and may start anywhere
    const bool vec = d % 4 == 0 && ((uintptr_t)table) % 16 == 0;
    if (dtype == KD_F32) {
        if (vec) embed_kernel<float, true><<<rows, 256, 0, s>>>((const float *)table, tokens, d, vocab, h);
        else embed_kernel<float, false><<<rows, 256, 0, s>>>((const float *)table, tokens, d, vocab, h);
    } else {
        if (vec) embed_kernel<bf16_t, true><<<rows, 256, 0, s>>>((const bf16_t *)table, tokens, d, vocab, h);
        else embed_kernel<bf16_t, false><<<rows, 256, 0, s>>>((const bf16_t *)table, tokens, d, vocab, h);
    }
}

// ------------------------------------------------------------------ RMSNorm
// out = h * rsqrt(mean(h^2) + eps) * gain; one block per row, statistics in fp32.
// Pending split-K slices of the previous projection are folded into h first (slice order).
// Rows of up to 4 * 256 * RMS_MAXV values (a multiple of 4) live in registers between the two passes.
static constexpr int RMS_MAXV = 6;

template <typename T> __device__ inline void store4(T *p, float4 v, uint32_t *sat);
template <> __device__ inline void store4<float>(float *p, float4 v, uint32_t *) { *(float4 *)p = v; }
template <> __device__ inline void store4<bf16_t>(bf16_t *p, float4 v, uint32_t *) {
    uint2 u = {pack2<bf16_t>(v.x, v.y), pack2<bf16_t>(v.z, v.w)};
    *(uint2 *)p = u;
}
template <> __device__ inline void store4<f16_t>(f16_t *p, float4 v, uint32_t *sat) {
    uint2 u = {pack2_sat<f16_t>(v.x, v.y, sat), pack2_sat<f16_t>(v.z, v.w, sat)};
    *(uint2 *)p = u;
}

template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_kernel(float *__restrict__ h, const int32_t *__restrict__ src_row,
                                                      const float *__restrict__ gain, int rows, int d, float eps,
                                                      T *__restrict__ out, const float *__restrict__ slices, int S,
                                                      uint32_t *__restrict__ sat) {
    __shared__ float part[4];
    const int r = blockIdx.x, tid = threadIdx.x;
    float *x = h + (int64_t)(src_row ? src_row[r] : r) * d;
    float ss = 0.f;
    for (int i = tid; i < d; i += 256) {
        float v = x[i];
        if (S > 1) {
            float add = 0.f;
            for (int z = 0; z < S; ++z) add += slices[((int64_t)z * rows + r) * d + i];
            v += add;
            x[i] = v;
        }
        ss += v * v;
    }
    ss = wave_sum(ss);
    if (tid % WAVE == 0) part[tid / WAVE] = ss;
    __syncthreads();
    const float tot = part[0] + part[1] + part[2] + part[3];
    const float rs = 1.0f / sqrtf(tot / (float)d + eps);
    T *o = out + (int64_t)r * d;
    for (int i = tid; i < d; i += 256) o[i] = from_f32_sat<T>(x[i] * rs * gain[i], sat);
}

// The same for rows that fit the registers, S slices known.  A decode step's launch is a few hundred rows, one trip to memory long: the
// loads of J pieces of a row and of all their slices are in flight at once, clamped past the row's end and not left out (a
// branch or a loop around them made a trip of every piece and of every fourth slice: rows x d x slices 256 x 1536 x 5 5.5 -> 5.1 us, 3
// x 1536 x 8 5.1 -> 4.2, 168 x 5120 x 6 10.3 -> 8.9; 8 slices of 256 x 4096, 34 MB, take 10.2).
template <typename T, int S>
__global__ __launch_bounds__(256) void rmsnorm4_kernel(float *__restrict__ h, const int32_t *__restrict__ src_row,
                                                       const float *__restrict__ gain, int rows, int d, float eps,
                                                       T *__restrict__ out, const float *__restrict__ slices,
                                                       uint32_t *__restrict__ sat) {
    constexpr int J = S == 1 ? RMS_MAXV : (S <= 4 ? 3 : 2);
    static_assert(RMS_MAXV % J == 0, "whole groups");
    __shared__ float part[4];
    const int r = blockIdx.x, tid = threadIdx.x, n4 = d / 4, wave0 = __builtin_amdgcn_readfirstlane(tid / WAVE) * WAVE;
    float4 *x = (float4 *)(h + (int64_t)(src_row ? src_row[r] : r) * d);
    const float4 *sp = (const float4 *)(slices + (int64_t)r * d);
    const int64_t zs = (int64_t)rows * n4;
    float ss = 0.f;
    float4 keep[RMS_MAXV];
#pragma unroll
    for (int j0 = 0; j0 < RMS_MAXV; j0 += J) {
        if (256 * j0 >= n4) break;   // (block-uniform)
        float4 t[J][S];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (wave0 + 256 * (j0 + j) >= n4) continue;   // (wave-uniform)
            const int i = min(tid + 256 * (j0 + j), n4 - 1);
            keep[j0 + j] = x[i];
            if (S > 1) {
#pragma unroll
                for (int z = 0; z < S; ++z) t[j][z] = sp[z * zs + i];
            }
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (wave0 + 256 * (j0 + j) >= n4) continue;
            const int i = tid + 256 * (j0 + j);
            float4 &v = keep[j0 + j];
            if (S > 1) {
                float4 add = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int z = 0; z < S; ++z) {
                    add.x += t[j][z].x; add.y += t[j][z].y; add.z += t[j][z].z; add.w += t[j][z].w;
                }
                v.x += add.x; v.y += add.y; v.z += add.z; v.w += add.w;
                if (i < n4) x[i] = v;
            }
            if (i < n4) ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        }
    }
    ss = wave_sum(ss);
    if (tid % WAVE == 0) part[tid / WAVE] = ss;
    __syncthreads();
    const float tot = part[0] + part[1] + part[2] + part[3];
    const float rs = 1.0f / sqrtf(tot / (float)d + eps);
    T *o = out + (int64_t)r * d;
#pragma unroll
    for (int j = 0; j < RMS_MAXV; ++j) {
        const int i = tid + 256 * j;
        if (i < n4) {
            const float4 g = ((const float4 *)gain)[i];
            float4 v = keep[j];
            v.x = v.x * rs * g.x; v.y = v.y * rs * g.y; v.z = v.z * rs * g.z; v.w = v.w * rs * g.w;
            store4<T>(o + 4 * i, v, sat);
        }
    }
}

template <typename T>
static void rmsnorm_t(float *h, const int32_t *src_row, const float *gain, int rows, int d, float eps, void *out, const float *slices, int S,
                      uint32_t *sat, hipStream_t s) {
    T *o = (T *)out;
#define PC_RMS(N) case N: rmsnorm4_kernel<T, N><<<rows, 256, 0, s>>>(h, src_row, gain, rows, d, eps, o, slices, sat); return
    if (d % 4 == 0 && d <= 4 * 256 * RMS_MAXV) {
        switch (std::max(S, 1)) { PC_RMS(1); PC_RMS(2); PC_RMS(3); PC_RMS(4); PC_RMS(5); PC_RMS(6); PC_RMS(7); PC_RMS(8); }
    }
#undef PC_RMS
    rmsnorm_kernel<T><<<rows, 256, 0, s>>>(h, src_row, gain, rows, d, eps, o, slices, S, sat);
}
void launch_rmsnorm(int dtype, float *h, const int32_t *src_row, const float *gain, int rows, int d, float eps,
                    void *out, const float *slices, int S, uint32_t *sat, hipStream_t s) {
    if (rows <= 0) return;
    if (dtype == KD_F32) rmsnorm_t<float>(h, src_row, gain, rows, d, eps, out, slices, S, sat, s);
    else if (dtype == KD_BF16) rmsnorm_t<bf16_t>(h, src_row, gain, rows, d, eps, out, slices, S, sat, s);
    else rmsnorm_t<f16_t>(h, src_row, gain, rows, d, eps, out, slices, S, sat, s);
}

// ------------------------------------------------------------------ RoPE + KV append
// The pair (i, i + hd/2) of every q and k head turns by the angle pos * theta^(-2i/hd) (cos/sin tables are
// built on the host in double).  Grid (rows, item chunks): a row's work items are its q pairs, then its k
// pairs, then its v elements; every thread takes exactly one, so all of a row's loads are in flight at once.
// Which product of a pair is rounded is written out: left to the compiler, it differed between the kernels below and from one number of
// slices to another, in 4 to 13 of 100000 values of half.
__device__ inline float turned_first(float x1, float x2, float c, float s) { return fmaf(x1, c, -(x2 * s)); }
__device__ inline float turned_second(float x1, float x2, float c, float s) { return fmaf(x2, c, x1 * s); }
template <typename T>
__global__ __launch_bounds__(256) void rope_append_kernel(const float *__restrict__ qkv, int S, int rows,
                                                          const int32_t *__restrict__ row_slot,
                                                          const int32_t *__restrict__ row_pos,
                                                          const int32_t *__restrict__ slot_len,
                                                          const float *__restrict__ rope_cos,
                                                          const float *__restrict__ rope_sin, int hq, KvGeom kv,
                                                          int layer, T *__restrict__ q_out,
                                                          uint32_t *__restrict__ sat, int perm) {
    const int r = blockIdx.x;
    const int hd = kv.head_dim, half = hd / 2, hkv = kv.n_kv_heads, bs = kv.block_size;
    const int nq = hq * half, nk = hkv * half, nv = hkv * hd;
    const int item = blockIdx.y * 256 + threadIdx.x;
    if (item >= nq + nk + nv) return;
    const int width = (hq + 2 * hkv) * hd;
    const float *row = qkv + (int64_t)r * width;
    const int64_t zs = (int64_t)rows * width;   // distance between K slices
    // perm: the weight rows of every q and k head were packed in the order the fused decode projection wants
    // (qkv_packed_dim): dim j of a head then sits at column qkv_packed_dim(j) of the head
    auto val = [&](int c) {
        float v = row[c];
        for (int z = 1; z < S; ++z) v += row[z * zs + c];
        return v;
    };
    auto qk_col = [&](int j) { return perm ? qkv_packed_dim(j, hd) : j; };
    const int slot = row_slot[r];
    const int pos = row_pos ? row_pos[r] : slot_len[slot];
    if (item < nq) {
        const int head = item / half, j = item % half;
        const float x1 = val(head * hd + qk_col(j)), x2 = val(head * hd + qk_col(j + half));
        const float c = rope_cos[(int64_t)pos * half + j], sgn = rope_sin[(int64_t)pos * half + j];
        T *qd = q_out + (int64_t)r * hq * hd + head * hd;
        qd[j] = from_f32_sat<T>(turned_first(x1, x2, c, sgn), sat);
        qd[j + half] = from_f32_sat<T>(turned_second(x1, x2, c, sgn), sat);
        return;
    }
    const int blk = kv.block_table[(int64_t)slot * kv.max_blocks_per_slot + pos / bs];
    const int tin = pos % bs;
    T *pool = (T *)kv.pool + (int64_t)layer * kv.layer_stride + (int64_t)blk * kv.block_elems();
    if (item < nq + nk) {   // k heads
        const int i = item - nq, head = i / half, j = i % half;
        const int koff = hq * hd;
        const float x1 = val(koff + head * hd + qk_col(j)), x2 = val(koff + head * hd + qk_col(j + half));
        const float c = rope_cos[(int64_t)pos * half + j], sgn = rope_sin[(int64_t)pos * half + j];
        T *kd = pool + (int64_t)head * kv.head_elems();
        kd[kv.k_index(tin, j)] = from_f32_sat<T>(turned_first(x1, x2, c, sgn), sat);
        kd[kv.k_index(tin, j + half)] = from_f32_sat<T>(turned_second(x1, x2, c, sgn), sat);
    } else {                // v heads
        const int i = item - nq - nk, head = i / hd, j = i % hd;
        const int voff = (hq + hkv) * hd;
        T *vd = pool + (int64_t)head * kv.head_elems();
        vd[kv.v_index(tin, j)] = from_f32_sat<T>(val(voff + head * hd + j), sat);
    }
}

// The same with four pairs (four dims of v) to a thread and S slices known: 16-byte loads of all slices in flight at once, where the kernel
// above waits for one slice after another (256 rows of the 8B shape 12.8 -> 11.8 us, 168 of 14B 9.7 -> 8.5).  Heads of a multiple of 16 (packed rows: 32),
// qkv on 16 bytes.
template <typename T, int S>
__global__ __launch_bounds__(256) void rope_append4_kernel(const float *__restrict__ qkv, int rows, const int32_t *__restrict__ row_slot,
                                                           const int32_t *__restrict__ row_pos, const int32_t *__restrict__ slot_len,
                                                           const float *__restrict__ rope_cos, const float *__restrict__ rope_sin, int hq,
                                                           KvGeom kv, int layer, T *__restrict__ q_out, uint32_t *__restrict__ sat, int perm) {
    const int r = blockIdx.x;
    const int hd = kv.head_dim, half = hd / 2, hkv = kv.n_kv_heads, bs = kv.block_size;
    const int nq = hq * half / 4, nk = hkv * half / 4, nv = hkv * hd / 4;
    const int item = blockIdx.y * 256 + threadIdx.x;
    if (item >= nq + nk + nv) return;
    const int width = (hq + 2 * hkv) * hd;
    const float *row = qkv + (int64_t)r * width;
    const int64_t zs = (int64_t)rows * width;
    const bool is_v = item >= nq + nk;
    // columns of the first and the second values of the pairs (v: of the four dims, twice)
    const int per = is_v ? hd / 4 : half / 4;
    const int i = is_v ? item - nq - nk : (item < nq ? item : item - nq);
    const int head = i / per, j = 4 * (i % per);
    const int base = (is_v ? (hq + hkv) * hd : (item < nq ? 0 : hq * hd)) + head * hd;
    const int c1 = base + (is_v || !perm ? j : qkv_packed_dim(j, hd)), c2 = is_v ? c1 : base + (perm ? qkv_packed_dim(j + half, hd) : j + half);
    float4 a[S], b[S];
#pragma unroll
    for (int z = 0; z < S; ++z) {
        a[z] = *(const float4 *)(row + z * zs + c1);
        b[z] = *(const float4 *)(row + z * zs + c2);
    }
    const int slot = row_slot[r];
    const int pos = row_pos ? row_pos[r] : slot_len[slot];
    const int blk = item < nq ? 0 : kv.block_table[(int64_t)slot * kv.max_blocks_per_slot + pos / bs];
    const int tin = pos % bs;
    float4 cs = {}, sn = {};
    if (!is_v) {
        cs = *(const float4 *)(rope_cos + (int64_t)pos * half + j);
        sn = *(const float4 *)(rope_sin + (int64_t)pos * half + j);
    }
    float4 x1 = a[0], x2 = b[0];
#pragma unroll
    for (int z = 1; z < S; ++z) {
        x1.x += a[z].x; x1.y += a[z].y; x1.z += a[z].z; x1.w += a[z].w;
        x2.x += b[z].x; x2.y += b[z].y; x2.z += b[z].z; x2.w += b[z].w;
    }
    T *pool = (T *)kv.pool + (int64_t)layer * kv.layer_stride + (int64_t)blk * kv.block_elems() + (int64_t)head * kv.head_elems();
    if (is_v) {
        pool[kv.v_index(tin, j)] = from_f32_sat<T>(x1.x, sat);
        pool[kv.v_index(tin, j + 1)] = from_f32_sat<T>(x1.y, sat);
        pool[kv.v_index(tin, j + 2)] = from_f32_sat<T>(x1.z, sat);
        pool[kv.v_index(tin, j + 3)] = from_f32_sat<T>(x1.w, sat);
        return;
    }
    const float4 y1 = {turned_first(x1.x, x2.x, cs.x, sn.x), turned_first(x1.y, x2.y, cs.y, sn.y),
                       turned_first(x1.z, x2.z, cs.z, sn.z), turned_first(x1.w, x2.w, cs.w, sn.w)};
    const float4 y2 = {turned_second(x1.x, x2.x, cs.x, sn.x), turned_second(x1.y, x2.y, cs.y, sn.y),
                       turned_second(x1.z, x2.z, cs.z, sn.z), turned_second(x1.w, x2.w, cs.w, sn.w)};
    T *q = q_out + (int64_t)r * hq * hd + head * hd;
    store4<T>(item < nq ? q + j : pool + kv.k_index(tin, j), y1, sat);                 // (four dims of a token are neighbours in K)
    store4<T>(item < nq ? q + j + half : pool + kv.k_index(tin, j + half), y2, sat);
}

template <typename T>
static void rope_append_t(const float *qkv, int S, const int32_t *row_slot, const int32_t *row_pos, const int32_t *slot_len, const float *rope_cos,
                          const float *rope_sin, int rows, int hq, KvGeom kv, int layer, T *q_out, uint32_t *sat, int perm, hipStream_t s) {
    const int hd = kv.head_dim, items = (hq + kv.n_kv_heads) * (hd / 2) + kv.n_kv_heads * hd;
    if (hd % 16 == 0 && (!perm || hd % 32 == 0) && (((uintptr_t)qkv) & 15) == 0) {
        const dim3 grid(rows, (items / 4 + 255) / 256);
#define PC_ROPE(N) \
    case N: rope_append4_kernel<T, N><<<grid, 256, 0, s>>>(qkv, rows, row_slot, row_pos, slot_len, rope_cos, rope_sin, hq, kv, layer, q_out, sat, perm); return
        switch (std::max(S, 1)) { PC_ROPE(1); PC_ROPE(2); PC_ROPE(3); PC_ROPE(4); PC_ROPE(5); PC_ROPE(6); PC_ROPE(7); PC_ROPE(8); }
#undef PC_ROPE
    }
    rope_append_kernel<T><<<dim3(rows, (items + 255) / 256), 256, 0, s>>>(qkv, S, rows, row_slot, row_pos, slot_len, rope_cos, rope_sin, hq, kv, layer,
                                                                          q_out, sat, perm);
}
void launch_rope_append(int dtype, const float *qkv, int S, const int32_t *row_slot, const int32_t *row_pos,
                        const int32_t *slot_len, const float *rope_cos, const float *rope_sin, int rows, int hq,
                        KvGeom kv, int layer, void *q_out, uint32_t *sat, int perm, hipStream_t s) {
    if (rows <= 0) return;
    if (dtype == KD_F32)
        rope_append_t<float>(qkv, S, row_slot, row_pos, slot_len, rope_cos, rope_sin, rows, hq, kv, layer, (float *)q_out, sat, perm, s);
    else if (dtype == KD_BF16)
        rope_append_t<bf16_t>(qkv, S, row_slot, row_pos, slot_len, rope_cos, rope_sin, rows, hq, kv, layer, (bf16_t *)q_out, sat, perm, s);
    else
        rope_append_t<f16_t>(qkv, S, row_slot, row_pos, slot_len, rope_cos, rope_sin, rows, hq, kv, layer, (f16_t *)q_out, sat, perm, s);
}

// ------------------------------------------------------------------ bookkeeping
__global__ void advance_len_kernel(int32_t *slot_len, const int32_t *row_slot, int rows) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < rows) slot_len[row_slot[i]] += 1;   // slots in a step are distinct
}
void launch_advance_len(int32_t *slot_len, const int32_t *row_slot, int rows, hipStream_t s) {
    if (rows <= 0) return;
    advance_len_kernel<<<(rows + 255) / 256, 256, 0, s>>>(slot_len, row_slot, rows);
}

__global__ void fill_i32_kernel(int32_t *p, int32_t v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
void launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    fill_i32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(p, v, n);
}

// copies whole KV blocks (all layers, all kv heads): pairs[2i] -> pairs[2i+1], 16 bytes a thread and 16 KB a workgroup (the block of a
// prompt's last tokens for each of 256 sequences, 3 layers of the 8B shape: 256 us two bytes a thread and
// a workgroup to a block of a layer, 70 so)
static constexpr int COPY_PIECES = 1024;   // of 16 bytes, per workgroup
__global__ __launch_bounds__(256) void copy_block_kernel(uint4 *__restrict__ pool, int64_t layer_pieces, int64_t block_pieces,
                                                         const int32_t *__restrict__ pairs) {
    const int pair = blockIdx.x, layer = blockIdx.y;
    const uint4 *src = pool + layer * layer_pieces + pairs[2 * pair] * block_pieces;
    uint4 *dst = pool + layer * layer_pieces + pairs[2 * pair + 1] * block_pieces;
    const int64_t first = (int64_t)blockIdx.z * COPY_PIECES + threadIdx.x;
    uint4 v[COPY_PIECES / 256];
#pragma unroll
    for (int u = 0; u < COPY_PIECES / 256; ++u)
        if (first + 256 * u < block_pieces) v[u] = src[first + 256 * u];
#pragma unroll
    for (int u = 0; u < COPY_PIECES / 256; ++u)
        if (first + 256 * u < block_pieces) dst[first + 256 * u] = v[u];
}
void launch_copy_block(int dtype, KvGeom kv, int n_layers, const int32_t *pairs, int n_pairs, hipStream_t s) {
    if (n_pairs <= 0) return;
    const int64_t size = dtype == KD_F32 ? 4 : 2;   // (blocks hold a multiple of 32 tokens, K and V: whole pieces)
    const int64_t pieces = kv.block_elems() * size / 16;
    const dim3 grid(n_pairs, n_layers, (unsigned)((pieces + COPY_PIECES - 1) / COPY_PIECES));
    copy_block_kernel<<<grid, 256, 0, s>>>((uint4 *)kv.pool, kv.layer_stride * size / 16, pieces, pairs);
}

// ------------------------------------------------------------------ weight repacking
// TS: the caller's element type, TD: the kernel dtype of the copy (bf16 -> half is a value conversion)
template <typename TS, typename TD> __device__ inline TD conv(TS v) { return from_f32<TD>(to_f32(v)); }

// head_perm > 0: rows come in heads of head_perm rows, and row j of a head goes to row qkv_packed_dim(j) of it
template <typename TS, typename TD>
__global__ void pack_rows_kernel(const TS *__restrict__ src, TD *__restrict__ dst, int64_t cols, int64_t dst_row0,
                                 int head_perm, int lg) {
    int64_t r = blockIdx.x, rd = r;
    if (head_perm > 0) rd = (r / head_perm) * head_perm + qkv_packed_dim((int)(r % head_perm), head_perm);
    for (int64_t i = threadIdx.x; i < cols; i += blockDim.x) dst[weight_at(dst_row0 + rd, i, cols, lg)] = conv<TS, TD>(src[r * cols + i]);
}
void launch_pack_rows(int kd, const void *src, void *dst, int64_t rows, int64_t cols, int64_t dst_row0, int head_perm, int lg,
                      hipStream_t s) {
    if (rows <= 0) return;
    if (kd == KD_F32)
        pack_rows_kernel<float, float><<<(unsigned)rows, 256, 0, s>>>((const float *)src, (float *)dst, cols, dst_row0, head_perm, lg);
    else if (kd == KD_BF16)
        pack_rows_kernel<bf16_t, bf16_t><<<(unsigned)rows, 256, 0, s>>>((const bf16_t *)src, (bf16_t *)dst, cols, dst_row0, head_perm, lg);
    else
        pack_rows_kernel<bf16_t, f16_t><<<(unsigned)rows, 256, 0, s>>>((const bf16_t *)src, (f16_t *)dst, cols, dst_row0, head_perm, lg);
}

// dst row 32t + c      = gate row 16t + c   (c < 16)
// dst row 32t + 16 + c = up   row 16t + c
template <typename TS, typename TD>
__global__ void pack_gate_up_kernel(const TS *__restrict__ gate, const TS *__restrict__ up, TD *__restrict__ dst, int d, int lg) {
    int64_t j = blockIdx.x;   // ffn row
    int64_t t = j / 16, c = j % 16;
    for (int i = threadIdx.x; i < d; i += blockDim.x) {
        dst[weight_at(32 * t + c, i, d, lg)] = conv<TS, TD>(gate[j * d + i]);
        dst[weight_at(32 * t + 16 + c, i, d, lg)] = conv<TS, TD>(up[j * d + i]);
    }
}
void launch_pack_gate_up(int kd, const void *gate, const void *up, void *dst, int d_ff, int d, int lg, hipStream_t s) {
    if (kd == KD_F32)
        pack_gate_up_kernel<float, float><<<d_ff, 256, 0, s>>>((const float *)gate, (const float *)up, (float *)dst, d, lg);
    else if (kd == KD_BF16)
        pack_gate_up_kernel<bf16_t, bf16_t><<<d_ff, 256, 0, s>>>((const bf16_t *)gate, (const bf16_t *)up, (bf16_t *)dst, d, lg);
    else
        pack_gate_up_kernel<bf16_t, f16_t><<<d_ff, 256, 0, s>>>((const bf16_t *)gate, (const bf16_t *)up, (f16_t *)dst, d, lg);
}

}  // namespace pc

// For tests, not part of the C ABI: one launch of the rotation (layer 0 of the cache).  1: launched; 0: not a call that it takes.
extern "C" int pc_internal_rope_append(int dtype, const float *qkv, int slices, const int32_t *row_slot, const int32_t *row_pos,
                                       const float *rope_cos, const float *rope_sin, int rows, int hq, const void *geom, int perm, void *q_out,
                                       void *stream) {
    using namespace pc;
    const KvGeom *kv = (const KvGeom *)geom;
    if (dtype < KD_F32 || dtype > KD_F16 || !qkv || !row_slot || !row_pos || !kv || !q_out || slices < 1 || slices > 8 || rows <= 0 ||
        kv->head_dim % 2 != 0 || (perm && kv->head_dim % 32 != 0))
        return 0;
    launch_rope_append(dtype, qkv, slices, row_slot, row_pos, nullptr, rope_cos, rope_sin, rows, hq, *kv, 0, q_out, nullptr, perm, (hipStream_t)stream);
    return 1;
}
