// Projection GEMMs with many rows (prefill, scoring, large decode batches; Section 3.1 policy pi_theta):
//   C[M,N] = A[M,K] * W[N,K]^T, fp32 accumulation, the epilogues of gemm.hip.
#include <algorithm>

#include "gemm_common.h"

namespace pc {

// 16x16x32 products whose accumulator lives in the accumulation registers (256 of a wave's 512 registers at one wave per
// SIMD).  Written out because the compiler, left to itself, keeps such accumulators in the other half and moves them back and
// forth (900 TFLOP/s at 8192^3 where this form reaches 1450).  `volatile` also keeps the order of the products and of the memory
// operations between them as they stand in the source.
// What the compiler does not see it does not keep apart either.  A product must not read a register less than two wait states
// after a vector-ALU instruction wrote it: its fragments come from LDS reads only, and where they are copied the copy is pinned
// to its place.  The results must not be read before the pipeline has drained (mma_drain).  tests/test_wait_states.py checks
// both on the generated code.
template <typename T> struct AccMma;
template <> struct AccMma<f16_t> {
    __device__ static inline void first(f16x8_t a, f16x8_t b, f32x4_t &c) {   // c = a b
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=a"(c) : "v"(a), "v"(b));
    }
    __device__ static inline void add(f16x8_t a, f16x8_t b, f32x4_t &c) {     // c += a b
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    }
};
template <> struct AccMma<bf16_t> {
    __device__ static inline void first(bf16x8_t a, bf16x8_t b, f32x4_t &c) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(a), "v"(b));
    }
    __device__ static inline void add(bf16x8_t a, bf16x8_t b, f32x4_t &c) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    }
};
__device__ inline f32x4_t acc_read(const f32x4_t &c) {
    f32x4_t v;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[0]) : "a"(c[0]));
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[1]) : "a"(c[1]));
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[2]) : "a"(c[2]));
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[3]) : "a"(c[3]));
    return v;
}
__device__ inline void mma_drain() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }
__device__ inline void code_fence() { asm volatile("" ::: "memory"); }

// Eight values to 16 bits, rounded to nearest even; what lies beyond the half range becomes infinite.
template <typename T> constexpr bool range_limited() { return false; }   // whether there is such a range
template <> constexpr bool range_limited<f16_t>() { return true; }
template <typename T> __device__ inline u32x4 pack8(const float (&x)[8]);
template <> __device__ inline u32x4 pack8<f16_t>(const float (&x)[8]) {
    typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
    u32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = __builtin_bit_cast(uint32_t, (f16x2){(_Float16)x[2 * e], (_Float16)x[2 * e + 1]});
    return r;
}
template <> __device__ inline u32x4 pack8<bf16_t>(const float (&x)[8]) {
    u32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = pack2<bf16_t>(x[2 * e], x[2 * e + 1]);
    return r;
}

// How the weight rows of a wave's strip are dealt to its column tiles, i.e. which output columns a lane ends up with.  Lane
// group g (lane / 16) of tile j holds, in element v, the product with weight row large_row(order, j, 4 g + v) of the strip.
enum LargeOrder {
    LO_PLAIN = 0,   // 16 j + r: four consecutive columns (fp32 stores of 16 bytes, row statistics)
    LO_PAIRED = 1,  // weight rows come in chunks of 32 = 16 + their 16 partners (gate and up; a head's dims and their rotary
                    // partners); four tiles (first, partner, first, partner) cover two chunks such that the lane's 2 x 4 values of
                    // either kind are eight consecutive ones: 16-byte stores of 16-bit results without a trip through LDS
};
PC_HD inline int large_row(int order, int j, int r) {
    if (order == LO_PLAIN) return 16 * j + r;
    const int o = 8 * (r / 4) + 4 * ((j / 2) % 2) + r % 4;           // place among the 32 firsts (partners) of the two chunks
    return 64 * (j / 4) + 32 * (o / 16) + 16 * (j % 2) + o % 16;
}

// Work decomposition: 256 threads, four waves in a square, one block per CU; a block computes a tile of 128 TMH/2 .. rows x
// columns after another (`run` of them), a wave a quarter of it, (32 TMH) x (32 TNH) outputs.
//
// Why this shape.  The products need 256 x 256 x 64 x 2 flop per 64 k, 2048 clocks of the matrix cores at best; the same tile on
// eight waves of 64 x 128 asks LDS for 192 KB of fragments per 64 k and 64 KB of fills, which takes about as long as the
// products and does not overlap with them entirely.  Four waves of 128 x 128 need 128 KB.  (8192^3 in half: eight waves 1190
// TFLOP/s, four 1450; the vendor's library 1476.)
//
// Data path: an operand tile of 64 k is cut into two units, the halves h = 0, 1 of every wave's rows (columns); A0, A1, W0, W1.
// A wave multiplies quadrant by quadrant, (A0 W0) (A0 W1) (A1 W1) (A1 W0), and while one quadrant's products run it reads the
// one unit that the next quadrant needs anew: W1, A1, then A0 and W0 of the next 64 k.  Units are fetched in that order too,
// two to a pair, into a ring of NP pairs in LDS (buffer loads that write LDS directly; the 16-byte chunk c of row r is stored at
// c ^ (r / 2) % 8, which makes fragment reads conflict free).  One barrier per pair: behind it the pair is there and the slot
// of the pair before it is free and takes the pair NP places on.  The ring runs on across output tiles: the last products of one
// run over the first loads of the next, so only a block's first tile waits for memory; a tile after that costs its products and
// its epilogue.  (Rows past the end read as zero through the buffer's bounds, stores past the end are dropped by them.)
template <typename T, int TMH, int TNH, int NP, int EPI>
__global__ __launch_bounds__(256, 1) void gemm_large_kernel(const T *__restrict__ A, const T *__restrict__ W, int lg,
                                                            void *__restrict__ Cv, int M, int N, int K, int mb, int nb,
                                                            int S, int bh, int run, uint32_t *__restrict__ sat,
                                                            typename GemmExtra<EPI>::type extra) {
#if defined(__HIP_DEVICE_COMPILE__)   // (the buffer descriptor's type does not exist in the host pass)
    constexpr int BM = 64 * TMH, BN = 64 * TNH, BK = 64, SM = BM / 2, SN = BN / 2;   // tile, K step, a wave's part
    constexpr int LA = BM / 64, LW = BN / 64, L = LA + LW;    // wave-wide 1 KB loads per wave for a unit of A, of W, for a pair
    constexpr int UA = SM * BK, PAIR = (SM + SN) * BK;        // elements
    constexpr bool SWIGLU = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_RS;
    constexpr int ORDER = (SWIGLU || EPI == EPI_QKV) ? LO_PAIRED : LO_PLAIN;
    static_assert(ORDER == LO_PLAIN || TNH % 2 == 0, "whole pairs of chunks per wave");
    static_assert(EPI == EPI_STORE_F32 || EPI == EPI_RESID_F32 || SWIGLU || EPI == EPI_QKV || EPI == EPI_LOGPROB, "epilogue");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    T *smem = (T *)smem_raw;
    constexpr size_t RING_BYTES = (size_t)NP * PAIR * sizeof(T);
    constexpr int V_PITCH = SN + 8;                           // (q/k/v: elements of a row of V under way to the cache)

    const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int wm = wave / 2, wn = wave % 2;

    struct Tile {   // (wave-uniform)
        int m0, n0, z, kt;
        const T *a, *w;
        uint32_t a_bytes, w_bytes;
    };
    const int KT = K / BK, per = (KT + S - 1) / S;
    auto locate = [&](int i, Tile &t) {
        int bm, bn;
        if (!gemm_band_tile(blockIdx.x, i, run, mb, nb, S, bh, &bm, &bn, &t.z)) return false;
        t.m0 = bm * BM;
        t.n0 = bn * BN;
        const int k0 = t.z * per;
        t.kt = min(KT, k0 + per) - k0;
        t.a = A + (int64_t)t.m0 * K + (int64_t)k0 * BK;
        t.w = W + (int64_t)t.n0 * K + (((int64_t)k0 * BK) << lg);   // (whole slabs)
        t.a_bytes = ((uint32_t)min(M - t.m0, BM) * (uint32_t)K - (uint32_t)(k0 * BK)) * 2u;   // up to the end of the last row
        t.w_bytes = ((uint32_t)min(N - t.n0, BN) * (uint32_t)K - ((uint32_t)(k0 * BK) << lg)) * 2u;
        return true;
    };

    // ---- global -> LDS: a wave-wide load fills 8 rows of 64 k; load i of wave w the unit's rows 32 i + 8 w .. + 7.
    // Row u of a unit of half h: rows (columns) of wave row (column) u / (S / 2), half h.
    const int lr = lane / 8, slot8 = lane % 8;
    uint32_t va[2][LA], vw[2][LW];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int u = 32 * i + 8 * wave + lr;
            const int row = (u / (SM / 2)) * SM + h * (SM / 2) + u % (SM / 2);
            va[h][i] = (uint32_t)row * (uint32_t)K * 2u + (uint32_t)(slot8 ^ ((u / 2) & 7)) * 16u;
        }
#pragma unroll
        for (int i = 0; i < LW; ++i) {
            const int u = 32 * i + 8 * wave + lr;
            const int in = h * (SN / 2) + u % (SN / 2);
            const int row = (u / (SN / 2)) * SN + large_row(ORDER, in / 16, in % 16);
            vw[h][i] = (uint32_t)weight_row(row, K, lg) * 2u + (uint32_t)(slot8 ^ ((u / 2) & 7)) * 16u;
        }
    }
    Tile cur, nxt;
    bool more = false;
    // load q of the unit of half h of K step t, counted from the current tile's first: steps past its end are the next tile's,
    // or nothing (a buffer of no bytes: the counter of loads in flight goes on, no memory is touched)
    auto load_a = [&](int t, int slot, int h, int q) {
        const bool in = t < cur.kt;
        const T *base = in ? cur.a : nxt.a;
        const uint32_t bytes = in ? cur.a_bytes : (more ? nxt.a_bytes : 0u);
        const int off = in ? t : (more ? t - cur.kt : 0);
        __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            r, (__attribute__((address_space(3))) void *)(smem + slot * PAIR + (32 * q + 8 * wave) * BK), 16, va[h][q], off * (BK * 2), 0, 0);
    };
    auto load_w = [&](int t, int slot, int h, int q) {
        const bool in = t < cur.kt;
        const T *base = in ? cur.w : nxt.w;
        const uint32_t bytes = in ? cur.w_bytes : (more ? nxt.w_bytes : 0u);
        const int off = in ? t : (more ? t - cur.kt : 0);
        __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            r, (__attribute__((address_space(3))) void *)(smem + slot * PAIR + UA + (32 * q + 8 * wave) * BK), 16, vw[h][q], off * (BK * 2) << lg, 0, 0);
    };

    // ---- LDS -> registers
    typedef typename Mma<T>::frag frag_t;
    const int fr = lane % 16, fg = lane / 16;
    int offa[2], offw[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const int o = fr * BK + (((4 * kk + fg) ^ ((fr / 2) & 7)) * 8);
        offa[kk] = o + wm * (SM / 2) * BK;
        offw[kk] = o + UA + wn * (SN / 2) * BK;
    }
    auto read_a = [&](int slot, frag_t (&f)[2][TMH], int q) {
        f[q / TMH][q % TMH] = *(const frag_t *)(smem + slot * PAIR + offa[q / TMH] + (q % TMH) * 16 * BK);
    };
    auto read_w = [&](int slot, frag_t (&f)[2][TNH], int q) {
        f[q / TNH][q % TNH] = *(const frag_t *)(smem + slot * PAIR + offw[q / TNH] + (q % TNH) * 16 * BK);
    };

    // ---- products
    f32x4_t acc[2 * TMH][2 * TNH];
    frag_t fa0[2][TMH], fa1[2][TMH], fbx[2][TNH], fby[2][TNH];
    constexpr int MM = 2 * TMH * TNH;   // products of a quadrant
    // one quadrant; NR fragment reads spread over its first half, NL loads over all of it
#define PC_QUADRANT(FIRST, FA, FB, HA, HB, NR, READ, NL, LOAD)                                              \
    do {                                                                                                    \
        constexpr int RS = (MM / 2) / (NR) > 1 ? (MM / 2) / (NR) : 1, LS = MM / (NL);               \
        _Pragma("unroll") for (int e = 0; e < MM; ++e) {                                                    \
            const int kk = e / (TMH * TNH), ti = (e / TNH) % TMH, tj = e % TNH;                             \
            f32x4_t &c = acc[HA * TMH + ti][HB * TNH + tj];                                                 \
            if (FIRST && kk == 0) AccMma<T>::first(FB[kk][tj], FA[kk][ti], c);                              \
            else AccMma<T>::add(FB[kk][tj], FA[kk][ti], c);                                                 \
            if (e % RS == RS - 1 && e / RS < (NR)) { const int q = e / RS; READ; }                          \
            if (e % LS == LS / 2 && e / LS < (NL)) { const int q = e / LS; LOAD; }                          \
        }                                                                                                   \
    } while (0)
    // The pair about to be read has landed when at most the loads of the NP - 2 pairs behind it are in flight.  (An epilogue's
    // stores count too; leaving them in flight over the first syncs of the next tile, or writing its results over the next
    // tile's first steps, gained nothing: what stores there are slow the loads wherever they stand.)
    auto sync = [&]() {
        wait_vmcnt_le<(NP - 2) * L>();
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's fragments are in registers
        code_fence();
        __builtin_amdgcn_s_barrier();         // (a bare one: __syncthreads() would drain the loads in flight)
        code_fence();
    };
    auto next = [&](int s) { return s + 1 == NP ? 0 : s + 1; };
    // Pairs in reading order: p = 2t: (W1, A1) of K step t; 2t + 1: (A0, W0) of step t + 1.  Behind the sync of pair p the slot of
    // pair p - 1 takes pair p - 1 + NP.
    constexpr int H0 = (NP % 2 == 0) ? 0 : 1, H1 = 1 - H0;   // the halves in pairs 2t - 1 + NP and 2t + NP
    auto step = [&](auto first, int t, int free, int s0, int s1, frag_t (&fb0)[2][TNH], frag_t (&fb1)[2][TNH]) {
        constexpr bool FIRST = decltype(first)::value;
        const int t0 = t + NP / 2, t1 = t + (NP + 1) / 2;
        sync();
        PC_QUADRANT(FIRST, fa0, fb0, 0, 0, 2 * TNH, read_w(s0, fb1, q), LA, load_a(t0, free, H0, q));
        PC_QUADRANT(FIRST, fa0, fb1, 0, 1, 2 * TMH, read_a(s0, fa1, q), LW, load_w(t0, free, H0, q));
        sync();
        PC_QUADRANT(FIRST, fa1, fb1, 1, 1, 2 * TMH, read_a(s1, fa0, q), LW, load_w(t1, s0, H1, q));
        PC_QUADRANT(FIRST, fa1, fb0, 1, 0, 2 * TNH, read_w(s1, fb1, q), LA, load_a(t1, s0, H1, q));
    };
#undef PC_QUADRANT
    if (!locate(0, cur)) return;
    nxt = cur;
    // q/k/v: sequence, position and cache block of the wave's rows, one or two to a lane.  Each is the address of the next; the
    // first tile's are fetched between its operand loads.
    constexpr int RL = EPI == EPI_QKV ? (SM + 63) / 64 : 1;
    int row_slot[RL], row_pos[RL], row_blk[RL];
    auto find_rows = [&](int stage) {
        if constexpr (EPI == EPI_QKV) {
#pragma unroll
            for (int r = 0; r < RL; ++r) {
                const int row = min(cur.m0 + wm * SM + 64 * r + lane, M - 1);
                if (stage == 0) row_slot[r] = extra.row_slot[row];
                if (stage == 1) row_pos[r] = extra.row_pos ? extra.row_pos[row] : extra.slot_len[row_slot[r]];
                if (stage == 2) row_blk[r] = extra.kv.block_table[(int64_t)row_slot[r] * extra.kv.max_blocks_per_slot + row_pos[r] / extra.kv.block_size];
            }
        }
    };
    // gate/up behind a norm: 1 / rms of the tile's rows, a thread to a row, from the row's sums of squares over 32 columns each.
    // Two tiles' worth in LDS: a wave may still be at the epilogue of one while the next one's are written.
    float *row_scale = (float *)(smem_raw + RING_BYTES);
    constexpr int RS_AHEAD = EPI == EPI_SWIGLU_RS ? 48 : 1;   // sums fetched at a time
    float sums[RS_AHEAD];
    auto fetch_sums = [&](int from) {   // (past the end: clamped, not left out; a branch around each load would make them wait for one another)
        if constexpr (EPI == EPI_SWIGLU_RS) {
            const int row = min(cur.m0 + tid, M - 1);
#pragma unroll
            for (int u = 0; u < RS_AHEAD; ++u) sums[u] = extra.ssq[(int64_t)min(from + u, extra.tiles - 1) * M + row];
        }
    };
    auto write_scale = [&](int which) {
        if constexpr (EPI == EPI_SWIGLU_RS) {
            float ss = 0.f;
            for (int from = 0;;) {
#pragma unroll
                for (int u = 0; u < RS_AHEAD; ++u) ss += from + u < extra.tiles ? sums[u] : 0.f;
                from += RS_AHEAD;
                if (from >= extra.tiles) break;
                fetch_sums(from);
            }
            if (tid < BM) row_scale[which * BM + tid] = 1.0f / sqrtf(ss / (float)extra.d + extra.eps);
        }
    };
    fetch_sums(0);
#pragma unroll
    for (int p = -1; p < NP - 1; ++p) {
        const int t = (p + 1) >> 1, h = (p & 1) ? 0 : 1;
        find_rows(p + 1);
#pragma unroll
        for (int q = 0; q < LA; ++q) load_a(t, p + 1, h, q);
#pragma unroll
        for (int q = 0; q < LW; ++q) load_w(t, p + 1, h, q);
    }
    write_scale(0);
    wait_vmcnt_le<(NP - 1) * L>();
    code_fence();
    __builtin_amdgcn_s_barrier();
    code_fence();
#pragma unroll
    for (int q = 0; q < 2 * TMH; ++q) read_a(0, fa0, q);
#pragma unroll
    for (int q = 0; q < 2 * TNH; ++q) read_w(0, fbx, q);

    int slot = 0;   // of the pair read last
    for (int i = 0;; ++i) {
        more = i + 1 < run && locate(i + 1, nxt);
        auto advance = [&](auto first, int t, frag_t (&fb0)[2][TNH], frag_t (&fb1)[2][TNH]) {
            const int s0 = next(slot), s1 = next(s0);
            step(first, t, slot, s0, s1, fb0, fb1);
            slot = s1;
        };
        advance(std::true_type{}, 0, fbx, fby);
        int t = 1;
        for (; t + 1 < cur.kt; t += 2) {
            advance(std::false_type{}, t, fby, fbx);
            advance(std::false_type{}, t + 1, fbx, fby);
        }
        if (t < cur.kt) {
            advance(std::false_type{}, t, fby, fbx);
        } else {   // an odd number of steps: the next tile's first W fragments are in the other set
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int j = 0; j < TNH; ++j) {
                    fbx[kk][j] = fby[kk][j];
                    asm volatile("" : "+v"(fbx[kk][j]));   // (made here, not between the products that read it)
                }
        }
        mma_drain();
#pragma unroll
        for (int i2 = 0; i2 < 2 * TMH; ++i2)
#pragma unroll
            for (int j = 0; j < 2 * TNH; ++j) asm volatile("" : "+a"(acc[i2][j]));
        if (!more) wait_vmcnt_le<0>();   // nothing may still be writing LDS when the block retires
        code_fence();

        // ---- epilogue: lane (ml, g) owns row ml of every row tile; of column tile j the four columns of large_row(j, 4g ..)
        // (rolled up by row tiles, their values taken out of the accumulation registers by a branch each: written out, an epilogue
        // is 10 to 20 KB of code that runs once per tile, and fetching it took longer than executing it)
        const int ml = lane % 16, g = lane / 16;
        auto take = [&](int i2, f32x4_t (&v)[2 * TNH]) {
#pragma unroll
            for (int k = 0; k < 2 * TMH; ++k)
                if (i2 == k) {
#pragma unroll
                    for (int j = 0; j < 2 * TNH; ++j) v[j] = acc_read(acc[k][j]);
                }
        };
        const int m0 = cur.m0 + wm * SM, n0 = cur.n0 + wn * SN;   // the wave's first row and column
        if constexpr (EPI == EPI_STORE_F32 || EPI == EPI_RESID_F32) {
            float *C = (float *)Cv + ((EPI == EPI_STORE_F32) ? (int64_t)cur.z * M * N : 0) + (int64_t)cur.m0 * N;
            __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc((void *)C, 0, (int)((uint32_t)min(M - cur.m0, BM) * (uint32_t)N * 4u), 0x00020000);
            auto place = [&](uint32_t row_off, int j) {   // of the lane's four columns of tile j
                const int col = n0 + 16 * j + 4 * g;
                return (int)(col < N ? row_off + (uint32_t)col * 4u : 0xFFFFFFF0u);
            };
            uint32_t row_off = (uint32_t)(wm * SM + ml) * (uint32_t)N * 4u;
            if constexpr (EPI == EPI_STORE_F32) {
#pragma unroll
                for (int i2 = 0; i2 < 2 * TMH; ++i2) {
#pragma unroll
                    for (int j = 0; j < 2 * TNH; ++j)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i2][j]), rc, place(row_off, j), 0, 0);
                    row_off += 16u * (uint32_t)N * 4u;
                }
            } else {
                constexpr int D = TMH;   // row tiles whose old values are under way
                u32x4 old[D][2 * TNH];
                const uint32_t tile_off = 16u * (uint32_t)N * 4u;
#pragma unroll
                for (int d = 0; d < D; ++d)
#pragma unroll
                    for (int j = 0; j < 2 * TNH; ++j)
                        old[d][j] = __builtin_amdgcn_raw_buffer_load_b128(rc, place(row_off + d * tile_off, j), 0, 0);
#pragma unroll
                for (int i2 = 0; i2 < 2 * TMH; ++i2) {
#pragma unroll
                    for (int j = 0; j < 2 * TNH; ++j) {
                        const f32x4_t sum = __builtin_bit_cast(f32x4_t, old[i2 % D][j]) + acc_read(acc[i2][j]);
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, sum), rc, place(row_off, j), 0, 0);
                        if (i2 + D < 2 * TMH)
                            old[i2 % D][j] = __builtin_amdgcn_raw_buffer_load_b128(rc, place(row_off + D * tile_off, j), 0, 0);
                    }
                    row_off += tile_off;
                }
            }
        } else if constexpr (SWIGLU) {
            const int ldc = N / 2;
            T *C = (T *)Cv + (int64_t)cur.m0 * ldc;
            __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc((void *)C, 0, (int)((uint32_t)min(M - cur.m0, BM) * (uint32_t)ldc * 2u), 0x00020000);
            uint32_t row_off = (uint32_t)(wm * SM + ml) * (uint32_t)ldc * 2u;
#pragma unroll 1
            for (int i2 = 0; i2 < 2 * TMH; ++i2) {
                f32x4_t x[2 * TNH];
                take(i2, x);
                if constexpr (EPI == EPI_SWIGLU_RS) {
                    const float scale = row_scale[(i % 2) * BM + wm * SM + 16 * i2 + ml];
#pragma unroll
                    for (int j = 0; j < 2 * TNH; ++j) x[j] *= scale;
                }
                // converted unchecked, and again with clamps and their count if anything of the row tile may be beyond the half range
                u32x4 out[TNH / 2];
                float sum = 0.f;
#pragma unroll
                for (int c = 0; c < TNH / 2; ++c) {
                    float y[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        y[e] = silu_mul(x[4 * c + 2 * (e / 4)][e % 4], x[4 * c + 2 * (e / 4) + 1][e % 4]);
                        sum += fabsf(y[e]);
                    }
                    out[c] = pack8<T>(y);
                }
                if (range_limited<T>() && !__all(sum <= 65504.f)) {
#pragma unroll
                    for (int c = 0; c < TNH / 2; ++c) {
                        // clamps are counted where stored
                        uint32_t *const count = n0 / 2 + 32 * c + 8 * g < ldc && m0 + 16 * i2 + ml < M ? sat : nullptr;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const f32x4_t &ga = x[4 * c + 2 * (e / 2)], &ua = x[4 * c + 2 * (e / 2) + 1];
                            out[c][e] = pack2_sat<T>(silu_mul(ga[2 * (e % 2)], ua[2 * (e % 2)]),
                                                     silu_mul(ga[2 * (e % 2) + 1], ua[2 * (e % 2) + 1]), count);
                        }
                    }
                }
#pragma unroll
                for (int c = 0; c < TNH / 2; ++c) {
                    const int col = n0 / 2 + 32 * c + 8 * g;
                    __builtin_amdgcn_raw_buffer_store_b128(out[c], rc, (int)(col < ldc ? row_off + (uint32_t)col * 2u : 0xFFFFFFF0u), 0, 0);
                }
                row_off += 16u * (uint32_t)ldc * 2u;
            }
        } else if constexpr (EPI == EPI_QKV) {
            // a wave's columns lie within one head (128 of them, or its first or second 64)
            static_assert(128 % SN == 0, "a strip lies within one head");
            if (n0 < N) {
                const int hkv = extra.kv.n_kv_heads, bs = extra.kv.block_size;
                const int qd = extra.hq * 128, kvd = hkv * 128;
                const int part = n0 < qd ? 0 : (n0 < qd + kvd ? 1 : 2);   // q, k, v (wave-uniform)
                const int pc0 = n0 - (part == 0 ? 0 : (part == 1 ? qd : qd + kvd));
                const int head = pc0 / 128, in = pc0 % 128;               // first column inside the head
                T *pool = (T *)extra.kv.pool + (int64_t)extra.layer * extra.kv.layer_stride + (int64_t)head * extra.kv.head_elems();
                auto of_row = [&](const int (&v)[RL], int r) {            // what lane r % 64 holds for row r of the wave's
                    int x = __shfl(v[0], r % 64, 64);
                    if constexpr (RL == 2) {
                        const int y = __shfl(v[1], r % 64, 64);
                        x = r < 64 ? x : y;
                    }
                    return x;
                };
                if (part == 2) {
                    // A token's 128 dims lie 16 bytes apart in the cache: whole rows are re-formed in LDS, so that one store covers 64
                    // dims of one token (8 cache lines) and not one dim of 16 tokens and 4 groups (64 lines)
                    T *stg = (T *)(smem_raw + RING_BYTES) + wave * 16 * V_PITCH;
#pragma unroll 1
                    for (int i2 = 0; i2 < 2 * TMH; ++i2) {
                        f32x4_t x[2 * TNH];
                        take(i2, x);
                        uint32_t *const count = m0 + 16 * i2 + ml < M ? sat : nullptr;   // clamps are counted where stored
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int c = 0; c < TNH / 2; ++c)
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const f32x4_t &x1 = x[4 * c + h], &x2 = x[4 * c + 2 + h];
                                const u32x2 lo = pack4_sat<T>(x1[0], x1[1], x1[2], x1[3], count);
                                const u32x2 hi = pack4_sat<T>(x2[0], x2[1], x2[2], x2[3], count);
                                *(u32x4 *)(stg + ml * V_PITCH + large_row(ORDER, 4 * c + h, 4 * g)) = (u32x4){lo[0], lo[1], hi[0], hi[1]};
                            }
                        __builtin_amdgcn_wave_barrier();
                        const int pos16 = of_row(row_pos, 16 * i2 + ml), blk16 = of_row(row_blk, 16 * i2 + ml);
                        const int left = min(16, M - m0 - 16 * i2);
#pragma unroll 1
                        for (int r4 = 0; r4 < left; r4 += 4)
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const int r = min(r4 + k, left - 1);   // (past the end: the last row once more)
                            const int tin = __builtin_amdgcn_readlane(pos16, r) % bs;
                            T *block = pool + (int64_t)__builtin_amdgcn_readlane(blk16, r) * extra.kv.block_elems();
#pragma unroll
                            for (int d = 0; d < SN / 64; ++d)
                                block[extra.kv.v_index(tin, in + 64 * d + lane)] = stg[r * V_PITCH + 64 * d + lane];
                        }
                    }
                } else {
                    f32x4_t cs[TNH / 2][2], sn[TNH / 2][2];               // of the lane's eight pair indices per chunk, for the row tile to come
                    auto rotation = [&](int pos) {
#pragma unroll
                        for (int c = 0; c < TNH / 2; ++c)
#pragma unroll
                            for (int s = 0; s < 2; ++s) {
                                const int64_t at = (int64_t)pos * 64 + in / 2 + 32 * c + 8 * g + 4 * s;
                                cs[c][s] = *(const f32x4_t *)(extra.rope_cos + at);
                                sn[c][s] = *(const f32x4_t *)(extra.rope_sin + at);
                            }
                    };
                    int pos = of_row(row_pos, ml);
                    rotation(pos);
#pragma unroll 1
                    for (int i2 = 0; i2 < 2 * TMH; ++i2) {
                        f32x4_t x[2 * TNH];
                        take(i2, x);
                        const int row = m0 + 16 * i2 + ml;
                        const int blk = of_row(row_blk, 16 * i2 + ml), tin = pos % bs;
                        uint32_t *const count = row < M ? sat : nullptr;
                        u32x2 lo[TNH / 2][2], hi[TNH / 2][2];
#pragma unroll
                        for (int c = 0; c < TNH / 2; ++c)
#pragma unroll
                            for (int s = 0; s < 2; ++s) {
                                const f32x4_t &x1 = x[4 * c + 2 * s], &x2 = x[4 * c + 2 * s + 1], &k = cs[c][s], &n = sn[c][s];
                                lo[c][s] = pack4_sat<T>(rotated_first(x1[0], x2[0], k[0], n[0]), rotated_first(x1[1], x2[1], k[1], n[1]),
                                                        rotated_first(x1[2], x2[2], k[2], n[2]), rotated_first(x1[3], x2[3], k[3], n[3]), count);
                                hi[c][s] = pack4_sat<T>(rotated_second(x1[0], x2[0], k[0], n[0]), rotated_second(x1[1], x2[1], k[1], n[1]),
                                                        rotated_second(x1[2], x2[2], k[2], n[2]), rotated_second(x1[3], x2[3], k[3], n[3]), count);
                            }
                        pos = of_row(row_pos, min(16 * i2 + 16, SM - 16) + ml);
                        rotation(pos);
                        if (row >= M) continue;
                        T *block = pool + (int64_t)blk * extra.kv.block_elems();
#pragma unroll
                        for (int c = 0; c < TNH / 2; ++c) {
                            const int j0 = in / 2 + 32 * c + 8 * g;
                            T *dst = part == 0 ? (T *)extra.q_out + ((int64_t)row * extra.hq + head) * 128 : block;
                            *(u32x4 *)(dst + (part == 0 ? j0 : extra.kv.k_index(tin, j0))) =   // (eight dims are contiguous in both)
                                (u32x4){lo[c][0][0], lo[c][0][1], lo[c][1][0], lo[c][1][1]};
                            *(u32x4 *)(dst + (part == 0 ? j0 + 64 : extra.kv.k_index(tin, j0 + 64))) =
                                (u32x4){hi[c][0][0], hi[c][0][1], hi[c][1][0], hi[c][1][1]};
                        }
                    }
                }
            }
        } else {
            // EPI_LOGPROB: maximum and, in double, sum of the exponentials of a row over the wave's strip of columns; the lane's
            // three partners (16, 32, 48 lanes on) hold the rest of the row's strip
            const int64_t strip = (int64_t)(n0 / SN);
            const int nq = 4 * g;
#pragma unroll 1
            for (int i2 = 0; i2 < 2 * TMH; ++i2) {
                f32x4_t x[2 * TNH];
                take(i2, x);
                const int row = m0 + 16 * i2 + ml;
                const int want = row < M ? extra.tokens[extra.token_index[row] + 1] - n0 - nq : -1;   // (column - nq) of the target
                if (__any(want >= 0 && want < SN)) {   // (rare: a row's target is in one of a thousand strips)
#pragma unroll
                    for (int j = 0; j < 2 * TNH; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (want == j * 16 + v && n0 + j * 16 < N) extra.target[row] = x[j][v];
                }
                float mx = -INFINITY;
#pragma unroll
                for (int j = 0; j < 2 * TNH; ++j) {
                    x[j] *= extra.inv_t;
                    if (n0 + j * 16 < N) mx = fmaxf(mx, fmaxf(fmaxf(x[j][0], x[j][1]), fmaxf(x[j][2], x[j][3])));   // N is a multiple of 16
                }
                mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                const float base = (mx == -INFINITY) ? 0.f : mx;
                double s = 0.0;
#pragma unroll
                for (int j = 0; j < 2 * TNH; ++j)
                    if (n0 + j * 16 < N) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) s += (double)exp_neg(x[j][v] - base);
                    }
                s += __shfl_xor(s, 16, 64);
                s += __shfl_xor(s, 32, 64);
                if (row < M && nq == 0) {
                    extra.part_max[strip * M + row] = mx;
                    extra.part_sum[strip * M + row] = s;
                }
            }
        }
        code_fence();
        if (!more) break;
        cur = nxt;
#pragma unroll
        for (int stage = 0; stage < 3; ++stage) find_rows(stage);
        fetch_sums(0);
        write_scale((i + 1) % 2);
    }
#endif
}

// The tiles, and in which of them an epilogue exists (one bit each).  LT_EIGHT: not here, but the 256 x 128 tile on eight waves of
// gemm_mfma, whose epilogues take fewer values per lane.
enum { LT_256x256, LT_256x192, LT_192x256, LT_256x128, LT_192x128, LT_128x128, LT_COUNT, LT_EIGHT = LT_COUNT };
constexpr int LARGE_SHAPES[LT_COUNT + 1][2] = {{256, 256}, {256, 192}, {192, 256}, {256, 128}, {192, 128}, {128, 128}, {256, 128}};
constexpr unsigned large_tiles(int epi) {
    return epi == EPI_STORE_F32 || epi == EPI_RESID_F32 ? (1u << LT_COUNT) - 1
           : epi == EPI_SWIGLU                          ? 1u << LT_256x256 | 1u << LT_192x256 | 1u << LT_192x128
           : epi == EPI_QKV                             ? 1u << LT_256x256 | 1u << LT_192x256 | 1u << LT_192x128
           : epi == EPI_SWIGLU_RS || epi == EPI_LOGPROB ? 1u << LT_256x256 | 1u << LT_192x256
                                                        : 0u;
}

template <typename T, int TMH, int TNH> struct LargeCfg {
    static constexpr int BM = 64 * TMH, BN = 64 * TNH, NP = 4;
    template <int E> static constexpr size_t smem() {   // a pair of units holds half of the rows, 2 bytes an element
        return (size_t)NP * (BM + BN) * 64 + (E == EPI_QKV ? (size_t)4 * 16 * (BN / 2 + 8) * 2 : 0) +
               (E == EPI_SWIGLU_RS ? (size_t)2 * BM * sizeof(float) : 0);
    }
    template <int E> static void set_attr() {
        (void)hipFuncSetAttribute((const void *)gemm_large_kernel<T, TMH, TNH, NP, E>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem<E>());
    }
    template <int E>
    static void launch(const void *A, WeightRef W, void *C, int M, int N, int K, int S, uint32_t *sat, hipStream_t s,
                       const typename GemmExtra<E>::type &extra) {
        const int mb = (M + BM - 1) / BM, nb = (N + BN - 1) / BN;
        int bh, run;
        const unsigned grid = gemm_band_grid(mb, nb, S, &bh, &run);
        gemm_large_kernel<T, TMH, TNH, NP, E><<<grid, 256, smem<E>(), s>>>((const T *)A, (const T *)W.p, W.lg, C, M, N, K, mb, nb, S, bh, run, sat, extra);
    }
};

// ---- which tile, how many K slices
// Estimated microseconds of a launch: rounds of blocks (one per CU) times K steps times the time of a step, plus what the first and
// each further tile of a block cost beside their steps, plus the fp32 results' way to the kernel that reads them.  A step takes
// longer the more CUs are busy (`load`: the clock falls under the matrix cores' power, 2.0 PFLOP/s on operands of zeros and 1.45 on
// random ones).  The constants are a least-squares fit, then moved a little for least regret, to the times of 1094 launches of 513 to
// 16384 rows x 512 to 151936 columns x 128 to 17408, each in every tile and up to 8 slices, with weights in plain rows whose values repeated (and let
// the clock rise).  Held against times on mixed values in slabs and, for residual projections, with the eight-wave tiles among the forms
// (profiles/large_tile_times.txt and resid_tile_times.txt, taken by kernel_bench tiles; tests/test_tile_choice.py) what runs takes 1.0 % longer on average than the
// fastest form, 9 % at worst from K = 1024 up (640 x 24576 x 4096, 138 us for 126) and 31 % below (16384 x 2368 x 256, 35 us for 27).  (One
// set of constants for all epilogues, fitted without the norm that reads the slices and to K of 1536 and more, was up to 28 % off there
// and 60 % below: 640 rows x 2560 x 9728 58.2 us for 44.5.)
struct LargeTime {
    double step, load, first, next;
};
static const LargeTime LARGE_TIMES[LT_COUNT + 1] = {{0.96, 0.274, 12.1, 2.98}, {0.78, 0.269, 11.1, 1.99}, {0.794, 0.235, 10.8, 2.03},
                                                    {0.591, 0.171, 8.87, 1.65}, {0.54, 0.150, 8.01, 1.03}, {0.478, 0.173, 7.85, 0.902},
                                                    {0.619, 0.248, 5.61, 4.05}};
struct LargeEpilogue {
    double first, next;   // times those of the tile
};
static LargeEpilogue large_epilogue(int id, int epi) {
    if (id == LT_EIGHT) return epi == EPI_QKV ? LargeEpilogue{2.34, 2.13} : LargeEpilogue{1.0, 1.0};
    switch (epi) {
        case EPI_RESID_F32: return {1.32, 2.97};
        case EPI_SWIGLU: case EPI_SWIGLU_RS: return {0.694, 1.61};
        case EPI_QKV: return {2.46, 2.88};
        case EPI_LOGPROB: return {1.24, 3.72};
        default: return {1.35, 2.79};
    }
}
// `decode`: q/k/v of rows that all belong to different sequences, whose keys and values go all over the cache.  `read_back`: fp32
// results of which a kernel behind this one reads all slices.
static double large_cost(int id, int S, int M, int N, int K, int epi, bool decode, bool read_back) {
    const LargeTime &t = LARGE_TIMES[id];
    const LargeEpilogue e = large_epilogue(id, S > 1 ? (int)EPI_STORE_F32 : epi);
    const int bm = LARGE_SHAPES[id][0], bn = LARGE_SHAPES[id][1];
    const int KT = K / 64, per = (KT + S - 1) / S;
    const int64_t tiles = (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * S, rounds = (tiles + 255) / 256;
    const double busy = (double)tiles / (256.0 * (double)rounds), mb = (double)M * N * 4e-6;
    return (double)rounds * per * t.step * (1.0 + t.load * busy * busy) + t.first * e.first + (double)(rounds - 1) * t.next * e.next +
           (read_back ? 0.39 * S * mb : 0.0) + (decode ? (id == LT_EIGHT ? 10.5 : 2.1) : 0.0);
}
// The tiles that a launch of this epilogue chooses from.  (The eight waves win where the epilogue is much of the launch: q/k/v, and
// gate/up of short reductions, 1280 rows x 6400 x 128 7.9 us against 9.6, x 768 15.5 against 18.5.)
static unsigned large_choice(int epi) {
    return large_tiles(epi) | (epi == EPI_SWIGLU || epi == EPI_QKV ? 1u << LT_EIGHT : 0u);
}
// (two steps at least to a slice: the ring reaches that far ahead)
static bool large_slices_ok(int S, int K) {
    const int KT = K / 64, per = (KT + S - 1) / S;
    return S == 1 || (per >= 4 && KT - (S - 1) * per >= 2);
}
static int large_pick(int max_slices, int M, int N, int K, int epi, int *S, bool decode = false, bool read_back = false) {
    int best = -1;
    double best_cost = 0.0;
    for (int id = 0; id <= LT_EIGHT; ++id)
        for (int n = 1; n <= max_slices && (large_choice(epi) >> id & 1); ++n) {
            if (!large_slices_ok(n, K)) continue;
            const double c = large_cost(id, n, M, N, K, epi, decode, read_back);
            if (best < 0 || c < best_cost) {
                best = id;
                best_cost = c;
                *S = n;
            }
        }
    // (gate/up in three whole rounds of the eight-wave tile where the larger one half-fills its second: 1024 x 24576 x 4096 168.5 us
    // against 176.8, 1280 x 19456 x 2560 112.8 and 117.1; on another card 153.0, 153.7 and 101.3, 104.4)
    auto fill = [&](int bm, int bn) {
        const int64_t tiles = (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        return (double)tiles / (256.0 * (double)((tiles + 255) / 256));
    };
    if (epi == EPI_SWIGLU && best == LT_256x256 && K >= 2048 && fill(256, 128) > 0.98 && fill(256, 256) < 0.77) best = LT_EIGHT;
    return best;
}

// The tile and the slices of a projection whose consumer adds up the latter, if there is room for them.
static int large_pick_sliced(int M, int N, int K, int epi, const float *slices, size_t slice_cap, int *S) {
    const int max_slices = slices ? (int)std::min<size_t>(8, slice_cap / ((size_t)M * N)) : 1;
    return large_pick(std::max(1, max_slices), M, N, K, epi, S, false, epi == EPI_RESID_F32 || slices);
}
int gemm_large_resid_slices(int M, int N, int K, const float *slices, size_t slice_cap) {
    int S = 1;
    (void)large_pick_sliced(M, N, K, EPI_RESID_F32, slices, slice_cap, &S);
    return S;
}

static bool large_ok(const void *A, WeightRef W, const void *C, int M, int N, int K, int epi) {
    // (two steps of K at least, the ring reaches that far ahead; rows of operands and results in whole 16-byte pieces, but fp32
    // results may start at any float: the logits are the caller's; a tile's bytes within a buffer descriptor's 32 bits)
    return K % 64 == 0 && K >= 128 && N % 16 == 0 && (((uintptr_t)A | (uintptr_t)W.p) & 15) == 0 && ((uintptr_t)C & (epi == EPI_STORE_F32 ? 3 : 15)) == 0 &&
           K <= (1 << 21) && N <= (1 << 21);
}

template <typename T> struct Large {
    template <typename F> static void with_tile(int id, F f) {
        switch (id) {
            case LT_256x256: f(LargeCfg<T, 4, 4>()); break;
            case LT_256x192: f(LargeCfg<T, 4, 3>()); break;
            case LT_192x256: f(LargeCfg<T, 3, 4>()); break;
            case LT_256x128: f(LargeCfg<T, 4, 2>()); break;
            case LT_192x128: f(LargeCfg<T, 3, 2>()); break;
            case LT_128x128: f(LargeCfg<T, 2, 2>()); break;
        }
    }
    template <int E, typename Cfg> static constexpr bool built() {
        for (int id = 0; id < LT_COUNT; ++id)
            if (LARGE_SHAPES[id][0] == Cfg::BM && LARGE_SHAPES[id][1] == Cfg::BN) return large_tiles(E) >> id & 1;
        return false;
    }
    template <int E> static void init_epilogue() {
        for (int id = 0; id < LT_COUNT; ++id)
            with_tile(id, [](auto cfg) {
                if constexpr (built<E, decltype(cfg)>()) decltype(cfg)::template set_attr<E>();
            });
    }
    static void init() {
        init_epilogue<EPI_STORE_F32>(); init_epilogue<EPI_RESID_F32>(); init_epilogue<EPI_SWIGLU>();
        init_epilogue<EPI_SWIGLU_RS>(); init_epilogue<EPI_QKV>(); init_epilogue<EPI_LOGPROB>();
    }
    template <int E>
    static void launch(int id, const void *A, WeightRef W, void *C, int M, int N, int K, int S, uint32_t *sat, hipStream_t s,
                       const typename GemmExtra<E>::type &extra) {
        with_tile(id, [&](auto cfg) {
            if constexpr (built<E, decltype(cfg)>()) decltype(cfg)::template launch<E>(A, W, C, M, N, K, S, sat, s, extra);
        });
    }
    static int gemm(const void *A, WeightRef W, void *C, int M, int N, int K, int epi, float *slices, size_t slice_cap, uint32_t *sat,
                    hipStream_t s, const GemmRowScale *row_scale) {
        int S = 1;
        if (epi == EPI_SWIGLU_RS || epi == EPI_SWIGLU) {
            const int id = large_pick(1, M, N, K, epi, &S);
            if (id == LT_EIGHT) return 0;
            if (epi == EPI_SWIGLU) launch<EPI_SWIGLU>(id, A, W, C, M, N, K, 1, sat, s, {});
            else launch<EPI_SWIGLU_RS>(id, A, W, C, M, N, K, 1, sat, s, *row_scale);
            return 1;
        }
        // (the vocabulary projection of a decode step, whose time is half the weights' way from memory, which the estimate leaves out:
        // the shortest tile that holds the rows in one or two blocks, its figures stand at the rule that leads here)
        if (M <= 512 && epi == EPI_STORE_F32 && !slices) {
            launch<EPI_STORE_F32>(M <= 256 ? LT_256x128 : (M <= 384 ? LT_192x256 : LT_256x256), A, W, C, M, N, K, 1, sat, s, {});
            return 1;
        }
        const int id = large_pick_sliced(M, N, K, epi, slices, slice_cap, &S);
        if (S > 1) launch<EPI_STORE_F32>(id, A, W, slices, M, N, K, S, sat, s, {});
        else if (epi == EPI_RESID_F32) launch<EPI_RESID_F32>(id, A, W, C, M, N, K, 1, sat, s, {});
        else launch<EPI_STORE_F32>(id, A, W, C, M, N, K, 1, sat, s, {});
        return S;
    }
    static bool qkv(const void *A, WeightRef W, int M, int N, int K, const GemmQkv &q, uint32_t *sat, hipStream_t s) {
        int S = 1;
        const int id = large_pick(1, M, N, K, EPI_QKV, &S, !q.row_pos);
        if (id == LT_EIGHT) return false;
        launch<EPI_QKV>(id, A, W, nullptr, M, N, K, 1, sat, s, q);
        return true;
    }
    static int logprob(const void *A, WeightRef W, int M, int N, int K, const GemmLogprob &lp, hipStream_t s) {
        int S = 1;
        launch<EPI_LOGPROB>(large_pick(1, M, N, K, EPI_LOGPROB, &S), A, W, nullptr, M, N, K, 1, nullptr, s, lp);
        return (N + 255) / 256 * 2;   // strips of 128 columns
    }
    // `extra`: the epilogue's own arguments, if it has any
    static void named(int id, int epi, const void *A, WeightRef W, void *C, int M, int N, int K, int S, const void *extra, uint32_t *sat,
                      hipStream_t s) {
        switch (epi) {
            case EPI_STORE_F32: launch<EPI_STORE_F32>(id, A, W, C, M, N, K, S, sat, s, {}); break;
            case EPI_RESID_F32: launch<EPI_RESID_F32>(id, A, W, C, M, N, K, 1, sat, s, {}); break;
            case EPI_SWIGLU: launch<EPI_SWIGLU>(id, A, W, C, M, N, K, 1, sat, s, {}); break;
            case EPI_SWIGLU_RS: launch<EPI_SWIGLU_RS>(id, A, W, C, M, N, K, 1, sat, s, *(const GemmRowScale *)extra); break;
            case EPI_QKV: launch<EPI_QKV>(id, A, W, nullptr, M, N, K, 1, sat, s, *(const GemmQkv *)extra); break;
            case EPI_LOGPROB: launch<EPI_LOGPROB>(id, A, W, nullptr, M, N, K, 1, nullptr, s, *(const GemmLogprob *)extra); break;
        }
    }
};

void gemm_large_init() {
    Large<bf16_t>::init();
    Large<f16_t>::init();
}

int launch_gemm_large(int dtype, const void *A, WeightRef W, void *C, int M, int N, int K, int epi, float *slices, size_t slice_cap,
                      uint32_t *sat, hipStream_t s, const GemmRowScale *row_scale) {
    const bool swiglu = epi == EPI_SWIGLU || epi == EPI_SWIGLU_RS;
    if ((epi != EPI_STORE_F32 && epi != EPI_RESID_F32 && !swiglu) || !large_ok(A, W, C, M, N, K, epi) || ((uintptr_t)slices & 15) != 0 ||
        (swiglu && N % 64 != 0) || (epi == EPI_SWIGLU_RS && !row_scale))
        return 0;
    if (dtype == KD_BF16) return Large<bf16_t>::gemm(A, W, C, M, N, K, epi, slices, slice_cap, sat, s, row_scale);
    return Large<f16_t>::gemm(A, W, C, M, N, K, epi, slices, slice_cap, sat, s, row_scale);
}

bool launch_gemm_large_qkv(int dtype, const void *A, WeightRef W, int M, int N, int K, const GemmQkv &q, uint32_t *sat, hipStream_t s) {
    if (!large_ok(A, W, nullptr, M, N, K, EPI_QKV)) return false;
    return dtype == KD_BF16 ? Large<bf16_t>::qkv(A, W, M, N, K, q, sat, s) : Large<f16_t>::qkv(A, W, M, N, K, q, sat, s);
}

int launch_gemm_large_logprob(int dtype, const void *A, WeightRef W, int M, int N, int K, const GemmLogprob &lp, hipStream_t s) {
    if (!large_ok(A, W, nullptr, M, N, K, EPI_LOGPROB)) return 0;
    return dtype == KD_BF16 ? Large<bf16_t>::logprob(A, W, M, N, K, lp, s) : Large<f16_t>::logprob(A, W, M, N, K, lp, s);
}

}   // namespace pc

namespace pc {
static int large_by_name(int dtype, int bm, int bn, int epi, int slices, const void *A, WeightRef w, void *C, int M, int N, int K, const void *extra,
                         uint32_t *sat, void *stream) {
    const bool swiglu = epi == EPI_SWIGLU || epi == EPI_SWIGLU_RS, own = epi == EPI_SWIGLU_RS || epi == EPI_QKV || epi == EPI_LOGPROB;
    for (int id = 0; id < LT_COUNT; ++id) {
        if (LARGE_SHAPES[id][0] != bm || LARGE_SHAPES[id][1] != bn || epi < 0 || !(large_tiles(epi) >> id & 1)) continue;
        if ((dtype != KD_BF16 && dtype != KD_F16) || !A || !w.p || (!C && epi != EPI_QKV && epi != EPI_LOGPROB) || (own && !extra) || M <= 0 ||
            N <= 0 || (w.lg && !weight_lg(dtype, N, K)) || !large_ok(A, w, C, M, N, K, epi) || (swiglu && N % 64 != 0) ||
            (epi == EPI_QKV && N % 128 != 0) || slices < 1 || (slices > 1 && epi != EPI_STORE_F32) || !large_slices_ok(slices, K))
            return 0;
        gemm_large_init();
        if (dtype == KD_BF16) Large<bf16_t>::named(id, epi, A, w, C, M, N, K, slices, extra, sat, (hipStream_t)stream);
        else Large<f16_t>::named(id, epi, A, w, C, M, N, K, slices, extra, sat, (hipStream_t)stream);
        return 1;
    }
    return 0;
}
}   // namespace pc
// For tests, not part of the C ABI: one launch in the tile of bm rows x bn columns, W in plain rows or (_slabs) in the order of the 16-bit
// copies (`extra`: the GemmRowScale, GemmQkv or GemmLogprob of such an epilogue).  1: launched; 0: no such tile with this epilogue, or not a
// call that the kernels take.
extern "C" int pc_internal_gemm_large(int dtype, int bm, int bn, int epi, int slices, const void *A, const void *W, void *C, int M, int N,
                                      int K, const void *extra, uint32_t *sat, void *stream) {
    return pc::large_by_name(dtype, bm, bn, epi, slices, A, pc::WeightRef(W, 0), C, M, N, K, extra, sat, stream);
}
extern "C" int pc_internal_gemm_large_slabs(int dtype, int bm, int bn, int epi, int slices, const void *A, const void *W, void *C, int M, int N,
                                            int K, const void *extra, uint32_t *sat, void *stream) {
    return pc::large_by_name(dtype, bm, bn, epi, slices, A, pc::WeightRef(W, pc::WEIGHT_SLAB), C, M, N, K, extra, sat, stream);
}
// The tile (its place in the list above; LT_EIGHT: gemm_mfma's) and the number of K slices that the estimate chooses, up to
// max_slices where there is room for slices (0: there is none).
extern "C" int pc_internal_gemm_large_pick(int epi, int decode, int max_slices, int M, int N, int K, int *slices) {
    *slices = 1;
    return pc::large_pick(max_slices > 1 ? max_slices : 1, M, N, K, epi, slices, decode != 0, max_slices > 0 || epi == pc::EPI_RESID_F32);
}
