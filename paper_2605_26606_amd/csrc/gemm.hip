// Projection GEMMs of the decoder (Section 3.1 policy pi_theta):
//   C[M,N] = A[M,K] * W[N,K]^T, fp32 accumulation, with fused epilogues.
// Three implementations here:
//   gemm_f32    fp32 matrix instructions, operands straight from memory (fp32 models)
//   gemm_simt   plain-ALU tiles, any dtype, any K
//   gemm_mfma   bf16 / f16 on the matrix cores (32x32x16 or 16x16x32 products),
//               operands streamed global -> LDS several K tiles ahead, one
//               barrier per K tile, output rows re-formed through LDS: up to 512
//               rows, and larger batches whose epilogue is most of the work
//               (gemm_large.hip takes the others)
#include <algorithm>

#include <type_traits>

#include "gemm_common.h"

namespace pc {

__device__ inline float silu_f(float x) { return x / (1.0f + expf(-x)); }

template <typename T> __device__ inline void store_out(T *p, float v, uint32_t *sat) { *p = from_f32_sat<T>(v, sat); }

// =====================================================================================
// plain-ALU GEMM: 64x64 tile, BK = 16, 256 threads, 4x4 outputs per thread at stride 16
// =====================================================================================
template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_simt_kernel(const T *__restrict__ A, const T *__restrict__ W, int lg,
                                                        void *__restrict__ Cv, int M, int N, int K,
                                                        uint32_t *__restrict__ sat) {
    constexpr int BM = 64, BN = 64, BK = 16;
    __shared__ float As[BK][BM + 4];
    __shared__ float Ws[BK][BN + 4];
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    float acc[4][4] = {};
    const int lr = tid / 4, lk = (tid % 4) * 4;   // load coordinates: row lr, k lk..lk+3
    for (int k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int k = k0 + lk + i;
            int am = m0 + lr, wn = n0 + lr;
            As[lk + i][lr] = (am < M && k < K) ? to_f32(A[(int64_t)am * K + k]) : 0.f;
            Ws[lk + i][lr] = (wn < N && k < K) ? to_f32(W[weight_at(wn, k, K, lg)]) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < BK; ++k) {
            float a[4], w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = As[k][ty + 16 * i];
                w[i] = Ws[k][tx + 16 * i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int row = m0 + ty + 16 * i;
        if (row >= M) continue;
        if (EPI == EPI_SWIGLU) {
            // this tile is two gate/up chunks: columns [0,16) gate, [16,32) the matching up, and again
            T *C = (T *)Cv;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (n0 + tx + 32 * j + 16 < N)
                    store_out(&C[(int64_t)row * (N / 2) + n0 / 2 + tx + 16 * j], silu_f(acc[i][2 * j]) * acc[i][2 * j + 1], sat);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int col = n0 + tx + 16 * j;
                if (col >= N) continue;
                if (EPI == EPI_STORE_F32) ((float *)Cv)[(int64_t)row * N + col] = acc[i][j];
                if (EPI == EPI_RESID_F32) ((float *)Cv)[(int64_t)row * N + col] += acc[i][j];
                if (EPI == EPI_STORE_T) store_out(&((T *)Cv)[(int64_t)row * N + col], acc[i][j], sat);
            }
        }
    }
}

template <typename T>
static void gemm_simt(const void *A, WeightRef W, void *C, int M, int N, int K, int epi, uint32_t *sat, hipStream_t s) {
    dim3 grid((N + 63) / 64, (M + 63) / 64);
    const T *a = (const T *)A, *w = (const T *)W.p;
    switch (epi) {
        case EPI_STORE_F32: gemm_simt_kernel<T, EPI_STORE_F32><<<grid, 256, 0, s>>>(a, w, W.lg, C, M, N, K, sat); break;
        case EPI_RESID_F32: gemm_simt_kernel<T, EPI_RESID_F32><<<grid, 256, 0, s>>>(a, w, W.lg, C, M, N, K, sat); break;
        case EPI_SWIGLU: gemm_simt_kernel<T, EPI_SWIGLU><<<grid, 256, 0, s>>>(a, w, W.lg, C, M, N, K, sat); break;
        default: gemm_simt_kernel<T, EPI_STORE_T><<<grid, 256, 0, s>>>(a, w, W.lg, C, M, N, K, sat); break;
    }
}

// =====================================================================================
// fp32 matrix-core GEMM for the sizes at which latency counts (fp32 models, K a multiple of 16)
// =====================================================================================
// v_mfma_f32_16x16x4_f32 (full fp32 products and sums): lane l holds A[l%16][k = l/16], B[k = l/16][l%16] and
// D[4*(l/16) + v][l%16].  A lane loads 16 consecutive bytes of its row, k = 16c + 4g .. + 3 (g = l/16), and the e-th
// instruction of a chunk takes the e-th of them on both sides: which k meet in one instruction does not matter.
// A block owns 16 TM x 16 TN outputs over the whole of K, its four waves take every fourth chunk of 16 k and add up
// through LDS in wave order.  No staging: at these sizes a launch is a few memory latencies long, so what counts is many
// blocks (TM = TN = 1: one tile each) and all loads of a wave in flight at once; the plain-ALU kernel's 64 x 64 tiles leave
// two to twelve blocks that walk K 16 at a time behind two barriers (32 rows,
// N = 128, K = 384: 47.7 -> 3.8 us; N = 2048, K = 1024: 125 -> 6.0 us; 4096 rows: 454 -> 231 us).
// NORM: the rows of A are RMS-normalised first, (h g rs) W^T = rs ((h g) W^T): the gain goes onto a row's pieces as they arrive, its
// sum of squares is taken from the same registers, the scale comes with the four waves' sums.  Every block of a row strip does that
// again, which costs next to nothing beside its loads.  (4 layers, a launch less per projection: 8 decode steps of 128 rows, d_model
// 128, 1113 -> 970 us, of 64 rows, d_model 512, 2643 -> 2603; prefill of 4096 rows, d_model 1024, 9.26 -> 7.85 ms, 512, 2.42 -> 2.23.)
template <int TM, int TN, int EPI, bool NORM>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ A, const float *__restrict__ W,
                                                       float *__restrict__ C, int M, int N, int K,
                                                       const float *__restrict__ gain, float eps) {
    static_assert(EPI != EPI_SWIGLU || TN == 2, "a gate tile and its up tile");
    constexpr int NT = TM * TN;
    __shared__ f32x4_t part[4][NT][64];
    __shared__ float squares[4][NORM ? 16 * TM : 1];
    float ss[TM] = {};
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64, i = lane % 16, g = lane / 16;
    const int m0 = blockIdx.y * 16 * TM;
    const int col0 = blockIdx.x * 16 * TN;   // (SwiGLU: a chunk of 16 gate rows and their 16 up rows)
    const float *pa[TM], *pw[TN];
#pragma unroll
    for (int t = 0; t < TM; ++t) pa[t] = A + (int64_t)min(m0 + 16 * t + i, M - 1) * K + 4 * g;
#pragma unroll
    for (int t = 0; t < TN; ++t) pw[t] = W + (int64_t)min(col0 + 16 * t + i, N - 1) * K + 4 * g;
    f32x4_t acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    constexpr int U = 4;                               // chunks in flight per wave
    const int chunks = K / 16;
    for (int c0 = wave; c0 < chunks; c0 += 4 * U) {
        f32x4_t fa[U][TM], fw[U][TN], fg[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + 4 * u;
#pragma unroll
            for (int t = 0; t < TM; ++t) fa[u][t] = c < chunks ? *(const f32x4_t *)(pa[t] + 16 * c) : (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < TN; ++t) fw[u][t] = c < chunks ? *(const f32x4_t *)(pw[t] + 16 * c) : (f32x4_t){0.f, 0.f, 0.f, 0.f};
            if (NORM) fg[u] = *(const f32x4_t *)(gain + 16 * min(c, chunks - 1) + 4 * g);
        }
        if (NORM) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int t = 0; t < TM; ++t) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) ss[t] = fmaf(fa[u][t][e], fa[u][t][e], ss[t]);
                    fa[u][t] *= fg[u];
                }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][a][e], fw[u][b][e], acc[a][b], 0, 0, 0);
    }
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) part[wave][a * TN + b][lane] = acc[a][b];
    if (NORM) {
#pragma unroll
        for (int a = 0; a < TM; ++a) {
            ss[a] += __shfl_xor(ss[a], 16, 64);
            ss[a] += __shfl_xor(ss[a], 32, 64);
            if (g == 0) squares[wave][16 * a + i] = ss[a];
        }
    }
    __syncthreads();
    // thread -> element wave of each lane's four: row 4 g + wave, column i of every tile
    auto sum = [&](int t) {
        float v = part[0][t][lane][wave];
#pragma unroll
        for (int w = 1; w < 4; ++w) v += part[w][t][lane][wave];
        return v;
    };
#pragma unroll
    for (int a = 0; a < TM; ++a) {
        const int at = 16 * a + 4 * g + wave, row = m0 + at;
        float scale = 1.f;
        if (NORM) scale = 1.0f / sqrtf((squares[0][at] + squares[1][at] + squares[2][at] + squares[3][at]) / (float)K + eps);
        if (EPI == EPI_SWIGLU) {
            const float gate = sum(a * TN) * scale, up = sum(a * TN + 1) * scale;
            const int out = blockIdx.x * 16 + i;
            if (row < M && out < N / 2) C[(int64_t)row * (N / 2) + out] = silu_f(gate) * up;
        } else {
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                const int col = col0 + 16 * b + i;
                const float v = sum(a * TN + b) * scale;
                if (row < M && col < N) {
                    if (EPI == EPI_RESID_F32) C[(int64_t)row * N + col] += v;
                    else C[(int64_t)row * N + col] = v;
                }
            }
        }
    }
}

template <int TM, int TN> static void gemm_f32_run(const float *A, const float *W, float *C, int M, int N, int K, int epi, hipStream_t s) {
    const int rows = (M + 16 * TM - 1) / (16 * TM);
    const dim3 grid((N + 16 * TN - 1) / (16 * TN), rows);
    if (epi == EPI_SWIGLU) gemm_f32_kernel<TM, 2, EPI_SWIGLU, false><<<dim3(N / 32, rows), 256, 0, s>>>(A, W, C, M, N, K, nullptr, 0.f);
    else if (epi == EPI_RESID_F32) gemm_f32_kernel<TM, TN, EPI_RESID_F32, false><<<grid, 256, 0, s>>>(A, W, C, M, N, K, nullptr, 0.f);
    else gemm_f32_kernel<TM, TN, EPI_STORE_F32, false><<<grid, 256, 0, s>>>(A, W, C, M, N, K, nullptr, 0.f);
}

// Whole 16-byte pieces of rows on both sides (the caller's lm_head may start anywhere).
static bool gemm_f32_ok(const void *A, const void *W, int N, int K, int epi) {
    return K % 16 == 0 && (((uintptr_t)A | (uintptr_t)W) & 15) == 0 && (epi != EPI_SWIGLU || N % 64 == 0);
}

// The largest tile that still gives every CU a block: below that the chip idles (32 rows x 2048 columns x 1024: 6 us with
// 256 blocks of 16 x 16, 12 us with 64 of 32 x 32, 28 us with 32 of 64 x 64), above it operands are re-read more often than
// they need be (1024 x 1024 x 4096: 225 / 138 / 100 us).
static int gemm_f32_tile(int M, int N, int epi) {
    auto blocks = [&](int t) {
        return (int64_t)((M + 16 * t - 1) / (16 * t)) * (epi == EPI_SWIGLU ? N / 32 : (N + 16 * t - 1) / (16 * t));
    };
    return blocks(4) >= 256 ? 4 : blocks(2) >= 256 ? 2 : 1;
}
static void gemm_f32(const float *A, const float *W, float *C, int M, int N, int K, int epi, hipStream_t s) {
    const int t = gemm_f32_tile(M, N, epi);
    if (t == 4) gemm_f32_run<4, 4>(A, W, C, M, N, K, epi, s);
    else if (t == 2) gemm_f32_run<2, 2>(A, W, C, M, N, K, epi, s);
    else gemm_f32_run<1, 1>(A, W, C, M, N, K, epi, s);
}

// (in every tile size: whether a row's norm is folded in must not depend on the batch that it is in)
bool gemm_f32_norm_ok(int dtype, int impl, const float *h, const float *gain, const void *W, int N, int K, int epi) {
    return dtype == KD_F32 && impl != 0 && (epi == EPI_STORE_F32 || epi == EPI_SWIGLU) && gemm_f32_ok(h, W, N, K, epi) && ((uintptr_t)gain & 15) == 0;
}
template <int T> static void gemm_f32_norm_run(const float *h, const float *gain, float eps, const float *W, float *C, int M, int N, int K, int epi, hipStream_t s) {
    const int rows = (M + 16 * T - 1) / (16 * T);
    if (epi == EPI_SWIGLU) gemm_f32_kernel<T, 2, EPI_SWIGLU, true><<<dim3(N / 32, rows), 256, 0, s>>>(h, W, C, M, N, K, gain, eps);
    else gemm_f32_kernel<T, T, EPI_STORE_F32, true><<<dim3((N + 16 * T - 1) / (16 * T), rows), 256, 0, s>>>(h, W, C, M, N, K, gain, eps);
}
void launch_gemm_f32_norm(const float *h, const float *gain, float eps, const void *W, float *C, int M, int N, int K, int epi, hipStream_t s) {
    if (M <= 0) return;
    const int t = gemm_f32_tile(M, N, epi);
    if (t == 4) gemm_f32_norm_run<4>(h, gain, eps, (const float *)W, C, M, N, K, epi, s);
    else if (t == 2) gemm_f32_norm_run<2>(h, gain, eps, (const float *)W, C, M, N, K, epi, s);
    else gemm_f32_norm_run<1>(h, gain, eps, (const float *)W, C, M, N, K, epi, s);
}

// =====================================================================================
// matrix-core GEMM (bf16 in, fp32 accumulate)
// =====================================================================================
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
static constexpr int N_XCD = 8;   // MI355X: 8 accelerator dies, each with its own L2; workgroup i runs on die i % 8

// One 32x32x16 product per instruction.  Operand layout (wave of 64 lanes):
//   a: lane l holds X[row = l%32][k = 8*(l/32) .. +7]
//   b: lane l holds Y[k = 8*(l/32) .. +7][col = l%32]
//   d: lane l, element v holds D[row = 8*(v/4) + 4*(l/32) + v%4][col = l%32]
// The kernel passes the WEIGHT fragment as a and the activation fragment as b (both are 8 consecutive k of one
// matrix row, contiguous in memory), so d is the transposed output tile: lane l holds output row l%32 and, per
// group of four elements, four consecutive output columns.
//
// Work decomposition: a 1-D grid; workgroup id -> (m block, n block, K slice) such that the m blocks
// that share a weight tile run on the same die back to back (the second one finds the tile in L2).
// K slices (S > 1) write plain fp32 slices [S][M][N] to `Cv`; whoever consumes them adds them up in
// slice order (no atomics, no fences: the kernel boundary orders the two).
//
// Data path: global memory -> LDS directly (global_load_lds_dwordx4, no register staging), NSTAGE
// tiles deep, one barrier per K tile; LDS -> registers one K step ahead of the products, also across tiles.  A wave-wide load lands as 1 KB of consecutive LDS (8 rows of
// 64 k); to keep the 128-bit fragment reads conflict free without padding, the 16-byte chunk c of
// row r is stored at chunk slot c ^ swz(r) (the lane fetches the chunk its slot must hold), where swz
// makes any 16 consecutive rows hit 16 different 16-byte bank groups.  K must be a multiple of 64 here.
// M16: the products are 16x16x32 instructions (a: A[row l%16][k = 8*(l/16) .. +7], b likewise,
// d[v]: D[row 4*(l/16) + v][col l%16]) instead of 32x32x16: the same fragment bytes per product volume, four
// times as many accumulator tiles per wave.
template <typename T, int BM, int BN, int WM, int WN, int NSTAGE, int BK, int EPI, bool M16 = false>
__global__ __launch_bounds__(64 * WM * WN) void gemm_mfma_kernel(const T *__restrict__ A, const T *__restrict__ W, int lg,
                                                        void *__restrict__ Cv, int M, int N, int K, int mb, int nb,
                                                        int S, int plain, uint32_t *__restrict__ sat,
                                                        typename GemmExtra<EPI>::type extra) {
    constexpr bool SWIGLU = (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_RS);
    constexpr int CPR = BK / 8;                           // 16-byte chunks per tile row
    constexpr int RPL = 64 / CPR;                         // tile rows one wave-wide load covers
    // rows that share a swizzle value (measured with a read-rate probe: 16-row fragment reads of 64-byte
    // rows want a new value every 2 rows, 267 -> 320 GB/s per CU)
    constexpr int SWZ_DIV = (M16 && BK == 32) ? 2 : 16 / CPR;
    constexpr int RT = M16 ? 16 : 32;                     // rows (columns) of one accumulator tile
    constexpr int CG = 64 / RT;                           // 16-byte k chunks one product consumes per row
    constexpr int AV = M16 ? 4 : 16;                      // accumulator values per lane and tile
    constexpr int TM = BM / WM / RT, TN = BN / WN / RT;
    typedef typename std::conditional<M16, f32x4_t, f32x16_t>::type acc_t;
    constexpr int NW = WM * WN;                           // waves per block
    constexpr int A_ITERS = BM / (RPL * NW), W_ITERS = BN / (RPL * NW);   // the waves move RPL*NW rows of BK k per pass
    constexpr int LOADS = A_ITERS + W_ITERS;              // load instructions per thread per K tile
    constexpr int STAGE_ELEMS = (BM + BN) * BK;
    static_assert(BK == 64 || BK == 32, "K tile");
    static_assert(BM % (RPL * NW) == 0 && BN % (RPL * NW) == 0, "whole passes");
    static_assert(!SWIGLU || (BN / WN) % 32 == 0, "SwiGLU needs whole gate/up chunks per wave");
    static_assert(NSTAGE * LOADS <= 63, "vmcnt is a 6-bit counter");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    T *smem = (T *)smem_raw;                     // [NSTAGE][A tile BM x 64 | W tile BN x 64]

    // ---- which tile
    const int id = blockIdx.x;
    int bm, bn, z;
    if (plain == 2) {
        // many row blocks, a multiple of 8 (prefill): every die owns mb/8 row blocks and walks all column blocks in
        // groups of 8, patch by patch of 4 row blocks x 8 column blocks.  The 32 blocks a die runs at a time then
        // share 4 activation slabs and 8 weight slabs (its L2 serves each K tile to 8 resp. 4 blocks), where plain
        // order gave a die 32 different weight slabs at once.
        if (!gemm_patch_tile(id, mb, nb, &bm, &bn)) return;
        z = 0;
    } else if (plain) {   // many row blocks (prefill): neighbours share the activation rows, plain order
        bn = id % nb;
        bm = id / nb;
        z = 0;
        if (bm >= mb) return;
    } else {
        const int die = id % N_XCD, j = id / N_XCD;
        const int unit = (j / mb) * N_XCD + die;           // (n block, K slice) pair
        if (unit >= nb * S) return;
        bm = j % mb;
        bn = unit % nb;
        z = unit / nb;
    }
    const int m0 = bm * BM, n0 = bn * BN;

    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int wm = wave / WN, wn = wave % WN;
    // the rows' RMSNorm scale from the partial sums of squares ssq[tile][row]: two threads per row, every load of a
    // thread in flight at once (a lane's neighbours read the neighbouring rows: whole cache lines per request)
    constexpr int RS_MAXT = 24;                        // tiles one thread sums per round
    __shared__ float s_rs[EPI == EPI_SWIGLU_RS ? BM : 1];
    __shared__ float s_rs_part[EPI == EPI_SWIGLU_RS ? BM : 1];
    const int KT = K / BK;
    const int per = (KT + S - 1) / S;
    const int kt0 = z * per, kt1 = min(KT, kt0 + per);

    // ---- global -> LDS: in pass i this wave fills rows (4i + wave)*8 .. +7; lane -> (row, slot)
    const int lr = lane / CPR, slot = lane % CPR;
    const T *pa[A_ITERS], *pw[W_ITERS];
#pragma unroll
    for (int i = 0; i < A_ITERS; ++i) {
        const int row = (NW * i + wave) * RPL + lr;
        const int chunk = slot ^ ((row / SWZ_DIV) & (CPR - 1));
        pa[i] = A + (int64_t)min(m0 + row, M - 1) * K + chunk * 8;   // rows past the end: clamped, results discarded
    }
#pragma unroll
    for (int i = 0; i < W_ITERS; ++i) {
        const int row = (NW * i + wave) * RPL + lr;
        const int chunk = slot ^ ((row / SWZ_DIV) & (CPR - 1));
        pw[i] = W + weight_row(min(n0 + row, N - 1), K, lg) + chunk * 8;
    }
    auto issue_tile = [&](int kt, int stage) {
        const int koff = min(kt, kt1 - 1) * BK;            // past the end: a redundant reload, keeps the count constant
        const int kw = BK == 64 ? koff << lg : ((koff >> 6) << (6 + lg)) + (koff & 63);
        T *sa = smem + stage * STAGE_ELEMS;
        T *sw = sa + BM * BK;
#pragma unroll
        for (int i = 0; i < A_ITERS; ++i)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(pa[i] + koff),
                                             (__attribute__((address_space(3))) void *)(sa + (NW * i + wave) * RPL * BK), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < W_ITERS; ++i)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(pw[i] + kw),
                                             (__attribute__((address_space(3))) void *)(sw + (NW * i + wave) * RPL * BK), 16, 0, 0);
    };

    auto issue_part = [&](int kt, int stage, int part, int parts) {   // the loads l of a tile with l * parts / LOADS == part
        const int koff = min(kt, kt1 - 1) * BK;            // past the end: a redundant reload, keeps the count constant
        const int kw = BK == 64 ? koff << lg : ((koff >> 6) << (6 + lg)) + (koff & 63);
        T *sa = smem + stage * STAGE_ELEMS;
        T *sw = sa + BM * BK;
#pragma unroll
        for (int i = 0; i < A_ITERS; ++i)
            if (i * parts / LOADS == part)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(pa[i] + koff),
                                                 (__attribute__((address_space(3))) void *)(sa + (NW * i + wave) * RPL * BK), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < W_ITERS; ++i)
            if ((A_ITERS + i) * parts / LOADS == part)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(pw[i] + kw),
                                                 (__attribute__((address_space(3))) void *)(sw + (NW * i + wave) * RPL * BK), 16, 0, 0);
    };
    acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jj = 0; jj < TN; ++jj)
#pragma unroll
            for (int v = 0; v < AV; ++v) acc[i][jj][v] = 0.f;
    // sums of the K slices behind the block, the current one's is in acc
    constexpr bool SLICES = EPI == EPI_RESID_SLICES;
    [[maybe_unused]] acc_t front[SLICES ? TM : 1][SLICES ? TN : 1] = {};
    auto end_slice = [&]() {
        if constexpr (SLICES) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int jj = 0; jj < TN; ++jj) {
                    front[i][jj] += acc[i][jj];
                    acc[i][jj] = acc_t{};
                }
        }
    };

    // fragment addressing: lane (fr, fg) reads chunk CG*kk + fg of its row, stored at slot chunk ^ swz(row)
    const int fr = lane % RT, fg = lane / RT;
    int arow[TM], aswz[TM], wrow[TN], wswz[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        arow[i] = wm * (BM / WM) + i * RT + fr;
        aswz[i] = (arow[i] / SWZ_DIV) & (CPR - 1);
    }
#pragma unroll
    for (int jj = 0; jj < TN; ++jj) {
        wrow[jj] = wn * (BN / WN) + jj * RT + fr;
        wswz[jj] = (wrow[jj] / SWZ_DIV) & (CPR - 1);
    }
    typedef typename Mma<T>::frag frag_t;
    auto load_frags = [&](const T *sa, const T *sw, int kk, frag_t (&fa)[TM], frag_t (&fb)[TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = *(const frag_t *)(sa + arow[i] * BK + (((CG * kk + fg) ^ aswz[i]) * 8));
#pragma unroll
        for (int jj = 0; jj < TN; ++jj) fb[jj] = *(const frag_t *)(sw + wrow[jj] * BK + (((CG * kk + fg) ^ wswz[jj]) * 8));
    };
    auto product = [&](frag_t a, frag_t b, acc_t c) -> acc_t {
        if constexpr (M16) return Mma<T>::m16(a, b, c);
        else return Mma<T>::m32(a, b, c);
    };
    // One K step (the products of 8*CG k values of every accumulator tile), software-pipelined ACROSS K tiles: while
    // the products of this step run on the fragments `ca`/`cb` already in registers, the fragments of the next step
    // are read into `na`/`nb` -- the next step of the same tile, or, in a tile's last step, the first step of the next
    // tile.  That read needs the next tile visible, so the block's one barrier per tile sits in front of the last
    // step (not at the top of the tile), and right behind it the stage just consumed is refilled.  No product then
    // waits for an LDS read issued just before it (the first version did, once per tile: with one step per tile the
    // matrix cores idled half the time).
    // Wave tiles of fewer than four accumulator tiles (the 128x64 and 64x64 blocks of the small decode projections)
    // keep the barrier at the top of the tile and prefetch within the tile only: with two products per step there
    // is nothing to hide the hand-over under, and the plain order measured faster there (decode down projection
    // 15.1 against 16.5 us).
    constexpr int KK = BK / (8 * CG);                     // steps per tile
    constexpr bool XT = (TM * TN >= 4);                   // pipelined across tiles
    auto kstep = [&](frag_t (&ca)[TM], frag_t (&cb)[TN], frag_t (&na)[TM], frag_t (&nb)[TN], int kt, int stage, int kk) {
        const T *sa = smem + stage * STAGE_ELEMS;
        const T *sw = sa + BM * BK;
        const int pstage = (stage == 0) ? NSTAGE - 1 : stage - 1;
        if constexpr (!XT) {
            if (kk == 0) {
                wait_vmcnt_le<(NSTAGE - 2) * LOADS>();    // this thread's loads of tile kt have landed
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();             // ... and everybody's; tile kt-1 is consumed
                asm volatile("" ::: "memory");
                load_frags(sa, sw, 0, ca, cb);
            }
            issue_part(kt - 1 + NSTAGE, pstage, kk, KK);  // the refill of tile kt-1's stage, spread over the steps
            if (kk + 1 < KK) load_frags(sa, sw, kk + 1, na, nb);
        } else if (kk == KK - 1) {
            wait_vmcnt_le<(NSTAGE - 2) * LOADS>();        // this thread's loads of tile kt+1 have landed
            __builtin_amdgcn_s_waitcnt(0xC07F);           // lgkmcnt(0): and its own reads of tile kt have returned
            // ... and everybody's: behind the barrier tile kt+1 is visible and tile kt's stage is free.  A bare
            // barrier: __syncthreads() would add a fence that drains every load in flight.
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const int nstage = (stage + 1 == NSTAGE) ? 0 : stage + 1;
            issue_part(kt + NSTAGE, stage, 0, KK);        // the refill of the stage just consumed starts here ...
            const T *nsa = smem + nstage * STAGE_ELEMS;
            load_frags(nsa, nsa + BM * BK, 0, na, nb);    // (behind the last tile: read and never used)
        } else {
            // ... and goes on over the next tile's other steps (a wave that has to hand the load unit six loads
            // in a row cannot issue matrix instructions meanwhile)
            issue_part(kt - 1 + NSTAGE, pstage, kk + 1, KK);
            load_frags(sa, sw, kk + 1, na, nb);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int jj = 0; jj < TN; ++jj)
                acc[i][jj] = product(cb[jj], ca[i], acc[i][jj]);   // weights as rows: the tile comes out transposed
        // instruction order asked of the compiler: after each matrix instruction one or two LDS fragment reads and
        // one global->LDS load, instead of all of them in a burst
#pragma unroll
        for (int g = 0; g < TM * TN; ++g) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, (TM + TN + TM * TN - 1) / (TM * TN), 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
    };

    // tile kt lives in stage (kt - kt0) % NSTAGE; the tile being consumed sits in registers, the next one in LDS,
    // NSTAGE-1 more are in flight
    // q/k/v: a lane keeps slot and position of one of the wave's rows, asked for around the first tile loads.  Looked up per row tile
    // behind the products, the chain slot -> length -> block or rotation -> store was a third of the launch (1024 decode rows x 2048 x
    // 1536 19.8 -> 16.4 us, 600 rows 18.6 -> 14.7).
    constexpr int WROWS = BM / WM;
    int row_slot = 0, row_pos = 0;
    [[maybe_unused]] const int own_row = min(m0 + wm * WROWS + lane % WROWS, M - 1);
    if constexpr (EPI == EPI_QKV) {
        static_assert(WROWS <= 64, "a lane per row");
        row_slot = extra.row_slot[own_row];
    }
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s) issue_tile(kt0 + s, s);
    if constexpr (XT) issue_part(kt0 + NSTAGE - 1, NSTAGE - 1, 0, KK);   // (its other parts: the first tile's steps)
    if constexpr (EPI == EPI_QKV) row_pos = extra.row_pos ? extra.row_pos[own_row] : extra.slot_len[row_slot];
    // (behind the first tile loads, so that the pipeline is already filling while the statistics arrive; these are
    // ordinary loads, younger than the tile loads: once they are back, so are the tiles.  Loads beyond the last partial sum
    // are clamped, not left out: a branch around each made them wait for one another, which cost gate/up 2.5 us at 96 rows of
    // the 1.5B shape and 8 us of the 8B one)
    if constexpr (EPI == EPI_SWIGLU_RS) {
        constexpr int PARTS = (64 * NW >= 2 * BM) ? 2 : 1;   // threads per row (each sums every PARTS-th round of tiles)
        static_assert(64 * NW >= BM, "a thread per row");
        const int r = tid % BM, part = tid / BM;
        float ss = 0.f;
        if (part < PARTS) {
            const int row = min(m0 + r, M - 1);
            for (int t0 = part * RS_MAXT; t0 < extra.tiles; t0 += PARTS * RS_MAXT) {
                float v[RS_MAXT];
#pragma unroll
                for (int u = 0; u < RS_MAXT; ++u) v[u] = extra.ssq[(int64_t)min(t0 + u, extra.tiles - 1) * M + row];
#pragma unroll
                for (int u = 0; u < RS_MAXT; ++u) ss += (t0 + u < extra.tiles) ? v[u] : 0.f;
            }
        }
        if (PARTS == 2) {
            if (part == 1) s_rs_part[r] = ss;
            __syncthreads();
            if (part == 0) ss += s_rs_part[r];
        }
        if (part == 0) s_rs[r] = 1.0f / sqrtf(ss / (float)extra.d + extra.eps);
        __syncthreads();
    }
    frag_t fa[2][TM], fb[2][TN];
    if constexpr (XT) {
        constexpr int PART0 = (LOADS + KK - 1) / KK;       // loads l with l * KK / LOADS == 0
        wait_vmcnt_le<(NSTAGE - 2) * LOADS + PART0>();     // the first tile has landed
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        load_frags(smem, smem + BM * BK, 0, fa[0], fb[0]);
    }
    int stage = 0;
    if constexpr (KK % 2 == 0) {   // an even number of steps per tile: the two fragment sets alternate within a tile
        int slice_end = kt1;
        if constexpr (SLICES) slice_end = kt0 + extra.per;
        for (int kt = kt0; kt < kt1; ++kt) {
            if constexpr (SLICES)
                if (kt == slice_end) {
                    end_slice();
                    slice_end += extra.per;
                }
#pragma unroll
            for (int kk = 0; kk < KK; kk += 2) {
                kstep(fa[0], fb[0], fa[1], fb[1], kt, stage, kk);
                kstep(fa[1], fb[1], fa[0], fb[0], kt, stage, kk + 1);
            }
            stage = (stage + 1 == NSTAGE) ? 0 : stage + 1;
        }
        if constexpr (SLICES)
            if (kt0 + extra.per < kt1) {
                end_slice();
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int jj = 0; jj < TN; ++jj) acc[i][jj] = front[i][jj];
            }
    } else {                       // one step per tile: they alternate from tile to tile
        static_assert(!SLICES, "ends of slices");
        static_assert(KK == 1 || KK % 2 == 0, "steps per tile");
        int kt = kt0;
        for (; kt + 1 < kt1; kt += 2) {
            kstep(fa[0], fb[0], fa[1], fb[1], kt, stage, 0);
            stage = (stage + 1 == NSTAGE) ? 0 : stage + 1;
            kstep(fa[1], fb[1], fa[0], fb[0], kt + 1, stage, 0);
            stage = (stage + 1 == NSTAGE) ? 0 : stage + 1;
        }
        if (kt < kt1) kstep(fa[0], fb[0], fa[1], fb[1], kt, stage, 0);
    }
    wait_vmcnt_le<0>();   // nothing may still be writing LDS when the block retires

    if constexpr (EPI == EPI_LOGPROB) {
        // A lane owns row ml of every row tile and 4 TN of the wave's columns, its three partners (16, 32, 48 lanes on) the
        // others: maximum, then the exponentials summed in double, both folded over the four.  One entry per row and wave
        // column strip leaves the block instead of the strip's logits (1024 rows x 151936: 15 MB for 622 MB, which the
        // softmax behind it had to read again).
        static_assert(M16, "lane layout of the 16x16x32 products");
        constexpr int WC = BN / WN;
        const int ml = lane % 16, nq = 4 * (lane / 16), col0 = n0 + wn * WC;
        const int64_t strip = (int64_t)bn * WN + wn;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row = m0 + wm * (BM / WM) + i * 16 + ml;
            const int want = row < M ? extra.tokens[extra.token_index[row] + 1] - col0 - nq : -1;   // (column - nq) of the target
            if (__any(want >= 0 && want < WC)) {   // (rare: a row's target is in one of a thousand strips)
#pragma unroll
                for (int jj = 0; jj < TN; ++jj)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (want == jj * 16 + v && col0 + jj * 16 < N) extra.target[row] = acc[i][jj][v];
            }
            float mx = -INFINITY;
#pragma unroll
            for (int jj = 0; jj < TN; ++jj)
                if (col0 + jj * 16 < N) {   // N is a multiple of 16: a tile is inside or outside
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        acc[i][jj][v] *= extra.inv_t;
                        mx = fmaxf(mx, acc[i][jj][v]);
                    }
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float base = (mx == -INFINITY) ? 0.f : mx;
            double s = 0.0;
#pragma unroll
            for (int jj = 0; jj < TN; ++jj)
                if (col0 + jj * 16 < N) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) s += (double)exp_neg(acc[i][jj][v] - base);
                }
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (row < M && nq == 0) {
                extra.part_max[strip * M + row] = mx;
                extra.part_sum[strip * M + row] = s;
            }
        }
        return;
    } else if constexpr (EPI == EPI_QKV) {
        // A wave's columns lie within one head.  q and k: columns come in blocks of 32, 16 dims and their 16 rotary partners
        // (dim + 64): two accumulator tiles that hold the same lanes' pairs.  The rotated 16-row tiles go through the wave's
        // piece of the idle LDS ring and leave as 16-byte pieces (eight dims: contiguous in q and in a key's cache fragment).
        // v: a token's dims lie 16 bytes apart in the cache; rows re-formed in LDS leave with neighbouring lanes on neighbouring
        // dims, 8 cache lines to a store instead of up to 64.  The fp32 q | k | v rows (134 MB per layer at 16384 rows of the 1.5B
        // shape, written and read again by a kernel of its own) never exist.
        static_assert(M16, "lane layout of the 16x16x32 products");
        constexpr int WC = BN / WN, HALF = WC / 2;
        constexpr int PITCH = WC * 2 + 16, LPR = WC / 8, PIECES = 16 * LPR;
        static_assert(WC % 32 == 0 && 128 % WC == 0, "whole 32-column blocks of one head");
        static_assert((size_t)NW * 16 * PITCH <= (size_t)NSTAGE * STAGE_ELEMS * sizeof(T), "staging fits the ring");
        const int ml = lane % 16, nq = 4 * (lane / 16), col0 = n0 + wn * WC;
        const int hkv = extra.kv.n_kv_heads, bs = extra.kv.block_size;
        const int qd = extra.hq * 128, kvd = hkv * 128;
        const int part = col0 < qd ? 0 : (col0 < qd + kvd ? 1 : 2);   // q, k, v (wave-uniform)
        const int pc0 = col0 - (part == 0 ? 0 : (part == 1 ? qd : qd + kvd));
        const int head = pc0 / 128, in = pc0 % 128;                   // first column inside the head
        const int row_tin = row_pos % bs;
        int row_blk = 0;
        if (part) row_blk = extra.kv.block_table[(int64_t)row_slot * extra.kv.max_blocks_per_slot + row_pos / bs];
        f32x4_t cs[TN / 2], sn[TN / 2];                               // of the lane's four pair indices per block, for the row tile to come
        auto rotation = [&](int i) {
            const int64_t at = (int64_t)__shfl(row_pos, 16 * i + ml, 64) * 64 + in / 2 + nq;
#pragma unroll
            for (int p2 = 0; p2 < TN / 2; ++p2) {
                cs[p2] = *(const f32x4_t *)(extra.rope_cos + at + 16 * p2);
                sn[p2] = *(const f32x4_t *)(extra.rope_sin + at + 16 * p2);
            }
        };
        if (part != 2) rotation(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();   // every wave has consumed its last fragments
        asm volatile("" ::: "memory");
        if (col0 >= N) return;
        unsigned char *stg = smem_raw + (size_t)wave * 16 * PITCH;
        T *pool = (T *)extra.kv.pool + (int64_t)extra.layer * extra.kv.layer_stride + (int64_t)head * extra.kv.head_elems();
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mt = m0 + wm * WROWS + i * 16, row = mt + ml;
            uint32_t *const count = row < M ? sat : nullptr;          // (rows past the end are copies of the last one)
            if (part == 2) {
#pragma unroll
                for (int jj = 0; jj < TN; ++jj)
                    *(u32x2 *)(stg + ml * PITCH + (16 * jj + nq) * 2) = pack4_sat<T>(acc[i][jj][0], acc[i][jj][1], acc[i][jj][2], acc[i][jj][3], count);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int it = 0; it < 16 * WC / 64; ++it) {
                    const int e = it * 64 + lane, r = e / WC, dim = e % WC;
                    const int rblk = __shfl(row_blk, 16 * i + r, 64), rtin = __shfl(row_tin, 16 * i + r, 64);
                    if (mt + r < M)
                        pool[(int64_t)rblk * extra.kv.block_elems() + extra.kv.v_index(rtin, in + dim)] = *(const T *)(stg + r * PITCH + dim * 2);
                }
                __builtin_amdgcn_wave_barrier();
                continue;
            }
#pragma unroll
            for (int p2 = 0; p2 < TN / 2; ++p2) {
                const f32x4_t &c = cs[p2], &n = sn[p2];
                const acc_t &x1 = acc[i][2 * p2], &x2 = acc[i][2 * p2 + 1];
                unsigned char *dst = stg + ml * PITCH + (16 * p2 + nq) * 2;
                *(u32x2 *)dst = pack4_sat<T>(rotated_first(x1[0], x2[0], c[0], n[0]), rotated_first(x1[1], x2[1], c[1], n[1]),
                                             rotated_first(x1[2], x2[2], c[2], n[2]), rotated_first(x1[3], x2[3], c[3], n[3]), count);
                *(u32x2 *)(dst + HALF * 2) = pack4_sat<T>(rotated_second(x1[0], x2[0], c[0], n[0]), rotated_second(x1[1], x2[1], c[1], n[1]),
                                                          rotated_second(x1[2], x2[2], c[2], n[2]), rotated_second(x1[3], x2[3], c[3], n[3]), count);
            }
            if (i + 1 < TM) rotation(i + 1);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < (PIECES + 63) / 64; ++it) {
                const int e = it * 64 + lane, r = (e / LPR) % 16, piece = e % LPR;
                const u32x4 val = *(const u32x4 *)(stg + r * PITCH + piece * 16);
                const int dim = in / 2 + (8 * piece) % HALF + 64 * ((8 * piece) / HALF);
                const int rblk = __shfl(row_blk, 16 * i + r, 64), rtin = __shfl(row_tin, 16 * i + r, 64);
                if (mt + r < M && (PIECES % 64 == 0 || e < PIECES)) {
                    if (part == 0)
                        *(u32x4 *)((T *)extra.q_out + ((int64_t)(mt + r) * extra.hq + head) * 128 + dim) = val;
                    else
                        *(u32x4 *)(pool + (int64_t)rblk * extra.kv.block_elems() + extra.kv.k_index(rtin, dim)) = val;
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        return;
    } else {
    // ---- epilogue
    // The products take the weights as the row operand, so the accumulators hold the TRANSPOSED tile: a lane owns ONE
    // output row m (m = lane % RT of the tile) and, per tile, runs of four consecutive output columns.  Written out
    // from there, an output row would leave in 2- or 4-byte pieces, one store instruction per value -- hundreds of
    // stores in flight per wave, which the store path takes far longer to retire than the bytes need (measured: a
    // fifth of the decode gate/up kernel).  Instead each wave turns RT output rows at a time into whole rows through
    // a private piece of the now idle LDS ring and stores them 16 bytes per lane, neighbouring lanes on
    // neighbouring addresses.  LDS instructions of one wave execute in order, so the hand-over needs no barrier.
    typedef typename std::conditional<(EPI == EPI_STORE_F32 || EPI == EPI_RESID_F32 || SLICES), float, T>::type OutT;
    constexpr int WCOLS = SWIGLU ? (BN / WN) / 2 : BN / WN;        // output columns of one wave
    constexpr int RB = WCOLS * (int)sizeof(OutT);                 // bytes of one output row of the wave
    constexpr int LPR = RB / 16;                                  // 16-byte pieces of one row
    constexpr int PIECES = RT * LPR, ITER = (PIECES + 63) / 64;   // pieces of the RT rows; store instructions for them
    constexpr int PITCH = RB + 16;                                // bytes; the pad spreads the rows over the banks
    constexpr int EPC = 16 / (int)sizeof(OutT);                   // output elements per 16-byte piece
    static_assert(RB % 16 == 0, "whole pieces");
    static_assert((size_t)NW * RT * PITCH <= (size_t)NSTAGE * STAGE_ELEMS * sizeof(T), "staging fits the ring");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();   // every wave has consumed its last fragments (they were waited for by the products)
    asm volatile("" ::: "memory");
    unsigned char *stg = smem_raw + (size_t)wave * RT * PITCH;
    const int ml = lane % RT, nq = 4 * (lane / RT);               // the lane's row of a tile; first column of its runs
    const int ldc = SWIGLU ? N / 2 : N;
    const int colbase = SWIGLU ? (n0 + wn * (BN / WN)) / 2 : n0 + wn * (BN / WN);
    OutT *Cbase = (OutT *)Cv + ((EPI == EPI_STORE_F32) ? (int64_t)z * M * N : 0);
    uint32_t *count = nullptr;                                    // clamped values are counted only where they are stored
    auto put4 = [&](int col, float v0, float v1, float v2, float v3) {   // four consecutive columns of row ml
        unsigned char *dst = stg + ml * PITCH + col * (int)sizeof(OutT);
        if constexpr (sizeof(OutT) == 4) {
            *(f32x4_t *)dst = (f32x4_t){v0, v1, v2, v3};
        } else {
            *(u32x2 *)dst = pack4_sat<T>(v0, v1, v2, v3, colbase + col < ldc ? count : nullptr);
        }
    };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        count = m0 + wm * (BM / WM) + i * RT + ml < M ? sat : nullptr;
        const float sc = (EPI == EPI_SWIGLU_RS) ? s_rs[wm * (BM / WM) + i * RT + ml] : 1.f;
        if constexpr (SWIGLU) {
            // a 32-wide chunk of weight rows = 16 gate rows, then the 16 matching up rows
            if constexpr (M16) {       // two tiles
#pragma unroll
                for (int p2 = 0; p2 < TN / 2; ++p2) {
                    const acc_t &ga = acc[i][2 * p2], &ua = acc[i][2 * p2 + 1];
                    put4(16 * p2 + nq, silu_mul(ga[0] * sc, ua[0] * sc), silu_mul(ga[1] * sc, ua[1] * sc),
                         silu_mul(ga[2] * sc, ua[2] * sc), silu_mul(ga[3] * sc, ua[3] * sc));
                }
            } else {                   // the two halves of a tile
#pragma unroll
                for (int jj = 0; jj < TN; ++jj)
#pragma unroll
                    for (int vg = 0; vg < 2; ++vg) {
                        const acc_t &ga = acc[i][jj];
                        put4(16 * jj + 8 * vg + nq, silu_mul(ga[4 * vg] * sc, ga[4 * vg + 8] * sc),
                             silu_mul(ga[4 * vg + 1] * sc, ga[4 * vg + 9] * sc),
                             silu_mul(ga[4 * vg + 2] * sc, ga[4 * vg + 10] * sc),
                             silu_mul(ga[4 * vg + 3] * sc, ga[4 * vg + 11] * sc));
                    }
            }
        } else {
#pragma unroll
            for (int jj = 0; jj < TN; ++jj)
#pragma unroll
                for (int vg = 0; vg < AV / 4; ++vg)
                    put4(jj * RT + (M16 ? 0 : 8 * vg) + nq, acc[i][jj][4 * vg], acc[i][jj][4 * vg + 1],
                         acc[i][jj][4 * vg + 2], acc[i][jj][4 * vg + 3]);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int e = it * 64 + lane, row = e / LPR, piece = e % LPR;
            if (PIECES % 64 != 0 && e >= PIECES) break;
            const u32x4 val = *(const u32x4 *)(stg + row * PITCH + piece * 16);
            const int gm = m0 + wm * (BM / WM) + i * RT + row, col = colbase + piece * EPC;
            if (gm < M && col < ldc) {
                OutT *dst = Cbase + (int64_t)gm * ldc + col;
                if constexpr (EPI == EPI_RESID_F32 || SLICES) {
                    const f32x4_t old = *(const f32x4_t *)dst, add = __builtin_bit_cast(f32x4_t, val);
                    *(f32x4_t *)dst = (f32x4_t){old[0] + add[0], old[1] + add[1], old[2] + add[2], old[3] + add[3]};
                } else {
                    *(u32x4 *)dst = val;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    }
}

template <typename T, int BM, int BN, int WM, int WN, int NSTAGE, int BK = 64, bool M16 = false> struct MfmaCfg {
    static constexpr size_t smem = (size_t)NSTAGE * (BM + BN) * BK * sizeof(T);
    static constexpr bool swiglu_ok = ((BN / WN) % 32 == 0);
    template <int E> static void set_attr() {
        (void)hipFuncSetAttribute((const void *)gemm_mfma_kernel<T, BM, BN, WM, WN, NSTAGE, BK, E, M16>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    }
    static void init() {
        set_attr<EPI_STORE_F32>();
        set_attr<EPI_RESID_F32>();
        set_attr<EPI_STORE_T>();
        if constexpr (swiglu_ok) {
            set_attr<EPI_SWIGLU>();
            set_attr<EPI_SWIGLU_RS>();
        }
    }
    template <int E>
    static void launch(const void *A, WeightRef W, void *C, int M, int N, int K, int split, uint32_t *sat, hipStream_t s,
                       const typename GemmExtra<E>::type &extra) {
        const int mb = (M + BM - 1) / BM, nb = (N + BN - 1) / BN;
        const int units = nb * split;
        // (log-probabilities: the vocabulary is so wide that a die keeps to one weight slab for all its row blocks where no
        // patches fit; in plain order every die streams all of the weights, 1640 rows x 151936 x 5120: 3001 against 2499 us)
        const int plain = (split == 1 && mb > 4) ? ((mb % N_XCD == 0) ? 2 : (E == EPI_LOGPROB ? 0 : 1)) : 0;
        const unsigned grid = plain ? (unsigned)(mb * nb) : (unsigned)((units + N_XCD - 1) / N_XCD * N_XCD * mb);
        gemm_mfma_kernel<T, BM, BN, WM, WN, NSTAGE, BK, E, M16><<<grid, 64 * WM * WN, smem, s>>>(
            (const T *)A, (const T *)W.p, W.lg, C, M, N, K, mb, nb, split, plain, sat, extra);
    }
    // split > 1 only with EPI_STORE_F32, C then being the slice buffer [split][M][N]
    static void run(const void *A, WeightRef W, void *C, int M, int N, int K, int epi, int split, uint32_t *sat, hipStream_t s,
                    const GemmRowScale *row_scale = nullptr) {
        switch (epi) {
            case EPI_STORE_F32: launch<EPI_STORE_F32>(A, W, C, M, N, K, split, sat, s, {}); break;
            case EPI_RESID_F32: launch<EPI_RESID_F32>(A, W, C, M, N, K, 1, sat, s, {}); break;
            case EPI_SWIGLU:
                if constexpr (swiglu_ok) launch<EPI_SWIGLU>(A, W, C, M, N, K, 1, sat, s, {});
                break;
            case EPI_SWIGLU_RS:
                if constexpr (swiglu_ok) launch<EPI_SWIGLU_RS>(A, W, C, M, N, K, 1, sat, s, *row_scale);
                break;
            default: launch<EPI_STORE_T>(A, W, C, M, N, K, 1, sat, s, {}); break;
        }
    }
    static void init_logprob() { set_attr<EPI_LOGPROB>(); }
    static void init_qkv() { set_attr<EPI_QKV>(); }
    static int strips(int N) { return (N + BN - 1) / BN * WN; }
    // K slices so that the launch has about `want_blocks` blocks, each with >= 4 K tiles
    static int pick_split(int M, int N, int K, size_t slice_cap_floats, int want_blocks) {
        const int64_t tiles = (int64_t)((N + BN - 1) / BN) * ((M + BM - 1) / BM);
        const int KT = K / BK;
        int64_t split = (want_blocks + tiles / 2) / tiles;
        // (never a second round for a few blocks: 6144 x 4096 at 400 rows 41.3 us with 288 blocks, 30.2 with 192)
        if (want_blocks <= 256) split = std::min<int64_t>(split, std::max<int64_t>(1, 256 / tiles));
        split = std::min<int64_t>(split, KT / 4);
        split = std::min<int64_t>(split, 8);
        split = std::min<int64_t>(split, (int64_t)(slice_cap_floats / ((size_t)M * N)));
        if (split < 2) return 1;
        const int per = (KT + (int)split - 1) / (int)split;
        return (KT + per - 1) / per;   // no empty slice
    }
};

// The tile configurations.  All on 16x16x32 products (0 to 13 % faster than 32x32x16 at every decode shape measured) except
// two whose wave tiles are a few 32x32 products only.
template <typename T> struct Gemm {
    // 256 x 128, 8 waves of 64 x 64: decode batches of 193 to 256 rows; q/k/v, gate/up and log-softmax of many rows
    typedef MfmaCfg<T, 256, 128, 4, 2, 3, 64, true> T256x128;
    typedef MfmaCfg<T, 256, 192, 4, 2, 2, 64, true> T256x192;
    typedef MfmaCfg<T, 256, 256, 4, 2, 4, 32, true> T256x256;   // short reductions of many rows; 64 x 128 per wave: three fragment reads per four products
    typedef MfmaCfg<T, 192, 128, 4, 2, 3, 64, true> T192x128;
    typedef MfmaCfg<T, 192, 192, 4, 2, 3, 64, true> T192x192;
    typedef MfmaCfg<T, 128, 128, 4, 2, 4, 64, true> T128x128;   // 8 waves of 32 x 64: up to 128 rows what counts is loads in flight
    typedef MfmaCfg<T, 128, 128, 4, 2, 2, 64, true> T128x128_2; // two stages, 64 KB of LDS: two blocks per CU
    typedef MfmaCfg<T, 128, 192, 4, 2, 3, 64, true> T128x192;
    typedef MfmaCfg<T, 64, 128, 2, 4, 3, 64, true> T64x128;     // 72 KB of LDS: two blocks per CU
    typedef MfmaCfg<T, 64, 192, 4, 2, 4, 64, true> T64x192;
    typedef MfmaCfg<T, 32, 64, 1, 4, 4, 64, true> T32x64;       // 48 KB of LDS: three blocks per CU
    typedef MfmaCfg<T, 32, 64, 1, 2, 4, 64, true> T32x64_2;     // the same with whole gate/up chunks per wave
    typedef MfmaCfg<T, 64, 64, 4, 2, 4, 64, true> T64x64;       // 8 waves of 16 x 32: residual projections of some hundred rows
    typedef MfmaCfg<T, 128, 64, 4, 2, 3, 64, true> T128x64_3;   // 8 waves of 32 x 32, 72 KB of LDS: the same for some more rows
    typedef MfmaCfg<T, 256, 160, 4, 1, 3, 64, true> T256x160;   // 4 waves of 64 x 160
    typedef MfmaCfg<T, 128, 64, 4, 2, 4, 64, true> T128x64;     // 8 waves of 32 x 32: long-K projections cut into K slices
    typedef MfmaCfg<T, 192, 64, 4, 2, 4, 64, true> T192x64;     // the same in wave tiles of 48 x 32
    typedef MfmaCfg<T, 64, 64, 2, 2, 4> M64x64;                 // wave tile 32 x 32: many blocks for the small projections
    static void init() {
        T256x128::init(); T256x192::init(); T256x256::init(); T192x128::init(); T192x192::init(); T128x128::init();
        T128x128_2::init(); T128x192::init(); T64x128::init(); T64x192::init(); T32x64::init();
        T32x64_2::init(); T128x64::init(); T192x64::init(); M64x64::init();
        T256x160::template set_attr<EPI_SWIGLU>();       // (gate/up only)
        T256x160::template set_attr<EPI_SWIGLU_RS>();
        T64x64::template set_attr<EPI_RESID_SLICES>();
        T128x64_3::template set_attr<EPI_RESID_SLICES>();
        T256x256::init_logprob();
        T256x128::init_logprob();
        T192x128::init_logprob();
        T128x128::init_logprob();
        T64x128::init_qkv();
        T128x128::init_qkv();
        T256x128::init_qkv();
        T256x256::init_qkv();
        T128x128_2::init_qkv();
    }
};
void gemm_init() {
    Gemm<bf16_t>::init();
    Gemm<f16_t>::init();
    gemm_large_init();
}

template <typename T>
static int gemm_mfma_dispatch(const void *A, WeightRef W, void *C, int M, int N, int K, int epi, float *slices,
                              size_t slice_cap_floats, uint32_t *sat, hipStream_t s, const GemmRowScale *row_scale);
static int large_min_k(bool swiglu) { return swiglu ? 128 : 256; }   // the shortest reduction that gemm_large.hip gets above 512 rows

// Residual projections of more than 512 rows whose blocks of 128 x 64 all run at once, one per CU: eight waves with little to do each
// and the whole reduction in one block, no slices for the norm behind to add up.  A block forms the sums of the slices that
// gemm_large.hip would cut and adds them in their order: the same bits (summed in one go, the logits of 1024 rows of the 1.5B shape, four
// layers, are 5.5e-4 of their size away, through the roundings to half that follow, and as far from 64-bit ones).  In 64 x 64 while there are no more than 320 of those
// (two fit a CU).  With that norm, us alone and as one of three streams, the best of gemm_large.hip's tiles and slices against these:
//   64 x 64    600 rows x 1536 x 1536  17.8 / 10.8, 13.7 / 8.5;  600 x 1024 x 2048  16.1 / 9.9, 14.4 / 7.8;  1024 x 512 x 256  10.5 / 6.2, 7.8 / 6.2
//              2000 x 512 x 2048  18.1 / 12.1, 16.7 / 10.3;  600 x 2048 x 1536 (320 blocks)  19.6 / 12.2, 16.7 / 9.9 (128 x 64: 17.8 / 10.4)
//   128 x 64   1024 x 1536 x 1536  20.7 / 14.1, 18.4 / 12.1 (64 x 64: 20.1 / 12.0);  768 x 2560 x 2048  23.0 / 17.1, 21.9 / 15.1;
//              2000 x 1024 x 1536  21.0 / 15.7, 18.6 / 13.6;  1024 x 2048 x 2048  22.8 / 18.1, 22.4 / 16.5
// Longer reductions are faster in slices of larger tiles: 1024 x 1536 x 3072  23.9 / 18.5, 26.2 / 18.8.
enum ResidTile { RESID_LARGE, RESID_64x64, RESID_128x64 };
static ResidTile resid_tile(int M, int N, int K, int epi) {
    if (epi != EPI_RESID_F32 || K < 256 || K > 2048 || (int64_t)((M + 127) / 128) * ((N + 63) / 64) > 256) return RESID_LARGE;
    return (int64_t)((M + 63) / 64) * ((N + 63) / 64) <= 320 ? RESID_64x64 : RESID_128x64;
}

int launch_gemm(int dtype, int impl, const void *A, WeightRef W, void *C, int M, int N, int K, int epi,
                float *slices, size_t slice_cap_floats, uint32_t *sat, hipStream_t s, const GemmRowScale *row_scale) {
    if (M <= 0 || N <= 0) return 1;
    if (dtype == KD_F32) {
        if (impl != 0 && gemm_f32_ok(A, W.p, N, K, epi)) gemm_f32((const float *)A, (const float *)W.p, (float *)C, M, N, K, epi, s);
        else gemm_simt<float>(A, W, C, M, N, K, epi, sat, s);
        return 1;
    }
    // (the matrix-core kernel stores whole 16-byte pieces of output rows; the SwiGLU ones need pairs of chunks)
    if (impl == 0 || (K % 64) != 0 || (N % 16) != 0 || ((epi == EPI_SWIGLU || epi == EPI_SWIGLU_RS) && (N % 64) != 0)) {
        if (dtype == KD_BF16) gemm_simt<bf16_t>(A, W, C, M, N, K, epi, sat, s);
        else gemm_simt<f16_t>(A, W, C, M, N, K, epi, sat, s);
        return 1;
    }
    // Four waves with a quarter of a large tile each (gemm_large.hip) win above 512 rows, on gate/up above 384 (512 rows x 17920 x
    // 1536 with the norm scale 51.2 -> 37.2 us against three 128-row blocks per CU, 24576 x 4096 108 -> 89) and on the vocabulary
    // projection above 192 (151936 x 1536 / 4096: 160 / 360 -> 157 / 336 us at 256 rows, 218 / 481 -> 206 / 425 at 384, 288 / 601 ->
    // 237 / 512 at 512; not yet at 256 rows of 5120: 444 -> 455, 580 -> 553 at 384); gate/up at 256 rows takes as long either way (27.9 and 27.1 us).
    // Not where the reduction is so short that the epilogue is most of it, which eight waves with half the values each get through
    // faster: gate/up 1024 rows x 6400, K = 64 6.8 against 7.7 us (7000 x 16384: 48.7, 49.5; K = 128: 58.1, 47.5); 600 x 512 / 1024 x 2048
    // with residual, K = 128 9.7 / 14.4 against 10.4 / 14.6, K = 256 11.2 / 16.0 against 11.3 / 15.5; 400 rows of gate/up x 6400, K = 256 6.1
    // against 10.3, K = 384 8.9 against 8.4; 384 x 65552 fp32, K = 128 28.2 against 31.8, K = 256 37.5 against 34.5.
    const int nb128 = (N + 127) / 128;
    const bool swiglu = epi == EPI_SWIGLU || epi == EPI_SWIGLU_RS;
    const bool large = M > 512   ? K >= large_min_k(swiglu) && resid_tile(M, N, K, epi) == RESID_LARGE
                       : swiglu  ? M > 384 && K >= 384
                                 : (M > 384 && nb128 >= 96) ||
                                       (M > 192 && nb128 >= 512 && epi == EPI_STORE_F32 && K >= 256 && (M > 256 || K <= 4096));
    if (large) {
        const int S = launch_gemm_large(dtype, A, W, C, M, N, K, epi, slices, slice_cap_floats, sat, s, row_scale);
        if (S) return S;
    }
    if (dtype == KD_BF16) return gemm_mfma_dispatch<bf16_t>(A, W, C, M, N, K, epi, slices, slice_cap_floats, sat, s, row_scale);
    return gemm_mfma_dispatch<f16_t>(A, W, C, M, N, K, epi, slices, slice_cap_floats, sat, s, row_scale);
}

// ---- q | k | v projection with rotary positions and cache append
// More than 512 rows.  What a tile costs here is its epilogue rather than its products, and eight waves share it better than four:
// while one round of blocks, one per CU, holds them, the smallest tile of gemm_mfma (us, against the best of gemm_large; since then its
// lookups moved ahead of the products: 1024 decode rows x 2048 x 1536 16.4, 600 rows 14.7 where it took 18.6; 128 x 128 21.9 and 19.8):
//   64 x 128    1024 rows x 2048 x 1536  16.8, 25.0 (decode, V all over the cache: 19.9, 26.5);  640 x 1536 x 1024  11.8, 19.7
//   128 x 128   2048 x 2048 x 1536  21.5, 25.7;  640 x 6144 x 4096  40.6, 47.4 (decode 46.6, 49.4);  1024 x 4096 x 2560  34.2, 36.9
// Beyond that gemm_large's estimate decides between its tiles and 256 x 128 (1024 x 7168 x 5120  74.1, 95.6;  4096 x 2048 x 1536
// 31.9, 43.8;  4096 x 6144 x 4096, three full rounds, 185, 199;  6144 x 6144 x 4096  289, 241;  700 decode rows 65.0, 56.5).  Reductions
// below 1024 stay on eight waves (3072 x 1536 x 256  12.6, 19.0;  3072 x 4096 x 768  37.4, 36.9): 256 x 256 for two rounds and more, 128 x 128 two to a CU where
// 256 x 128 would leave half the chip idle.
// With few rows and a wide output a kernel of its own for the rotation is faster, behind K slices: three row blocks of 192 that
// 128 x 128 tiles cannot replace fill two thirds of the chip (576 rows x 7168 x 5120: 62.6 us, 72.1 in 192 x 128 tiles; 640 rows: 67.8,
// 64.9); on eight waves up to three row blocks of 256 (69.9 against 76.0 us at 513 rows x 7168, 82.9 and 84.1 at 768, 91.9 and 87.4 at 896).
enum QkvRoute { QKV_SEPARATE, QKV_64x128, QKV_128x128, QKV_256x128, QKV_256x256, QKV_128x128_2, QKV_LARGE };
static QkvRoute qkv_route(int M, int N, int K) {
    const int64_t nb128 = (N + 127) / 128, mb = (M + 255) / 256;
    if ((M + 63) / 64 * nb128 <= 256) return QKV_64x128;
    if ((M + 127) / 128 * nb128 <= 256) return QKV_128x128;
    if (K >= 1024) return M <= 576 ? QKV_SEPARATE : QKV_LARGE;
    if (M <= 768 && 3 * nb128 >= 160) return QKV_SEPARATE;
    if (mb * ((N + 255) / 256) >= 2 * 256) return QKV_256x256;
    return mb * nb128 >= 160 ? QKV_256x128 : QKV_128x128_2;
}
template <typename T> static void gemm_qkv_t(QkvRoute r, const void *A, WeightRef W, int M, int N, int K, const GemmQkv &qkv, uint32_t *sat, hipStream_t s) {
    typedef Gemm<T> G;
    if (r == QKV_64x128) G::T64x128::template launch<EPI_QKV>(A, W, nullptr, M, N, K, 1, sat, s, qkv);
    else if (r == QKV_128x128) G::T128x128::template launch<EPI_QKV>(A, W, nullptr, M, N, K, 1, sat, s, qkv);
    else if (r == QKV_256x256) G::T256x256::template launch<EPI_QKV>(A, W, nullptr, M, N, K, 1, sat, s, qkv);
    else if (r == QKV_128x128_2) G::T128x128_2::template launch<EPI_QKV>(A, W, nullptr, M, N, K, 1, sat, s, qkv);
    else G::T256x128::template launch<EPI_QKV>(A, W, nullptr, M, N, K, 1, sat, s, qkv);
}
bool launch_gemm_qkv(int dtype, int impl, const void *A, WeightRef W, int M, int K, const GemmQkv &qkv, uint32_t *sat,
                     hipStream_t s) {
    const int N = (qkv.hq + 2 * qkv.kv.n_kv_heads) * qkv.kv.head_dim;
    if (dtype == KD_F32 || impl == 0 || qkv.kv.head_dim != 128 || K % 64 != 0 || M <= 512) return false;
    const QkvRoute r = qkv_route(M, N, K);
    if (r == QKV_SEPARATE) return false;
    if (r == QKV_LARGE && launch_gemm_large_qkv(dtype, A, W, M, N, K, qkv, sat, s)) return true;
    if (dtype == KD_BF16) gemm_qkv_t<bf16_t>(r, A, W, M, N, K, qkv, sat, s);
    else gemm_qkv_t<f16_t>(r, A, W, M, N, K, qkv, sat, s);
    return true;
}

// ---- log-probabilities straight from the vocabulary projection: a scoring pass wrote 622 MB of logits per 1024 rows of the
// 1.5B shape for a softmax kernel to read once (157 us); now all rows of a chunk go through one launch of the large tiles
// (scoring 20 sequences of 700 to 1280 tokens on 4 layers: 19.97 -> 17.90 ms)
static bool logprob_shape_ok(int dtype, int impl, int N, int K) { return dtype != KD_F32 && impl != 0 && K % 64 == 0 && N % 16 == 0; }
static constexpr int LOGPROB_STRIP = 64;   // the narrowest strip of the configurations below

int logprob_fused_rows(int dtype, int impl, int N, int K, size_t scratch_bytes) {
    if (!logprob_shape_ok(dtype, impl, N, K)) return 0;
    const size_t strips = ((size_t)N + 255) / 256 * (256 / LOGPROB_STRIP);
    return (int)std::min<size_t>(scratch_bytes / (strips * (sizeof(double) + sizeof(float)) + sizeof(float)), 1 << 20);
}

// 16 rows per block, 64 threads to a row that share its strips (a few rows must not mean a few blocks: the strips are
// thousands); maxima first, then the sums: no chain through the loads
__global__ __launch_bounds__(1024) void logprob_merge_kernel(GemmLogprob lpa, int M, int N, int strips, float *__restrict__ out) {
    __shared__ float s_m[64][16];
    __shared__ double s_s[64][16];
    const int r = threadIdx.x % 16, part = threadIdx.x / 16, row = blockIdx.x * 16 + r;
    float m = -INFINITY;
    if (row < M) {
#pragma unroll 4
        for (int t = part; t < strips; t += 64) m = fmaxf(m, lpa.part_max[(int64_t)t * M + row]);
    }
    s_m[part][r] = m;
    __syncthreads();
    float mx = -INFINITY;
#pragma unroll 8
    for (int w = 0; w < 64; ++w) mx = fmaxf(mx, s_m[w][r]);
    const float base = (mx == -INFINITY) ? 0.f : mx;
    double s = 0.0;
    if (row < M) {
#pragma unroll 4
        for (int t = part; t < strips; t += 64)
            s += lpa.part_sum[(int64_t)t * M + row] * (double)expf(lpa.part_max[(int64_t)t * M + row] - base);
    }
    s_s[part][r] = s;
    __syncthreads();
    if (part != 0 || row >= M) return;
    double z = 0.0;
#pragma unroll 8
    for (int w = 0; w < 64; ++w) z += s_s[w][r];
    const int target = lpa.tokens[lpa.token_index[row] + 1];
    out[row] = (target >= 0 && target < N) ? (float)((double)(lpa.target[row] * lpa.inv_t) - (double)mx - log(z)) : -INFINITY;
}

template <typename T>
static void gemm_logprob_t(const void *A, WeightRef W, int M, int N, int K, GemmLogprob lpa, float *out, hipStream_t s) {
    typedef Gemm<T> G;
    int strips = 0;
    auto run = [&](auto cfg) {
        strips = decltype(cfg)::strips(N);
        decltype(cfg)::template launch<EPI_LOGPROB>(A, W, nullptr, M, N, K, 1, nullptr, s, lpa);
    };
    // (short reductions: the epilogue is most of it and eight waves get through it faster: 4500 rows x 151936 x 256 616 us against
    // 820, 3072 x 151936 x 512 586 against 688, 1400 and 2048 x 151936 x 768 418 and 586 against 429 and 566)
    if (M > 512 && K >= 1024) strips = launch_gemm_large_logprob(std::is_same<T, bf16_t>::value ? KD_BF16 : KD_F16, A, W, M, N, K, lpa, s);
    if (strips == 0) {
        if ((int64_t)((M + 255) / 256) * ((N + 255) / 256) >= 2 * 256 && M > 512) run(typename G::T256x256());
        else if (M <= 128) run(typename G::T128x128());
        else if (M <= 192) run(typename G::T192x128());
        else run(typename G::T256x128());
    }
    logprob_merge_kernel<<<(M + 15) / 16, 1024, 0, s>>>(lpa, M, N, strips, out);
}

void launch_gemm_logprob(int dtype, const void *A, WeightRef W, int M, int N, int K, float temperature,
                         const int32_t *tokens, const int32_t *token_index, void *scratch, float *out, hipStream_t s) {
    if (M <= 0) return;
    const size_t strips = ((size_t)N + 255) / 256 * (256 / LOGPROB_STRIP);
    double *sums = (double *)scratch;
    float *maxima = (float *)(sums + strips * M);
    const GemmLogprob lpa{1.0f / temperature, tokens, token_index, maxima, maxima + strips * M, sums};
    if (dtype == KD_BF16) gemm_logprob_t<bf16_t>(A, W, M, N, K, lpa, out, s);
    else gemm_logprob_t<f16_t>(A, W, M, N, K, lpa, out, s);
}

template <typename T>
static int gemm_mfma_dispatch(const void *A, WeightRef W, void *C, int M, int N, int K, int epi, float *slices,
                              size_t slice_cap_floats, uint32_t *sat, hipStream_t s, const GemmRowScale *row_scale) {
    // Rules from sweeps of the configurations over the projection shapes of the 1.5B, 8B and 14B models at 3 to 16384 rows.
    typedef Gemm<T> G;
    const bool swiglu = epi == EPI_SWIGLU || epi == EPI_SWIGLU_RS;
    const bool can_split = slices && (epi == EPI_STORE_F32 || epi == EPI_RESID_F32);
    auto whole = [&](auto cfg) {
        decltype(cfg)::run(A, W, C, M, N, K, epi, 1, sat, s, row_scale);
        return 1;
    };
    auto sliced = [&](auto cfg, int want_blocks) {   // K slices where they bring the launch nearer to want_blocks
        typedef decltype(cfg) Cfg;
        const int split = can_split ? Cfg::pick_split(M, N, K, slice_cap_floats, want_blocks) : 1;
        if (split > 1) Cfg::run(A, W, slices, M, N, K, EPI_STORE_F32, split, sat, s);
        else Cfg::run(A, W, C, M, N, K, epi, 1, sat, s);
        return split;
    };
    if (M > 512) {
        const ResidTile resid = resid_tile(M, N, K, epi);
        if (resid != RESID_LARGE) {
            const int S = gemm_large_resid_slices(M, N, K, slices, slice_cap_floats);
            const GemmSlices sums{(K / 64 + S - 1) / S};
            if (resid == RESID_64x64) G::T64x64::template launch<EPI_RESID_SLICES>(A, W, C, M, N, K, 1, sat, s, sums);
            else G::T128x64_3::template launch<EPI_RESID_SLICES>(A, W, C, M, N, K, 1, sat, s, sums);
            return 1;
        }
        if (K >= large_min_k(swiglu)) return whole(typename G::T256x128());   // (gate/up that gemm_large.hip left to this tile; widths beyond its limit)
        // 256 x 256 tiles where they still come in several rounds per CU, 256 x 128 below that
        if ((int64_t)((M + 255) / 256) * ((N + 255) / 256) >= 2 * 256) return whole(typename G::T256x256());
        // (a few row blocks against a narrow projection leave most CUs without a tile: smaller ones, and K slices)
        if ((int64_t)((M + 255) / 256) * ((N + 127) / 128) < 160 && can_split) return sliced(typename G::T128x128_2(), 240);
        return whole(typename G::T256x128());
    }
    // blocks of one round of the chip, one per CU
    auto one_round = [&](int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn) <= 256; };
    // decode: the weights are streamed once; fill the chip with blocks, by K slices where N is small
    const int nb128 = (N + 127) / 128, nb192 = (N + 191) / 192;
    if (swiglu || nb128 >= 96) {   // wide outputs: no K slices needed
        // 128-column tiles that need a second, nearly empty round of blocks (one per CU) where 192-column ones fit the first
        // (14B gate/up, 34816 columns: 272 blocks against 182; 112 / 119 / 162 / 159 us against 74 / 84 / 90 / 132 us at
        // 60 / 116 / 168 / 256 rows)
        const bool second_round = nb128 > 256 && nb192 <= 256;
        if (M <= 32 && !second_round) return swiglu ? whole(typename G::T32x64_2()) : whole(typename G::T32x64());
        // (a 64-row tile buys the vocabulary projection 5 %, gate/up nothing: at 60 rows 22.7 us for 21.7 with the norm scale)
        if (M <= 64 && (second_round || !swiglu)) return second_round ? whole(typename G::T64x192()) : whole(typename G::T64x128());
        if (M <= 128) return second_round ? whole(typename G::T128x192()) : whole(typename G::T128x128());
        if (M <= 192) return second_round ? whole(typename G::T192x192()) : whole(typename G::T192x128());
        if (M <= 256) {
            // Where one row block of 128 columns is more than a round, the narrowest tile that is not (34816 x 5120: 256 x 192 127 us,
            // 256 x 160 106.5; 17920 x 1536 in two row blocks of 128 x 160, 224 CUs instead of 140, is 25.8 us for 28.3 alone, but
            // decode steps on several streams, which fill the idle CUs, take 3 % longer: the same work costs more CU time)
            if (swiglu && second_round && one_round(256, 160)) {
                if (epi == EPI_SWIGLU) G::T256x160::template launch<EPI_SWIGLU>(A, W, C, M, N, K, 1, sat, s, {});
                else G::T256x160::template launch<EPI_SWIGLU_RS>(A, W, C, M, N, K, 1, sat, s, *row_scale);
                return 1;
            }
            return second_round ? whole(typename G::T256x192()) : whole(typename G::T256x128());   // a weight tile is fetched by exactly one block
        }
        // two 192-row blocks instead of two of 256 (380 rows: 24576 x 4096 70 us against 119 us, 17920 x 1536 27 us against 33
        // us with three 128-row blocks)
        if (M <= 384) return whole(typename G::T192x192());
        // (up to 512 rows, gate/up of a short reduction: 400 rows x 6400 x 256 6.1 us, 8.2 in 256 x 128, 7.5 with three 128-row blocks per
        // CU; beyond one round 256 x 128, 400 x 16384 x 256 9.8, 11.6 and 10.4)
        if (swiglu && K < 384 && one_round(128, 128)) return whole(typename G::T128x128());
        return whole(typename G::T256x128());
    }
    // The smallest batches stream the weights and little else: rows loaded for nothing (a tile of 128 for 3) cost as much of
    // the load path as the weights (4096 x 12288 at 3 rows: 20 us against 27 us, 1536 x 8960: 6.6 against 9.5 us)
    if (M <= 32) return sliced(typename G::T32x64(), 480);
    if ((int64_t)N * K >= (int64_t)8 << 20 && nb128 >= 24) {
        // mid-width outputs with large weights (q/k/v, o and down projections of the 8B / 14B models): 128-column
        // tiles cut into about 240 blocks by K slices (8B down at 256 rows: 38 us against 48 us with 128x64 tiles); the tile is
        // as tall as the batch needs (8B down at 60 rows: 22 us, 29 us with 128-row tiles; 14B q/k/v at 168: 25 us, 30 us
        // with 256-row ones)
        if (M <= 64) return sliced(typename G::T64x128(), 240);
        // A shorter reduction is cheaper in few slices of smaller tiles, also for the norm that adds them up (us with that norm: 4096 x
        // 4096 in 4 slices of 128 x 128 24.0 at 256 rows, in 8 of 256 x 128 27.3; 21.5 against 23.2 at 168; 29.2 against 30.0 at 400);
        // wider outputs gain nothing (5120 x 5120 on two cards: 34.0 and 33.7 against 35.9 and 33.1 at 256 rows, 31.1 against 30.8 at 168,
        // 29.3 against 28.9 at 129), nor do longer reductions (6144 x 4096 at 168: 22.3 for 22.2 without a norm; 4096 x 12288 at 256: 41.4
        // for 40.8)
        if (K <= 5120 && nb128 <= 32 && ((M > 128 && M <= 256) || M > 384)) return sliced(typename G::T128x128(), 240);
        if (M <= 128) return sliced(typename G::T128x128(), 240);
        if (M <= 192) return sliced(typename G::T192x128(), 240);
        if (M > 256 && M <= 384) return sliced(typename G::T192x192(), 240);   // 8B down at 380 rows: 44 us against 49 us
        return sliced(typename G::T256x128(), 240);
    }
    if ((int64_t)N * K >= (int64_t)8 << 20) {   // narrow output, long K (the 1.5B model's down projection)
        if (M <= 64) return sliced(typename G::M64x64(), 240);   // 8.2 us against 10.4 us with 128-row tiles at 60 rows
        // (4 waves of 64x32 took 16.1 us for 15.8 at 256 rows and 12.0 for 11.8 at 116)
        if (M <= 256) return sliced(typename G::T128x64(), 240);
        // One block per CU and 32 CUs to a die: with three and four row blocks of 128 x 64 the slices no longer come out even
        // over the dies (1536 x 8960 at 420 rows: 72 slices, 9 to a die, 36 blocks on its CUs).  Two row blocks up to 384
        // (17.2 us at 300 rows, 18.8 with three of 128), then four of twice the width (420 rows: 20.2 us against 35.5 us with
        // 128 x 64, 22.2 us with 256 x 64; the same order for 2048 x 6144 and 2560 x 4096)
        if (M <= 384) return sliced(typename G::T192x64(), 240);
        return sliced(typename G::T128x128(), 240);
    }
    return sliced(typename G::M64x64(), 192);
}

}  // namespace pc

// For tests, not part of the C ABI: a projection of 16-bit operands in the tile that the library chooses, W in slabs or in plain rows.  The
// number of K slices, 1: the result is in C; 0: not such a call.
extern "C" int pc_internal_gemm(int dtype, int epi, const void *A, const void *W, int slabs, void *C, int M, int N, int K, float *slices,
                                size_t slice_cap_floats, uint32_t *sat, void *stream) {
    using namespace pc;
    if ((dtype != KD_BF16 && dtype != KD_F16) || (epi != EPI_STORE_F32 && epi != EPI_RESID_F32 && epi != EPI_SWIGLU) || !A || !W || !C || M <= 0 ||
        N <= 0 || N % 64 != 0 || K <= 0 || K % 64 != 0 || (((uintptr_t)A | (uintptr_t)W | (uintptr_t)C | (uintptr_t)slices) & 15) != 0)
        return 0;
    gemm_init();
    return launch_gemm(dtype, 1, A, WeightRef(W, slabs ? WEIGHT_SLAB : 0), C, M, N, K, epi, slices, slice_cap_floats, sat, (hipStream_t)stream, nullptr);
}
// For tests, not part of the C ABI: the ResidTile of a residual projection and the QkvRoute of a q/k/v projection of more than 512 rows, and
// one launch in the tile of a q/k/v route, W in plain rows or (_slabs) in the order of the 16-bit copies (`extra`: a GemmQkv).  1: launched;
// 0: not a tile of this file, or not a call that the kernels take.
extern "C" int pc_internal_resid_tile(int M, int N, int K) { return pc::resid_tile(M, N, K, pc::EPI_RESID_F32); }
extern "C" int pc_internal_qkv_route(int M, int N, int K) { return pc::qkv_route(M, N, K); }
namespace pc {
static int qkv_by_route(int dtype, int route, const void *A, WeightRef w, int M, int N, int K, const void *extra, uint32_t *sat, void *stream) {
    if ((dtype != KD_BF16 && dtype != KD_F16) || route <= QKV_SEPARATE || route >= QKV_LARGE || !A || !w.p || !extra || M <= 0 || N <= 0 ||
        N % 128 != 0 || K <= 0 || K % 64 != 0 || (((uintptr_t)A | (uintptr_t)w.p) & 15) != 0)
        return 0;
    gemm_init();
    if (dtype == KD_BF16) gemm_qkv_t<bf16_t>((QkvRoute)route, A, w, M, N, K, *(const GemmQkv *)extra, sat, (hipStream_t)stream);
    else gemm_qkv_t<f16_t>((QkvRoute)route, A, w, M, N, K, *(const GemmQkv *)extra, sat, (hipStream_t)stream);
    return 1;
}
}  // namespace pc
extern "C" int pc_internal_gemm_qkv(int dtype, int route, const void *A, const void *W, int M, int N, int K, const void *extra, uint32_t *sat,
                                    void *stream) {
    return pc::qkv_by_route(dtype, route, A, pc::WeightRef(W, 0), M, N, K, extra, sat, stream);
}
extern "C" int pc_internal_gemm_qkv_slabs(int dtype, int route, const void *A, const void *W, int M, int N, int K, const void *extra,
                                          uint32_t *sat, void *stream) {
    return pc::qkv_by_route(dtype, route, A, pc::WeightRef(W, pc::WEIGHT_SLAB), M, N, K, extra, sat, stream);
}
