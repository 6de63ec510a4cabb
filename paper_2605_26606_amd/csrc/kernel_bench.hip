// Standalone driver for the two kernels that dominate a decode step: it launches the library's own
// decode-attention kernel and projection GEMMs, in the launch configurations of the 1.5B-shaped
// workload, with synthetic cache contents, and times them with HIP events.  Used for tuning and for
// hardware-counter runs (rocprofv3 --pmc), which need a plain process without HIP graphs.
//
//   kernel_bench attn [n_seqs group prompt_len gen_len block_size grouped_only event_study]   (defaults 256 4 256 512 64 0 0)
//       event_study: also brackets single launches with an event pair, as the library's per-launch timing does,
//       next to pairs around nothing / one / two empty kernels and around two launches
//   kernel_bench gemm
//   kernel_bench tiles [launch ...]                         (projections of more than 512 rows in every tile and K slicing:
//       what the choice of gemm_large.hip is fitted to; launches as listed in bench_tiles, all by default)
//   kernel_bench copy                                       (a plain 1 GiB copy: the counters' known-size reference)
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "attention.hip"   // (elementwise.hip is linked)
#include "gemm.hip"
#include "gemm_large.hip"

namespace pc {
void set_error(const char *, ...) {}
}
using namespace pc;

#define CK(x)                                                                          \
    do {                                                                               \
        hipError_t e_ = (x);                                                           \
        if (e_ != hipSuccess) {                                                        \
            fprintf(stderr, "%s: %s\n", #x, hipGetErrorString(e_));                    \
            return 1;                                                                  \
        }                                                                              \
    } while (0)

__global__ void fill_half_kernel(uint16_t *p, size_t n, uint32_t seed) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        // (well mixed: of values that repeat every 1024, as a product alone gives them, fewer bits change from one product to the next, the
        // matrix cores draw less power and the chip holds a higher clock, by an amount that depends on the order of the weights)
        uint32_t h = (uint32_t)i ^ seed;
        for (int r = 0; r < 3; ++r) {
            h *= 2654435761u;
            h ^= h >> 15;
        }
        p[i] = 0x2800 | (h & 0x3FF) | ((h >> 3) & 0x8000);   // +-(0.03 .. 0.06) as IEEE half
    }
}
__global__ void copy_kernel(const float4 *__restrict__ src, float4 *__restrict__ dst, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

__global__ void null_kernel() {}

static int bench_attention(int n, int group, int lp, int gen, int bs, bool grouped_only, bool event_study) {
    const int L = 28, hq = 12, hkv = 2, hd = 128;
    const int P = n / group, ctx = lp + gen;
    const int pre_blocks = lp / bs, own_blocks = (ctx + bs - 1) / bs - pre_blocks, per_slot = pre_blocks + own_blocks;
    const int64_t n_blocks = (int64_t)P * pre_blocks + (int64_t)n * own_blocks;
    const int64_t block_elems = (int64_t)hkv * 2 * bs * hd;
    void *pool;
    CK(hipMalloc(&pool, (size_t)(L * n_blocks * block_elems * 2)));
    fill_half_kernel<<<(unsigned)((L * n_blocks * block_elems + 255) / 256), 256>>>((uint16_t *)pool,
                                                                                    (size_t)(L * n_blocks * block_elems), 9);
    std::vector<int32_t> table((size_t)n * per_slot), len(n, ctx - 1), slot(n);
    for (int s = 0; s < n; ++s) {
        slot[s] = s;
        for (int b = 0; b < pre_blocks; ++b) table[(size_t)s * per_slot + b] = (s / group) * pre_blocks + b;
        for (int b = 0; b < own_blocks; ++b) table[(size_t)s * per_slot + pre_blocks + b] = P * pre_blocks + s * own_blocks + b;
    }
    int32_t *d_table, *d_len, *d_slot;
    CK(hipMalloc(&d_table, table.size() * 4));
    CK(hipMalloc(&d_len, n * 4));
    CK(hipMalloc(&d_slot, n * 4));
    CK(hipMemcpy(d_table, table.data(), table.size() * 4, hipMemcpyHostToDevice));
    CK(hipMemcpy(d_len, len.data(), n * 4, hipMemcpyHostToDevice));
    CK(hipMemcpy(d_slot, slot.data(), n * 4, hipMemcpyHostToDevice));
    void *q, *out;
    float *scratch;
    CK(hipMalloc(&q, (size_t)n * hq * hd * 2));
    CK(hipMalloc(&out, (size_t)n * hq * hd * 2));
    fill_half_kernel<<<(n * hq * hd + 255) / 256, 256>>>((uint16_t *)q, (size_t)n * hq * hd, 3);
    CK(hipMalloc(&scratch, attention_decode_scratch_floats(n, hq, hd) * 4));
    KvGeom kv;
    kv.pool = pool;
    kv.layer_stride = n_blocks * block_elems;
    kv.block_size = bs;
    kv.n_kv_heads = hkv;
    kv.head_dim = hd;
    kv.max_blocks_per_slot = per_slot;
    kv.block_table = d_table;
    const int splits = attention_decode_splits(n, hkv, ctx + 64);
    hipEvent_t e0, e1;
    CK(hipEventCreate(&e0));
    CK(hipEventCreate(&e1));
    for (int g : {group, 1}) {
        if (grouped_only && g != group) continue;
        auto layer = [&](int l) {   // the merge pass only runs when the context is split
            launch_attention_decode_mfma(KD_F16, q, d_slot, d_len, n, hq, kv, l, splits, g, scratch, out, nullptr, 0);
            launch_attention_decode_merge(KD_F16, d_slot, d_len, n, hq, hkv, splits, scratch, out, nullptr, 0);
        };
        for (int l = 0; l < L; ++l) layer(l);
        CK(hipDeviceSynchronize());
        const int reps = 3;
        CK(hipEventRecord(e0, 0));
        for (int r = 0; r < reps; ++r)
            for (int l = 0; l < L; ++l) layer(l);
        CK(hipEventRecord(e1, 0));
        CK(hipEventSynchronize(e1));
        float ms;
        CK(hipEventElapsedTime(&ms, e0, e1));
        const double us = ms * 1e3 / (reps * L);
        const double alg = ((double)P * lp + (double)n * gen) * 2 * hkv * hd * 2;       // prefix once per prompt
        const double raw = (double)n * ctx * 2 * hkv * hd * 2;                          // prefix once per sequence
        printf("attention n=%d group=%d(order %d) block %d ctx=%d+%d splits=%d: %.2f us/launch  algorithmic %.1f MB -> %.0f GB/s  "
               "(per-sequence bytes %.1f MB -> %.0f GB/s)  %s\n",
               n, group, g, bs, lp, gen, splits, us, alg / 1e6, alg / us / 1e3, raw / 1e6, raw / us / 1e3,
               hipGetErrorString(hipGetLastError()));
        if (event_study && g == group) {
            // what an event pair reads around k launches of a kernel, averaged
            auto pair_us = [&](int k, bool attn, double *out_us) -> int {
                const int reps = 3;
                double tot = 0;
                for (int r = 0; r < reps; ++r)
                    for (int l = 0; l < L; ++l) {
                        CK(hipEventRecord(e0, 0));
                        for (int c = 0; c < k; ++c) {
                            if (attn) layer(l);
                            else null_kernel<<<1, 64>>>();
                        }
                        CK(hipEventRecord(e1, 0));
                        CK(hipEventSynchronize(e1));
                        float one;
                        CK(hipEventElapsedTime(&one, e0, e1));
                        tot += one;
                    }
                *out_us = tot * 1e3 / (reps * L);
                return 0;
            };
            double p0, n1, n2, a1, a2;
            if (pair_us(0, false, &p0) || pair_us(1, false, &n1) || pair_us(2, false, &n2) || pair_us(1, true, &a1) ||
                pair_us(2, true, &a2))
                return 1;
            printf("event pair around: nothing %.2f us, one empty kernel %.2f us, two empty kernels %.2f us, "
                   "one attention launch %.2f us, two attention launches %.2f us\n", p0, n1, n2, a1, a2);
            printf("  attention launch: %.2f us by (pair - empty pair), %.2f us by (two launches - one launch)\n", a1 - p0,
                   a2 - a1);
        }
    }
    return 0;
}

template <typename Cfg>
static int run_gemm(const char *name, int M, int N, int K, int epi, int split, std::vector<void *> &Ws, void *A, void *C,
                    float *slices) {
    Cfg::init();
    hipEvent_t e0, e1;
    CK(hipEventCreate(&e0));
    CK(hipEventCreate(&e1));
    const int ring = (int)Ws.size();
    const int lg = weight_lg(KD_F16, N, K);   // (the order of a model's copies; the values are the same everywhere)
    for (int i = 0; i < 3; ++i) Cfg::run(A, {Ws[i % ring], lg}, split > 1 ? (void *)slices : C, M, N, K, epi, split, nullptr, 0);
    CK(hipDeviceSynchronize());
    const int iters = 24;
    CK(hipEventRecord(e0, 0));
    for (int i = 0; i < iters; ++i) Cfg::run(A, {Ws[i % ring], lg}, split > 1 ? (void *)slices : C, M, N, K, epi, split, nullptr, 0);
    CK(hipEventRecord(e1, 0));
    CK(hipEventSynchronize(e1));
    float ms;
    CK(hipEventElapsedTime(&ms, e0, e1));
    const double us = ms * 1000 / iters;
    printf("gemm %-28s M=%5d N=%6d K=%5d slices=%2d: %8.2f us  weights %.2f TB/s  %.1f TFLOP/s  %s\n", name, M, N, K, split,
           us, (double)N * K * 2 / us / 1e6, 2.0 * M * N * K / us / 1e6, hipGetErrorString(hipGetLastError()));
    return 0;
}

// the tile that the library's own dispatch picks
struct Dispatched {
    static void init() { gemm_init(); }
    static void run(const void *A, WeightRef W, void *C, int M, int N, int K, int epi, int, uint32_t *sat, hipStream_t s) {
        launch_gemm(KD_F16, 1, A, W, C, M, N, K, epi, nullptr, 0, sat, s);
    }
};

static int bench_gemm() {
    typedef f16_t T;
    const size_t NK = (size_t)17920 * 1536;
    void *A, *C;
    float *slices;
    CK(hipMalloc(&A, (size_t)16384 * 8960 * 2));
    fill_half_kernel<<<(unsigned)(((size_t)16384 * 8960 + 255) / 256), 256>>>((uint16_t *)A, (size_t)16384 * 8960, 1);
    std::vector<void *> Ws(12);   // a ring larger than the caches: every launch streams its weights from HBM
    for (size_t i = 0; i < Ws.size(); ++i) {
        CK(hipMalloc(&Ws[i], NK * 2));
        fill_half_kernel<<<(unsigned)((NK + 255) / 256), 256>>>((uint16_t *)Ws[i], NK, 77 + (uint32_t)i);
    }
    CK(hipMalloc(&C, (size_t)16384 * 17920 * 4));
    CK(hipMalloc(&slices, (size_t)32 << 20));
    CK(hipDeviceSynchronize());
    int rc = 0;
    rc |= run_gemm<Gemm<T>::T256x128>("decode gate/up (SwiGLU)", 256, 17920, 1536, EPI_SWIGLU, 1, Ws, A, C, slices);
    rc |= run_gemm<Gemm<T>::T128x64>("decode down", 256, 1536, 8960, EPI_STORE_F32, 5, Ws, A, C, slices);
    rc |= run_gemm<Gemm<T>::M64x64>("decode o-proj", 256, 1536, 1536, EPI_STORE_F32, 2, Ws, A, C, slices);
    rc |= run_gemm<Gemm<T>::M64x64>("decode qkv", 256, 2048, 1536, EPI_STORE_F32, 2, Ws, A, C, slices);
    rc |= run_gemm<Dispatched>("prefill gate/up (SwiGLU)", 16384, 17920, 1536, EPI_SWIGLU, 1, Ws, A, C, slices);
    rc |= run_gemm<Dispatched>("prefill down (+residual)", 16384, 1536, 8960, EPI_RESID_F32, 1, Ws, A, C, slices);
    return rc;
}

// One line per launch: name, rows, columns, K, "dec" (every row a sequence of its own, as in a decode step) or "pre" (prompts), then
// the best of five times in us of every form that computes it: tile[/K slices], m...: a tile of gemm_mfma.  A projection onto the
// residual stream includes the norm behind it, which reads the slices.  Weights come from memory, activations are hot.
static int bench_tiles(int n_only, char **only) {
    typedef f16_t T;
    typedef Gemm<T> G;
    typedef Large<T> L;
    const int RMAX = 16384, SLOTS = 1024, PER_SLOT = 32, BS = 64, HKV = 8;
    const size_t W_BYTES = (size_t)3 << 30, SLICE_CAP = (size_t)8 << 20;
    char *A, *W, *C, *out;
    float *slices, *table_f, *gain;
    void *pool;
    CK(hipMalloc(&A, (size_t)RMAX * 17408 * 2));
    CK(hipMalloc(&W, W_BYTES));
    CK(hipMalloc(&C, (size_t)RMAX * 17920 * 4));
    CK(hipMalloc(&out, (size_t)RMAX * 17920 * 2));
    CK(hipMalloc(&slices, SLICE_CAP * 4));
    CK(hipMalloc(&table_f, 4096 * 64 * 4));   // rotary cosines and sines
    CK(hipMalloc(&gain, RMAX * 4));
    CK(hipMalloc(&pool, (size_t)SLOTS * PER_SLOT * BS * HKV * 128 * 2 * 2));
    fill_half_kernel<<<(unsigned)((size_t)RMAX * 17408 / 256), 256>>>((uint16_t *)A, (size_t)RMAX * 17408, 1);
    fill_half_kernel<<<(unsigned)(W_BYTES / 2 / 256), 256>>>((uint16_t *)W, W_BYTES / 2, 77);
    CK(hipMemset(C, 0, (size_t)RMAX * 17920 * 4));
    CK(hipMemset(table_f, 0, 4096 * 64 * 4));
    CK(hipMemset(gain, 0, RMAX * 4));
    std::vector<int32_t> blocks((size_t)SLOTS * PER_SLOT), id(RMAX + 8), prompt(RMAX), in_prompt(RMAX), seq(RMAX), len(SLOTS), token(RMAX + 8);
    for (size_t i = 0; i < blocks.size(); ++i) blocks[i] = (int)((i * 7919 + 13) % blocks.size());   // (7919 is prime: a permutation)
    for (int i = 0; i < RMAX; ++i) {
        prompt[i] = i / 512;
        in_prompt[i] = i % 512;
        seq[i] = i % SLOTS;
    }
    for (int i = 0; i < SLOTS; ++i) len[i] = 300 + i * 37 % 1200;
    for (int i = 0; i < RMAX + 8; ++i) {
        id[i] = i;
        token[i] = i * 977 % 150000;
    }
    auto up = [](const std::vector<int32_t> &v) {
        int32_t *p = nullptr;
        if (hipMalloc(&p, v.size() * 4) != hipSuccess || hipMemcpy(p, v.data(), v.size() * 4, hipMemcpyHostToDevice) != hipSuccess) exit(1);
        return p;
    };
    int32_t *d_blocks = up(blocks), *d_id = up(id), *d_prompt = up(prompt), *d_in = up(in_prompt), *d_seq = up(seq), *d_len = up(len),
            *d_token = up(token);
    KvGeom kv{pool, 0, BS, HKV, 128, PER_SLOT, d_blocks};
    gemm_init();
    hipEvent_t e0, e1;
    CK(hipEventCreate(&e0));
    CK(hipEventCreate(&e1));
    struct Launch { const char *name; int epi, N, K, hq = 0, hkv = 0; };
    std::vector<Launch> launches = {
        {"qkv1.5", EPI_QKV, 2048, 1536, 12, 2}, {"qkv8", EPI_QKV, 6144, 4096, 32, 8}, {"qkv14", EPI_QKV, 7168, 5120, 40, 8},
        {"qkv1k", EPI_QKV, 1536, 1024, 8, 2}, {"qkv2.5k", EPI_QKV, 4096, 2560, 16, 8}, {"o1.5", EPI_RESID_F32, 1536, 1536},
        {"o8", EPI_RESID_F32, 4096, 4096}, {"o14", EPI_RESID_F32, 5120, 5120}, {"down1.5", EPI_RESID_F32, 1536, 8960},
        {"down8", EPI_RESID_F32, 4096, 12288}, {"down14", EPI_RESID_F32, 5120, 17408}, {"o2.5k", EPI_RESID_F32, 2560, 2048},
        {"down2.5k", EPI_RESID_F32, 2560, 9728}, {"gu1.5", EPI_SWIGLU, 17920, 1536}, {"gu8", EPI_SWIGLU, 24576, 4096},
        {"gu14", EPI_SWIGLU, 34816, 5120}, {"gu2.5k", EPI_SWIGLU, 19456, 2560}, {"head1.5", EPI_STORE_F32, 151936, 1536},
        {"head8", EPI_STORE_F32, 151936, 4096}, {"head14", EPI_STORE_F32, 151936, 5120}, {"head32k", EPI_STORE_F32, 32000, 2048},
        {"lp1.5", EPI_LOGPROB, 151936, 1536}, {"lp8", EPI_LOGPROB, 151936, 4096}, {"lp32k", EPI_LOGPROB, 32000, 2048}};
    for (int K : {128, 256, 512, 768}) {   // short reductions, as far down as these tiles are used
        for (int N : {2368, 6400, 16384}) launches.push_back({"gu_k", EPI_SWIGLU, N, K});
        if (K < 256) continue;
        for (int N : {512, 2048}) launches.push_back({"o_k", EPI_RESID_F32, N, K});
        for (int N : {32768, 65552}) launches.push_back({"head_k", EPI_STORE_F32, N, K});
    }
    const int rows[] = {513, 576, 640, 704, 768, 832, 896, 960, 1024, 1152, 1280, 1408, 1536, 1792, 2048, 2560, 3072, 3500, 4096, 5000,
                        6144, 7000, 8192, 10000, 12288, 16384};
    for (const Launch &l : launches)
        for (int M : rows)
            for (int decode = l.epi == EPI_QKV && M <= SLOTS; decode >= 0; --decode) {
                const double about = 2.0 * M * l.N * l.K / 0.9e9 + (double)l.N * l.K * 2 / 4.5e6 + 8;
                bool wanted = n_only == 0;
                for (int i = 0; i < n_only; ++i) wanted |= !strcmp(only[i], l.name);
                if (!wanted || about > 2500 || (l.epi == EPI_STORE_F32 && M > 1024)) continue;
                struct Form { std::string name; int tile, S; double us; };   // tile >= 100: gemm_mfma's
                std::vector<Form> forms;
                for (int t = 0; t < LT_COUNT; ++t)
                    for (int S = 1; S <= (l.epi == EPI_RESID_F32 ? 8 : 1); ++S) {
                        const int bm = LARGE_SHAPES[t][0], bn = LARGE_SHAPES[t][1];
                        const int64_t tiles = (int64_t)((M + bm - 1) / bm) * ((l.N + bn - 1) / bn) * S;
                        if (!(large_tiles(l.epi) >> t & 1) || !large_slices_ok(S, l.K) || (size_t)S * M * l.N > (S > 1 ? SLICE_CAP : (size_t)-1)) continue;
                        if ((S > 1 && tiles > 520) || (tiles > 256 * 24 && bm * bn < 192 * 192)) continue;
                        forms.push_back({std::to_string(bm) + "x" + std::to_string(bn) + (S > 1 ? "/" + std::to_string(S) : ""), t, S, 1e9});
                    }
                if (l.epi == EPI_QKV) {
                    forms.push_back({"m64x128", 100, 1, 1e9});
                    forms.push_back({"m128x128", 101, 1, 1e9});
                }
                if (l.epi == EPI_QKV || l.epi == EPI_SWIGLU) forms.push_back({"m256x128", 102, 1, 1e9});
                if (l.epi == EPI_RESID_F32 && l.K <= 3072) {   // (blocks that run in two rounds at most)
                    auto blocks = [&](int bm) { return (int64_t)((M + bm - 1) / bm) * ((l.N + 63) / 64); };
                    if (blocks(64) <= 1024) forms.push_back({"m64x64", 103, 1, 1e9});
                    if (blocks(128) <= 512) forms.push_back({"m128x64", 104, 1, 1e9});
                }
                const int slices_of = gemm_large_resid_slices(M, l.N, l.K, slices, SLICE_CAP);
                const GemmSlices sums{(l.K / 64 + slices_of - 1) / slices_of};
                const GemmQkv q{decode ? d_seq : d_prompt, decode ? nullptr : d_in, d_len, table_f, table_f, kv, 0, l.hq, out};
                kv.n_kv_heads = l.hkv;
                const size_t strips = ((size_t)l.N + 255) / 256 * 4;
                float *maxima = (float *)(C + strips * M * 8);
                const GemmLogprob lp{1.0f, d_token, d_id, maxima, maxima + strips * M, (double *)C};
                auto run = [&](const Form &f, const char *rows) {
                    const WeightRef w(rows, weight_lg(KD_F16, l.N, l.K));   // the order of a model's copies
                    if (l.epi == EPI_QKV) {
                        GemmQkv a = q;
                        a.kv = kv;
                        if (f.tile == 100) G::T64x128::launch<EPI_QKV>(A, w, nullptr, M, l.N, l.K, 1, nullptr, 0, a);
                        else if (f.tile == 101) G::T128x128::launch<EPI_QKV>(A, w, nullptr, M, l.N, l.K, 1, nullptr, 0, a);
                        else if (f.tile == 102) G::T256x128::launch<EPI_QKV>(A, w, nullptr, M, l.N, l.K, 1, nullptr, 0, a);
                        else L::launch<EPI_QKV>(f.tile, A, w, nullptr, M, l.N, l.K, 1, nullptr, 0, a);
                    } else if (f.tile == 103) {
                        G::T64x64::launch<EPI_RESID_SLICES>(A, w, C, M, l.N, l.K, 1, nullptr, 0, sums);
                    } else if (f.tile == 104) {
                        G::T128x64_3::launch<EPI_RESID_SLICES>(A, w, C, M, l.N, l.K, 1, nullptr, 0, sums);
                    } else if (f.tile == 102) {
                        G::T256x128::launch<EPI_SWIGLU>(A, w, out, M, l.N, l.K, 1, nullptr, 0, {});
                    } else if (l.epi == EPI_LOGPROB) {
                        L::named(f.tile, EPI_LOGPROB, A, w, nullptr, M, l.N, l.K, 1, &lp, nullptr, 0);
                    } else {
                        L::named(f.tile, f.S > 1 ? EPI_STORE_F32 : l.epi, A, w, f.S > 1 ? (void *)slices : l.epi == EPI_SWIGLU ? (void *)out : (void *)C,
                                 M, l.N, l.K, f.S, nullptr, nullptr, 0);
                    }
                    if (l.epi == EPI_RESID_F32) launch_rmsnorm(KD_F16, (float *)C, nullptr, gain, M, l.N, 1e-6f, out, slices, f.S, nullptr, 0);
                };
                const size_t w_size = (size_t)l.N * l.K * 2;
                const int ring = (int)(W_BYTES / w_size), iters = (int)std::max(3.0, std::min(30.0, 900.0 / about));
                int at = 0;
                for (int rep = 0; rep < 5; ++rep)
                    for (Form &f : forms) {
                        if (rep == 0) run(f, W + (size_t)(at++ % ring) * w_size);
                        CK(hipEventRecord(e0, 0));
                        for (int i = 0; i < iters; ++i) run(f, W + (size_t)(at++ % ring) * w_size);
                        CK(hipEventRecord(e1, 0));
                        CK(hipEventSynchronize(e1));
                        CK(hipGetLastError());
                        float ms;
                        CK(hipEventElapsedTime(&ms, e0, e1));
                        f.us = std::min(f.us, ms * 1e3 / iters);
                    }
                double best = 1e9;
                for (const Form &f : forms) best = std::min(best, f.us);
                printf("%s %d %d %d %s |", l.name, M, l.N, l.K, decode ? "dec" : "pre");
                for (const Form &f : forms)
                    if (f.us < 1.6 * best) printf(" %s=%.2f", f.name.c_str(), f.us);
                printf("\n");
                fflush(stdout);
            }
    return 0;
}

static int bench_copy() {
    const size_t bytes = (size_t)1 << 30, n = bytes / 16;
    float4 *src, *dst;
    CK(hipMalloc((void **)&src, bytes));
    CK(hipMalloc((void **)&dst, bytes));
    CK(hipMemset(src, 1, bytes));
    for (int i = 0; i < 3; ++i) copy_kernel<<<(unsigned)((n + 255) / 256), 256>>>(src, dst, n);
    CK(hipDeviceSynchronize());
    printf("copy_kernel: 3 launches, each reads 1 GiB (1048576 KiB) and writes 1 GiB\n");
    return 0;
}

int main(int argc, char **argv) {
    const char *what = argc > 1 ? argv[1] : "attn";
    if (!strcmp(what, "attn")) {
        const int n = argc > 2 ? atoi(argv[2]) : 256, g = argc > 3 ? atoi(argv[3]) : 4;
        const int lp = argc > 4 ? atoi(argv[4]) : 256, gen = argc > 5 ? atoi(argv[5]) : 512;
        const int bs = argc > 6 ? atoi(argv[6]) : 64;
        if (n <= 0 || g <= 0 || n % g || lp <= 0 || (bs != 32 && bs != 64 && bs != 128) || lp % bs || gen <= 0) {
            fprintf(stderr, "bad sizes\n");
            return 2;
        }
        return bench_attention(n, g, lp, gen, bs, argc > 7 && atoi(argv[7]) != 0, argc > 8 && atoi(argv[8]) != 0);
    }
    if (!strcmp(what, "gemm")) return bench_gemm();
    if (!strcmp(what, "tiles")) return bench_tiles(argc - 2, argv + 2);
    if (!strcmp(what, "copy")) return bench_copy();
    fprintf(stderr, "usage: kernel_bench attn|gemm|tiles|copy\n");
    return 2;
}
