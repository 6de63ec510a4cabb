// Token sampling o_t ~ softmax(logits / T) (Section 3.1; Section 4.2: T = 1.0,
// top_p = 1.0) by inverse CDF with a Philox4x32-10 uniform.
//
// One block of 16 waves per row.  The row is read from HBM once: every wave
// keeps an online (max, sum) of a contiguous segment, the block locates the
// segment whose cumulative weight crosses u*Z, then narrows it twice more
// (16 sub-segments, then an in-order wavefront scan), re-reading only that
// segment.  Sums are accumulated in double so that the selected token agrees
// with an in-order double-precision CDF except within rounding of a boundary.
//
// A pass over a row costs its instructions about as much as its memory: 19 a token, of which the weight's exponential is eleven and its
// way into the sum two.  With expf's range tests, a branch or a select per token for the end of the row and the EOS id and
// a rescaling under selects they were 26: 256 rows of 151936 logits, passes on three streams, 35.3 -> 27.9 us; 1024 rows back to back
// 154 -> 125 us (5.0 TB/s, the copy rate).
//
// Nucleus truncation (top_p < 1): the tokens in order of decreasing probability (ties: lower id first) until their
// cumulative mass reaches top_p keep their weight, the rest get none; the passes above then run on the kept tokens.
// The first pass of the scheme above gives the maximum and Z of the whole row; there are two ways from there to the cut:
//   binned (nucleus_binned): the first pass also files the tokens that can matter in bins of 1/32 of a scaled logit, with
//     a count and a sum of 25-bit fractions in ONE 64-bit LDS integer add; the bin in which the mass from the top crosses
//     top_p Z is known then.  A second pass sums the float weights in front of that bin and lists the bin's own tokens in
//     LDS, where the exact cut is found.  It, and the pass over the kept tokens, leave out the granules (256 tokens) whose
//     maximum is behind the cut.  The row is read once, and as much of it as has kept tokens twice more.
//   radix (any row): a select over an order-preserving 32-bit key of the logit, four passes of 8 bits with a histogram of
//     the mass per bucket (double, one histogram per wave, added up in wave order).  The row is read four times and the few
//     buckets in use make the LDS adds collide.  Taken when the binned way cannot be: more than 5120 tokens in the
//     crossing bin (logits almost all alike), scaled logits beyond 1e5, more than 2^18 tokens.
//   Both decide on the same float weights and the same Z, so they keep the same tokens.
// The kept tokens then go through the first pass again: tokens and log-probabilities are those of plain sampling with all
// other tokens masked, to the last bit.
//   1024 rows of 151936 logits, T = 0.7, top_p = 0.95 (a read of the rows at the copy rate: 121 us): 1509 us by the radix way; 469 us binned
//   with a binning pass of its own and no granules left out, 202 us so, where a few dozen tokens hold most of the mass; 565 and 464
//   where the cut is in the bulk of the vocabulary.  (Filing costs the first pass 8 us a row while two share a CU, the pass it replaces
//   was 20.)  Rows that fall back have paid for the bins: 1901 and 1859 us with logits rounded to whole numbers.
#include <type_traits>

#include "pc_internal.h"

namespace pc {

static constexpr int WAVE = 64;
static constexpr int SAMPLE_WAVES = 16;

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies
__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                                     uint32_t out[4]) {
    const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(M0, c0), lo0 = M0 * c0;
        const uint32_t hi1 = __umulhi(M1, c2), lo1 = M1 * c2;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += W0; k1 += W1;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

__device__ inline double wave_sum_d(double v) {
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    return v;
}
__device__ inline float wave_max_f32(float v) {
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, WAVE));
    return v;
}

// order-preserving key of a float: a < b  <=>  okey(a) < okey(b)
__device__ inline uint32_t okey(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ inline float key_logit(uint32_t key) { return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key); }
// Largest of the wave's 64 values, in every lane, without a trip through LDS: rows of 16 lanes, then over the rows.
__device__ inline float wave_max_all(float v) {
    auto fold = [&](auto ctrl) {   // (lanes without a source keep their own)
        const int o = __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false);
        v = fmaxf(v, __int_as_float(o));
    };
    fold(std::integral_constant<int, 0x111>{});   // row_shr 1, 2, 4, 8
    fold(std::integral_constant<int, 0x112>{});
    fold(std::integral_constant<int, 0x114>{});
    fold(std::integral_constant<int, 0x118>{});
    fold(std::integral_constant<int, 0x142>{});   // row_bcast 15, 31
    fold(std::integral_constant<int, 0x143>{});
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), WAVE - 1));
}
// exp(d) for -103 <= d <= 0 as 2^(d log2 e), with Cody and Waite's two-piece constant: log2 e is a float and the float nearest to what that one
// leaves; the product with the first is split exactly into its rounded value and the rest of it (fma), the nearest whole number goes into the
// exponent, and what is left, at most 1/2 and a little, is the argument of the hardware's 2^x.  To the bit what expf gives (a test compares
// the two).  expf also asks whether the result under- or overflows, four of its fourteen instructions; the passes over a row are bound by
// them as much as by memory.
__device__ inline float exp_weight_near(float d) {
#pragma clang fp contract(off)
    const float hi = d * 0x1.715476p+0f;
    const float lo = fmaf(d, 0x1.4ae0bep-26f, fmaf(d, 0x1.715476p+0f, -hi));
    const float n = rintf(hi);
    return ldexpf(__builtin_amdgcn_exp2f((hi - n) + lo), (int)n);
}
__device__ inline float exp_weight(float d) {   // any d <= 0, minus infinity too
    const float w = exp_weight_near(d);
    return d < -103.2789306640625f ? 0.f : w;   // (the logarithm of the smallest float)
}
// Running sum over the wave's lanes, up to and with the own one, without LDS.
template <int CTRL, int ROWS> __device__ inline double dpp_or_zero(double v) {
    const unsigned long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo));
}
__device__ inline double wave_scan_d(double v) {
    v += dpp_or_zero<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8: within rows of 16 lanes
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v);   // row_bcast 15 into rows 1 and 3, 31 into rows 2 and 3
    v += dpp_or_zero<0x143, 0xc>(v);
    return v;
}
__device__ inline double readlane_d(double v, int lane) {
    const unsigned long long b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, lane), hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// A scaled logit, rounded: not to be contracted with what is subtracted from it, so that all ways to a weight round alike.
__device__ inline float scale_logit(float raw, float inv_t) {
#pragma clang fp contract(off)
    return raw * inv_t;
}
// The same with the EOS id's bias, rounded once.
__device__ inline float scale_logit(float raw, int idx, float inv_t, int eos_id, float eos_bias) {
    return idx == eos_id ? fmaf(raw, inv_t, eos_bias) : scale_logit(raw, inv_t);
}

// The kept set of a nucleus: logit key above kstar, or equal to it with an id up to tie_limit.
struct Nucleus {
    bool on;
    uint32_t kstar;
    int tie_limit;
    float eos_key_add;   // the EOS bias in logit units (bias * temperature): the key of the EOS id is logit + this
};
__device__ inline uint32_t logit_key(float raw, int idx, int eos_id, float eos_key_add) {
    return okey(idx == eos_id ? raw + eos_key_add : raw);
}

template <int VEC> __device__ inline void load_vec(const float *__restrict__ x, float (&v)[VEC]) {
    if (VEC == 4) {
        const float4 t = *(const float4 *)x;
        v[0] = t.x; v[1 % VEC] = t.y; v[2 % VEC] = t.z; v[3 % VEC] = t.w;
    } else {
        v[0] = *x;
    }
}

// The logits of VEC tokens from idx on; those from `end` on are not there (ok false, 0).
template <int VEC> __device__ inline void load_raw(const float *__restrict__ x, int idx, int end, float (&v)[VEC], bool (&ok)[VEC]) {
    if (VEC == 4 && idx + 3 < end) {
        load_vec<VEC>(x + idx, v);
#pragma unroll
        for (int c = 0; c < VEC; ++c) ok[c] = true;
    } else {
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            ok[c] = (idx + c) < end;
            v[c] = ok[c] ? x[idx + c] : 0.f;
        }
    }
}
template <int VEC>
__device__ inline void load_scaled(const float *__restrict__ x, int idx, int end, float inv_t, int eos_id,
                                   float eos_bias, float (&v)[VEC], bool (&ok)[VEC], const Nucleus &nu) {
    load_raw<VEC>(x, idx, end, v, ok);
    if (nu.on) {
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            const uint32_t key = logit_key(v[c], idx + c, eos_id, nu.eos_key_add);
            ok[c] = ok[c] && (key > nu.kstar || (key == nu.kstar && idx + c <= nu.tie_limit));
        }
    }
#pragma unroll
    for (int c = 0; c < VEC; ++c) v[c] = scale_logit(v[c], idx + c, inv_t, eos_id, eos_bias);
}

__device__ inline int round_up(int a, int b) { return (a + b - 1) / b * b; }

// The fold of one lane: m the maximum, ref the same, or 0 while all tokens so far are masked (no weight); s the sum of
// weights relative to ref.  A masked token counts as minus infinity.
struct Fold {
    float m = -INFINITY, ref = 0.f;
    double s = 0.0;
    // KEPT_ONLY: tokens for which ok is false count as masked, all others are within 100 of the row's maximum (the kept tokens of a
    // nucleus: no weight underflows)
    template <int VEC, bool KEPT_ONLY = false> __device__ void take(const float (&v)[VEC], const bool *ok = nullptr) {
        float lm = m;
#pragma unroll
        for (int c = 0; c < VEC; ++c) lm = fmaxf(lm, !KEPT_ONLY || ok[c] ? v[c] : -INFINITY);
        const float next = lm == -INFINITY ? 0.f : lm;
        // (no branch: some lane of the wave has a new maximum nearly always.  Without one the factor is 1, and so it is while s is 0 and
        // ref no maximum yet, which may lie above the first)
        s *= (double)exp_weight(fminf(ref - next, 0.f));
        m = lm;
        ref = next;
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            // (of masked tokens too: a branch around each would be a chain of its own)
            const float w = KEPT_ONLY ? exp_weight_near(v[c] - ref) : exp_weight(v[c] - ref);
            s += (double)(!KEPT_ONLY || ok[c] ? w : 0.f);
        }
    }
};

// ---- the binned way to the nucleus
static constexpr int NUC_BINS = 4096;          // four per thread
static constexpr float NUC_PER_UNIT = 32.0f;   // bins per unit of scaled logit
static constexpr int NUC_LIST = 5120;          // tokens of the crossing bin that fit the list (with the bins 72 KB, 78.6 of the kernel's all: two blocks
                                               // fit the 160 KB of a CU)
static constexpr int NUC_COUNT_SHIFT = 44;     // a bin: count above, sum of weights as integers below (2^18 tokens fit either)
static constexpr int NUC_GRANULE = 256;        // tokens of a wave's segment whose maximum is kept, so that later passes skip them
static constexpr int NUC_GRANULES = 64;        // per wave
static constexpr int NUC_MAX_VOCAB = SAMPLE_WAVES * NUC_GRANULES * NUC_GRANULE;   // 2^18

struct NucleusBins {
    union {
        struct {
            unsigned long long bin[NUC_BINS];
            uint2 list[NUC_LIST];                      // key, id
        };
        struct {
            double hist[SAMPLE_WAVES][256];
            int cnt[SAMPLE_WAVES][256];
            double comb[256];
            int ccnt[256];
        } radix;
    };
    double wave_sum[SAMPLE_WAVES];
    uint32_t wave_lo[SAMPLE_WAVES], wave_hi[SAMPLE_WAVES];
    double above;
    unsigned long long sel_bin;
    int sel, n;
    uint32_t seen;                                     // key of the largest scaled logit that any wave has seen
    uint32_t opening;                                  // the same of the first strides only: not written to while the waves read it
    float granule_max[SAMPLE_WAVES][NUC_GRANULES];     // largest scaled logit
};

// From the bins (each thread owns four, in order of falling logit): the first one at which above + the running mass reaches
// `want` (NUC_BINS if none does) into sb.sel, its word into sb.sel_bin and the mass in front of it into sb.above.  place_of(i) is the
// place of bin i in that order, scale(i) turns its integer sum into mass and falls by the factor `ratio` from one bin to the next.  Every
// thread must call it; nobody reads the bins behind its last barrier, they may be cleared there.
template <typename At, typename Scale>
__device__ inline void nucleus_cross(NucleusBins &sb, double above, double want, double ratio, At place_of, Scale scale) {
    const int tid = threadIdx.x, lane = tid % WAVE, wave = tid / WAVE;
    double m[4], own = 0.0, unit = scale(4 * tid);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned long long b = sb.bin[place_of(4 * tid + i)];
        m[i] = (b >> NUC_COUNT_SHIFT) ? (double)(b & ((1ull << NUC_COUNT_SHIFT) - 1)) * unit : 0.0;
        own += m[i];
        unit *= ratio;
    }
    const double incl = wave_scan_d(own);
    if (tid == 0) sb.sel = NUC_BINS;
    if (lane == WAVE - 1) sb.wave_sum[wave] = incl;
    __syncthreads();
    const double front = wave_scan_d(lane < wave ? sb.wave_sum[lane % SAMPLE_WAVES] : 0.0);   // (lane 63: of all waves in front)
    double run = above + readlane_d(front, WAVE - 1) + (incl - own);
    int mine = -1;
    double at = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (mine < 0 && m[i] > 0.0 && run + m[i] >= want) {
            mine = 4 * tid + i;
            at = run;
        }
        run += m[i];
    }
    if (mine >= 0) atomicMin(&sb.sel, mine);
    __syncthreads();
    if (mine >= 0 && mine == sb.sel) {
        sb.above = at;
        sb.sel_bin = sb.bin[place_of(mine)];
    }
    __syncthreads();
}

// How many of the c tied tokens at the cut it takes, whose masses sum to `comb` and in front of which lies `run`; -1: all.
__device__ inline int ties_to_keep(double want, double run, double comb, int c) {
    const double wt = comb / (double)c;
    int r = (int)ceil((want - run) / wt);
    r = max(1, min(r, c));
    while (r > 1 && run + (double)(r - 1) * wt >= want) --r;
    while (r < c && run + (double)r * wt < want) ++r;
    return r >= c ? -1 : r;
}

// The place of a token among the bins: its logit in bins, rounded to a whole number n by one fma, as PLACE_BASE + n (exact while
// |n| < 2^22), so that the low bits of the word are n modulo NUC_BINS.  The bins lie in a ring: they can be filled before the
// row's maximum is known.  (The EOS id's bias counts like in its key, so tokens with the same key have the same place.)
static constexpr float PLACE_BASE = 12582912.0f;   // 1.5 * 2^23
__device__ inline float place(float key_logit, float per_logit) { return fmaf(key_logit, per_logit, PLACE_BASE); }
struct NucleusFile {
    uint32_t at;
    unsigned int mass;   // relative to the bin's middle, times 2^25
    __device__ NucleusFile(float key_logit, float per_logit) {
        const float p = place(key_logit, per_logit);
        const float off = fmaf(key_logit, per_logit, -(p - PLACE_BASE));   // at most 1/2
        mass = (unsigned int)__builtin_amdgcn_exp2f(fmaf(off, 1.4426950408889634f / NUC_PER_UNIT, 25.0f));
        at = __float_as_uint(p) & (NUC_BINS - 1);
    }
    __device__ void add(NucleusBins &sb) const { atomicAdd(&sb.bin[at], (1ull << NUC_COUNT_SHIFT) + mass); }
};

// The granules in `mask`, four strides of a wave's segment [b, e) at a time: the lane's first token in each (at), whether it is
// in the segment (in), its raw logits.  Strides are as load_scaled's: the lane owns VEC consecutive tokens of WAVE * VEC.
// Returns whether the four strides are plain: all of them in the segment, none with the EOS id (wave-uniform).
template <int VEC>
__device__ inline bool next_granules(unsigned long long &mask, const float *__restrict__ x, int b, int e, int eos_id, int lane,
                                     int (&at)[4], bool (&in)[4], float (&raw)[4][VEC]) {
    bool plain = true;
#pragma unroll
    for (int u = 0; u < 4; ++u) {   // (VEC 4: a stride is a granule; else four are)
        const int first = mask ? b + __builtin_ctzll(mask) * NUC_GRANULE + (VEC == 4 ? 0 : u * WAVE) : e;
        if (VEC == 4 || u == 3) mask &= mask - 1;   // (0 stays 0)
        plain = plain && first + WAVE * VEC <= e && !(eos_id >= first && eos_id < first + WAVE * VEC);
        at[u] = first + lane * VEC;
        // (clamped, not left out: a branch around each load would make them wait for one another)
        in[u] = at[u] < e;          // (with VEC = 4 segments end on multiples of four)
        load_vec<VEC>(x + min(at[u], e - VEC), raw[u]);
    }
    return plain;
}

// The cut at mass `want` = top_p Z of a row with maximum M and sum Z: kstar and the number of its ties to keep (-1: all), and
// which granules of the wave's segment [b, e) have a token that may be kept.  The bins hold the tokens within `reach` of M, some of those
// further down, and none at or below `filed`, so that their ring has not gone round if M is not too far above that (else see below).
// False: not found this way, nothing is left behind (the caller's arithmetic decides either way, see the end of pass 2).
template <int VEC>
__device__ inline bool nucleus_binned(const float *__restrict__ x, int vocab, int b, int e, float inv_t, float top_p, int eos_id,
                                      float eos_bias, float eos_key_add, float M, double Z, double want, float filed, float reach,
                                      NucleusBins &sb, uint32_t &kstar, int &keep_ties, unsigned long long &granules) {
    constexpr int BLOCK = SAMPLE_WAVES * WAVE;
    const int tid = threadIdx.x, lane = tid % WAVE, wave = tid / WAVE;
    // (beyond these sizes places are no longer exact, or an EOS logit and its bias may cancel)
    if (vocab > NUC_MAX_VOCAB || !(fabsf(M) < 1e5f) || !(Z >= 0.5 && Z < 1e9)) return false;
    if (eos_id >= 0 && !(fabsf(eos_bias) < 1e5f) && eos_bias != -INFINITY) return false;
    const float per_logit = NUC_PER_UNIT * inv_t;
    auto scaled = [&](float raw, int idx) { return scale_logit(raw, idx, inv_t, eos_id, eos_bias); };
    const int top = (int)rintf(M * NUC_PER_UNIT) + 2;   // no place is above it, whatever the rounding of the scaled maximum
    const int n_granules = (e - b + NUC_GRANULE - 1) / NUC_GRANULE;   // (b <= e)
    auto with_place = [&](float n) {   // granules with a token at place n or above (places and maxima differ by rounding only)
        return __ballot(lane < n_granules && sb.granule_max[wave][lane % NUC_GRANULES] * NUC_PER_UNIT >= n - 2.f);
    };
    // The bins were filled while the maximum was found.  Did their ring go round (block-uniform; a maximum 100 units of scaled
    // logit above all that was seen of the row at first)?  Then once more, from what is within reach of it.
    if (!((M - filed) * NUC_PER_UNIT < (float)(NUC_BINS - 16))) {
#pragma unroll
        for (int i = 0; i < NUC_BINS / BLOCK; ++i) sb.bin[tid + i * BLOCK] = 0ull;
        __syncthreads();
        const float from = M - reach;   // (reach is at most 32)
        for (unsigned long long mask = with_place(from * NUC_PER_UNIT); mask;) {
            int at[4];
            bool in[4];
            float raw[4][VEC];
            (void)next_granules<VEC>(mask, x, b, e, eos_id, lane, at, in, raw);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = 0; c < VEC; ++c)
                    if (in[u] && scaled(raw[u][c], at[u] + c) > from)
                        NucleusFile(at[u] + c == eos_id ? raw[u][c] + eos_key_add : raw[u][c], per_logit).add(sb);
        }
        __syncthreads();
    }
    if (tid == 0) sb.n = 0;
    // ---- pass 1 is done: which bin the cut is in
    nucleus_cross(sb, 0.0, want, 0.96923323447634408185 /* exp(-1/32) */, [&](int i) { return (top - i) & (NUC_BINS - 1); },
                  [&](int i) { return (1.0 / 33554432.0) * exp((double)(top - i) / (double)NUC_PER_UNIT - (double)M); });
    const int sel = sb.sel;
    if (sel == NUC_BINS || (int)(sb.sel_bin >> NUC_COUNT_SHIFT) > NUC_LIST) return false;
    // ---- pass 2: the mass in front of that bin, its tokens into the list
    const float place_sel = PLACE_BASE + (float)(top - sel);
    granules = with_place((float)(top - sel));
    double s = 0.0;
    for (unsigned long long mask = granules; mask;) {
        int at[4];
        bool in[4];
        float raw[4][VEC];
        const bool plain = next_granules<VEC>(mask, x, b, e, eos_id, lane, at, in, raw);
        uint32_t hits = 0u;   // the lane's tokens in the bin
        auto weigh = [&](auto is_plain) {
            constexpr bool PLAIN = decltype(is_plain)::value;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
#pragma unroll
                for (int c = 0; c < VEC; ++c) {
                    const float v = PLAIN ? scale_logit(raw[u][c], inv_t) : scaled(raw[u][c], at[u] + c);
                    float key = raw[u][c];
                    if (!PLAIN && at[u] + c == eos_id) key += eos_key_add;
                    if (!PLAIN && !in[u]) key = -INFINITY;
                    const float p = place(key, per_logit);
                    hits |= p == place_sel ? 1u << (4 * u + c) : 0u;
                    // (every token's weight, and none in place of those behind: a branch around each would be a chain of its own)
                    const float w = exp_weight_near(v - M);
                    s += (double)(p > place_sel ? w : 0.f);
                }
                __builtin_amdgcn_sched_barrier(0);   // (a stride at a time: all of them at once do not fit the registers)
            }
        };
        if (plain) weigh(std::true_type{});
        else weigh(std::false_type{});
        if (hits) {
            for (int k = atomicAdd(&sb.n, __popc(hits)); hits; ++k, hits &= hits - 1) {
                const int u = __builtin_ctz(hits) / 4, c = __builtin_ctz(hits) % 4;
                if (k < NUC_LIST) sb.list[k].y = (uint32_t)((u == 0 ? at[0] : (u == 1 ? at[1] : (u == 2 ? at[2] : at[3]))) + c);
            }
        }
    }
    s = wave_sum_d(s);
    if (lane == 0) sb.wave_sum[wave] = s;
    // Behind this barrier every wave has filed its tokens.
    __syncthreads();
    const int n_list = sb.n;
    if (n_list > NUC_LIST || n_list == 0) return false;
    uint32_t lo = 0xffffffffu, hi = 0u;
    for (int k = tid; k < n_list; k += BLOCK) {   // (a thread's own entries, from here on)
        const int id = (int)sb.list[k].y;
        const uint32_t key = logit_key(x[id], id, eos_id, eos_key_add);
        sb.list[k].x = key;
        lo = min(lo, key);
        hi = max(hi, key);
    }
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, WAVE));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, WAVE));
    }
    if (lane == 0) {
        sb.wave_lo[wave] = lo;
        sb.wave_hi[wave] = hi;
    }
    __syncthreads();
    double above = 0.0;
    lo = 0xffffffffu;
    hi = 0u;
#pragma unroll 4
    for (int w = 0; w < SAMPLE_WAVES; ++w) {
        lo = min(lo, sb.wave_lo[w]);
        hi = max(hi, sb.wave_hi[w]);
        above += sb.wave_sum[w];
    }
    // From here on the weights are the ones that every other way to the cut takes, expf(v - M), and their sums are exact: the
    // list's, all within 2 % of the bin's middle, as integers of at most 2^28.  The cut is the list's if it is reached within it.
    if (!(above < want)) return false;
    const float unit = ldexpf(1.0f, 26 - ilogbf(expf((float)(top - sel) * (1.0f / NUC_PER_UNIT) - M)));
    auto weight = [&](uint32_t key, int id) {
        const float raw = id == eos_id ? x[id] : key_logit(key);
        return (unsigned int)(expf(scaled(raw, id) - M) * unit);
    };
    // ---- the list's cut: 4096 parts of its key range, then of that part's, until a part is one key
    for (;;) {
        const int shift = max(0, 32 - 12 - (hi > lo ? __clz((int)(hi - lo)) : 32));
#pragma unroll
        for (int i = 0; i < NUC_BINS / BLOCK; ++i) sb.bin[tid + i * BLOCK] = 0ull;
        __syncthreads();
        for (int k = tid; k < n_list; k += BLOCK) {
            const uint2 t = sb.list[k];
            if (t.x >= lo && t.x <= hi)
                atomicAdd(&sb.bin[NUC_BINS - 1 - (int)((t.x - lo) >> shift)], (1ull << NUC_COUNT_SHIFT) + weight(t.x, (int)t.y));
        }
        __syncthreads();
        nucleus_cross(sb, above, want, 1.0, [](int i) { return i; }, [&](int) { return 1.0 / (double)unit; });
        const int part = sb.sel;
        if (part == NUC_BINS) return false;
        above = sb.above;
        lo += (uint32_t)(NUC_BINS - 1 - part) << shift;
        const unsigned long long bin = sb.sel_bin;
        if (shift > 0 && (bin >> NUC_COUNT_SHIFT) == 1ull) {   // (mostly) one token is left: it is the cut
            for (int k = tid; k < n_list; k += BLOCK) {
                const uint32_t key = sb.list[k].x;
                if (key >= lo && key - lo < (1u << shift) && key <= hi) sb.seen = key;
            }
            __syncthreads();
            kstar = sb.seen;
            keep_ties = -1;
            return true;
        }
        if (shift == 0) {
            kstar = lo;
            keep_ties = ties_to_keep(want, above, (double)(bin & ((1ull << NUC_COUNT_SHIFT) - 1)) / (double)unit,
                                     (int)(bin >> NUC_COUNT_SHIFT));
            return true;
        }
        hi = min(hi, lo + ((1u << shift) - 1u));
    }
}

// ROOMY: a launch of at most half a block per CU keeps the segment sums in registers; larger ones read them from LDS four at a time and
// fit two blocks per CU (with the longer passes of before, back to back: 107 rows 17.7 us, 19.3 without; 256 rows 34 us against 43 us, 1024
// rows 149 against 178).
template <int VEC, bool TOPP, bool ROOMY>
__global__ __launch_bounds__(SAMPLE_WAVES *WAVE, ROOMY ? 4 : 8) void sample_kernel(
    const float *__restrict__ logits, const int32_t *__restrict__ logit_row, int vocab, float inv_t, float top_p,
    float eos_key_add, uint64_t seed,
    const uint64_t *__restrict__ seq_uid, const int32_t *__restrict__ step, int step_base, int eos_id, float eos_bias,
    int32_t *__restrict__ tokens_out, float *__restrict__ logprob_out, uint8_t *__restrict__ finished,
    int32_t *__restrict__ hist_tokens, float *__restrict__ hist_logprob, const int32_t *__restrict__ hist_index) {
    __shared__ float s_wm[SAMPLE_WAVES];
    __shared__ double s_ws[SAMPLE_WAVES];
    __shared__ double s_sub[SAMPLE_WAVES], s_seg[SAMPLE_WAVES];
    __shared__ float s_u;
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid % WAVE, wave = tid / WAVE;
    if (finished && finished[row]) {   // block-uniform
        if (tid == 0) {
            tokens_out[row] = eos_id;
            if (logprob_out) logprob_out[row] = 0.f;
            const int hi = hist_index ? hist_index[row] : row;
            if (hist_tokens) hist_tokens[hi] = eos_id;
            if (hist_logprob) hist_logprob[hi] = 0.f;
        }
        return;
    }
    const float *x = logits + (int64_t)(logit_row ? logit_row[row] : row) * vocab;
    if (tid == 0) {
        const uint64_t uid = seq_uid[row];
        const uint32_t st = (uint32_t)(step_base + (step ? step[row] : 0));
        uint32_t r[4];
        philox4x32_10(st, (uint32_t)uid, (uint32_t)(uid >> 32), 0u, (uint32_t)seed, (uint32_t)(seed >> 32), r);
        s_u = ((float)(r[0] >> 9) + 0.5f) * (1.0f / 8388608.0f);   // exact in fp32, inside (0,1)
    }
    constexpr int STRIDE = WAVE * VEC, SEG_UNROLL = ROOMY ? SAMPLE_WAVES : 4;
    Nucleus nu{false, 0u, 0x7fffffff, eos_key_add};
    // ---- level 1: online (max, sum) per contiguous wave segment
    const int seg = round_up((vocab + SAMPLE_WAVES - 1) / SAMPLE_WAVES, STRIDE);
    const int wb = min(vocab, wave * seg), we = min(vocab, wb + seg);
    auto finish = [&](const Fold &f) {
        const float wm = wave_max_f32(f.m);
        const double ws = wave_sum_d(f.m == -INFINITY ? 0.0 : f.s * (double)expf(f.m - wm));
        if (lane == 0) {
            s_wm[wave] = wm;
            s_ws[wave] = ws;
        }
    };
    // four strides are fetched before the first is folded in (the fold is a serial chain, and a load
    // per link would leave the memory latency exposed at every step); the order of the arithmetic is
    // that of the plain loop
    constexpr int AHEAD = 4;
    auto level1 = [&]() {
        Fold f;
        for (int base = wb; base < we; base += AHEAD * STRIDE) {
            float v[AHEAD][VEC];
            bool ok[AHEAD][VEC];
            if (!nu.on && base + AHEAD * STRIDE <= we && !(eos_id >= base && eos_id < base + AHEAD * STRIDE)) {   // (wave-uniform)
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) load_vec<VEC>(x + base + u * STRIDE + lane * VEC, v[u]);
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
#pragma unroll
                    for (int c = 0; c < VEC; ++c) v[u][c] = scale_logit(v[u][c], inv_t);
                    f.take(v[u]);
                }
            } else {
#pragma unroll
                for (int u = 0; u < AHEAD; ++u)
                    load_scaled<VEC>(x, base + u * STRIDE + lane * VEC, we, inv_t, eos_id, eos_bias, v[u], ok[u], nu);
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
#pragma unroll
                    for (int c = 0; c < VEC; ++c) v[u][c] = ok[u][c] ? v[u][c] : -INFINITY;
                    f.take(v[u]);
                }
            }
        }
        finish(f);
    };
    if constexpr (!TOPP) level1();
    if constexpr (TOPP) {
        __shared__ NucleusBins sb;
        // ---- nucleus: the key kstar and the id limit among its ties at which the mass from the top reaches top_p Z
        __shared__ uint32_t s_prefix;
        __shared__ double s_above;
        __shared__ int s_keep_ties, s_tie_limit, s_wcount[SAMPLE_WAVES];
        // Level 1, and in the same pass the bins: tokens of a weight below half of (1 - top_p) Z / vocab lie behind the cut, all of
        // them together, and need no bin.  Z is at least the largest weight, and the largest logit at least the largest
        // seen so far, by any wave: the first stride of every segment is looked at ahead, the rest is published as it comes.
        const float reach = 1.0f - logf(0.5f * (1.0f - top_p) / (float)vocab);
        // No token whose scaled logit is at or below this is in a bin.  Those above it are if they were within reach of the largest logit
        // seen when their turn came; the others lie behind the cut.
        float filed = -INFINITY;
        {
            constexpr int BLOCK = SAMPLE_WAVES * WAVE;
            const float per_logit = NUC_PER_UNIT * inv_t;
#pragma unroll
            for (int i = 0; i < NUC_BINS / BLOCK; ++i) sb.bin[tid + i * BLOCK] = 0ull;
            if (tid == 0) sb.seen = sb.opening = okey(-INFINITY);
            __syncthreads();
            {
                float v[VEC], lm = -INFINITY;
                bool ok[VEC];
                load_scaled<VEC>(x, wb + lane * VEC, we, inv_t, eos_id, eos_bias, v, ok, nu);
#pragma unroll
                for (int c = 0; c < VEC; ++c)
                    if (ok[c]) lm = fmaxf(lm, v[c]);
                lm = wave_max_all(lm);
                if (lane == 0) atomicMax(&sb.opening, okey(lm));
            }
            __syncthreads();
            // (all waves have to agree on `filed`, which decides whether the bins are filled again; no barrier keeps a fast wave from
            // publishing what it sees next before a slow one is here, so that goes to another word)
            float seen = key_logit(sb.opening);
            filed = seen - reach;
            // Rows that nucleus_binned refuses whatever the bins hold: too long, or a maximum beyond 1e5 at the first look (block-uniform).
            // (1024 x 151936 beyond 1e5: 3803 us with the bins filled, 3720 without; 256 rows of 300000 tokens 770, 727)
            if (vocab > NUC_MAX_VOCAB || !(seen < 1e5f)) {
                level1();
            } else {
                Fold f;
                auto chunk = [&](auto plain, int base) {   // plain: whole strides without the EOS id
                    constexpr bool PLAIN = decltype(plain)::value;
                    float raw[AHEAD][VEC], v[AHEAD][VEC];
                    const uint32_t others = __hip_atomic_load(&sb.seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) {
                        const int idx = base + u * STRIDE + lane * VEC;
                        if (PLAIN) load_vec<VEC>(x + idx, raw[u]);
                        else {
#pragma unroll
                            for (int c = 0; c < VEC; ++c) raw[u][c] = idx + c < we ? x[idx + c] : 0.f;
                        }
                    }
                    float top[AHEAD];
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) {
                        const int idx = base + u * STRIDE + lane * VEC;
                        top[u] = -INFINITY;
#pragma unroll
                        for (int c = 0; c < VEC; ++c) {
                            v[u][c] = PLAIN ? scale_logit(raw[u][c], inv_t) : scale_logit(raw[u][c], idx + c, inv_t, eos_id, eos_bias);
                            if (!PLAIN && idx + c == eos_id) raw[u][c] += eos_key_add;   // (from here on: the key's logit)
                            if (!PLAIN && idx + c >= we) v[u][c] = -INFINITY;
                            top[u] = fmaxf(top[u], v[u][c]);
                        }
                    }
                    const float before = seen;
                    const int granule = (base - wb) / NUC_GRANULE;   // (beyond the last one only where the bins are not used)
                    if (VEC == 4) {
#pragma unroll
                        for (int u = 0; u < AHEAD; ++u) {
                            top[u] = wave_max_all(top[u]);
                            seen = fmaxf(seen, top[u]);
                            if (lane == 0 && granule + u < NUC_GRANULES) sb.granule_max[wave][granule + u] = top[u];
                        }
                    } else {
                        const float t = wave_max_all(fmaxf(fmaxf(top[0], top[1]), fmaxf(top[2], top[3])));
                        seen = fmaxf(seen, t);
                        if (lane == 0 && granule < NUC_GRANULES) sb.granule_max[wave][granule] = t;
                    }
                    if (lane == 0 && seen > before) atomicMax(&sb.seen, okey(seen));
                    seen = fmaxf(seen, key_logit(others));
                    const float from = seen - reach;
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) {
                        f.take(v[u]);
                        if (VEC > 1 && !(top[u] > from)) continue;   // (wave-uniform)
#pragma unroll
                        for (int c = 0; c < VEC; ++c) {
                            const NucleusFile t(raw[u][c], per_logit);
                            if (v[u][c] > from) t.add(sb);
                        }
                    }
                };
                for (int base = wb; base < we; base += AHEAD * STRIDE) {
                    if (base + AHEAD * STRIDE <= we && !(eos_id >= base && eos_id < base + AHEAD * STRIDE))
                        chunk(std::true_type{}, base);
                    else
                        chunk(std::false_type{}, base);
                }
                finish(f);
            }
        }
        __syncthreads();
        float M0 = -INFINITY;
#pragma unroll
        for (int w = 0; w < SAMPLE_WAVES; ++w) M0 = fmaxf(M0, s_wm[w]);
        double Z0 = 0.0;
#pragma unroll 4
        for (int w = 0; w < SAMPLE_WAVES; ++w) Z0 += (s_wm[w] == -INFINITY) ? 0.0 : s_ws[w] * (double)expf(s_wm[w] - M0);
        const double want = (double)top_p * Z0;
        int keep_ties;
        unsigned long long granules = 0ull;   // of the wave's segment, those with a token that may be kept
        const bool binned = nucleus_binned<VEC>(x, vocab, wb, we, inv_t, top_p, eos_id, eos_bias, eos_key_add, M0, Z0, want, filed,
                                                reach, sb, nu.kstar, keep_ties, granules);
        if (!binned) {
        auto &s_hist = sb.radix.hist;
        auto &s_cnt = sb.radix.cnt;
        auto &s_comb = sb.radix.comb;
        auto &s_ccnt = sb.radix.ccnt;
        __syncthreads();
        if (tid == 0) {
            s_prefix = 0u;
            s_above = 0.0;
        }
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            for (int bkt = lane; bkt < 256; bkt += WAVE) {
                s_hist[wave][bkt] = 0.0;
                s_cnt[wave][bkt] = 0;
            }
            __syncthreads();
            const uint32_t prefix = s_prefix;
            for (int base = tid * VEC; base < vocab; base += SAMPLE_WAVES * WAVE * VEC) {
                float v[VEC];
                bool ok[VEC];
                float raw[VEC];
#pragma unroll
                for (int c = 0; c < VEC; ++c) raw[c] = (base + c < vocab) ? x[base + c] : 0.f;
                load_scaled<VEC>(x, base, vocab, inv_t, eos_id, eos_bias, v, ok, nu);
#pragma unroll
                for (int c = 0; c < VEC; ++c) {
                    if (!ok[c]) continue;
                    const uint32_t key = logit_key(raw[c], base + c, eos_id, eos_key_add);
                    if (pass > 0 && (key >> (shift + 8)) != prefix) continue;
                    const int bkt = (key >> shift) & 255;
                    atomicAdd(&s_hist[wave][bkt], (double)expf(v[c] - M0));
                    atomicAdd(&s_cnt[wave][bkt], 1);
                }
            }
            __syncthreads();
            if (tid < 256) {   // the waves' histograms in wave order
                double h = 0.0;
                int cn = 0;
#pragma unroll
                for (int w = 0; w < SAMPLE_WAVES; ++w) {
                    h += s_hist[w][tid];
                    cn += s_cnt[w][tid];
                }
                s_comb[tid] = h;
                s_ccnt[tid] = cn;
            }
            __syncthreads();
            if (tid == 0) {   // from the top bucket down: where the cumulative mass reaches the wanted one
                double run = s_above;
                int sel = -1, lowest = 0;
                for (int bkt = 255; bkt >= 0; --bkt) {
                    if (s_ccnt[bkt] == 0) continue;
                    lowest = bkt;
                    if (run + s_comb[bkt] >= want) {
                        sel = bkt;
                        break;
                    }
                    run += s_comb[bkt];
                }
                if (sel < 0) {   // rounding left the total short of top_p Z: every token stays
                    sel = lowest;
                    run -= s_comb[lowest];
                }
                s_above = run;
                s_prefix = (prefix << 8) | (uint32_t)sel;
                if (pass == 3) {   // ties at the cut: as many as it takes, lowest ids first
                    s_keep_ties = ties_to_keep(want, run, s_comb[sel], s_ccnt[sel]);
                }
            }
            __syncthreads();
        }
        nu.kstar = s_prefix;
        keep_ties = s_keep_ties;
        }
        nu.tie_limit = 0x7fffffff;
        if (keep_ties > 0) {   // (block-uniform, rare) only the first keep_ties of the tied ids stay: find the id of the last one
            int seen = 0;      // ties in the ids before this chunk (same value in every thread)
            int limit = -1;
            for (int base = 0; base < vocab && limit < 0; base += SAMPLE_WAVES * WAVE) {
                const int idx = base + tid;
                const bool tie = idx < vocab && logit_key(x[idx], idx, eos_id, eos_key_add) == nu.kstar;
                const unsigned long long bal = __ballot(tie);
                if (lane == 0) s_wcount[wave] = __popcll(bal);
                __syncthreads();
                int before = 0, total = 0;
#pragma unroll
                for (int w = 0; w < SAMPLE_WAVES; ++w) {
                    if (w < wave) before += s_wcount[w];
                    total += s_wcount[w];
                }
                if (seen + total >= keep_ties) {   // the last kept tie is in this chunk
                    const int rank = seen + before + __popcll(bal & ((1ull << lane) - 1ull));   // ties before this id
                    if (tie && rank == keep_ties - 1) s_tie_limit = idx;
                    limit = 0;
                }
                seen += total;
                __syncthreads();
            }
            nu.tie_limit = s_tie_limit;
        }
        nu.on = true;
        __syncthreads();
        // the same pass over the kept tokens only
        if (!binned) {
            level1();
        } else {   // by the granules that have any: what is left out would add nothing, so the sums are level1's, to the last bit
            Fold f;
            const float cut = key_logit(nu.kstar);
            const bool by_value = nu.tie_limit == 0x7fffffff && cut != 0.f;   // (the keys tell the zeros apart)
            while (granules) {
                int at[AHEAD];
                bool in[AHEAD];
                float v[AHEAD][VEC];
                const bool plain = next_granules<VEC>(granules, x, wb, we, eos_id, lane, at, in, v);
                if (plain && by_value) {
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) {
                        bool ok[VEC];
#pragma unroll
                        for (int c = 0; c < VEC; ++c) {
                            ok[c] = v[u][c] >= cut;
                            v[u][c] = scale_logit(v[u][c], inv_t);
                        }
                        f.take<VEC, true>(v[u], ok);
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) {
                        bool ok[VEC];
#pragma unroll
                        for (int c = 0; c < VEC; ++c) {
                            const int idx = at[u] + c;
                            const uint32_t key = logit_key(v[u][c], idx, eos_id, eos_key_add);
                            ok[c] = in[u] && (key > nu.kstar || (key == nu.kstar && idx <= nu.tie_limit));
                            v[u][c] = scale_logit(v[u][c], idx, inv_t, eos_id, eos_bias);
                        }
                        f.take<VEC, true>(v[u], ok);
                    }
                }
            }
            finish(f);
        }
    }
    __syncthreads();
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < SAMPLE_WAVES; ++w) M = fmaxf(M, s_wm[w]);
    if (tid < SAMPLE_WAVES) s_seg[tid] = (s_wm[tid] == -INFINITY) ? 0.0 : s_ws[tid] * (double)expf(s_wm[tid] - M);
    __syncthreads();
    double Z = 0.0;
#pragma unroll SEG_UNROLL
    for (int w = 0; w < SAMPLE_WAVES; ++w) Z += s_seg[w];
    const double target = (double)s_u * Z;
    int k = -1;
    double before = 0.0, run = 0.0;
#pragma unroll SEG_UNROLL
    for (int w = 0; w < SAMPLE_WAVES; ++w) {
        const double sw = s_seg[w];
        if (k < 0 && run + sw > target) {
            k = w;
            before = run;
        }
        run += sw;
    }
    if (k < 0) {   // rounding left no crossing: the last segment with weight
        run = 0.0;
#pragma unroll SEG_UNROLL
        for (int w = 0; w < SAMPLE_WAVES; ++w) {
            const double sw = s_seg[w];
            if (sw > 0.0) {
                k = w;
                before = run;
            }
            run += sw;
        }
        if (k < 0) k = 0;   // no weight anywhere (a row of minus infinities or NaNs): some token of the row
    }
    double rem = target - before;
    const int kb = min(vocab, k * seg), ke = min(vocab, kb + seg);
    // ---- level 2: 16 sub-segments of segment k
    const int sub = round_up((seg + SAMPLE_WAVES - 1) / SAMPLE_WAVES, STRIDE);
    {
        const int b = min(ke, kb + wave * sub), e = min(ke, b + sub);
        double s = 0.0;
        for (int base = b; base < e; base += STRIDE) {
            float v[VEC];
            bool ok[VEC];
            load_scaled<VEC>(x, base + lane * VEC, e, inv_t, eos_id, eos_bias, v, ok, nu);
#pragma unroll
            for (int c = 0; c < VEC; ++c)
                if (ok[c]) s += (double)expf(v[c] - M);
        }
        s = wave_sum_d(s);
        if (lane == 0) s_sub[wave] = s;
    }
    __syncthreads();
    if (wave != 0) return;
    int j = -1;
    before = 0.0;
    run = 0.0;
#pragma unroll SEG_UNROLL
    for (int w = 0; w < SAMPLE_WAVES; ++w) {
        const double sw = s_sub[w];
        if (j < 0 && run + sw > rem) {
            j = w;
            before = run;
        }
        run += sw;
    }
    if (j < 0) {
        run = 0.0;
#pragma unroll SEG_UNROLL
        for (int w = 0; w < SAMPLE_WAVES; ++w) {
            if (s_sub[w] > 0.0) {
                j = w;
                before = run;
            }
            run += s_sub[w];
        }
        if (j < 0) j = 0;
    }
    rem -= before;
    // ---- level 3: wave 0 scans sub-segment j in index order
    const int jb = min(ke, kb + j * sub), je = min(ke, jb + sub);
    double running = 0.0;
    int token = -1, last_pos = -1;
    float tok_x = 0.f;
    for (int base = jb; base < je && token < 0; base += STRIDE) {
        float v[VEC];
        bool ok[VEC];
        const int idx = base + lane * VEC;
        load_scaled<VEC>(x, idx, je, inv_t, eos_id, eos_bias, v, ok, nu);
        double pre[VEC], lsum = 0.0;
        int my_last = -1;
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            const double w = ok[c] ? (double)expf(v[c] - M) : 0.0;
            lsum += w;
            pre[c] = lsum;
            if (w > 0.0) my_last = idx + c;
        }
        double incl = lsum;
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            const double t = __shfl_up(incl, o, WAVE);
            if (lane >= o) incl += t;
        }
        const double excl = running + (incl - lsum);
        int cross = -1;
#pragma unroll
        for (int c = VEC - 1; c >= 0; --c)
            if (ok[c] && excl + pre[c] > rem) cross = c;
        const unsigned long long bal = __ballot(cross >= 0);
        if (bal) {
            const int src = __ffsll((long long)bal) - 1;
            const int t = __shfl(idx + (cross < 0 ? 0 : cross), src, WAVE);
            float xv = 0.f;
#pragma unroll
            for (int c = 0; c < VEC; ++c)
                if (c == cross) xv = v[c];
            tok_x = __shfl(xv, src, WAVE);
            token = t;
        }
        running += __shfl(incl, WAVE - 1, WAVE);
        // remember the last index that carried weight, for the no-crossing case
        int ml = my_last;
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) ml = max(ml, __shfl_xor(ml, o, WAVE));
        last_pos = max(last_pos, ml);
    }
    if (token < 0) {
        token = last_pos >= 0 ? last_pos : max(0, je - 1);
        tok_x = scale_logit(x[token], token, inv_t, eos_id, eos_bias);
    }
    if (lane == 0) {
        tokens_out[row] = token;
        const float lp = (float)((double)tok_x - (double)M - log(Z));
        if (logprob_out) logprob_out[row] = lp;
        if (finished && token == eos_id) finished[row] = 1;
        const int hi = hist_index ? hist_index[row] : row;
        if (hist_tokens) hist_tokens[hi] = token;
        if (hist_logprob) hist_logprob[hi] = lp;
    }
}

void launch_sample(const float *logits, const int32_t *logit_row, int n, int vocab, float temperature, float top_p,
                   uint64_t seed, const uint64_t *seq_uid, const int32_t *step, int step_base, int eos_id, float eos_bias,
                   int32_t *tokens_out, float *logprob_out, uint8_t *finished, int32_t *hist_tokens,
                   float *hist_logprob, const int32_t *hist_index, hipStream_t s) {
    if (n <= 0) return;
    const float inv_t = 1.0f / temperature;
    const bool vec = (vocab % 4 == 0) && (((uintptr_t)logits) % 16 == 0);
    const float key_add = (eos_id >= 0) ? eos_bias * temperature : 0.f;
    const bool roomy = n <= 128;   // one block per row, 256 CUs
#define PC_SAMPLE(V, TP, RM)                                                                                      \
    sample_kernel<V, TP, RM><<<n, SAMPLE_WAVES * WAVE, 0, s>>>(logits, logit_row, vocab, inv_t, top_p, key_add, seed, seq_uid, \
                                                           step, step_base, eos_id, eos_bias, tokens_out, logprob_out,      \
                                                           finished, hist_tokens, hist_logprob, hist_index)
    if (top_p < 1.0f) {
        if (vec) PC_SAMPLE(4, true, false);
        else PC_SAMPLE(1, true, false);
    } else {
        if (roomy) {
            if (vec) PC_SAMPLE(4, false, true);
            else PC_SAMPLE(1, false, true);
        } else {
            if (vec) PC_SAMPLE(4, false, false);
            else PC_SAMPLE(1, false, false);
        }
    }
#undef PC_SAMPLE
}

// log softmax(logits / T) at a given token per row (teacher-forced scoring: Section 3.1, the per-token
// factors of Eq. 2's ratio).  One block of 16 waves per row, the row is read once: online (max, sum) per
// thread, combined over the block; sums in double.  The target of row r is tokens[token_index[r] + 1]:
// the token that follows the position whose logits the row holds.
template <int VEC>
__global__ __launch_bounds__(SAMPLE_WAVES *WAVE) void logprob_kernel(const float *__restrict__ logits, int vocab,
                                                                      float inv_t,
                                                                      const int32_t *__restrict__ tokens,
                                                                      const int32_t *__restrict__ token_index,
                                                                      float *__restrict__ out) {
    __shared__ float s_wm[SAMPLE_WAVES];
    __shared__ double s_ws[SAMPLE_WAVES];
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid % WAVE, wave = tid / WAVE;
    const float *x = logits + (int64_t)row * vocab;
    float m = -INFINITY;
    double s = 0.0;
    for (int base = tid * VEC; base < vocab; base += SAMPLE_WAVES * WAVE * VEC) {
        float v[VEC];
        bool ok[VEC];
        load_raw<VEC>(x, base, vocab, v, ok);
#pragma unroll
        for (int c = 0; c < VEC; ++c) v[c] *= inv_t;
        float lm = -INFINITY;
#pragma unroll
        for (int c = 0; c < VEC; ++c)
            if (ok[c]) lm = fmaxf(lm, v[c]);
        if (lm > m) {
            s *= (double)expf(m - lm);
            m = lm;
        }
#pragma unroll
        for (int c = 0; c < VEC; ++c)
            if (ok[c]) s += (double)expf(v[c] - m);
    }
    const float wm = wave_max_f32(m);
    const double ws = wave_sum_d(m == -INFINITY ? 0.0 : s * (double)expf(m - wm));
    if (lane == 0) {
        s_wm[wave] = wm;
        s_ws[wave] = ws;
    }
    __syncthreads();
    if (tid == 0) {
        float M = -INFINITY;
        for (int w = 0; w < SAMPLE_WAVES; ++w) M = fmaxf(M, s_wm[w]);
        double Z = 0.0;
        for (int w = 0; w < SAMPLE_WAVES; ++w) Z += (s_wm[w] == -INFINITY) ? 0.0 : s_ws[w] * (double)expf(s_wm[w] - M);
        const int target = tokens[token_index[row] + 1];
        float lp = -INFINITY;
        if (target >= 0 && target < vocab) lp = (float)((double)(x[target] * inv_t) - (double)M - log(Z));
        out[row] = lp;
    }
}

void launch_logprob(const float *logits, int n, int vocab, float temperature, const int32_t *tokens,
                    const int32_t *token_index, float *out, hipStream_t s) {
    if (n <= 0) return;
    const float inv_t = 1.0f / temperature;
    const bool vec = (vocab % 4 == 0) && (((uintptr_t)logits) % 16 == 0);
    if (vec)
        logprob_kernel<4><<<n, SAMPLE_WAVES * WAVE, 0, s>>>(logits, vocab, inv_t, tokens, token_index, out);
    else
        logprob_kernel<1><<<n, SAMPLE_WAVES * WAVE, 0, s>>>(logits, vocab, inv_t, tokens, token_index, out);
}

// For tests: a[i] = exp_weight(d[i]), b[i] = expf(d[i])
__global__ void exp_weight_kernel(const float *__restrict__ d, float *__restrict__ a, float *__restrict__ b, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    a[i] = exp_weight(d[i]);
    b[i] = expf(d[i]);
}

}  // namespace pc

// For tests, not part of the C ABI.
extern "C" void pc_internal_exp_weight(const float *d, float *a, float *b, int n, void *stream) {
    if (n > 0) pc::exp_weight_kernel<<<(n + 255) / 256, 256, 0, (hipStream_t)stream>>>(d, a, b, n);
}
