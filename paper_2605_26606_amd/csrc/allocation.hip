// Pilot-Commit allocation on the device: per-prompt reward statistics (Eq. 3,
// Section 3.3 pilot success rate), the pilot filter with eviction flags and the
// stable compaction of the commit set (Section 3.3, Algorithm 1), and
// group-relative advantages (Section 3.1).  KBs of data: latency only.
#include "pc_internal.h"

namespace pc {

static constexpr int WAVE = 64;

// Sixteen lanes per group: a group's rewards arrive in one or two wide loads instead of a chain of single ones (three
// dependent passes over 32 rewards by one thread took longer than the launch), sums in double, lanes in a fixed order.
// 1024 groups of 32: statistics 7.6 -> 2.6 us, advantages 15.8 -> 2.7 us; 3 groups of 5000: 747 -> 98 and 1561 -> 118 us.
// The first GROUP_KEEP rewards of a lane stay in registers between the passes.
static constexpr int GROUP_LANES = 16, GROUP_KEEP = 4;

__device__ inline double group_sum(double v) {
#pragma unroll
    for (int o = GROUP_LANES / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, GROUP_LANES);
    return v;
}

struct GroupRewards {
    const float *r;
    int b, e, j;                       // the group's range, this lane
    float keep[GROUP_KEEP];
    __device__ GroupRewards(const float *rewards, const int32_t *off, int p, int lane) : r(rewards), b(off[p]), e(off[p + 1]), j(lane) {
#pragma unroll
        for (int k = 0; k < GROUP_KEEP; ++k) {
            const int i = b + j + GROUP_LANES * k;
            keep[k] = i < e ? r[i] : 0.f;
        }
    }
    template <typename F> __device__ void each(F f) const {   // f(index, reward) for this lane's rewards, ascending
#pragma unroll
        for (int k = 0; k < GROUP_KEEP; ++k) {
            const int i = b + j + GROUP_LANES * k;
            if (i < e) f(i, keep[k]);
        }
        for (int i = b + j + GROUP_LANES * GROUP_KEEP; i < e; i += GROUP_LANES) f(i, r[i]);
    }
    __device__ double mean() const {
        double s = 0.0;
        each([&](int, float v) { s += (double)v; });
        s = group_sum(s);
        return e > b ? s / (double)(e - b) : 0.0;
    }
    __device__ double variance(double mu) const {
        double s = 0.0;
        each([&](int, float v) {
            const double d = (double)v - mu;
            s += d * d;
        });
        s = group_sum(s);
        return e > b ? s / (double)(e - b) : 0.0;
    }
};

__global__ __launch_bounds__(256) void group_stats_kernel(const float *__restrict__ rewards, const int32_t *__restrict__ off, int P,
                                   int32_t *__restrict__ n_pos, int32_t *__restrict__ n_tot, float *__restrict__ mean,
                                   float *__restrict__ var) {
    const int lane = threadIdx.x % GROUP_LANES, p = blockIdx.x * (256 / GROUP_LANES) + threadIdx.x / GROUP_LANES;
    if (p >= P) return;                // whole groups of lanes leave together
    const GroupRewards g(rewards, off, p, lane);
    int pos = 0;
    g.each([&](int, float v) { pos += (v != 0.0f); });
#pragma unroll
    for (int o = GROUP_LANES / 2; o > 0; o >>= 1) pos += __shfl_xor(pos, o, GROUP_LANES);
    const double mu = g.mean(), v = g.variance(mu);
    if (lane == 0) {
        if (n_pos) n_pos[p] = pos;
        if (n_tot) n_tot[p] = g.e - g.b;
        if (mean) mean[p] = (float)mu;
        if (var) var[p] = (float)v;
    }
}

static unsigned group_blocks(int P) { return (unsigned)((P + 256 / GROUP_LANES - 1) / (256 / GROUP_LANES)); }

void launch_group_stats(const float *rewards, const int32_t *off, int P, int32_t *n_pos, int32_t *n_tot, float *mean,
                        float *var, hipStream_t s) {
    if (P <= 0) return;
    group_stats_kernel<<<group_blocks(P), 256, 0, s>>>(rewards, off, P, n_pos, n_tot, mean, var);
}

// One block walks the batch in chunks of 1024 prompts; the kept prompts are
// compacted in batch order (ballot ranks inside a wave, a 16-entry prefix
// across waves, a running count across chunks).
// VAR: the filter for rewards that are not binary: `p_hat` is the pilot mean, `var` the pilot variance, lo / hi are
// the variance thresholds on the approaching (mean <= pivot) and on the leaving side (mean > pivot).
template <bool VAR>
__global__ __launch_bounds__(1024) void select_commit_kernel(const float *__restrict__ p_hat,
                                                             const float *__restrict__ var, int P, float lo, float hi,
                                                             float pivot, float solve, int b_t, uint8_t *__restrict__ cls,
                                                             uint8_t *__restrict__ evict,
                                                             int32_t *__restrict__ commit_idx,
                                                             int32_t *__restrict__ surplus_idx,
                                                             int32_t *__restrict__ counts) {
    __shared__ int w_keep[16], w_easy[16], w_hard[16];
    const int tid = threadIdx.x, lane = tid % WAVE, wave = tid / WAVE;
    int kept_before = 0, n_easy = 0, n_hard = 0;
    for (int q0 = 0; q0 < P; q0 += 1024) {
        const int q = q0 + tid;
        int c = -1;
        if (q < P) {
            const float ph = p_hat[q];
            if (VAR) {
                const float vr = var[q];
                const bool approaching = ph <= pivot;
                const bool kept = approaching ? (vr >= lo) : (vr >= hi);
                c = kept ? 1 : (approaching ? 0 : 2);
            } else {
                c = (ph > hi) ? 2 : (ph < lo) ? 0 : 1;
            }
            if (cls) cls[q] = (uint8_t)c;
            if (evict) evict[q] = (ph >= solve) ? 1 : 0;
        }
        const unsigned long long bk = __ballot(c == 1), be = __ballot(c == 2), bh = __ballot(c == 0);
        if (lane == 0) {
            w_keep[wave] = __popcll(bk);
            w_easy[wave] = __popcll(be);
            w_hard[wave] = __popcll(bh);
        }
        __syncthreads();
        int wave_off = 0, chunk_keep = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) wave_off += w_keep[w];
            chunk_keep += w_keep[w];
            n_easy += w_easy[w];
            n_hard += w_hard[w];
        }
        if (c == 1) {
            const int rank = kept_before + wave_off + __popcll(bk & ((1ull << lane) - 1ull));
            if (b_t <= 0 || rank < b_t)
                commit_idx[rank] = q;
            else if (surplus_idx)
                surplus_idx[rank - b_t] = q;
        }
        kept_before += chunk_keep;
        __syncthreads();
    }
    if (tid == 0) {
        const int n_commit = (b_t <= 0) ? kept_before : min(kept_before, b_t);
        counts[0] = n_commit;
        counts[1] = kept_before - n_commit;
        counts[2] = n_easy;
        counts[3] = n_hard;
    }
}

void launch_select_commit(const float *p_hat, int P, float lo, float hi, float solve, int b_t, uint8_t *cls,
                          uint8_t *evict, int32_t *commit_idx, int32_t *surplus_idx, int32_t *counts, hipStream_t s) {
    select_commit_kernel<false><<<1, 1024, 0, s>>>(p_hat, nullptr, P, lo, hi, 0.f, solve, b_t, cls, evict, commit_idx,
                                                   surplus_idx, counts);
}

void launch_select_commit_var(const float *mean, const float *var, int P, float var_hard, float var_easy, float pivot,
                              float solve, int b_t, uint8_t *cls, uint8_t *evict, int32_t *commit_idx, int32_t *surplus_idx,
                              int32_t *counts, hipStream_t s) {
    select_commit_kernel<true><<<1, 1024, 0, s>>>(mean, var, P, var_hard, var_easy, pivot, solve, b_t, cls, evict,
                                                  commit_idx, surplus_idx, counts);
}

__global__ __launch_bounds__(256) void advantages_kernel(const float *__restrict__ rewards, const int32_t *__restrict__ off, int P, float eps,
                                  float *__restrict__ adv, float *__restrict__ mu_out, float *__restrict__ sigma_out) {
    const int lane = threadIdx.x % GROUP_LANES, p = blockIdx.x * (256 / GROUP_LANES) + threadIdx.x / GROUP_LANES;
    if (p >= P) return;
    const GroupRewards g(rewards, off, p, lane);
    const double mu = g.mean(), sigma = sqrt(g.variance(mu)), den = sigma + (double)eps;
    g.each([&](int i, float v) {
        const double d = (double)v - mu;
        adv[i] = (d == 0.0) ? 0.0f : (float)(d / den);
    });
    if (lane == 0) {
        if (mu_out) mu_out[p] = (float)mu;
        if (sigma_out) sigma_out[p] = (float)sigma;
    }
}

void launch_advantages(const float *rewards, const int32_t *off, int P, float eps, float *adv, float *mu, float *sigma,
                       hipStream_t s) {
    if (P <= 0) return;
    advantages_kernel<<<group_blocks(P), 256, 0, s>>>(rewards, off, P, eps, adv, mu, sigma);
}

}  // namespace pc
