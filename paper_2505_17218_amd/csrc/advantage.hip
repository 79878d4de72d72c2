// GRPO group advantage with the gradient-filter compaction, and the live-row
// compaction of ragged decoding.  Both are tiny (N <= a few thousand): one
// workgroup of 1024 threads walks the input in chunks, and a ballot / mbcnt
// prefix inside each wave plus an LDS scan across the 16 waves gives every
// kept element its output slot, so kept indices come out in ascending order
// with no atomics (deterministic).
//
// Group statistics (groups of G <= 64): samples are spread over "virtual
// lanes", P2 = next power of two >= G lanes per group with the tail zero, so a
// group sits in an aligned run of P2 lanes of one wave and an xor butterfly
// (offsets 1, 2, 4, ...) forms the pairwise sum, adjacent pairs first.  Groups
// with 64 < G <= 1024 use the same tree in LDS, one group at a time; larger
// groups (up to 65536, e.g. the single-path baseline over a whole batch) give
// each thread a power-of-two run of the group, summed pairwise with a binary
// counter, then the LDS tree over the threads: the same tree, level by level.
// Modes: mean-centred (Eq. (4)), / (std + eps) with ddof 0 or 1, and the
// leave-one-out baseline r - (S - r) / (G - 1).
// Built with -ffp-contract=off: see sampler_math.h.
#include "common.h"
#include "kernels.h"
#include "sampler_math.h"

namespace dash {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;

// Exclusive prefix of `flag` over the workgroup, in thread order; returns the
// prefix and writes the total to *total.  `scan` is LDS of kWaves ints.
DASH_DEV int block_excl_scan(bool flag, int* scan, int* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t bal = __ballot(flag);
    const int in_wave = __popcll(bal & ((1ull << lane) - 1ull));
    __syncthreads();
    if (lane == 0) scan[w] = __popcll(bal);
    __syncthreads();
    int before = 0, tot = 0;
    for (int i = 0; i < kWaves; ++i) {
        const int c = scan[i];
        before += i < w ? c : 0;
        tot += c;
    }
    *total = tot;
    return before + in_wave;
}

constexpr int kModeLoo = 3;

// Leave-one-out advantage from the reward x and its group's sum S.
DASH_DEV float adv_loo(float x, float S, int G) { return x - div_rn(S - x, (float)(G - 1)); }

DASH_DEV float adv_of(float d, float ss, int G, int mode, float eps) {
    if (mode == 0) return d;
    const int ddof = mode == 2 ? 1 : 0;
    float sd = 0.f;
    if (G - ddof > 0) sd = sqrt_rn(div_rn(ss, (float)(G - ddof)));
    return div_rn(d, sd + eps);
}

__global__ void __launch_bounds__(kThreads) adv_filter_wave_k(const float* __restrict__ r, int n_groups, int G, int P2,
                                                              int mode, float eps, float tau, float* __restrict__ adv,
                                                              int32_t* __restrict__ kept, int32_t* __restrict__ count) {
    __shared__ int scan[kWaves];
    const int total_v = n_groups * P2;
    int base = 0;
    for (int c0 = 0; c0 < total_v; c0 += kThreads) {
        const int v = c0 + threadIdx.x;
        const int grp = v / P2, j = v % P2;
        const bool valid = v < total_v && j < G;
        const int n = grp * G + j;
        const float x = valid ? r[n] : 0.f;
        float s = x;
        for (int o = 1; o < P2; o <<= 1) s = s + __shfl_xor(s, o, 64);
        const float mu = div_rn(s, (float)G);
        const float d = x - mu;
        float q = valid ? d * d : 0.f;
        if (mode != 0 && mode != kModeLoo)
            for (int o = 1; o < P2; o <<= 1) q = q + __shfl_xor(q, o, 64);
        const float a = mode == kModeLoo ? adv_loo(x, s, G) : adv_of(d, q, G, mode, eps);
        const bool keep = valid && fabsf(a) >= tau;
        if (valid) adv[n] = a;
        int tot;
        const int at = block_excl_scan(keep, scan, &tot);
        if (keep) kept[base + at] = n;
        base += tot;
    }
    if (threadIdx.x == 0) *count = base;
}

__global__ void __launch_bounds__(kThreads) adv_filter_lds_k(const float* __restrict__ r, int n_groups, int G, int P2,
                                                             int mode, float eps, float tau, float* __restrict__ adv,
                                                             int32_t* __restrict__ kept, int32_t* __restrict__ count) {
    __shared__ float buf[kThreads];
    __shared__ int scan[kWaves];
    const int j = threadIdx.x;
    int base = 0;
    for (int grp = 0; grp < n_groups; ++grp) {
        const bool valid = j < G;
        const int n = grp * G + j;
        const float x = valid ? r[n] : 0.f;
        if (j < P2) buf[j] = x;
        __syncthreads();
        for (int half = P2 >> 1; half >= 1; half >>= 1) {  // a[i] = a[2i] + a[2i+1]
            float t = 0.f;
            if (j < half) t = buf[2 * j] + buf[2 * j + 1];
            __syncthreads();
            if (j < half) buf[j] = t;
            __syncthreads();
        }
        const float S = buf[0];
        const float mu = div_rn(S, (float)G);
        const float d = x - mu;
        __syncthreads();
        if (j < P2) buf[j] = valid ? d * d : 0.f;
        __syncthreads();
        for (int half = P2 >> 1; half >= 1; half >>= 1) {
            float t = 0.f;
            if (j < half) t = buf[2 * j] + buf[2 * j + 1];
            __syncthreads();
            if (j < half) buf[j] = t;
            __syncthreads();
        }
        const float a = mode == kModeLoo ? adv_loo(x, S, G) : adv_of(d, buf[0], G, mode, eps);
        __syncthreads();
        const bool keep = valid && fabsf(a) >= tau;
        if (valid) adv[n] = a;
        int tot;
        const int at = block_excl_scan(keep, scan, &tot);
        if (keep) kept[base + at] = n;
        base += tot;
    }
    if (threadIdx.x == 0) *count = base;
}

constexpr int kMaxRunLog = 6;  // runs of up to 64 samples per thread: groups up to 65536

// Pairwise sum of val(0 .. kThreads * c - 1) (c a power of two <= 2^kMaxRunLog):
// thread t sums its run [t c, (t + 1) c) with a binary counter (a finished pair
// of 2^k-sums merges left + right, as one level of the tree), then LDS adds
// adjacent thread results level by level.  Returns the total in every thread.
template <typename F>
DASH_DEV float block_pairwise_sum(F val, int c, float* buf) {
    const int t = threadIdx.x;
    float st[kMaxRunLog];
    float run = 0.f;
    for (int i = 0; i < c; ++i) {
        float v = val(t * c + i);
        bool placed = false;
#pragma unroll
        for (int k = 0; k < kMaxRunLog; ++k) {
            if (!placed) {
                if ((i >> k) & 1) {
                    v = st[k] + v;
                } else {
                    st[k] = v;
                    placed = true;
                }
            }
        }
        run = v;  // after the last element every level has merged: the run's total
    }
    __syncthreads();
    buf[t] = run;
    __syncthreads();
    for (int half = kThreads >> 1; half >= 1; half >>= 1) {
        float x = 0.f;
        if (t < half) x = buf[2 * t] + buf[2 * t + 1];
        __syncthreads();
        if (t < half) buf[t] = x;
        __syncthreads();
    }
    const float total = buf[0];
    __syncthreads();
    return total;
}

__global__ void __launch_bounds__(kThreads) adv_filter_big_k(const float* __restrict__ r, int n_groups, int G, int P2,
                                                             int mode, float eps, float tau, float* __restrict__ adv,
                                                             int32_t* __restrict__ kept, int32_t* __restrict__ count) {
    __shared__ float buf[kThreads];
    __shared__ int scan[kWaves];
    const int c = P2 / kThreads;
    int base = 0;
    for (int grp = 0; grp < n_groups; ++grp) {
        const float* rg = r + (size_t)grp * G;
        const float S = block_pairwise_sum([&](int j) { return j < G ? rg[j] : 0.f; }, c, buf);
        const float mu = div_rn(S, (float)G);
        float ss = 0.f;
        if (mode != 0 && mode != kModeLoo)
            ss = block_pairwise_sum(
                [&](int j) {
                    if (j >= G) return 0.f;
                    const float d = rg[j] - mu;
                    return d * d;
                },
                c, buf);
        for (int c0 = 0; c0 < G; c0 += kThreads) {
            const int j = c0 + threadIdx.x;
            const bool valid = j < G;
            const float x = valid ? rg[j] : 0.f;
            const float a = mode == kModeLoo ? adv_loo(x, S, G) : adv_of(x - mu, ss, G, mode, eps);
            const bool keep = valid && fabsf(a) >= tau;
            if (valid) adv[(size_t)grp * G + j] = a;
            int tot;
            const int at = block_excl_scan(keep, scan, &tot);
            if (keep) kept[base + at] = grp * G + j;
            base += tot;
        }
    }
    if (threadIdx.x == 0) *count = base;
}

__global__ void __launch_bounds__(kThreads)
live_compact_k(const int32_t* __restrict__ tok, const int32_t* __restrict__ slot, const int32_t* __restrict__ pos,
               const int32_t* __restrict__ step, const int32_t* __restrict__ uid, const int32_t* __restrict__ budget,
               int eos_id, int n, int32_t* __restrict__ tok_o, int32_t* __restrict__ slot_o,
               int32_t* __restrict__ pos_o, int32_t* __restrict__ step_o, int32_t* __restrict__ uid_o,
               int32_t* __restrict__ count) {
    __shared__ int scan[kWaves];
    int base = 0;
    for (int c0 = 0; c0 < n; c0 += kThreads) {
        const int i = c0 + threadIdx.x;
        bool live = false;
        if (i < n) live = (step[i] + 1 < budget[uid[i]]) && !(eos_id >= 0 && tok[i] == eos_id);
        int tot;
        const int at = block_excl_scan(live, scan, &tot);
        if (live) {
            const int o = base + at;
            tok_o[o] = tok[i];
            slot_o[o] = slot[i];
            pos_o[o] = pos[i] + 1;
            step_o[o] = step[i] + 1;
            uid_o[o] = uid[i];
        }
        base += tot;
    }
    if (threadIdx.x == 0) *count = base;
}

// Loss over the kept samples, float64, reproducible bit for bit.  A wave sums a sample's
// per-token values (loss_row_sum: lanes over tokens, then the lanes by an xor tree); the
// samples' terms are then added by one workgroup, thread t taking kept samples t, t + 1024,
// ... in order and the threads as a pairwise tree.  Surrogate: A S (PG, no old log-probs)
// or PPO's min(rho A, clip(rho, 1 - eps, 1 + eps) A) with rho = exp(S - S_old); the KL
// sums (if given) enter with weight beta.  stats[4 n ..] = (S, S_old, KL, dloss/dS).
//
// The rows are what there is to read (12 MB for 1024 samples of 1024 tokens), so they are
// read by a launch of their own, a wave per sample over the whole GPU, which leaves the
// sums in the caller's stats (or seq_lp) for the one-workgroup sum.  One thread per sample
// in a single workgroup took 560 us at 1024 x 1024 (three rows, 614 kept, mean length
// 512): uncoalesced 4-byte reads and a serial chain of adds on one CU; the two launches
// take 7.4 and 3.6 us (the call 593 -> 24 us, half of it the host).  Without an output that holds
// the sums the one workgroup's waves read the rows too.
struct LossArgs {
    const float *lp, *lp_old, *kl;
    int64_t ld;
    int T;
    const int32_t* len;
    const float* adv;
    const int32_t *kept, *kept_count;
    int n_total;
    double clip_eps, beta;
    double *loss, *seq_lp, *stats;
};

// Sum of row[0 .. L-1] over the wave, the same value in every lane.  (t runs up to 575 past L:
// unsigned, so that it doesn't wrap at the largest L.)
DASH_DEV double loss_row_sum(const float* __restrict__ row, int L) {
    const uint32_t n = (uint32_t)L;
    double acc = 0.0;
    uint32_t t = threadIdx.x & 63;
    for (; t + 7 * 64 < n; t += 8 * 64) {  // eight loads in flight per lane
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = row[t + 64 * j];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc += (double)v[j];
    }
    for (; t < n; t += 64) acc += (double)row[t];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) acc += __shfl_xor(acc, o, 64);
    return acc;
}

struct LossRow {
    double S, S_old, kl;
};

DASH_DEV LossRow loss_row(const LossArgs& a, int n) {
    const int L = a.len ? min(max(a.len[n], 0), a.T) : a.T;
    LossRow r;
    r.S = loss_row_sum(a.lp + (int64_t)n * a.ld, L);
    r.S_old = a.lp_old ? loss_row_sum(a.lp_old + (int64_t)n * a.ld, L) : r.S;
    r.kl = a.kl ? loss_row_sum(a.kl + (int64_t)n * a.ld, L) : 0.0;
    return r;
}

// The sample's surrogate and the loss's derivative with respect to S.
DASH_DEV double loss_surrogate(const LossArgs& a, const LossRow& r, double A, double& w) {
    const double N = (double)a.n_total;
    if (!a.lp_old) {
        w = -A / N;
        return A * r.S;
    }
    const double rho = exp(r.S - r.S_old);
    const double un = rho * A;
    const double cl = fmin(fmax(rho, 1.0 - a.clip_eps), 1.0 + a.clip_eps) * A;
    w = un <= cl ? -A * rho / N : 0.0;
    return fmin(un, cl);
}

constexpr int kLossRowWaves = 4;  // samples per workgroup of the row launch

__global__ void __launch_bounds__(64 * kLossRowWaves) loss_rows_k(LossArgs a) {
    const int K = *a.kept_count;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int k = blockIdx.x * kLossRowWaves + wave; k < K; k += gridDim.x * kLossRowWaves) {
        const int n = a.kept[k];
        const LossRow r = loss_row(a, n);
        if ((threadIdx.x & 63) == 0) {
            if (a.seq_lp) a.seq_lp[n] = r.S;
            if (a.stats) {
                double w;
                loss_surrogate(a, r, (double)a.adv[n], w);
                double* st = a.stats + 4 * (int64_t)n;
                st[0] = r.S;
                st[1] = r.S_old;
                st[2] = r.kl;
                st[3] = w;
            }
        }
    }
}

// FROM: where the samples' sums come from: 0 read here, 1 from stats, 2 from seq_lp (S alone).
template <int FROM>
__global__ void __launch_bounds__(kThreads) loss_sum_k(LossArgs a) {
    __shared__ double buf[kThreads], kbuf[kThreads];
    __shared__ LossRow rows[FROM == 0 ? kThreads : 1];
    const int K = *a.kept_count;
    const int tid = threadIdx.x;
    const double N = (double)a.n_total;
    double acc = 0.0, kacc = 0.0;
    for (int k0 = 0; k0 < K; k0 += kThreads) {
        if constexpr (FROM == 0) {
            for (int i = tid >> 6; i < min(kThreads, K - k0); i += kWaves) {
                const LossRow r = loss_row(a, a.kept[k0 + i]);
                if ((tid & 63) == 0) rows[i] = r;
            }
            __syncthreads();
        }
        if (k0 + tid < K) {
            const int n = a.kept[k0 + tid];
            LossRow r;
            if constexpr (FROM == 0) {
                r = rows[tid];
            } else if constexpr (FROM == 1) {
                const double* st = a.stats + 4 * (int64_t)n;
                r = LossRow{st[0], st[1], st[2]};
            } else {
                r = LossRow{a.seq_lp[n], 0.0, 0.0};
            }
            double w;
            acc += loss_surrogate(a, r, (double)a.adv[n], w);
            kacc += r.kl;
        }
        if constexpr (FROM == 0) __syncthreads();  // rows are refilled next
    }
    buf[tid] = acc;
    kbuf[tid] = kacc;
    __syncthreads();
    for (int half = kThreads >> 1; half >= 1; half >>= 1) {
        double x = 0.0, y = 0.0;
        if (tid < half) {
            x = buf[2 * tid] + buf[2 * tid + 1];
            y = kbuf[2 * tid] + kbuf[2 * tid + 1];
        }
        __syncthreads();
        if (tid < half) {
            buf[tid] = x;
            kbuf[tid] = y;
        }
        __syncthreads();
    }
    if (tid == 0) {
        double l = -buf[0] / N;
        if (a.kl) l += a.beta * kbuf[0] / N;
        *a.loss = l;
    }
}

}  // namespace

hipError_t launch_policy_loss(const float* lp, const float* lp_old, const float* kl, int64_t ld, int T,
                              const int32_t* len, const float* adv, const int32_t* kept, const int32_t* kept_count,
                              int n_total, double clip_eps, double beta, double* loss, double* seq_lp, double* stats,
                              hipStream_t st) {
    const LossArgs a{lp, lp_old, kl, ld, T, len, adv, kept, kept_count, n_total, clip_eps, beta, loss, seq_lp, stats};
    if (seq_lp && !stats && (lp_old || kl)) return hipErrorInvalidValue;
    // the sums' way from the row launch to the final one: stats, or seq_lp where S is all there is
    const int from = stats ? 1 : seq_lp ? 2 : 0;
    if (from) {
        const int blocks = n_total / kLossRowWaves < 2048 ? n_total / kLossRowWaves + 1 : 2048;
        loss_rows_k<<<blocks, 64 * kLossRowWaves, 0, st>>>(a);
    }
    if (from == 1)
        loss_sum_k<1><<<1, kThreads, 0, st>>>(a);
    else if (from == 2)
        loss_sum_k<2><<<1, kThreads, 0, st>>>(a);
    else
        loss_sum_k<0><<<1, kThreads, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_pg_loss(const float* lp, int64_t ld, int T, const int32_t* len, const float* adv,
                          const int32_t* kept, const int32_t* kept_count, int n_total, double* loss, double* seq_lp,
                          hipStream_t st) {
    return launch_policy_loss(lp, nullptr, nullptr, ld, T, len, adv, kept, kept_count, n_total, 0.0, 0.0, loss, seq_lp,
                              nullptr, st);
}

hipError_t launch_group_advantage_filter(const float* r, int n_groups, int group, int mode, float eps, float tau,
                                         float* adv, int32_t* kept, int32_t* count, hipStream_t st) {
    int P2 = 1;
    while (P2 < group) P2 <<= 1;
    if (P2 > (kThreads << kMaxRunLog)) return hipErrorInvalidValue;
    if (P2 <= 64)
        adv_filter_wave_k<<<1, kThreads, 0, st>>>(r, n_groups, group, P2, mode, eps, tau, adv, kept, count);
    else if (P2 <= kThreads)
        adv_filter_lds_k<<<1, kThreads, 0, st>>>(r, n_groups, group, P2, mode, eps, tau, adv, kept, count);
    else
        adv_filter_big_k<<<1, kThreads, 0, st>>>(r, n_groups, group, P2, mode, eps, tau, adv, kept, count);
    return hipGetLastError();
}

hipError_t launch_live_compact(const int32_t* tok, const int32_t* slot, const int32_t* pos, const int32_t* step,
                               const int32_t* uid, const int32_t* budget, int eos_id, int n, int32_t* tok_o,
                               int32_t* slot_o, int32_t* pos_o, int32_t* step_o, int32_t* uid_o, int32_t* count,
                               hipStream_t st) {
    live_compact_k<<<1, kThreads, 0, st>>>(tok, slot, pos, step, uid, budget, eos_id, n, tok_o, slot_o, pos_o, step_o,
                                           uid_o, count);
    return hipGetLastError();
}

}  // namespace dash
