// Sampling stage: guidance, temperature / top-k warp, inverse-CDF draws, the accept /
// reject scan with residual resampling, and the commit of a step.
//
// The functions of one row are in sample_rows.h.
#include <mutex>
#include "sample_rows.h"

namespace hawk {

namespace {

// ---------------------------------------------------------------------------- kernels

__global__ void plan_kernel(const int32_t* n, int32_t* k_eff, int32_t* draft, int32_t* step,
                            unsigned long long* counters, int B, int N, int k, int kstride) {
    int b = threadIdx.x;
    if (b == 0) {
        step[0] += 1;
        bool any = false;
        for (int j = 0; j < B; ++j) any = any || n[j] < N;
        if (any) counters[3] += 1ull;  // lock-step iterations that still had work
    }
    if (b >= B) return;
    int nb = n[b];
    k_eff[b] = nb < N ? min(k, N - nb - 1) : -1;
    for (int i = 0; i < kstride; ++i) draft[b * kstride + i] = -1;
}

// Token 0 of every prompt from the logits of the last condition row.
__global__ __launch_bounds__(NT) void first_token_kernel(const float* logit_s, float* logit_b, int32_t* grid,
                                                         int32_t* n, SampParams P, UniformSrc us) {
    __shared__ Shared sh;
    const int b = blockIdx.x;
    float* row = logit_b + (size_t)b * P.kstride * P.Vs;
    combine_row(logit_s + (size_t)b * P.Vs, P.use_cfg ? logit_s + (size_t)(P.B + b) * P.Vs : nullptr,
                P.cfg_scale, row, P.Vs);
    WarpStat st = warp_stats(row, P.Vs, P.inv_t, P.top_k, P.greedy, sh);
    float u = pick_uniform(us, us.fin, b, b, kSlotFinal);
    int idx = inv_cdf([&](int j) { return weight_of(st, row, P.inv_t, j); }, P.Vs, st.total, u, sh);
    if (threadIdx.x == 0) {
        grid[(size_t)b * P.N] = P.samp_lo + idx;
        n[b] = 1;
    }
}

// Draft i (1-based): guide, warp, then draw the token by inverse CDF - or, when a table
// of forced tokens is given, take the token from it (teacher-forced drafting; with
// point_mass the draft distribution becomes the point mass on that token).  Keeps the
// guided row and its warp statistics for the accept test of the verify step.
__global__ __launch_bounds__(NT) void draft_sample_kernel(const float* dlogit_s, float* dlogit_b, const int32_t* n,
                                                          const int32_t* k_eff, int32_t* draft, WarpStat* qstat,
                                                          int i, int k, SampParams P, UniformSrc us, ForcedSrc fs) {
    __shared__ Shared sh;
    const int b = blockIdx.x;
    if (i > k_eff[b]) return;
    float* row = dlogit_b + ((size_t)b * P.kstride + (i - 1)) * P.Vs;
    combine_row(dlogit_s + (size_t)b * P.Vs, P.use_cfg ? dlogit_s + (size_t)(P.B + b) * P.Vs : nullptr,
                P.cfg_scale, row, P.Vs);
    WarpStat st = warp_stats(row, P.Vs, P.inv_t, P.top_k, P.greedy, sh);
    int tok;
    if (fs.table) {
        tok = fs.table[(size_t)b * fs.stride + (fs.relative ? n[b] : 0) + (i - 1)];
        if (fs.point_mass) { st.onehot = tok - P.samp_lo; st.total = 1.0; }
    } else {
        float u = pick_uniform(us, us.draft, b * k + (i - 1), b, kSlotDraft + (i - 1));
        tok = P.samp_lo + inv_cdf([&](int j) { return weight_of(st, row, P.inv_t, j); }, P.Vs, st.total, u, sh);
    }
    if (threadIdx.x == 0) {
        draft[b * P.kstride + (i - 1)] = tok;
        qstat[b * P.kstride + (i - 1)] = st;
    }
}

// Guided target row r of prompt b and its warp statistics.
__global__ __launch_bounds__(NT) void verify_stats_kernel(const float* logit_s, float* logit_b,
                                                          const int32_t* k_eff, WarpStat* pstat, int k,
                                                          SampParams P) {
    __shared__ Shared sh;
    const int r = blockIdx.x, b = blockIdx.y;
    if (r > k_eff[b]) return;
    float* row = logit_b + ((size_t)b * P.kstride + r) * P.Vs;
    combine_row(logit_s + ((size_t)b * (k + 1) + r) * P.Vs,
                P.use_cfg ? logit_s + ((size_t)(P.B + b) * (k + 1) + r) * P.Vs : nullptr, P.cfg_scale, row, P.Vs);
    WarpStat st = warp_stats(row, P.Vs, P.inv_t, P.top_k, P.greedy, sh);
    if (threadIdx.x == 0) pstat[b * P.kstride + r] = st;
}

// Accept scan, residual / bonus draw and commit for prompt b.
__global__ __launch_bounds__(NT) void accept_commit_kernel(
    const float* logit_b, const float* dlogit_b, const WarpStat* pstat, const WarpStat* qstat, const int32_t* k_eff,
    const int32_t* draft, int32_t* grid, int32_t* n, const uint32_t* hid, uint32_t* hprev, int hid_words,
    int32_t* out_na, int32_t* out_tok, unsigned long long* counters, int k, int n_seq_streams, SampParams P,
    UniformSrc us) {
    __shared__ Shared sh;
    const int b = blockIdx.x;
    const int ke = k_eff[b];
    if (threadIdx.x <= k) out_tok[b * (k + 1) + threadIdx.x] = -1;
    if (ke < 0) {
        if (threadIdx.x == 0) out_na[b] = -1;
        return;
    }
    // accept scan (every thread computes the same thing)
    int a = 0;
    for (; a < ke; ++a) {
        const int dj = draft[b * P.kstride + a] - P.samp_lo;
        const WarpStat ps = pstat[b * P.kstride + a], qs = qstat[b * P.kstride + a];
        const double pd = weight_of(ps, logit_b + ((size_t)b * P.kstride + a) * P.Vs, P.inv_t, dj) / ps.total;
        const double qd = weight_of(qs, dlogit_b + ((size_t)b * P.kstride + a) * P.Vs, P.inv_t, dj) / qs.total;
        const float u = pick_uniform(us, us.acc, b * k + a, b, kSlotAcc + a);
        if (!((double)u * qd < pd)) break;
    }
    const float uf = pick_uniform(us, us.fin, b, b, kSlotFinal);
    const float* prow = logit_b + ((size_t)b * P.kstride + a) * P.Vs;
    const WarpStat ps = pstat[b * P.kstride + a];
    int y;
    auto wp = [&](int j) { return weight_of(ps, prow, P.inv_t, j); };
    if (a < ke) {
        const float* qrow = dlogit_b + ((size_t)b * P.kstride + a) * P.Vs;
        const WarpStat qs = qstat[b * P.kstride + a];
        auto res = [&](int j) {
            double r = weight_of(ps, prow, P.inv_t, j) / ps.total - weight_of(qs, qrow, P.inv_t, j) / qs.total;
            return r > 0.0 ? r : 0.0;
        };
        const Seg sg = my_segment(P.Vs);
        double s = 0.0;
        for (int j = sg.j0; j < sg.j1; ++j) s += res(j);
        const double R = block_sum_d(s, sh);
        y = (R > 0.0) ? inv_cdf(res, P.Vs, R, uf, sh) : inv_cdf(wp, P.Vs, ps.total, uf, sh);
    } else {
        y = inv_cdf(wp, P.Vs, ps.total, uf, sh);
    }
    // commit: tokens, counters, hidden state of row a for the next draft
    const int nb = n[b];
    for (int s = b; s < n_seq_streams; s += P.B) {
        const uint32_t* src = hid + ((size_t)s * (k + 1) + a) * hid_words;
        uint32_t* dst = hprev + (size_t)s * hid_words;
        for (int i = threadIdx.x; i < hid_words; i += NT) dst[i] = src[i];
    }
    __syncthreads();  // every thread has read n[b] before it changes
    if (threadIdx.x == 0) {
        for (int i = 0; i < a; ++i) {
            int t = draft[b * P.kstride + i];
            grid[(size_t)b * P.N + nb + i] = t;
            out_tok[b * (k + 1) + i] = t;
        }
        grid[(size_t)b * P.N + nb + a] = P.samp_lo + y;
        out_tok[b * (k + 1) + a] = P.samp_lo + y;
        out_na[b] = a;
        n[b] = nb + a + 1;
        atomicAdd(&counters[0], 1ull);
        atomicAdd(&counters[1], (unsigned long long)a);
        atomicAdd(&counters[2], (unsigned long long)(a + 1));
    }
}

__global__ void force_setup_kernel(const int32_t* n_from, const int32_t* forced, int32_t* n, int32_t* k_eff,
                                   int32_t* draft, int B, int cnt, int kstride) {
    int b = threadIdx.x;
    if (b >= B) return;
    n[b] = n_from[b];
    k_eff[b] = cnt - 1;
    for (int i = 0; i < kstride; ++i) draft[b * kstride + i] = i < cnt - 1 ? forced[b * cnt + i] : -1;
}

__global__ void force_commit_kernel(const int32_t* forced, int32_t* grid, int32_t* n, const uint32_t* hid,
                                    uint32_t* hprev, int hid_words, int B, int N, int cnt, int n_seq_streams) {
    const int b = blockIdx.x;
    const int nb = n[b];
    for (int s = b; s < n_seq_streams; s += B) {
        const uint32_t* src = hid + ((size_t)s * cnt + (cnt - 1)) * hid_words;
        uint32_t* dst = hprev + (size_t)s * hid_words;
        for (int i = threadIdx.x; i < hid_words; i += blockDim.x) dst[i] = src[i];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 0; i < cnt; ++i) grid[(size_t)b * N + nb + i] = forced[b * cnt + i];
        n[b] = nb + cnt;
    }
}

template <int E>
__global__ __launch_bounds__(NT) void first_token_fast(const float* logit_s, float* logit_b, int32_t* grid, int32_t* n,
                                                       SampParams P, UniformSrc us) {
    __shared__ FastShared fs;
    __shared__ CompactList L;
    const int b = blockIdx.x;
    float z[E];
    load_row<E>(logit_s + (size_t)b * P.Vs, P.use_cfg ? logit_s + (size_t)(P.B + b) * P.Vs : nullptr, P.cfg_scale,
                P.inv_t, logit_b + (size_t)b * P.kstride * P.Vs, P.Vs, z);
    const float u = pick_uniform(us, us.fin, b, b, kSlotFinal);
    int idx = 0;
    (void)warp_and_draw<E>(z, P.Vs, P.top_k, P.greedy, fs, L, &u, &idx);
    if (threadIdx.x == 0) {
        grid[(size_t)b * P.N] = P.samp_lo + idx;
        n[b] = 1;
    }
}

template <int E>
__global__ __launch_bounds__(NT) void draft_sample_fast(const float* dlogit_s, float* dlogit_b, const int32_t* n,
                                                        const int32_t* k_eff, int32_t* draft, WarpStat* qstat, int i,
                                                        int k, SampParams P, UniformSrc us, ForcedSrc fsrc) {
    __shared__ FastShared fs;
    __shared__ CompactList L;
    const int b = blockIdx.x;
    if (i > k_eff[b]) return;
    float z[E];
    load_row<E>(dlogit_s + (size_t)b * P.Vs, P.use_cfg ? dlogit_s + (size_t)(P.B + b) * P.Vs : nullptr, P.cfg_scale,
                P.inv_t, dlogit_b + ((size_t)b * P.kstride + (i - 1)) * P.Vs, P.Vs, z);
    const float u = fsrc.table ? 0.f : pick_uniform(us, us.draft, b * k + (i - 1), b, kSlotDraft + (i - 1));
    int drawn = 0;
    WarpStat st = warp_and_draw<E>(z, P.Vs, P.top_k, P.greedy, fs, L, fsrc.table ? nullptr : &u, &drawn);
    int tok;
    if (fsrc.table) {
        tok = fsrc.table[(size_t)b * fsrc.stride + (fsrc.relative ? n[b] : 0) + (i - 1)];
        if (fsrc.point_mass) { st.onehot = tok - P.samp_lo; st.total = 1.0; }
    } else {
        tok = P.samp_lo + drawn;
    }
    if (threadIdx.x == 0) {
        draft[b * P.kstride + (i - 1)] = tok;
        qstat[b * P.kstride + (i - 1)] = st;
    }
}

template <int E>
__global__ __launch_bounds__(NT) void verify_stats_fast(const float* logit_s, float* logit_b, const int32_t* k_eff,
                                                        WarpStat* pstat, int32_t* llen, int32_t* lidx, double* lw, int k,
                                                        SampParams P) {
    __shared__ FastShared fs;
    __shared__ CompactList L;
    const int r = blockIdx.x, b = blockIdx.y;
    if (r > k_eff[b]) return;
    float z[E];
    load_row<E>(logit_s + ((size_t)b * (k + 1) + r) * P.Vs,
                P.use_cfg ? logit_s + ((size_t)(P.B + b) * (k + 1) + r) * P.Vs : nullptr, P.cfg_scale, P.inv_t,
                logit_b + ((size_t)b * P.kstride + r) * P.Vs, P.Vs, z);
    const ListStore store = list_at(llen, lidx, lw, (size_t)b * P.kstride + r);
    const WarpStat st = warp_and_draw<E>(z, P.Vs, P.top_k, P.greedy, fs, L, nullptr, nullptr, store);
    if (threadIdx.x == 0) pstat[b * P.kstride + r] = st;
}

template <int E>
__global__ __launch_bounds__(NT) void accept_commit_fast(
    const float* logit_b, const float* dlogit_b, const WarpStat* pstat, const WarpStat* qstat, int32_t* llen, int32_t* lidx,
    double* lw, const int32_t* k_eff, const int32_t* draft, int32_t* grid, int32_t* n, const uint32_t* hid, uint32_t* hprev,
    int hid_words, int32_t* out_na, int32_t* out_tok, unsigned long long* counters, int k, int n_seq_streams, SampParams P,
    UniformSrc us) {
    __shared__ Slots sl;
    __shared__ Shared sh;
    const int b = blockIdx.x, lane = threadIdx.x & 63, th = (int)threadIdx.x;
    const int ke = k_eff[b];
    if (threadIdx.x <= k) out_tok[b * (k + 1) + threadIdx.x] = -1;
    if (ke < 0) {
        if (threadIdx.x == 0) out_na[b] = -1;
        return;
    }
    if (threadIdx.x == 0) sl.pick = 0x7FFFFFFF;
    // Accept scan: the tests do not depend on each other, so lane i of every wave makes test i and the
    // first rejection is where the scan stops (k <= 63).
    bool rejected = false;
    if (lane < ke) {
        const int dj = draft[b * P.kstride + lane] - P.samp_lo;
        const WarpStat ps = pstat[b * P.kstride + lane], qs = qstat[b * P.kstride + lane];
        const double pd = weight_of(ps, logit_b + ((size_t)b * P.kstride + lane) * P.Vs, P.inv_t, dj) / ps.total;
        const double qd = weight_of(qs, dlogit_b + ((size_t)b * P.kstride + lane) * P.Vs, P.inv_t, dj) / qs.total;
        const float u = pick_uniform(us, us.acc, b * k + lane, b, kSlotAcc + lane);
        rejected = !((double)u * qd < pd);
    }
    const unsigned long long rej = __ballot(rejected);
    const int a = rej ? (int)__ffsll(rej) - 1 : ke;
    const float uf = pick_uniform(us, us.fin, b, b, kSlotFinal);
    const float* prow = logit_b + ((size_t)b * P.kstride + a) * P.Vs;
    const WarpStat ps = pstat[b * P.kstride + a];
    int y;
    bool resid = false;
    if (use_list(P.top_k, P.Vs, P.greedy)) {
        // the kept entries of p (a superset of the residual's support) as the list verify_stats_fast left; q only where p > 0
        const ListStore src = list_at(llen, lidx, lw, (size_t)b * P.kstride + a);
        const int Kc = *src.len;
        int idx[kLH];
        double w[kLH], c[kLH];
#pragma unroll
        for (int h = 0; h < kLH; ++h) {
            const int i = (int)threadIdx.x + h * NT;
            idx[h] = -1;
            w[h] = 0.0;
            if (i < Kc) { idx[h] = src.idx[i]; w[h] = src.w[i]; }
        }
        int at = 0;
        __syncthreads();   // sl.pick is set
        if (a < ke) {
            const float* qrow = dlogit_b + ((size_t)b * P.kstride + a) * P.Vs;
            const WarpStat qs = qstat[b * P.kstride + a];
            double r[kLH];
#pragma unroll
            for (int h = 0; h < kLH; ++h) {
                r[h] = 0.0;
                if (idx[h] >= 0) {
                    const double v = w[h] / ps.total - weight_of(qs, qrow, P.inv_t, idx[h]) / qs.total;
                    r[h] = v > 0.0 ? v : 0.0;
                }
            }
            const double R = list_scan(r, Kc, c, sl.scan[0]);
            if (R > 0.0) {
                resid = true;
                at = list_pick(r, c, (double)uf * R, sl, sh);
            }
        }
        if (!resid) {
            (void)list_scan(w, Kc, c, sl.scan[1]);
            at = list_pick(w, c, (double)uf * ps.total, sl, sh);
        }
        y = Kc > 0 ? src.idx[at] : 0;
    } else {
        double w[E];
#pragma unroll
        for (int e = 0; e < E; ++e) w[e] = entry<E>(e, th) < P.Vs ? weight_of(ps, prow, P.inv_t, entry<E>(e, th)) : 0.0;
        if (a < ke) {
            const float* qrow = dlogit_b + ((size_t)b * P.kstride + a) * P.Vs;
            const WarpStat qs = qstat[b * P.kstride + a];
            double res[E], s = 0.0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const double q = entry<E>(e, th) < P.Vs ? weight_of(qs, qrow, P.inv_t, entry<E>(e, th)) / qs.total : 0.0;
                const double r = w[e] / ps.total - q;
                res[e] = r > 0.0 ? r : 0.0;
                s += res[e];
            }
            const double R = sum1(s, sl.sum);
            if (R > 0.0) {
                resid = true;
                y = inv_cdf_row<E>(res, R, uf, sl, sh);
            }
        }
        if (!resid) y = inv_cdf_row<E>(w, ps.total, uf, sl, sh);
    }
    const int nb = n[b];
    for (int s2 = b; s2 < n_seq_streams; s2 += P.B) {
        const uint32_t* src = hid + ((size_t)s2 * (k + 1) + a) * hid_words;
        uint32_t* dst = hprev + (size_t)s2 * hid_words;
        for (int i = threadIdx.x; i < hid_words; i += NT) dst[i] = src[i];
    }
    for (int i = threadIdx.x; i < a; i += NT) {
        const int t = draft[b * P.kstride + i];
        grid[(size_t)b * P.N + nb + i] = t;
        out_tok[b * (k + 1) + i] = t;
    }
    __syncthreads();   // every thread has read n[b] before it changes
    if (threadIdx.x == 0) {
        grid[(size_t)b * P.N + nb + a] = P.samp_lo + y;
        out_tok[b * (k + 1) + a] = P.samp_lo + y;
        out_na[b] = a;
        n[b] = nb + a + 1;
        atomicAdd(&counters[0], 1ull);
        atomicAdd(&counters[1], (unsigned long long)a);
        atomicAdd(&counters[2], (unsigned long long)(a + 1));
    }
}

// Several candidates at one position, each from a proposal of its own (Method, "Sampling and
// Verification", the recursion over consecutive rejections; appendix "Theoretical
// Justification", general form): p^(1) = p; candidate i is accepted iff u_i q_i(s_i) < p^(i)(s_i),
// otherwise p^(i+1) = norm(max(0, p^(i) - q_i)) (unchanged if that residual has no mass); after m
// rejections the token comes from p^(m+1) by inverse CDF.  One workgroup per position, the
// running target in registers (E fp64 values per thread), every proposal row read once.
// Candidates of a row: m, or the row's own count (clamped to 0 .. m) if the caller gives one.
__device__ __forceinline__ int row_candidates(const int32_t* m_rows, int row, int m) {
    return m_rows ? max(0, min(m, m_rows[row])) : m;
}

// The same recursion with the running target held as a list (the thread's entries in registers): top-k
// leaves at most kTopCap entries of p with mass, max(0, p - q) lives on those, and fp64 exponentials are
// evaluated for list entries only.
struct WalkShared {
    double pick;
    double R[2][NW];   // residual sums, alternating between candidates
};

// Candidate i of a position against the running target (list entries idx, w of this thread):
// accepts, or moves on to the residual.  qs, qrow: the proposal's statistics and logits.  True: accepted.
__device__ __forceinline__ bool walk_step(const int (&idx)[kLH], double (&w)[kLH], const WarpStat& qs, const float* qrow, float inv_t,
                                          int s_in, int n, float u, int parity, WalkShared& ws, double* resid_out) {
    const bool s_ok = (unsigned)s_in < (unsigned)n;   // a token outside the slice is rejected, never read
    const int s = s_ok ? s_in : 0;
    const float ls = qrow[s];                         // same address for every lane
    double res[kLH];
    float lq[kLH];
#pragma unroll
    for (int h = 0; h < kLH; ++h) lq[h] = idx[h] >= 0 ? qrow[idx[h]] : 0.f;
    auto weight = [&](float l, int j) {
        if (qs.onehot >= 0) return j == qs.onehot ? 1.0 : 0.0;
        const float z = l * inv_t;
        return kept(qs, z, j) ? exp((double)z - (double)qs.zmax) : 0.0;
    };
    const double qd = s_ok ? weight(ls, s) / qs.total : 1.0;
#pragma unroll
    for (int h = 0; h < kLH; ++h) {
        res[h] = 0.0;
        if (idx[h] >= 0) {
            if (idx[h] == s) ws.pick = w[h];
            const double r = w[h] - weight(lq[h], idx[h]) / qs.total;
            res[h] = r > 0.0 ? r : 0.0;
        }
    }
    const double R = sum1(sum3(res), ws.R[parity]);   // its barrier also publishes pick
    const double pd = s_ok ? ws.pick : 0.0;
    if (resid_out && threadIdx.x == 0) *resid_out = R;
    if ((double)u * qd < pd) return true;
    if (R > 0.0) {
#pragma unroll
        for (int h = 0; h < kLH; ++h) w[h] = res[h] / R;
    }
    __syncthreads();   // every thread has read pick
    if (threadIdx.x == 0) ws.pick = 0.0;   // p^(i)(s) if s has no mass left
    __syncthreads();
    return false;
}

// The end of a walk: the token of the accepted candidate, or a draw from the running target.
__device__ __forceinline__ void walk_finish(const int (&idx)[kLH], const double (&w)[kLH], int Kp, int acc, int mr, int tok, float u,
                                            int row, int m, Slots& sl, Shared& sh, int32_t* out_index, int32_t* out_token,
                                            double* out_resid) {
    int at = -1;
    if (acc == mr) {
        double c[kLH];
        const double total = list_scan(w, Kp, c, sl.scan[0]);
        at = list_pick(w, c, (double)u * total, sl, sh);
    }
#pragma unroll
    for (int h = 0; h < kLH; ++h)
        if (at == (int)threadIdx.x + h * NT) out_token[row] = idx[h];   // the drawn entry's owner
    if (threadIdx.x == 0) {
        out_index[row] = acc;
        if (at < 0) out_token[row] = tok;
        if (out_resid)
            for (int i = (acc == mr ? mr : acc + 1); i < m; ++i) out_resid[(size_t)row * m + i] = -1.0;   // steps not evaluated
    }
}

template <int E>
__global__ __launch_bounds__(NT) void multi_verify_list_kernel(const float* p_logits, const float* q_logits,
                                                               const int32_t* cand, const float* u_acc,
                                                               const float* u_final, const int32_t* m_rows, int m,
                                                               int n, float inv_t, int top_k, int32_t* out_index,
                                                               int32_t* out_token, double* out_resid) {
    __shared__ FastShared fs;
    __shared__ CompactList L;    // kept entries of the row at hand
    __shared__ WalkShared ws;
    const int row = blockIdx.x;
    const int mr = row_candidates(m_rows, row, m);
    int Kp = 0, acc = mr, tok = -1;
    int idx[kLH];
    double w[kLH];
    if (threadIdx.x == 0) ws.pick = 0.0;
    // One loop over the target row (i = -1) and the proposal rows, so that the top-k selection has
    // a single call site and is inlined with its LDS operands (a second copy would be called
    // through generic pointers).
    for (int i = -1; i < mr; ++i) {
        const float* qrow = i < 0 ? p_logits + (size_t)row * n : q_logits + ((size_t)row * m + i) * n;
        const int th = this_thread();
        float z[E];
        load_row<E>(qrow, nullptr, 0.f, inv_t, nullptr, n, z, th);
        WarpStat qs;
        Threshold t;
        const int Kq = select_list<E>(z, n, top_k, fs, L, t, qs, th);
        int iq[kLH];
        double wq[kLH];
        list_weights(L, Kq, qs.zmax, t, iq, wq);
        qs.total = sum1(sum3(wq), fs.s.sum);
        if (i < 0) {   // p^(1): the kept entries of the target, normalised
            Kp = Kq;
#pragma unroll
            for (int h = 0; h < kLH; ++h) {
                idx[h] = iq[h];
                w[h] = wq[h] / qs.total;
            }
            continue;
        }
        const int s = cand[(size_t)row * m + i];
        if (walk_step(idx, w, qs, qrow, inv_t, s, n, u_acc[(size_t)row * m + i], i & 1, ws,
                      out_resid ? &out_resid[(size_t)row * m + i] : nullptr)) {
            acc = i;
            tok = s;
            break;
        }
    }
    walk_finish(idx, w, Kp, acc, mr, tok, u_final[row], row, m, fs.s, fs.sh, out_index, out_token, out_resid);
}

// The same in two launches when the caller lends room for the rows' statistics: the top-k
// selection of the target row and of every proposal row runs in a workgroup of its own (all of
// them in parallel), and the walk over the candidates then gathers the target's kept entries again
// (writing them out instead made no difference: tree step 173.0 ms an image against 173.6).
// 64 registers, so that two rows share a compute unit and one's barriers and loads are covered by the other.
template <int E>
__global__ __launch_bounds__(NT, 8) void multi_row_stats_kernel(const float* p_logits, const float* q_logits,
                                                             const int32_t* m_rows, int m, int n, float inv_t,
                                                             int top_k, WarpStat* stats) {
    __shared__ FastShared fs;
    __shared__ CompactList L;
    const int j = blockIdx.x, row = blockIdx.y;   // j = 0: the target row, j >= 1: proposal j - 1
    if (j > row_candidates(m_rows, row, m)) return;
    const float* l = j == 0 ? p_logits + (size_t)row * n : q_logits + ((size_t)row * m + (j - 1)) * n;
    float z[E];
    load_row<E>(l, nullptr, 0.f, inv_t, nullptr, n, z);
    WarpStat st;
    Threshold t;
    const int Kc = select_list<E>(z, n, top_k, fs, L, t, st);
    int idx[kLH];
    double w[kLH];
    list_weights(L, Kc, st.zmax, t, idx, w);
    st.total = sum1(sum3(w), fs.s.sum);
    if (threadIdx.x == 0) stats[(size_t)row * (m + 1) + j] = st;
}

template <int E>
__global__ __launch_bounds__(NT) void multi_verify_walk_kernel(const float* p_logits, const float* q_logits,
                                                               const int32_t* cand, const float* u_acc,
                                                               const float* u_final, const int32_t* m_rows, int m,
                                                               int n, float inv_t, const WarpStat* stats, int32_t* out_index,
                                                               int32_t* out_token, double* out_resid) {
    __shared__ Slots sl;
    __shared__ Shared sh;
    __shared__ CompactList L;
    __shared__ WalkShared ws;
    const int row = blockIdx.x, th = (int)threadIdx.x;
    const int mr = row_candidates(m_rows, row, m);
    const WarpStat ps = stats[(size_t)row * (m + 1)];
    if (threadIdx.x == 0) { ws.pick = 0.0; sl.pick = 0x7FFFFFFF; }
    int idx[kLH], Kp;
    double w[kLH];
    float z[E];
    load_row<E>(p_logits + (size_t)row * n, nullptr, 0.f, inv_t, nullptr, n, z);
    const Threshold t = {key_to_float(ps.tau), ps.tie_cut};
    unsigned hi[E], lim = 1u;
    if (ps.onehot < -1) {   // the list the selection had: everything from the threshold's bin up
        float gmin = INFINITY;
#pragma unroll
        for (int e = 0; e < E; ++e) gmin = fminf(gmin, z[e]);
        gmin = -block_max_f(-gmin, sh);
        linear_bins<E>(z, gmin, ps.zmax, hi);
        lim = (unsigned)(-2 - ps.onehot);
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) hi[e] = keeps(t, z[e], entry<E>(e, th)) ? 1u : 0u;
    }
    count_entries<E>(hi, lim, sl);
    __syncthreads();
    Kp = place_entries<E>(hi, lim, z, n, L, sl, th);
    __syncthreads();
    list_weights(L, Kp, ps.zmax, t, idx, w);
#pragma unroll
    for (int h = 0; h < kLH; ++h) w[h] /= ps.total;
    int acc = mr, tok = -1;
    for (int i = 0; i < mr; ++i) {
        const WarpStat qs = stats[(size_t)row * (m + 1) + 1 + i];
        const int s = cand[(size_t)row * m + i];
        if (walk_step(idx, w, qs, q_logits + ((size_t)row * m + i) * n, inv_t, s, n, u_acc[(size_t)row * m + i], i & 1, ws,
                      out_resid ? &out_resid[(size_t)row * m + i] : nullptr)) {
            acc = i;
            tok = s;
            break;
        }
    }
    walk_finish(idx, w, Kp, acc, mr, tok, u_final[row], row, m, sl, sh, out_index, out_token, out_resid);
}

// The same with every entry of the target kept, for rows that do not take the list form (top-k beyond
// kTopCap, or all entries).  The running target lives in LDS (entry e of thread t at [e][t], read and written by
// its owner only): as E more fp64 values in registers beside the selection's and the proposal's it spilled (326
// registers at E = 16).  16384 entries, two candidates, top-k 16384 / 2500: 86.5 / 97.7 us with the target in
// registers, 58.3 / 61.6 us here.
template <int E>
__global__ __launch_bounds__(NT) void multi_verify_kernel(const float* p_logits, const float* q_logits,
                                                          const int32_t* cand, const float* u_acc,
                                                          const float* u_final, const int32_t* m_rows, int m, int n,
                                                          float inv_t, int top_k, int32_t* out_index,
                                                          int32_t* out_token, double* out_resid) {
    __shared__ FastShared fs;
    __shared__ double pick[2];
    __shared__ double target[E][NT];
    const int row = blockIdx.x;
    const int mr = row_candidates(m_rows, row, m);
    int acc = mr, tok = -1;
    for (int i = -1; i < mr; ++i) {   // i = -1: the target row (one call site of the selection, see multi_verify_list_kernel)
        const int th = this_thread();
        if (threadIdx.x == 0) {   // a candidate outside the slice has no owner: p = 0, q = 1 rejects it
            pick[0] = 0.0;
            pick[1] = 1.0;
        }
        float z[E];
        load_row<E>(i < 0 ? p_logits + (size_t)row * n : q_logits + ((size_t)row * m + i) * n, nullptr, 0.f, inv_t, nullptr, n, z, th);
        double q[E];
        const WarpStat qs = dense_row<E>(z, n, top_k, 0, fs, q, th);
        __syncthreads();   // the sum's words are used again below; pick[] is initialised
        if (i < 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                target[e][th] = q[e] / qs.total;
                __builtin_amdgcn_sched_barrier(0);   // one division at a time, here and below: interleaved ones spill
            }
            continue;
        }
        const int s = cand[(size_t)row * m + i];
        double rs = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            q[e] /= qs.total;
            const double p = target[e][th];
            if (entry<E>(e, th) == s) {   // the owner of the candidate's entry publishes p^(i)(s), q_i(s)
                pick[0] = p;
                pick[1] = q[e];
            }
            const double r = p - q[e];
            q[e] = r > 0.0 ? r : 0.0;   // q now holds max(0, p^(i) - q_i)
            rs += q[e];
            __builtin_amdgcn_sched_barrier(0);
        }
        const double R = sum1(rs, fs.s.scan[0][0]);   // its barrier also publishes pick[]
        const double pd = pick[0], qd = pick[1];
        if (out_resid && threadIdx.x == 0) out_resid[(size_t)row * m + i] = R;
        const bool accept = (double)u_acc[(size_t)row * m + i] * qd < pd;
        __syncthreads();   // pick[] is rewritten by the next candidate
        if (accept) {
            acc = i;
            tok = s;
            break;
        }
        if (R > 0.0) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                target[e][th] = q[e] / R;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    if (acc == mr) {
        double p[E], sp = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            p[e] = target[e][threadIdx.x];
            sp += p[e];
        }
        __syncthreads();
        const double total = sum1(sp, fs.s.sum);
        tok = inv_cdf_row<E>(p, total, u_final[row], fs.s, fs.sh);
    }
    if (threadIdx.x == 0) {
        out_index[row] = acc;
        out_token[row] = tok;
        if (out_resid)
            for (int i = (acc == mr ? mr : acc + 1); i < m; ++i) out_resid[(size_t)row * m + i] = -1.0;   // steps not evaluated
    }
}

// The same where every row is the point mass on its arg-max (greedy): the target stays the point mass it
// is - a proposal's point mass elsewhere leaves max(0, p - q) = p with mass 1, the same one leaves nothing -, so a
// row costs its arg-max and the recursion is a comparison of indices.  16384 entries, two candidates: 93.2 us as fp64
// weights per entry, 11.7 us here.
template <int E>
__global__ __launch_bounds__(NT) void multi_verify_greedy_kernel(const float* p_logits, const float* q_logits, const int32_t* cand,
                                                                 const float* u_acc, const int32_t* m_rows, int m, int n, float inv_t,
                                                                 int32_t* out_index, int32_t* out_token, double* out_resid) {
    __shared__ unsigned long long key[2][NW];   // alternating: a row's exchange may be read while the next one is written
    const int row = blockIdx.x;
    const int mr = row_candidates(m_rows, row, m);
    int acc = mr, best = 0;
    for (int i = -1; i < mr; ++i) {
        const int th = this_thread();
        float z[E];
        load_row<E>(i < 0 ? p_logits + (size_t)row * n : q_logits + ((size_t)row * m + i) * n, nullptr, 0.f, inv_t, nullptr, n, z, th);
        const int top = arg_max<E>(z, n, key[i & 1], th);
        if (i < 0) {
            best = top;
            continue;
        }
        const int s = cand[(size_t)row * m + i];
        // a candidate outside the slice: p = 0, q = 1 rejects it
        const double pd = s == best ? 1.0 : 0.0, qd = (s == top || (unsigned)s >= (unsigned)n) ? 1.0 : 0.0;
        if (out_resid && threadIdx.x == 0) out_resid[(size_t)row * m + i] = top == best ? 0.0 : 1.0;
        if ((double)u_acc[(size_t)row * m + i] * qd < pd) {
            acc = i;
            break;
        }
    }
    if (threadIdx.x == 0) {
        out_index[row] = acc;
        out_token[row] = acc < mr ? cand[(size_t)row * m + acc] : best;
        if (out_resid)
            for (int i = (acc == mr ? mr : acc + 1); i < m; ++i) out_resid[(size_t)row * m + i] = -1.0;   // steps not evaluated
    }
}

// One draw per row from the row's warped distribution (inverse CDF over ascending index): the
// candidates of a sampling pool.  Rows whose entry of `skip` is negative give -1.
template <int E>
__global__ __launch_bounds__(NT) void sample_rows_kernel(const float* logits, const int32_t* skip, const float* u, int n,
                                                         float inv_t, int top_k, int greedy, int32_t* out_token) {
    __shared__ FastShared fs;
    __shared__ CompactList L;
    const int row = blockIdx.x;
    if (skip && skip[row] < 0) {
        if (threadIdx.x == 0) out_token[row] = -1;
        return;
    }
    float z[E];
    load_row<E>(logits + (size_t)row * n, nullptr, 0.f, inv_t, nullptr, n, z);
    const float ur = u[row];
    int drawn = 0;
    (void)warp_and_draw<E>(z, n, top_k, greedy, fs, L, &ur, &drawn);
    if (threadIdx.x == 0) out_token[row] = drawn;
}

}  // namespace

void launch_plan(hawk_ctx* c, int k) {
    plan_kernel<<<1, 64 * ((c->B + 63) / 64), 0, c->stream>>>(wsp<int32_t>(c, c->off.n), wsp<int32_t>(c, c->off.k_eff),
                                                            wsp<int32_t>(c, c->off.draft),
                                                            wsp<int32_t>(c, c->off.step),
                                                            wsp<unsigned long long>(c, c->off.counters), c->B, c->N,
                                                            k, c->kmax + 1);
}

// Entries per thread of the register-resident kernels for this vocabulary slice (0: too large).
static int entries_per_thread(int n) { return n <= 4 * NT ? 4 : (n <= 8 * NT ? 8 : (n <= 16 * NT ? 16 : 0)); }
static int fast_e(const hawk_ctx* c) { return entries_per_thread(c->Vs); }

void launch_first_token(hawk_ctx* c, const UniformSrc& us) {
    if (fast_e(c)) {
        auto kern = fast_e(c) == 4 ? first_token_fast<4> : (fast_e(c) == 8 ? first_token_fast<8> : first_token_fast<16>);
        kern<<<c->B, NT, 0, c->stream>>>(wsp<float>(c, c->off.logit_s), wsp<float>(c, c->off.logit_b),
                                         wsp<int32_t>(c, c->off.grid), wsp<int32_t>(c, c->off.n), samp_params(c), us);
        return;
    }
    first_token_kernel<<<c->B, NT, 0, c->stream>>>(wsp<float>(c, c->off.logit_s), wsp<float>(c, c->off.logit_b),
                                                   wsp<int32_t>(c, c->off.grid), wsp<int32_t>(c, c->off.n),
                                                   samp_params(c), us);
}

void launch_draft_sample(hawk_ctx* c, int i, int k, const UniformSrc& us, const DraftMode& dm) {
    const ForcedSrc fs = forced_src(c, k, dm);
    if (fast_e(c)) {
        auto kern = fast_e(c) == 4 ? draft_sample_fast<4> : (fast_e(c) == 8 ? draft_sample_fast<8> : draft_sample_fast<16>);
        kern<<<c->B, NT, 0, c->stream>>>(wsp<float>(c, c->off.dlogit_s), wsp<float>(c, c->off.dlogit_b),
                                         wsp<int32_t>(c, c->off.n), wsp<int32_t>(c, c->off.k_eff),
                                         wsp<int32_t>(c, c->off.draft), wsp<WarpStat>(c, c->off.qstat), i, k,
                                         samp_params(c), us, fs);
        return;
    }
    draft_sample_kernel<<<c->B, NT, 0, c->stream>>>(wsp<float>(c, c->off.dlogit_s), wsp<float>(c, c->off.dlogit_b),
                                                    wsp<int32_t>(c, c->off.n), wsp<int32_t>(c, c->off.k_eff),
                                                    wsp<int32_t>(c, c->off.draft), wsp<WarpStat>(c, c->off.qstat), i,
                                                    k, samp_params(c), us, fs);
}

void launch_verify_stats(hawk_ctx* c, int k) {
    if (fast_e(c)) {
        auto kern = fast_e(c) == 4 ? verify_stats_fast<4> : (fast_e(c) == 8 ? verify_stats_fast<8> : verify_stats_fast<16>);
        kern<<<dim3(k + 1, c->B), NT, 0, c->stream>>>(wsp<float>(c, c->off.logit_s), wsp<float>(c, c->off.logit_b),
                                                      wsp<int32_t>(c, c->off.k_eff), wsp<WarpStat>(c, c->off.pstat),
                                                      wsp<int32_t>(c, c->off.llen), wsp<int32_t>(c, c->off.lidx), wsp<double>(c, c->off.lw), k,
                                                      samp_params(c));
        return;
    }
    verify_stats_kernel<<<dim3(k + 1, c->B), NT, 0, c->stream>>>(
        wsp<float>(c, c->off.logit_s), wsp<float>(c, c->off.logit_b), wsp<int32_t>(c, c->off.k_eff),
        wsp<WarpStat>(c, c->off.pstat), k, samp_params(c));
}

void launch_accept_commit(hawk_ctx* c, int k, const UniformSrc& us) {
    if (fast_e(c)) {
        auto kern = fast_e(c) == 4 ? accept_commit_fast<4> : (fast_e(c) == 8 ? accept_commit_fast<8> : accept_commit_fast<16>);
        kern<<<c->B, NT, 0, c->stream>>>(
            wsp<float>(c, c->off.logit_b), wsp<float>(c, c->off.dlogit_b), wsp<WarpStat>(c, c->off.pstat),
            wsp<WarpStat>(c, c->off.qstat), wsp<int32_t>(c, c->off.llen), wsp<int32_t>(c, c->off.lidx), wsp<double>(c, c->off.lw),
            wsp<int32_t>(c, c->off.k_eff), wsp<int32_t>(c, c->off.draft), wsp<int32_t>(c, c->off.grid), wsp<int32_t>(c, c->off.n), wsp<uint32_t>(c, c->off.x),
            wsp<uint32_t>(c, c->off.hprev), (int)(c->d * c->asz / 4), wsp<int32_t>(c, c->off.out_na),
            wsp<int32_t>(c, c->off.out_tok), wsp<unsigned long long>(c, c->off.counters), k, c->S, samp_params(c), us);
        return;
    }
    accept_commit_kernel<<<c->B, NT, 0, c->stream>>>(
        wsp<float>(c, c->off.logit_b), wsp<float>(c, c->off.dlogit_b), wsp<WarpStat>(c, c->off.pstat),
        wsp<WarpStat>(c, c->off.qstat), wsp<int32_t>(c, c->off.k_eff), wsp<int32_t>(c, c->off.draft),
        wsp<int32_t>(c, c->off.grid), wsp<int32_t>(c, c->off.n), wsp<uint32_t>(c, c->off.x),
        wsp<uint32_t>(c, c->off.hprev), (int)(c->d * c->asz / 4), wsp<int32_t>(c, c->off.out_na),
        wsp<int32_t>(c, c->off.out_tok), wsp<unsigned long long>(c, c->off.counters), k, c->S, samp_params(c), us);
}

void launch_force_setup(hawk_ctx* c, int cnt) {
    force_setup_kernel<<<1, 64 * ((c->B + 63) / 64), 0, c->stream>>>(
        wsp<int32_t>(c, c->off.u_draft), wsp<int32_t>(c, c->off.forced), wsp<int32_t>(c, c->off.n),
        wsp<int32_t>(c, c->off.k_eff), wsp<int32_t>(c, c->off.draft), c->B, cnt, c->kmax + 1);
}

void launch_force_commit(hawk_ctx* c, int cnt) {
    force_commit_kernel<<<c->B, 256, 0, c->stream>>>(wsp<int32_t>(c, c->off.forced), wsp<int32_t>(c, c->off.grid),
                                                     wsp<int32_t>(c, c->off.n), wsp<uint32_t>(c, c->off.x),
                                                     wsp<uint32_t>(c, c->off.hprev), (int)(c->d * c->asz / 4), c->B,
                                                     c->N, cnt, c->S);
}

int launch_sample_rows(const float* logits, const int32_t* skip, const float* u, int rows, int n, float temperature,
                       int top_k, int32_t* out_token, hipStream_t stream) {
    const int E = entries_per_thread(n);
    if (!E) return HAWK_EINVAL;
    const int greedy = (temperature == 0.0f || top_k == 1) ? 1 : 0;
    const float inv_t = greedy ? 1.0f : 1.0f / temperature;
    const int tk = top_k < n ? top_k : n;
    auto kern = E == 4 ? sample_rows_kernel<4> : (E == 8 ? sample_rows_kernel<8> : sample_rows_kernel<16>);
    kern<<<rows, NT, 0, stream>>>(logits, skip, u, n, inv_t, tk, greedy, out_token);
    return hipGetLastError() == hipSuccess ? HAWK_OK : HAWK_EDEVICE;
}

size_t multi_verify_workspace_bytes(int rows, int m) { return (size_t)rows * (m + 1) * sizeof(WarpStat); }
size_t list_len_bytes(size_t rows) { return rows * sizeof(int32_t); }
size_t list_idx_bytes(size_t rows) { return rows * kCap * sizeof(int32_t); }
size_t list_w_bytes(size_t rows) { return rows * kCap * sizeof(double); }

int launch_multi_verify(const float* p_logits, const float* q_logits, const int32_t* cand, const float* u_acc,
                        const float* u_final, const int32_t* m_rows, int rows, int m, int n, float temperature, int top_k,
                        int32_t* out_index, int32_t* out_token, double* out_resid, void* workspace,
                        size_t workspace_bytes, hipStream_t stream) {
    const int E = entries_per_thread(n);
    if (!E) return HAWK_EINVAL;
    const int greedy = (temperature == 0.0f || top_k == 1) ? 1 : 0;
    const float inv_t = greedy ? 1.0f : 1.0f / temperature;
    const int tk = top_k < n ? top_k : n;
    if (use_list(tk, n, greedy) && workspace && workspace_bytes >= multi_verify_workspace_bytes(rows, m)) {
        WarpStat* stats = static_cast<WarpStat*>(workspace);
        auto k1 = E == 4 ? multi_row_stats_kernel<4> : (E == 8 ? multi_row_stats_kernel<8> : multi_row_stats_kernel<16>);
        auto k2 = E == 4 ? multi_verify_walk_kernel<4> : (E == 8 ? multi_verify_walk_kernel<8> : multi_verify_walk_kernel<16>);
        k1<<<dim3(m + 1, rows), NT, 0, stream>>>(p_logits, q_logits, m_rows, m, n, inv_t, tk, stats);
        k2<<<rows, NT, 0, stream>>>(p_logits, q_logits, cand, u_acc, u_final, m_rows, m, n, inv_t, stats, out_index,
                                    out_token, out_resid);
    } else if (use_list(tk, n, greedy)) {
        auto kern = E == 4 ? multi_verify_list_kernel<4> : (E == 8 ? multi_verify_list_kernel<8> : multi_verify_list_kernel<16>);
        kern<<<rows, NT, 0, stream>>>(p_logits, q_logits, cand, u_acc, u_final, m_rows, m, n, inv_t, tk, out_index, out_token,
                                      out_resid);
    } else if (greedy) {
        auto kern = E == 4 ? multi_verify_greedy_kernel<4> : (E == 8 ? multi_verify_greedy_kernel<8> : multi_verify_greedy_kernel<16>);
        kern<<<rows, NT, 0, stream>>>(p_logits, q_logits, cand, u_acc, m_rows, m, n, inv_t, out_index, out_token, out_resid);
    } else {
        auto kern = E == 4 ? multi_verify_kernel<4> : (E == 8 ? multi_verify_kernel<8> : multi_verify_kernel<16>);
        kern<<<rows, NT, 0, stream>>>(p_logits, q_logits, cand, u_acc, u_final, m_rows, m, n, inv_t, tk, out_index, out_token,
                                      out_resid);
    }
    return hipGetLastError() == hipSuccess ? HAWK_OK : HAWK_EDEVICE;
}

// ---- hawk_multi_verify for callers that cannot allocate: the rows' statistics live in a fixed array in
// device memory instead of a caller-provided workspace.  Every GPU holds its own copy of the array at
// its own address, looked up once per device; host code only ever uses that address.
constexpr int kStaticStatRows = 4096;   // logit rows (positions x (candidates + 1)) one call may have
static __device__ __align__(256) unsigned char scratch[(size_t)kStaticStatRows * sizeof(WarpStat)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU (null: not looked up yet)

int scratch_address(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return HAWK_EDEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return HAWK_EDEVICE;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return HAWK_OK;
}
}  // namespace

int launch_multi_verify_static(const float* p_logits, const float* q_logits, const int32_t* cand, const float* u_acc,
                               const float* u_final, const int32_t* m_rows, int rows, int m, int n, float temperature,
                               int top_k, int32_t* out_index, int32_t* out_token, double* out_resid, hipStream_t stream) {
    if ((long long)rows * (m + 1) > kStaticStatRows) return HAWK_ENOMEM;
    void* ws = nullptr;
    const int rc = scratch_address(&ws);
    if (rc != HAWK_OK) return rc;
    // every record the second launch reads is written by the first launch of the same call, so
    // nothing in the array has to be cleared between calls
    return launch_multi_verify(p_logits, q_logits, cand, u_acc, u_final, m_rows, rows, m, n, temperature, top_k, out_index,
                               out_token, out_resid, ws, multi_verify_workspace_bytes(rows, m), stream);
}

}  // namespace hawk
