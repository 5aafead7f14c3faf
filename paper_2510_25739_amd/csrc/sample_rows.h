// Device functions of the sampling stage: guidance, temperature / top-k warp and inverse-CDF draws of one logit row by one
// workgroup of 1024 threads.  sampling.hip's kernels and the draft chain's (chain.hip) are made of them.
//
// Decisions (which logits survive top-k, where a uniform falls in a CDF, whether a draft is
// accepted) are taken on fp32 logits with fp64 weights exp(z - zmax) and fp64 sums, so
// that they do not depend on the order of summation beyond the last bits of an fp64.
// One workgroup of 1024 threads handles one logit row.  In the generic form thread t owns the contiguous
// index segment [t*E, (t+1)*E), which makes every scan an in-order prefix over token indices; the
// register-resident form owns chunks of four and scans a list in index order.
// Reductions use cross-lane moves, then one LDS exchange across the 16 waves.
#pragma once

#include "hawk_internal.h"

namespace hawk {

namespace {

constexpr int NT = kSampThreads;
constexpr int NW = NT / 64;

struct Shared {
    unsigned hist[256];
    double dred[NW];
    int ired[NW];
    float fred[NW];
    // broadcast slots
    unsigned b_prefix, b_remaining, b_count_eq;
    int b_int;
};

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__device__ __forceinline__ float gen_uniform(uint64_t seed, uint32_t seq, uint32_t step, uint32_t slot) {
    uint64_t ctr = ((uint64_t)seq << 44) | ((uint64_t)step << 8) | (uint64_t)(slot & 0xFFu);
    uint64_t z = mix64(seed + 0x9E3779B97F4A7C15ull);
    z = mix64(z + 0x9E3779B97F4A7C15ull * (ctr + 1));
    return (float)(z >> 40) * (1.0f / 16777216.0f);
}
__device__ __forceinline__ float pick_uniform(const UniformSrc& u, const float* table, int idx, int b, int slot) {
    return u.use_gen ? gen_uniform(u.seed, (uint32_t)b, (uint32_t)u.step[0], (uint32_t)slot) : table[idx];
}

// Order-preserving key of a float (larger value <=> larger key); -0 and +0 share a key.
__device__ __forceinline__ unsigned fkey(float z) {
    unsigned u = __float_as_uint(z);
    if ((u << 1) == 0u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Cross-lane moves inside the VALU (DPP) instead of LDS-crossbar shuffles: within a row of 16
// lanes by quad permutes and mirrors, across the four rows by lane broadcasts.
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) { return __builtin_bit_cast(float, dpp_i<CTRL>(__builtin_bit_cast(int, v))); }
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)dpp_i<CTRL>((int)(unsigned)b), hi = (unsigned)dpp_i<CTRL>((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ float lane_f(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double lane_d(double v, int l) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// 0xB1 = quad_perm [1,0,3,2], 0x4E = quad_perm [2,3,0,1], 0x141 = row_half_mirror, 0x140 = row_mirror:
// after the four steps every lane of a row holds the row's result.
#define ROW_ALLREDUCE(v, OP, DPP)         \
    v = OP(v, DPP<0xB1>(v));              \
    v = OP(v, DPP<0x4E>(v));              \
    v = OP(v, DPP<0x141>(v));             \
    v = OP(v, DPP<0x140>(v));
__device__ __forceinline__ double addd(double a, double b) { return a + b; }
__device__ __forceinline__ int mini(int a, int b) { return min(a, b); }
__device__ __forceinline__ int maxi(int a, int b) { return max(a, b); }

__device__ __forceinline__ double wave_sum_d(double v) {
    ROW_ALLREDUCE(v, addd, dpp_d)
    return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}
__device__ __forceinline__ float wave_max_f(float v) {
    ROW_ALLREDUCE(v, fmaxf, dpp_f)
    return fmaxf(fmaxf(lane_f(v, 0), lane_f(v, 16)), fmaxf(lane_f(v, 32), lane_f(v, 48)));
}
__device__ __forceinline__ float wave_min_f(float v) {
    ROW_ALLREDUCE(v, fminf, dpp_f)
    return fminf(fminf(lane_f(v, 0), lane_f(v, 16)), fminf(lane_f(v, 32), lane_f(v, 48)));
}
__device__ __forceinline__ float addf(float a, float b) { return a + b; }
__device__ __forceinline__ float wave_sum_f(float v) {
    ROW_ALLREDUCE(v, addf, dpp_f)
    return (lane_f(v, 0) + lane_f(v, 16)) + (lane_f(v, 32) + lane_f(v, 48));
}
__device__ __forceinline__ int wave_min_i(int v) {
    ROW_ALLREDUCE(v, mini, dpp_i)
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
__device__ __forceinline__ int wave_max_i(int v) {
    ROW_ALLREDUCE(v, maxi, dpp_i)
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
// Inclusive prefix sums over the lanes of the wave, in lane order: row_shr 1, 2, 4, 8 with zero
// fill inside each row of 16 (0x111, 0x112, 0x114, 0x118), then the totals of the rows before.
__device__ __forceinline__ double wave_incl_scan_d(double v) {
    v += dpp_d<0x111>(v);
    v += dpp_d<0x112>(v);
    v += dpp_d<0x114>(v);
    v += dpp_d<0x118>(v);
    const double r0 = lane_d(v, 15), r1 = lane_d(v, 31), r2 = lane_d(v, 47);
    const int row = (threadIdx.x & 63) >> 4;
    return v + (row == 0 ? 0.0 : row == 1 ? r0 : row == 2 ? r0 + r1 : (r0 + r1) + r2);
}
__device__ __forceinline__ int wave_incl_scan_i(int v) {
    v += dpp_i<0x111>(v);
    v += dpp_i<0x112>(v);
    v += dpp_i<0x114>(v);
    v += dpp_i<0x118>(v);
    const int r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31), r2 = __builtin_amdgcn_readlane(v, 47);
    const int row = (threadIdx.x & 63) >> 4;
    return v + (row == 0 ? 0 : row == 1 ? r0 : row == 2 ? r0 + r1 : r0 + r1 + r2);
}

// All block primitives below return the same value to every thread and may be called
// back to back (each starts with a barrier that protects the exchange buffer).
__device__ double block_sum_d(double v, Shared& sh) {
    v = wave_sum_d(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.dred[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += sh.dred[w];
    return t;
}
__device__ float block_max_f(float v, Shared& sh) {
    v = wave_max_f(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.fred[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = sh.fred[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) t = fmaxf(t, sh.fred[w]);
    return t;
}
__device__ int block_min_i(int v, Shared& sh) {
    v = wave_min_i(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.ired[threadIdx.x >> 6] = v;
    __syncthreads();
    int t = sh.ired[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) t = min(t, sh.ired[w]);
    return t;
}
__device__ int block_max_i(int v, Shared& sh) {
    v = wave_max_i(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.ired[threadIdx.x >> 6] = v;
    __syncthreads();
    int t = sh.ired[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) t = max(t, sh.ired[w]);
    return t;
}
// Exclusive prefix sums over the threads of the block, in thread order.
__device__ double block_excl_scan_d(double v, Shared& sh) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double inc = wave_incl_scan_d(v);
    __syncthreads();
    if (lane == 63) sh.dred[wave] = inc;
    __syncthreads();
    double base = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) base += w < wave ? sh.dred[w] : 0.0;
    return base + (inc - v);
}
__device__ int block_excl_scan_i(int v, Shared& sh) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int inc = wave_incl_scan_i(v);
    __syncthreads();
    if (lane == 63) sh.ired[wave] = inc;
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) base += w < wave ? sh.ired[w] : 0;
    return base + (inc - v);
}

struct Seg { int j0, j1; };
__device__ __forceinline__ Seg my_segment(int n) {
    int e = (n + NT - 1) / NT;
    Seg s;
    s.j0 = min(n, (int)threadIdx.x * e);
    s.j1 = min(n, s.j0 + e);
    return s;
}

// Guided logits of one row into `out` (also the row every later pass reads).
__device__ void combine_row(const float* lc, const float* lu, float scale, float* out, int n) {
    for (int j = threadIdx.x; j < n; j += NT) out[j] = lu ? fmaf(scale, lc[j] - lu[j], lu[j]) : lc[j];
    __syncthreads();
}

__device__ __forceinline__ bool kept(const WarpStat& st, float z, int j) {
    unsigned k = fkey(z);
    return k > st.tau || (k == st.tau && j <= st.tie_cut);
}
__device__ __forceinline__ double weight_of(const WarpStat& st, const float* l, float inv_t, int j) {
    if (st.onehot >= 0) return j == st.onehot ? 1.0 : 0.0;
    float z = l[j] * inv_t;
    return kept(st, z, j) ? exp((double)z - (double)st.zmax) : 0.0;
}

// Temperature / top-k warp of the row l[0..n): arg-max point mass if greedy, otherwise
// z = l * inv_t, keep the top_k largest z (equal values: lower index first).
__device__ WarpStat warp_stats(const float* l, int n, float inv_t, int top_k, int greedy, Shared& sh) {
    const Seg sg = my_segment(n);
    WarpStat st;
    st.total = 1.0; st.zmax = 0.f; st.tau = 0u; st.tie_cut = 0x7FFFFFFF; st.onehot = -1;
    if (greedy) {
        float best = -INFINITY;
        for (int j = sg.j0; j < sg.j1; ++j) best = fmaxf(best, l[j]);
        float gmax = block_max_f(best, sh);
        int idx = 0x7FFFFFFF;
        for (int j = sg.j0; j < sg.j1; ++j)
            if (l[j] == gmax) { idx = j; break; }
        st.onehot = block_min_i(idx, sh);
        return st;
    }
    const int K = min(top_k, n);
    if (K < n) {
        unsigned prefix = 0u, mask = 0u, remaining = (unsigned)K, count_eq = 0u;
        for (int shift = 24; shift >= 0; shift -= 8) {
            __syncthreads();
            if (threadIdx.x < 256) sh.hist[threadIdx.x] = 0u;
            __syncthreads();
            for (int j = sg.j0; j < sg.j1; ++j) {
                unsigned key = fkey(l[j] * inv_t);
                if ((key & mask) == prefix) atomicAdd(&sh.hist[(key >> shift) & 255u], 1u);
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                unsigned cum = 0u;
                for (int bin = 255; bin >= 0; --bin) {
                    unsigned h = sh.hist[bin];
                    if (cum + h >= remaining) {
                        sh.b_prefix = prefix | ((unsigned)bin << shift);
                        sh.b_remaining = remaining - cum;
                        sh.b_count_eq = h;
                        break;
                    }
                    cum += h;
                }
            }
            __syncthreads();
            prefix = sh.b_prefix;
            remaining = sh.b_remaining;
            count_eq = sh.b_count_eq;
            mask |= 255u << shift;
        }
        st.tau = prefix;
        if (remaining < count_eq) {  // keep only the first `remaining` entries equal to tau
            int c = 0;
            for (int j = sg.j0; j < sg.j1; ++j) c += fkey(l[j] * inv_t) == prefix;
            int before = block_excl_scan_i(c, sh);
            __syncthreads();
            if (before < (int)remaining && before + c >= (int)remaining) {
                int seen = before;
                for (int j = sg.j0; j < sg.j1; ++j)
                    if (fkey(l[j] * inv_t) == prefix && ++seen == (int)remaining) { sh.b_int = j; break; }
            }
            __syncthreads();
            st.tie_cut = sh.b_int;
        }
    }
    float zm = -INFINITY;
    for (int j = sg.j0; j < sg.j1; ++j) zm = fmaxf(zm, l[j] * inv_t);
    st.zmax = block_max_f(zm, sh);
    double s = 0.0;
    for (int j = sg.j0; j < sg.j1; ++j) s += weight_of(st, l, inv_t, j);
    st.total = block_sum_d(s, sh);
    return st;
}

// Inverse-CDF draw over ascending index from weights w(j) >= 0 given by a functor:
// first j whose running sum exceeds u * total, else the last j with positive weight.
template <class WF>
__device__ int inv_cdf(WF w, int n, double total, float u, Shared& sh) {
    const Seg sg = my_segment(n);
    double s = 0.0;
    for (int j = sg.j0; j < sg.j1; ++j) s += w(j);
    double c = block_excl_scan_d(s, sh);
    const double target = (double)u * total;
    int cand = 0x7FFFFFFF, last = -1;
    for (int j = sg.j0; j < sg.j1; ++j) {
        double wj = w(j);
        if (wj > 0.0) {
            c += wj;
            last = j;
            if (c > target) { cand = j; break; }
        }
    }
    cand = block_min_i(cand, sh);
    if (cand != 0x7FFFFFFF) return cand;
    return block_max_i(last, sh);
}

// ---------------------------------------------------------------------------- register-resident rows
//
// Fast variants for rows of at most 1024 * E entries: a thread keeps its E scaled logits in
// registers for the whole kernel (one coalesced read of the row).  Same decisions, to the bit, as
// the generic functions above.
//
// What bounds them is a chain of about a dozen phases on one compute unit, 0.35 to 1.3 us each, which wait for each other at
// barriers: with two thirds of the entries kept out of the histogram a draw is not faster.  What bounded them before was
// its instruction issue: a wave's vector instruction takes
// four cycles and a SIMD has four of the block's sixteen waves, so one instruction per entry of a
// 16384-entry row is 256 cycles (0.1 us), and work that every wave repeats costs four times as much as
// work of one wave.  So:
//   - entry e of thread t is index (e / 4) * 4096 + 4 t + e % 4 (E / 4 chunks of 16 KB): a wave's
//     request is one contiguous kilobyte;
//   - places past the end of the row hold NaN, which no comparison of values keeps, so that no entry needs a
//     bounds check.  They share bin 0 with the smallest entries: find_bin takes them off its count, and a list
//     cut at bin 0 ends at the row's n-th entry (place_entries; they come last in index order);
//   - an entry's bin of the first, linear cut of the value range is computed once and kept; the entries
//     at or above the threshold's bin go to a list in LDS with one comparison each, their places counted
//     from lane masks; which of the few entries of the threshold's bin itself survive is settled meanwhile,
//     and those that do not get weight zero;
//   - every block-wide exchange has LDS words of its own and costs one barrier (behind the writes).
// Draw from a 16384-entry row at top-k 1000 (sample_rows_kernel, kernel trace): 19.3 us with bounds checks, per-thread
// segments and per-wave histograms, 9.4 us like this.
// A word of Slots may be written again once every thread has passed a barrier after reading it.

constexpr int kBins = NT;    // bins of the first, linear cut of the value range
constexpr float kMinRange = 1e-30f;   // narrower rows take the radix select: 1024 / range must be finite, or bins are not
constexpr int kCand = 256;   // entries of the threshold's bin that are ranked directly
constexpr int kTopCap = 2048;               // largest top-k that takes the list form
constexpr int kCap = kTopCap + kCand;       // entries of a list: the kept ones and the rest of the threshold's bin
constexpr int kLH = (kCap + NT - 1) / NT;   // list entries per thread: t, NT + t, 2 NT + t
static_assert(NW == 16, "per-wave values are folded by one row of 16 lanes");

struct alignas(16) Slots {
    float2 mm[NW];           // minimum / maximum of a wave
    unsigned long long key[NW];
    double sum[NW];
    double scan[2][4][NW];
    int cnt[4 * NW];         // [chunk][wave]
    int pick;
};
struct FastShared {
    unsigned hist[kBins];
    float cand_z[kCand];
    int cand_idx[kCand];
    unsigned cand_rank[kCand];   // candidates that come before each one (see rank_candidates)
    unsigned cand_n;
    int bin, want, count;        // the threshold's bin, how many of its entries are kept, how many it has
    float tau_z;
    int tie_cut;
    Slots s;
    Shared sh;
};
// The entries a top-k row keeps: z > tz, or z == tz up to index cut.
struct Threshold { float tz; int cut; };
__device__ __forceinline__ bool keeps(const Threshold& t, float z, int j) { return z > t.tz || (z == t.tz && j <= t.cut); }
__device__ __forceinline__ float key_to_float(unsigned k) { return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k); }

// Index of entry e of thread t.  The functions below take t from their caller: a kernel that runs them in a loop
// over rows passes a value of that iteration (this_thread), or the compiler keeps every entry's address and bounds
// check in registers across the loop, and spills.
template <int E> __device__ __forceinline__ int entry(int e, int t) { return (e >> 2) * (4 * NT) + t * 4 + (e & 3); }
__device__ __forceinline__ int this_thread() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

// Sum over the block of one double per thread.  One barrier.
__device__ __forceinline__ double sum1(double v, double (&slot)[NW]) {
    v = wave_sum_d(v);
    if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = slot[threadIdx.x & 15];
    ROW_ALLREDUCE(t, addd, dpp_d)
    return t;
}
__device__ __forceinline__ unsigned long long maxu64(unsigned long long a, unsigned long long b) { return a > b ? a : b; }
template <int CTRL> __device__ __forceinline__ unsigned long long dpp_u64(unsigned long long v) {
    return ((unsigned long long)(unsigned)dpp_i<CTRL>((int)(v >> 32)) << 32) | (unsigned)dpp_i<CTRL>((int)(unsigned)v);
}
// Largest of one 64-bit key per thread.  One barrier.
__device__ __forceinline__ unsigned long long max1(unsigned long long v, unsigned long long (&slot)[NW]) {
    ROW_ALLREDUCE(v, maxu64, dpp_u64)
    const unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    unsigned long long m = 0ull;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        m = maxu64(m, ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)hi, 16 * r) << 32) |
                          (unsigned)__builtin_amdgcn_readlane((int)lo, 16 * r));
    if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = m;
    __syncthreads();
    unsigned long long t = slot[threadIdx.x & 15];
    ROW_ALLREDUCE(t, maxu64, dpp_u64)
    return t;
}
// Folds the per-wave totals in `slot`: `base` = sum of the waves before this one, returns the block's total.
__device__ __forceinline__ double wave_base_d(const double* slot, int wave, double& base) {
    double v = slot[threadIdx.x & 15];
    v += dpp_d<0x111>(v);
    v += dpp_d<0x112>(v);
    v += dpp_d<0x114>(v);
    v += dpp_d<0x118>(v);
    const double b = lane_d(v, wave > 0 ? wave - 1 : 0);
    base = wave > 0 ? b : 0.0;
    return lane_d(v, 15);
}
__device__ __forceinline__ int wave_base_i(const int* slot, int wave, int& base) {
    int v = slot[threadIdx.x & 15];
    v += dpp_i<0x111>(v);
    v += dpp_i<0x112>(v);
    v += dpp_i<0x114>(v);
    v += dpp_i<0x118>(v);
    const int b = __builtin_amdgcn_readlane(v, wave > 0 ? wave - 1 : 0);
    base = wave > 0 ? b : 0;
    return __builtin_amdgcn_readlane(v, 15);
}

// Ranks of all gathered candidates at once (fs.cand_rank[i] = candidates that come before candidate
// i - larger value first, lower index first among equals -, zeroed by the caller): the cnt x cnt
// comparisons are spread over the block - NT / cnt threads share a candidate, each compares it with a
// slice of the list and adds its count with one LDS atomic.  All threads call; ends with a barrier.
__device__ __forceinline__ void rank_candidates(FastShared& fs, unsigned cnt) {
    const unsigned per = max(1u, (unsigned)NT / cnt), len = (cnt + per - 1u) / per;
    const unsigned i = threadIdx.x % cnt, c = threadIdx.x / cnt;
    if (c < per) {
        const float mine = fs.cand_z[i];
        const int mi = fs.cand_idx[i];
        const unsigned j1 = min(cnt, (c + 1u) * len);
        unsigned part = 0u;
        for (unsigned j = c * len; j < j1; ++j) {
            const float r = fs.cand_z[j];
            part += (r > mine || (r == mine && fs.cand_idx[j] < mi)) ? 1u : 0u;
        }
        if (part) atomicAdd(&fs.cand_rank[i], part);
    }
    __syncthreads();
}

// The row's guided, scaled logits into registers (and the guided row to `out`); NaN past the end.
template <int E>
__device__ __forceinline__ void load_row(const float* lc, const float* lu, float scale, float inv_t, float* out, int n,
                                         float (&z)[E], int th = (int)threadIdx.x) {
    const float nan = __uint_as_float(0x7FC00000u);
    if ((n & 3) == 0 && ((reinterpret_cast<uintptr_t>(lc) | reinterpret_cast<uintptr_t>(lu) | reinterpret_cast<uintptr_t>(out)) & 15) == 0) {
        float4 a[E / 4], u[E / 4];
#pragma unroll
        for (int q = 0; q < E / 4; ++q) {
            const int j = entry<E>(4 * q, th);
            a[q] = make_float4(nan, nan, nan, nan);
            if (j < n) a[q] = *reinterpret_cast<const float4*>(lc + j);
            if (lu && j < n) u[q] = *reinterpret_cast<const float4*>(lu + j);
        }
#pragma unroll
        for (int q = 0; q < E / 4; ++q) {
            const int j = entry<E>(4 * q, th);
            if (lu && j < n) {
                a[q].x = fmaf(scale, a[q].x - u[q].x, u[q].x); a[q].y = fmaf(scale, a[q].y - u[q].y, u[q].y);
                a[q].z = fmaf(scale, a[q].z - u[q].z, u[q].z); a[q].w = fmaf(scale, a[q].w - u[q].w, u[q].w);
            }
            if (out && j < n) *reinterpret_cast<float4*>(out + j) = a[q];
            z[4 * q] = a[q].x * inv_t; z[4 * q + 1] = a[q].y * inv_t; z[4 * q + 2] = a[q].z * inv_t; z[4 * q + 3] = a[q].w * inv_t;
        }
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = entry<E>(e, th);
            z[e] = nan;
            if (j < n) {
                const float l = lu ? fmaf(scale, lc[j] - lu[j], lu[j]) : lc[j];
                if (out) out[j] = l;
                z[e] = l * inv_t;
            }
        }
    }
}

// Exact radix select on the order-preserving keys, for rows the linear cut does not thin out (ties,
// odd distributions, infinite logits): the value of the K-th largest entry and up to which index entries
// equal to it are kept (fs.tau_z, fs.tie_cut; ends with a barrier).
template <int E>
__device__ __forceinline__ void radix_select(const float (&z)[E], int n, int K, FastShared& fs, int th) {
    Shared& sh = fs.sh;
    const int lane = threadIdx.x & 63, wave = wave_id();
    unsigned prefix = 0u, mask = 0u, remaining = (unsigned)K, count_eq = 0u;
    for (int shift = 24; shift >= 0; shift -= 8) {
        __syncthreads();
        if (threadIdx.x < 256) fs.hist[threadIdx.x] = 0u;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const unsigned k = fkey(z[e]);
            if (entry<E>(e, th) < n && (k & mask) == prefix) atomicAdd(&fs.hist[(k >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (wave == 0) {  // lane owns bins 4*lane .. 4*lane+3; suffix sums from the top bin down
            const unsigned cs[4] = {fs.hist[lane * 4], fs.hist[lane * 4 + 1], fs.hist[lane * 4 + 2], fs.hist[lane * 4 + 3]};
            const unsigned own = cs[0] + cs[1] + cs[2] + cs[3];
            const unsigned inc = (unsigned)wave_incl_scan_i((int)own);
            unsigned cum = (unsigned)__builtin_amdgcn_readlane((int)inc, 63) - inc;   // entries in higher lanes' bins
#pragma unroll
            for (int q = 3; q >= 0; --q) {
                if (cum < remaining && cum + cs[q] >= remaining) {   // exactly one lane and bin
                    sh.b_prefix = prefix | ((unsigned)(lane * 4 + q) << shift);
                    sh.b_remaining = remaining - cum;
                    sh.b_count_eq = cs[q];
                }
                cum += cs[q];
            }
        }
        __syncthreads();
        prefix = sh.b_prefix;
        remaining = sh.b_remaining;
        count_eq = sh.b_count_eq;
        mask |= 255u << shift;
    }
    if (threadIdx.x == 0) {
        fs.tau_z = __uint_as_float((prefix & 0x80000000u) ? (prefix ^ 0x80000000u) : ~prefix);
        fs.tie_cut = 0x7FFFFFFF;
    }
    __syncthreads();
    if (remaining < count_eq) {   // keep only the first `remaining` entries equal to the threshold, in index order
        int before = 0;           // equal entries of the chunks already passed
#pragma unroll
        for (int q = 0; q < E / 4; ++q) {
            int c = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) c += (entry<E>(4 * q + e, th) < n && fkey(z[4 * q + e]) == prefix) ? 1 : 0;
            const int at = before + block_excl_scan_i(c, sh);
            int seen = at;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (entry<E>(4 * q + e, th) < n && fkey(z[4 * q + e]) == prefix && ++seen == (int)remaining) fs.tie_cut = entry<E>(4 * q + e, th);
            __syncthreads();
            if (threadIdx.x == NT - 1) sh.b_int = at + c;
            __syncthreads();
            before = sh.b_int;
        }
    }
    __syncthreads();
}

// Arg-max of the row, lowest index first: the largest (key, ~index).  One barrier.
template <int E>
__device__ __forceinline__ int arg_max(const float (&z)[E], int n, unsigned long long (&slot)[NW], int th) {
    unsigned long long best = 0ull;
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (entry<E>(e, th) < n) best = maxu64(best, ((unsigned long long)fkey(z[e]) << 32) | (0xFFFFFFFFu - (unsigned)entry<E>(e, th)));
    best = max1(best, slot);
    return (int)(0xFFFFFFFFu - (unsigned)best);
}

// Clears the words a selection counts in, then the smallest and largest entry of the row.  One barrier.
template <int E>
__device__ __forceinline__ void row_minmax(const float (&z)[E], float& gmin, float& gmax, FastShared& fs) {
    gmin = INFINITY;
    gmax = -INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e) { gmin = fminf(gmin, z[e]); gmax = fmaxf(gmax, z[e]); }
    gmin = wave_min_f(gmin);
    gmax = wave_max_f(gmax);
    if ((threadIdx.x & 63) == 0) fs.s.mm[threadIdx.x >> 6] = make_float2(gmin, gmax);
    fs.hist[threadIdx.x] = 0u;
    if (threadIdx.x < (unsigned)kCand) fs.cand_rank[threadIdx.x] = 0u;
    if (threadIdx.x == 0) { fs.cand_n = 0u; fs.s.pick = 0x7FFFFFFF; }
    __syncthreads();
    const float2 m = fs.s.mm[threadIdx.x & 15];
    gmin = m.x; gmax = m.y;
    ROW_ALLREDUCE(gmin, fminf, dpp_f)
    ROW_ALLREDUCE(gmax, fmaxf, dpp_f)
    gmin = lane_f(gmin, 0);
    gmax = lane_f(gmax, 0);
}

// One wave: the highest bin b of fs.hist with (entries in bins >= b) >= K (fs.bin), how many of its
// entries are among the K largest (fs.want) and how many it has (fs.count; `pads` places past the end of the
// row were counted in bin 0).  Lane l holds bins 256 j + 4 l .. + 3 of the four quarters j.
__device__ __forceinline__ void find_bin(FastShared& fs, int K, int pads) {
    const int lane = threadIdx.x & 63;
    int4 c[4];
    int tot[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        c[j] = *reinterpret_cast<const int4*>(&fs.hist[j * 256 + lane * 4]);
        int t = (c[j].x + c[j].y) + (c[j].z + c[j].w);
        t += dpp_i<0xB1>(t); t += dpp_i<0x4E>(t); t += dpp_i<0x141>(t); t += dpp_i<0x140>(t);
        tot[j] = (__builtin_amdgcn_readlane(t, 0) + __builtin_amdgcn_readlane(t, 16)) +
                 (__builtin_amdgcn_readlane(t, 32) + __builtin_amdgcn_readlane(t, 48));
    }
    int above = 0, qsel = 0;
    int4 cc = c[0];
    bool hit = false;
#pragma unroll
    for (int j = 3; j >= 1; --j)
        if (!hit) {
            if (above + tot[j] >= K) { hit = true; qsel = j; cc = c[j]; }
            else above += tot[j];
        }
    const int inc = wave_incl_scan_i((cc.x + cc.y) + (cc.z + cc.w));
    int cum = above + __builtin_amdgcn_readlane(inc, 63) - inc;   // entries in bins above this lane's
    const int cs[4] = {cc.x, cc.y, cc.z, cc.w};
#pragma unroll
    for (int q = 3; q >= 0; --q) {
        if (cum < K && cum + cs[q] >= K) {   // exactly one lane and bin
            const int b = qsel * 256 + lane * 4 + q;
            fs.bin = b;
            fs.want = K - cum;
            fs.count = cs[q] - (b == 0 ? pads : 0);
        }
        cum += cs[q];
    }
}

// At most 64 candidates, one per lane: wave w compares them with candidates w, w + 16, .. and adds up how many
// of those come before each one (larger value first, lower index first among equals); behind the next
// barrier the one that `want - 1` others precede is the threshold (ranked_threshold).
__device__ __forceinline__ void rank_by_waves(FastShared& fs, int cnt) {
    const int lane = threadIdx.x & 63;
    const float mz = lane < cnt ? fs.cand_z[lane] : 0.f;
    const int mi = lane < cnt ? fs.cand_idx[lane] : 0;
    unsigned part = 0u;
    for (int j = wave_id(); j < cnt; j += NW) {
        const float oz = fs.cand_z[j];
        const int oi = fs.cand_idx[j];
        part += (oz > mz || (oz == mz && oi < mi)) ? 1u : 0u;
    }
    if (lane < cnt && part) atomicAdd(&fs.cand_rank[lane], part);
}
__device__ __forceinline__ Threshold ranked_threshold(const FastShared& fs, bool pending) {
    Threshold t = {fs.tau_z, fs.tie_cut};
    if (pending) {
        const int lane = threadIdx.x & 63;
        const unsigned long long hit = __ballot(lane < fs.count && fs.cand_rank[lane] + 1u == (unsigned)fs.want);
        const int l = (int)__ffsll(hit) - 1;   // exactly one lane
        t.tz = lane_f(fs.cand_z[lane], l);
        t.cut = __builtin_amdgcn_readlane(fs.cand_idx[lane], l);
    }
    return t;
}

// Bins of the row's entries, linear between its smallest and largest one (places past the end: bin 0).
template <int E>
__device__ __forceinline__ void linear_bins(const float (&z)[E], float gmin, float gmax, unsigned (&bin)[E]) {
    const float scale = ((float)kBins - 0.01f) / (gmax - gmin);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const float f = (z[e] - gmin) * scale;
        asm("v_cvt_u32_f32 %0, %1" : "=v"(bin[e]) : "v"(f));   // NaN converts to 0
    }
}

// The cut of a row at its K-th largest entry (K < n).  On return hi[e] is larger than `lim` or equal to it
// for every kept entry e and for the entries that share the threshold's bin; the exact threshold is in
// fs.tau_z / fs.tie_cut, or, if `pending`, still to be found by rank_by_waves (behind a barrier) and
// ranked_threshold (behind another).  tag: -2 - (the threshold's bin), -1 if hi holds the exact
// decision (WarpStat::onehot of such a row: any negative value means no point mass, and the tag lets another
// kernel gather the same list).
template <int E>
__device__ __forceinline__ void cut_row(const float (&z)[E], int n, int K, FastShared& fs, float& gmax, unsigned (&hi)[E],
                                        unsigned& lim, bool& pending, int& tag, int th) {
    float gmin;
    row_minmax<E>(z, gmin, gmax, fs);
    pending = false;
    tag = -1;
    if (gmax - gmin > kMinRange && gmin > -INFINITY && gmax < INFINITY) {
        linear_bins<E>(z, gmin, gmax, hi);
#pragma unroll
        for (int e = 0; e < E; ++e) atomicAdd(&fs.hist[hi[e]], 1u);
        __syncthreads();
        if (threadIdx.x < 64) find_bin(fs, K, E * NT - n);
        __syncthreads();
        lim = (unsigned)__builtin_amdgcn_readfirstlane(fs.bin);
        const int cnt = __builtin_amdgcn_readfirstlane(fs.count);
        if (cnt <= kCand) {
            tag = -2 - (int)lim;
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (hi[e] == lim && entry<E>(e, th) < n) {
                    const unsigned at = atomicAdd(&fs.cand_n, 1u);
                    fs.cand_z[at] = z[e];
                    fs.cand_idx[at] = entry<E>(e, th);
                }
            if (cnt <= 64) {
                pending = true;
                return;
            }
            const unsigned want = (unsigned)fs.want;
            __syncthreads();
            rank_candidates(fs, (unsigned)cnt);
            if (threadIdx.x < (unsigned)cnt && fs.cand_rank[threadIdx.x] + 1u == want) {
                fs.tau_z = fs.cand_z[threadIdx.x];
                fs.tie_cut = fs.cand_idx[threadIdx.x];
            }
            __syncthreads();
            return;
        }
    }
    radix_select<E>(z, n, K, fs, th);
    const Threshold t = {fs.tau_z, fs.tie_cut};
    lim = 1u;
#pragma unroll
    for (int e = 0; e < E; ++e) hi[e] = keeps(t, z[e], entry<E>(e, th)) ? 1u : 0u;
}

// When top-k keeps at most kTopCap entries, they are gathered - in index order - into a list in LDS
// and the fp64 exponentials are evaluated for those only (the other 15 of 16 entries of a 16384-entry
// row would cost a software exp each for a weight of zero).  Thread t owns entries t, NT + t, 2 NT + t.
struct CompactList {
    int2 e[kCap];   // index, scaled logit (bits)
};

__host__ __device__ __forceinline__ bool use_list(int top_k, int n, int greedy) { return !greedy && top_k < n && top_k <= kTopCap; }

// Per-wave counts of the entries with hi[e] >= lim, for place_entries behind the next barrier.
template <int E>
__device__ __forceinline__ void count_entries(const unsigned (&hi)[E], unsigned lim, Slots& sl) {
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
        int c = 0;
#pragma unroll
        for (int e = 4 * q; e < 4 * q + 4; ++e) c += __popcll(__ballot(hi[e] >= lim));
        if ((threadIdx.x & 63) == 0) sl.cnt[q * NW + (threadIdx.x >> 6)] = c;
    }
}
// Writes those entries into the list in index order; returns their number without the places past the end of
// the row (n entries): where lim is bin 0 these are counted too, behind every entry of the row.
template <int E>
__device__ __forceinline__ int place_entries(const unsigned (&hi)[E], unsigned lim, const float (&z)[E], int n, CompactList& L, const Slots& sl, int th) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int v = lane < 4 * E ? sl.cnt[lane] : 0;   // chunk-major, wave-minor: the order of the indices
    const int inc = wave_incl_scan_i(v);
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
        int at = __builtin_amdgcn_readlane(inc - v, q * NW + wave);
#pragma unroll
        for (int e = 4 * q; e < 4 * q + 4; ++e) {   // entries of the lanes before this one
            const unsigned long long m = __ballot(hi[e] >= lim);
            at = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, (unsigned)at));
        }
#pragma unroll
        for (int e = 4 * q; e < 4 * q + 4; ++e)
            if (hi[e] >= lim) {
                if (at < kCap) L.e[at] = make_int2(entry<E>(e, th), __float_as_int(z[e]));
                ++at;
            }
    }
    return min(__builtin_amdgcn_readlane(inc, 4 * E - 1), min(n, kCap));
}

// The list of a top-k row: its length, its largest entry and the exact threshold.
template <int E>
__device__ __forceinline__ int select_list(const float (&z)[E], int n, int K, FastShared& fs, CompactList& L, Threshold& t, WarpStat& st,
                                           int th = (int)threadIdx.x) {
    unsigned hi[E], lim;
    bool pending;
    cut_row<E>(z, n, K, fs, st.zmax, hi, lim, pending, st.onehot, th);
    count_entries<E>(hi, lim, fs.s);
    __syncthreads();
    if (pending) rank_by_waves(fs, fs.count);
    const int Kc = place_entries<E>(hi, lim, z, n, L, fs.s, th);
    __syncthreads();
    t = ranked_threshold(fs, pending);
    st.tau = fkey(t.tz);
    st.tie_cut = t.cut;
    return Kc;
}

// Weights exp(z - zmax) of the thread's list entries (0 past the end and for entries that are not kept).
__device__ __forceinline__ void list_weights(const CompactList& L, int Kc, float zmax, const Threshold& t, int (&idx)[kLH], double (&w)[kLH]) {
#pragma unroll
    for (int h = 0; h < kLH; ++h) {
        const int i = (int)threadIdx.x + h * NT;
        w[h] = 0.0;
        idx[h] = -1;
        if (i < Kc) {
            const int2 v = L.e[i];
            idx[h] = v.x;
            const float z = __int_as_float(v.y);
            if (keeps(t, z, v.x)) w[h] = exp((double)z - (double)zmax);
        }
    }
}
__device__ __forceinline__ double sum3(const double (&w)[kLH]) {
    double s = w[0];
#pragma unroll
    for (int h = 1; h < kLH; ++h) s += w[h];
    return s;
}

// Running sums of the list weights w: c[h] = sum of all entries up to and including the thread's own
// entry h; returns the total.  One barrier.
__device__ __forceinline__ double list_scan(const double (&w)[kLH], int Kc, double (&c)[kLH], double (&s)[4][NW]) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    double inc[kLH];
#pragma unroll
    for (int h = 0; h < kLH; ++h)
        if (h * NT < Kc) {
            inc[h] = wave_incl_scan_d(w[h]);
            if (lane == 63) s[h][threadIdx.x >> 6] = inc[h];
        }
    __syncthreads();
    double before = 0.0;
#pragma unroll
    for (int h = 0; h < kLH; ++h) {
        c[h] = 0.0;
        if (h * NT < Kc) {
            double base;
            const double t = wave_base_d(s[h], wave, base);
            c[h] = before + base + inc[h];
            before += t;
        }
    }
    return before;
}

// Inverse-CDF draw from running sums c of list weights w: the first entry whose running sum exceeds
// target, else the last one with weight.  sl.pick holds 0x7FFFFFFF on entry (set before the last
// barrier).  Returns the position in the list; all threads call.
__device__ __forceinline__ int list_pick(const double (&w)[kLH], const double (&c)[kLH], double target, Slots& sl, Shared& sh) {
    int cand = 0x7FFFFFFF, last = -1;
#pragma unroll
    for (int h = kLH - 1; h >= 0; --h)
        if (w[h] > 0.0) {
            last = max(last, (int)threadIdx.x + h * NT);
            if (c[h] > target) cand = (int)threadIdx.x + h * NT;
        }
    cand = wave_min_i(cand);
    if ((threadIdx.x & 63) == 0 && cand != 0x7FFFFFFF) atomicMin(&sl.pick, cand);
    __syncthreads();
    cand = sl.pick;
    if (cand != 0x7FFFFFFF) return cand;
    return max(0, block_max_i(last, sh));
}

// Inverse-CDF draw from the dense per-thread weights w (ascending index order).
template <int E>
__device__ __forceinline__ int inv_cdf_row(const double (&w)[E], double total, float u, Slots& sl, Shared& sh, int th = (int)threadIdx.x) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    double s[E / 4], inc[E / 4];
    __syncthreads();   // the slots may still be read by an earlier exchange
    if (threadIdx.x == 0) sl.pick = 0x7FFFFFFF;
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
        s[q] = (w[4 * q] + w[4 * q + 1]) + (w[4 * q + 2] + w[4 * q + 3]);
        inc[q] = wave_incl_scan_d(s[q]);
        if (lane == 63) sl.scan[0][q][threadIdx.x >> 6] = inc[q];
    }
    __syncthreads();
    const double target = (double)u * total;
    int cand = 0x7FFFFFFF, last = -1;
    double before = 0.0;
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
        double base;
        const double t = wave_base_d(sl.scan[0][q], wave, base);
        double c = before + base + (inc[q] - s[q]);
        before += t;
#pragma unroll
        for (int e = 4 * q; e < 4 * q + 4; ++e)
            if (w[e] > 0.0) {
                c += w[e];
                last = entry<E>(e, th);
                if (c > target && cand == 0x7FFFFFFF) cand = entry<E>(e, th);
            }
    }
    cand = wave_min_i(cand);
    if (lane == 0 && cand != 0x7FFFFFFF) atomicMin(&sl.pick, cand);
    __syncthreads();
    cand = sl.pick;
    if (cand != 0x7FFFFFFF) return cand;
    return block_max_i(last, sh);
}

// The statistics (with total) of a row that does not take the list form - greedy, every entry kept, or more
// than kTopCap kept - and the weight of every entry of the thread.
template <int E>
__device__ __forceinline__ WarpStat dense_row(const float (&z)[E], int n, int top_k, int greedy, FastShared& fs, double (&w)[E],
                                             int th = (int)threadIdx.x) {
    WarpStat st;
    st.total = 1.0; st.zmax = 0.f; st.tau = 0x007FFFFFu; st.tie_cut = -1; st.onehot = -1;  // keeps every finite entry
    if (greedy) {
        st.onehot = arg_max<E>(z, n, fs.s.key, th);
#pragma unroll
        for (int e = 0; e < E; ++e) w[e] = (entry<E>(e, th) == st.onehot) ? 1.0 : 0.0;
        return st;
    }
    Threshold t = {-INFINITY, -1};
    if (top_k < n) {
        unsigned hi[E], lim;
        bool pending;
        int tag;
        cut_row<E>(z, n, top_k, fs, st.zmax, hi, lim, pending, tag, th);
        __syncthreads();
        if (pending) rank_by_waves(fs, fs.count);
        __syncthreads();
        t = ranked_threshold(fs, pending);
        st.tau = fkey(t.tz);
        st.tie_cut = t.cut;
    } else {
        float gmin;
        row_minmax<E>(z, gmin, st.zmax, fs);
    }
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        w[e] = keeps(t, z[e], entry<E>(e, th)) ? exp((double)z[e] - (double)st.zmax) : 0.0;
        s += w[e];
        __builtin_amdgcn_sched_barrier(0);   // one exponential at a time: interleaved ones spill
    }
    st.total = sum1(s, fs.s.sum);
    return st;
}

// Where a row's list goes for the kernel that needs it next: its length, then per entry the index and the weight
// (kCap entries each).
struct ListStore { int32_t* len; int32_t* idx; double* w; };

// One row, start to finish: the warp's statistics (with total) and, if u != null, a draw; its list, if it has
// one, also goes to `store` when that is given.
template <int E>
__device__ __forceinline__ WarpStat warp_and_draw(const float (&z)[E], int n, int top_k, int greedy, FastShared& fs, CompactList& L,
                                                  const float* u, int* drawn, const ListStore store = {nullptr, nullptr, nullptr}) {
    WarpStat st;
    if (use_list(top_k, n, greedy)) {
        Threshold t;
        const int Kc = select_list<E>(z, n, top_k, fs, L, t, st);
        int idx[kLH];
        double w[kLH], c[kLH];
        list_weights(L, Kc, st.zmax, t, idx, w);
        if (store.len) {
            if (threadIdx.x == 0) *store.len = Kc;
#pragma unroll
            for (int h = 0; h < kLH; ++h)
                if (idx[h] >= 0) {
                    store.idx[threadIdx.x + h * NT] = idx[h];
                    store.w[threadIdx.x + h * NT] = w[h];
                }
        }
        if (u) {
            st.total = list_scan(w, Kc, c, fs.s.scan[0]);
            const int at = list_pick(w, c, (double)*u * st.total, fs.s, fs.sh);
            *drawn = Kc > 0 ? L.e[at].x : 0;   // NaN logits may leave nothing: still a token of the slice
        } else {
            st.total = sum1(sum3(w), fs.s.sum);
        }
        return st;
    }
    double w[E];
    st = dense_row<E>(z, n, top_k, greedy, fs, w);
    if (u) *drawn = st.onehot >= 0 ? st.onehot : inv_cdf_row<E>(w, st.total, *u, fs.s, fs.sh);
    return st;
}

__device__ __forceinline__ ListStore list_at(int32_t* len, int32_t* idx, double* w, size_t row) {
    ListStore l;
    l.len = len + row; l.idx = idx + row * kCap; l.w = w + row * kCap;
    return l;
}

}  // namespace

}  // namespace hawk
