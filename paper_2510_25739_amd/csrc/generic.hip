// Generic (any-shape) kernels of the target decoder and the draft head.
//
// Two arithmetic configurations, selected by the weight dtype of the context:
//   fp32 blobs: fp32 weights, fp64 activations / accumulators / KV cache (exact-parity set); products and the attention
//               over heads of 32, 64 and 128 are in fp32.hip;
//   bf16 blobs: bf16 weights, fp16 KV cache (same bytes as bf16, 3 more mantissa bits: the
//               cache's rounding is what dominates the logit error), fp32 activations and
//               accumulators.
// One wave computes one output column of a skinny GEMM for up to RT rows, streaming its
// weight row with 16-byte loads; this is the fallback path of bf16 contexts, which otherwise run in xcd.hip,
// stream.hip and rows.hip.
#include <string.h>

#include "hawk_internal.h"

namespace hawk {

struct CfgF32 {
    using WT = float; using AT = double; using KT = double;
};
struct CfgBF16 {
    using WT = uint16_t; using AT = float; using KT = _Float16;
    static constexpr int VE = 8;
};

__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {  // round to nearest even
    uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ void load_w(const uint16_t* p, float* out) {
    uint4 v = *reinterpret_cast<const uint4*>(p);
    out[0] = bf16_to_f32(v.x & 0xFFFFu); out[1] = bf16_to_f32(v.x >> 16);
    out[2] = bf16_to_f32(v.y & 0xFFFFu); out[3] = bf16_to_f32(v.y >> 16);
    out[4] = bf16_to_f32(v.z & 0xFFFFu); out[5] = bf16_to_f32(v.z >> 16);
    out[6] = bf16_to_f32(v.w & 0xFFFFu); out[7] = bf16_to_f32(v.w >> 16);
}
__device__ __forceinline__ double w1(const float* p, size_t i) { return (double)p[i]; }
__device__ __forceinline__ float w1(const uint16_t* p, size_t i) { return bf16_to_f32(p[i]); }
__device__ __forceinline__ double kload(const double* p, size_t i) { return p[i]; }
__device__ __forceinline__ float kload(const _Float16* p, size_t i) { return (float)p[i]; }
__device__ __forceinline__ void kstore(double* p, size_t i, double v) { p[i] = v; }
__device__ __forceinline__ void kstore(_Float16* p, size_t i, float v) { p[i] = (_Float16)v; }

template <typename T> __device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
template <typename T> __device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { T t = __shfl_xor(v, o, 64); v = t > v ? t : v; }
    return v;
}
// Sum over a 256-thread block; every thread gets the result. red: >= 4 entries of LDS.
template <typename T> __device__ __forceinline__ T block_sum256(T v, T* red) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}
template <typename T> __device__ __forceinline__ T block_max256(T v, T* red) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    T a = red[0] > red[1] ? red[0] : red[1], b = red[2] > red[3] ? red[2] : red[3];
    return a > b ? a : b;
}

// Row R of a pass -> sequence, row within the sequence, prompt, absolute position.
// pos: position (rotary angle); slot: index of the row's entry in the cache (= pos except for tree rows).
struct RowInfo { int s, r, b, pos, slot; bool valid; };
__device__ __forceinline__ RowInfo row_info(const RowMap& m, int R) {
    RowInfo o;
    o.s = R / m.rows_per_seq;
    o.r = R - o.s * m.rows_per_seq;
    o.b = o.s % m.batch;
    if (m.mode == 0) {
        o.pos = o.r;
        o.valid = true;
    } else {
        int ke = m.k_eff[o.b];
        o.valid = o.r <= ke;
        o.pos = o.valid ? m.n_cond + m.n[o.b] - 1 + (m.mode == 2 ? m.tree_depth[o.r] : o.r) : 0;
    }
    o.slot = (m.mode == 2 && o.valid) ? m.n_cond + m.n[o.b] - 1 + o.r : o.pos;
    return o;
}

// ------------------------------------------------------------------ rows in

// X[R] = E[token of row R]: row 0 of a sequence is the last committed token, row r > 0
// is draft r-1.
template <class Cfg>
__global__ void embed_rows_kernel(typename Cfg::AT* X, const typename Cfg::WT* E, RowMap map,
                                  const int32_t* grid, const int32_t* draft, int N, int kstride, int d) {
    RowInfo ri = row_info(map, blockIdx.x);
    int tok = 0;
    if (ri.valid) tok = ri.r == 0 ? grid[(size_t)ri.b * N + map.n[ri.b] - 1] : draft[ri.b * kstride + ri.r - 1];
    if (tok < 0) tok = 0;
    for (int i = threadIdx.x; i < d; i += blockDim.x)
        X[(size_t)blockIdx.x * d + i] = w1(E, (size_t)tok * d + i);
}

template <class Cfg>
__global__ void cond_rows_kernel(typename Cfg::AT* X, const float* cond, size_t total) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < total) X[i] = (typename Cfg::AT)cond[i];
}

template <class Cfg>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const typename Cfg::AT* X, const typename Cfg::WT* g,
                                                      typename Cfg::AT* out, int d, size_t in_stride,
                                                      float eps) {
    using AT = typename Cfg::AT;
    __shared__ AT red[4];
    const AT* x = X + (size_t)blockIdx.x * in_stride;
    AT ss = 0;
    for (int i = threadIdx.x; i < d; i += 256) ss += x[i] * x[i];
    ss = block_sum256(ss, red);
    AT r = (AT)1 / sqrt(ss / (AT)d + (AT)eps);
    for (int i = threadIdx.x; i < d; i += 256) {
        const AT v = x[i] * r * w1(g, i);
        out[(size_t)blockIdx.x * d + i] = v;
    }
}

// The same for fp32 activations and bf16 gains with the row held in registers (V float4 per
// thread: d <= 1024 V, d % 4 == 0, rows 16-byte aligned): one pass over the row instead of two
// loops of dependent scalar loads.
template <int V>
__global__ __launch_bounds__(256) void rmsnorm_rows_kernel(const float* X, const uint16_t* g, float* out, int d,
                                                           size_t in_stride, float eps) {
    __shared__ float red[4];
    const float4* x = reinterpret_cast<const float4*>(X + (size_t)blockIdx.x * in_stride);
    const int n4 = d / 4;
    float4 v[V];
    uint2 gw[V];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const int q = threadIdx.x + i * 256;
        v[i] = q < n4 ? x[q] : make_float4(0.f, 0.f, 0.f, 0.f);
        gw[i] = q < n4 ? reinterpret_cast<const uint2*>(g)[q] : make_uint2(0u, 0u);
    }
#pragma unroll
    for (int i = 0; i < V; ++i) ss += v[i].x * v[i].x + v[i].y * v[i].y + v[i].z * v[i].z + v[i].w * v[i].w;
    ss = block_sum256(ss, red);
    const float r = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const int q = threadIdx.x + i * 256;
        if (q < n4) {
            float4 o;
            o.x = v[i].x * r * __uint_as_float(gw[i].x << 16);
            o.y = v[i].y * r * __uint_as_float(gw[i].x & 0xFFFF0000u);
            o.z = v[i].z * r * __uint_as_float(gw[i].y << 16);
            o.w = v[i].w * r * __uint_as_float(gw[i].y & 0xFFFF0000u);
            reinterpret_cast<float4*>(out + (size_t)blockIdx.x * d)[q] = o;
        }
    }
}

// ------------------------------------------------------------------ skinny GEMM

template <class Cfg, int RT, typename OT>
__global__ __launch_bounds__(256) void gemm_rows_kernel(const typename Cfg::AT* A, int lda,
                                                        const typename Cfg::WT* W, int N, int K,
                                                        OT* Y, int ldy, int M, int accumulate) {
    using AT = typename Cfg::AT;
    constexpr int VE = Cfg::VE;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n = blockIdx.x * 4 + wave;
    if (n >= N) return;
    const int r0 = blockIdx.y * RT;
    AT acc[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r] = 0;
    const typename Cfg::WT* wrow = W + (size_t)n * K;
    for (int c = lane * VE; c < K; c += 64 * VE) {
        AT w[VE];
        load_w(wrow + c, w);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if (r0 + r < M) {
                const AT* a = A + (size_t)(r0 + r) * lda + c;
#pragma unroll
                for (int e = 0; e < VE; ++e) acc[r] += w[e] * a[e];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r] = wave_sum(acc[r]);
    if (lane == 0) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
            if (r0 + r < M) {
                OT* y = Y + (size_t)(r0 + r) * ldy + n;
                *y = (OT)((accumulate ? (AT)*y : (AT)0) + acc[r]);
            }
    }
}

// ------------------------------------------------------------------ rotary + cache append

// In place on QKV[R] = [q | k | v]: rotates q and k (pair (2j, 2j+1) of each head by
// pos * inv_freq[j]) and writes k, v to the cache at (sequence, pos).
template <class Cfg>
__global__ void rope_append_kernel(typename Cfg::AT* QKV, typename Cfg::KT* Kc, typename Cfg::KT* Vc,
                                   RowMap map, const double* inv_freq, int layer, int d, int hd,
                                   int Smax, int Tmax) {
    using AT = typename Cfg::AT;
    RowInfo ri = row_info(map, blockIdx.x);
    if (!ri.valid) return;
    AT* q = QKV + (size_t)blockIdx.x * 3 * d;
    AT* k = q + d;
    AT* v = k + d;
    // cache layout [layer][sequence][head][position][hd]: one head's entries are contiguous
    const int H = d / hd;
    auto at = [&](int e) {   // element e of the row (feature index within d)
        const int h = e / hd;
        return ((((size_t)layer * Smax + ri.s) * H + h) * Tmax + ri.slot) * hd + (e - h * hd);
    };
    // the angles depend on the position and the pair index within a head only: one sincos per pair
    // index and row, shared by all heads through LDS (hd <= 512)
    __shared__ double tab_c[256], tab_s[256];
    for (int j = threadIdx.x; j < hd / 2; j += blockDim.x) sincos((double)ri.pos * inv_freq[j], &tab_s[j], &tab_c[j]);
    __syncthreads();
    constexpr int U = 4;   // pairs per thread in flight
    for (int p0 = threadIdx.x; p0 < d / 2; p0 += U * blockDim.x) {
        AT qa[U], qb[U], ka[U], kb[U], va[U], vb[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p0 + u * blockDim.x;
            if (p < d / 2) {
                qa[u] = q[2 * p]; qb[u] = q[2 * p + 1];
                ka[u] = k[2 * p]; kb[u] = k[2 * p + 1];
                va[u] = v[2 * p]; vb[u] = v[2 * p + 1];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p0 + u * blockDim.x;
            if (p < d / 2) {
                const int j = p % (hd / 2);
                const AT c = (AT)tab_c[j], sn = (AT)tab_s[j];
                q[2 * p] = qa[u] * c - qb[u] * sn;
                q[2 * p + 1] = qa[u] * sn + qb[u] * c;
                kstore(Kc, at(2 * p), ka[u] * c - kb[u] * sn);
                kstore(Kc, at(2 * p + 1), ka[u] * sn + kb[u] * c);
                kstore(Vc, at(2 * p), va[u]);
                kstore(Vc, at(2 * p + 1), vb[u]);
            }
        }
    }
}

// ------------------------------------------------------------------ attention

// One workgroup per (head, row): the row attends cache entries 0..pos of its sequence
// (its own entry included), i.e. causal inside the block of new rows.  Tree rows: entries up to
// the root's, then of the new entries only the row's ancestors and its own.
template <class Cfg>
__global__ __launch_bounds__(256) void attention_kernel(const typename Cfg::AT* QKV, const typename Cfg::KT* Kc,
                                                        const typename Cfg::KT* Vc, typename Cfg::AT* O,
                                                        RowMap map, int layer, int d, int hd, int Smax, int Tmax) {
    using AT = typename Cfg::AT;
    extern __shared__ double smem_raw[];
    AT* sc = reinterpret_cast<AT*>(smem_raw);  // [Tmax] scores, then [hd] q, then [256] partials
    AT* sq = sc + Tmax;
    AT* part = sq + hd;
    __shared__ AT red[4];
    const int R = blockIdx.y, h = blockIdx.x, tid = threadIdx.x;
    RowInfo ri = row_info(map, R);
    if (!ri.valid) return;
    const size_t base = ((((size_t)layer * Smax + ri.s) * (d / hd) + h) * Tmax) * hd;   // this head's entries, contiguous
    for (int i = tid; i < hd; i += 256) sq[i] = QKV[(size_t)R * 3 * d + (size_t)h * hd + i];
    __syncthreads();
    const AT scale = (AT)1 / sqrt((AT)hd);
    const int root = ri.slot - ri.r;   // tree rows: entry of node 0
    const unsigned long long anc = map.mode == 2 ? (map.tree_anc[ri.r] | (1ull << ri.r)) : ~0ull;
    AT mx = -INFINITY;
    for (int t = tid; t <= ri.slot; t += 256) {
        AT s = 0;
        for (int i = 0; i < hd; ++i) s += sq[i] * kload(Kc, base + (size_t)t * hd + i);
        s *= scale;
        if (map.mode == 2 && t > root && !((anc >> (t - root)) & 1ull)) s = -INFINITY;   // not on the row's path
        sc[t] = s;
        mx = s > mx ? s : mx;
    }
    mx = block_max256(mx, red);
    AT den = 0;
    for (int t = tid; t <= ri.slot; t += 256) {
        AT e = exp(sc[t] - mx);
        sc[t] = e;
        den += e;
    }
    den = block_sum256(den, red);  // also orders the sc[] writes before the reads below
    const int i = tid % hd, sl = tid / hd, nsl = 256 / hd;
    AT acc = 0;
    for (int t = sl; t <= ri.slot; t += nsl) acc += sc[t] * kload(Vc, base + (size_t)t * hd + i);
    part[tid] = acc;
    __syncthreads();
    if (tid < hd) {
        AT o = 0;
        for (int s2 = 0; s2 < nsl; ++s2) o += part[s2 * hd + tid];
        o /= den;
        O[(size_t)R * d + (size_t)h * hd + tid] = o;
    }
}

template <class Cfg>
__global__ void swiglu_kernel(typename Cfg::AT* U, int m, size_t total) {
    using AT = typename Cfg::AT;
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    size_t row = idx / m, i = idx - row * m;
    AT a = U[row * 2 * m + i], b = U[row * 2 * m + m + i];
    const AT v = a / ((AT)1 + exp(-a)) * b;
    U[row * 2 * m + i] = v;
}

// ------------------------------------------------------------------ draft head input

// DIN[s] = [previous head output (target hidden for the first draft) | E[left] | E[up]]
// for draft i (1-based) of every sequence.
template <class Cfg>
__global__ void draft_input_kernel(typename Cfg::AT* DIN, const typename Cfg::AT* prev,
                                   const typename Cfg::WT* E, const int32_t* n_arr, const int32_t* k_eff,
                                   const int32_t* grid, const int32_t* draft, int i, int B, int N, int IW,
                                   int kstride, int d) {
    using AT = typename Cfg::AT;
    const int s = blockIdx.x, b = s % B;
    AT* out = DIN + (size_t)s * 3 * d;
    if (i > k_eff[b]) {
        for (int c = threadIdx.x; c < 3 * d; c += blockDim.x) out[c] = 0;
        return;
    }
    const int n = n_arr[b], t = n - 1 + i;
    const int left = (i == 1) ? grid[(size_t)b * N + n - 1] : draft[b * kstride + i - 2];
    const int up = (t >= IW) ? grid[(size_t)b * N + t - IW] : -1;
    for (int c = threadIdx.x; c < d; c += blockDim.x) {
        out[c] = prev[(size_t)s * d + c];
        out[d + c] = w1(E, (size_t)left * d + c);
        out[2 * d + c] = up >= 0 ? w1(E, (size_t)up * d + c) : (AT)0;
    }
}

template <class Cfg>
__global__ void keep_hprev_prefill_kernel(typename Cfg::AT* hprev, const typename Cfg::AT* X, int C, int d) {
    const int s = blockIdx.x;
    for (int c = threadIdx.x; c < d; c += blockDim.x)
        hprev[(size_t)s * d + c] = X[((size_t)s * C + C - 1) * d + c];
}

// ------------------------------------------------------------------ launchers

#define DISPATCH(ctx, CALL)                       \
    do {                                          \
        if ((ctx)->cfg.dtype == HAWK_FP32) {      \
            using Cfg = CfgF32;                   \
            CALL;                                 \
        } else {                                  \
            using Cfg = CfgBF16;                  \
            CALL;                                 \
        }                                         \
    } while (0)

template <class Cfg> static const typename Cfg::WT* wptr(hawk_ctx* c, size_t blob_off) {
    return reinterpret_cast<const typename Cfg::WT*>(c->ws + c->off.blob + blob_off);
}

void launch_embed_rows(hawk_ctx* c, const RowMap& map, int M) {
    DISPATCH(c, (embed_rows_kernel<Cfg><<<M, 256, 0, c->stream>>>(
                    wsp<typename Cfg::AT>(c, c->off.x), wptr<Cfg>(c, c->w.E), map, wsp<int32_t>(c, c->off.grid),
                    wsp<int32_t>(c, c->off.draft), c->N, c->kmax + 1, c->d)));
}

void launch_cond_rows(hawk_ctx* c, int M) {
    size_t total = (size_t)M * c->d;
    DISPATCH(c, (cond_rows_kernel<Cfg><<<(unsigned)((total + 255) / 256), 256, 0, c->stream>>>(
                    wsp<typename Cfg::AT>(c, c->off.x), wsp<float>(c, c->off.cond), total)));
}

void launch_rmsnorm(hawk_ctx* c, size_t off_in, size_t in_stride, size_t off_gain, size_t off_out, int M) {
    using Cfg = CfgBF16;
    if (c->d % 4 == 0 && in_stride % 4 == 0 && off_in % 16 == 0 && off_out % 16 == 0 && (c->off.blob + off_gain) % 8 == 0 &&
        c->d <= 8192) {
        const float* X = wsp<float>(c, off_in);
        const uint16_t* g = reinterpret_cast<const uint16_t*>(c->ws + c->off.blob + off_gain);
        float* out = wsp<float>(c, off_out);
        if (c->d <= 2048)
            rmsnorm_rows_kernel<2><<<M, 256, 0, c->stream>>>(X, g, out, c->d, in_stride, c->cfg.rms_eps);
        else if (c->d <= 4096)
            rmsnorm_rows_kernel<4><<<M, 256, 0, c->stream>>>(X, g, out, c->d, in_stride, c->cfg.rms_eps);
        else
            rmsnorm_rows_kernel<8><<<M, 256, 0, c->stream>>>(X, g, out, c->d, in_stride, c->cfg.rms_eps);
        return;
    }
    rmsnorm_kernel<Cfg><<<M, 256, 0, c->stream>>>(
                    wsp<typename Cfg::AT>(c, off_in), wptr<Cfg>(c, off_gain), wsp<typename Cfg::AT>(c, off_out),
                    c->d, in_stride, c->cfg.rms_eps);
}

void launch_gemm(hawk_ctx* c, size_t off_a, int lda, size_t w_off, int N, int K, size_t off_y, int ldy,
                 int M, bool accumulate, bool out_f32) {
    // bf16 products that the matrix cores take although the context as a whole does not run in rows.hip (d no multiple of 32),
    // or that have no tile-major weights there
    if (c->off.split && K % 32 == 0 && N % 16 == 0 && ldy % 4 == 0 && lda % 4 == 0 && 4 * plane_halves(M, K) <= c->split_bytes) {
        RowsGemm g;
        memset(&g, 0, sizeof g);
        uint16_t* hi = wsp<uint16_t>(c, c->off.split);
        g.hi = hi; g.lo = hi + plane_halves(M, K);
        g.W = wptr<CfgBF16>(c, w_off); g.mode = accumulate ? kGemmResidual : kGemmPlain;
        g.M = M; g.N = N; g.K = K; g.Y = wsp<float>(c, off_y); g.ldy = ldy;
        launch_rows_split(c->stream, wsp<float>(c, off_a), lda, M, K, hi, hi + plane_halves(M, K));
        launch_rows_gemm(c->stream, g);
        return;
    }
    using Cfg = CfgBF16;
    constexpr int RT = 8;
    dim3 grid((N + 3) / 4, (M + RT - 1) / RT);
    if (out_f32) {
        gemm_rows_kernel<Cfg, RT, float><<<grid, 256, 0, c->stream>>>(
                        wsp<typename Cfg::AT>(c, off_a), lda, wptr<Cfg>(c, w_off), N, K, wsp<float>(c, off_y), ldy,
                        M, accumulate ? 1 : 0);
    } else {
        gemm_rows_kernel<Cfg, RT, typename Cfg::AT><<<grid, 256, 0, c->stream>>>(
                        wsp<typename Cfg::AT>(c, off_a), lda, wptr<Cfg>(c, w_off), N, K,
                        wsp<typename Cfg::AT>(c, off_y), ldy, M, accumulate ? 1 : 0);
    }
}

void launch_rope_append(hawk_ctx* c, const RowMap& map, int layer, int M) {
    DISPATCH(c, (rope_append_kernel<Cfg><<<M, 256, 0, c->stream>>>(
                    wsp<typename Cfg::AT>(c, c->off.qkv), wsp<typename Cfg::KT>(c, c->off.kc),
                    wsp<typename Cfg::KT>(c, c->off.vc), map, wsp<double>(c, c->off.inv_freq), layer, c->d, c->hd,
                    c->Smax, c->Tmax)));
}

void launch_attention(hawk_ctx* c, const RowMap& map, int layer, int M) {
    dim3 grid(c->H, M);
    DISPATCH(c, (attention_kernel<Cfg><<<grid, 256, (size_t)(c->Tmax + c->hd + 256) * sizeof(typename Cfg::AT),
                                         c->stream>>>(
                    wsp<typename Cfg::AT>(c, c->off.qkv), wsp<typename Cfg::KT>(c, c->off.kc),
                    wsp<typename Cfg::KT>(c, c->off.vc), wsp<typename Cfg::AT>(c, c->off.o), map, layer, c->d, c->hd,
                    c->Smax, c->Tmax)));
}

void launch_swiglu(hawk_ctx* c, int M) {
    using Cfg = CfgBF16;
    size_t total = (size_t)M * c->m;
    swiglu_kernel<Cfg><<<(unsigned)((total + 255) / 256), 256, 0, c->stream>>>(
                    wsp<typename Cfg::AT>(c, c->off.u), c->m, total);
}

void launch_draft_input(hawk_ctx* c, int i) {
    using Cfg = CfgBF16;
    // draft i writes its head output to g1 (i odd) / g0 (i even); draft i > 1 reads draft i-1's
    size_t prev = (i == 1) ? c->off.hprev : (((i - 1) & 1) ? c->off.g1 : c->off.g0);
    draft_input_kernel<Cfg><<<c->S, 256, 0, c->stream>>>(
                    wsp<typename Cfg::AT>(c, c->off.din), wsp<typename Cfg::AT>(c, prev), wptr<Cfg>(c, c->w.E),
                    wsp<int32_t>(c, c->off.n), wsp<int32_t>(c, c->off.k_eff), wsp<int32_t>(c, c->off.grid),
                    wsp<int32_t>(c, c->off.draft), i, c->B, c->N, c->gw, c->kmax + 1, c->d);
}

void launch_keep_hprev_prefill(hawk_ctx* c) {
    DISPATCH(c, (keep_hprev_prefill_kernel<Cfg><<<c->S, 256, 0, c->stream>>>(
                    wsp<typename Cfg::AT>(c, c->off.hprev), wsp<typename Cfg::AT>(c, c->off.x), c->C, c->d)));
}

}  // namespace hawk
