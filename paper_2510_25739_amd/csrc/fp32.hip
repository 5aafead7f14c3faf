// The fp32 configuration (fp32 weights; fp64 activations, accumulators and cache): five launches per decoder layer.
//
// Models of this configuration are a few MB, so a pass is a chain of launches, each near its latency: norms, rotation,
// cache append, SwiGLU and the draft head's gather happen inside the products and the attention (45 -> 27 launches for a
// step of the 2-layer, 256-wide model with four drafts), every load of a wave is requested ahead of its arithmetic,
// and sums over lanes are register moves.
#include <string.h>

#include "hawk_internal.h"

namespace hawk {

namespace {

template <int CTRL> __device__ __forceinline__ double dpp_move(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double lane_value(double v, int l) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l), hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Sum over groups of L lanes (8, 16, 32), the same value in every lane of a group.
template <int L> __device__ __forceinline__ double group_sum(double v) {
    v += dpp_move<0xB1>(v);     // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);     // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);    // row_half_mirror
    if (L >= 16) v += dpp_move<0x140>(v);   // row_mirror
    if (L >= 32) v += __shfl_xor(v, 16);
    return v;
}
__device__ __forceinline__ double wave_total(double v) {
    v = group_sum<16>(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Four sums over the wave at once: lanes 16 g .. 16 g + 15 get that of value quad_of(g).  Two lane swaps fold two values into
// one register each, so that the steps within rows of 16 lanes are taken once for all four (21 instructions instead of 100).
__device__ __forceinline__ int quad_of(int g) { return (g >> 1) | ((g & 1) << 1); }
__device__ __forceinline__ double fold32(double a, double b) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) + __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double fold16(double a, double b) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) + __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double quad_total(double v0, double v1, double v2, double v3) {
    return group_sum<16>(fold16(fold32(v0, v1), fold32(v2, v3)));
}

// ------------------------------------------------------------------------------------------ products

enum { kNormed = 0, kLogits, kSwiglu, kResidual, kDraft };
struct Product {
    const double* A;           // [M] rows, lda apart (kDraft: the previous head output)
    size_t lda;
    const float* W;            // [N][K] (kSwiglu: [2 N][K], W1 rows then W3 rows)
    int N, K, M;
    const float* gain;         // kNormed, kLogits, kSwiglu: A is normalised (over K) and times gain
    double eps;
    double* Y;                 // results, ldy apart (kResidual: added to)
    int ldy;
    float* logits;             // kLogits: where the results go instead, as fp32
    const float* E;            // kDraft: row s of A is [previous head output | E[left] | E[up]] of draft i of sequence s
    const int32_t *n, *k_eff, *grid, *draft;
    int i, B, cells, IW, kstride;
};

// One wave: NC columns (kSwiglu: NC / 2 of W1 and the matching ones of W3) over up to RT rows; KW waves of a workgroup
// split K.  A normalised row's factor commutes with the product: the sum of squares is taken on the way.
template <int MODE, int RT, int NC, int KW>
__global__ __launch_bounds__(256) void product_kernel(Product g) {
    __shared__ double part[4][(RT + 3) / 4 * 4 * NC];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int kw = wave % KW, r0 = blockIdx.y * RT;
    constexpr int OUT = MODE == kSwiglu ? NC / 2 : NC;   // results of a row
    const int n0 = (blockIdx.x * (4 / KW) + wave / KW) * OUT;
    constexpr bool NORM = MODE == kNormed || MODE == kLogits || MODE == kSwiglu;
    const float* w[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) w[j] = g.W + (size_t)(j / OUT * g.N + min(n0 + j % OUT, g.N - 1)) * g.K;
    const double* a[RT];
    const float *left[RT], *up[RT];   // kDraft (null: zeros)
    bool on[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int row = min(r0 + r, g.M - 1);
        a[r] = g.A + (size_t)row * g.lda;
        on[r] = true;
        left[r] = up[r] = nullptr;
        if (MODE == kDraft) {
            const int b = row % g.B;
            on[r] = g.i <= g.k_eff[b];
            if (on[r]) {
                const int n = g.n[b], t = n - 1 + g.i;
                const int lt = g.i == 1 ? g.grid[(size_t)b * g.cells + n - 1] : g.draft[b * g.kstride + g.i - 2];
                const int ut = t >= g.IW ? g.grid[(size_t)b * g.cells + t - g.IW] : -1;
                const int d = g.K / 3;
                left[r] = g.E + (size_t)lt * d;
                if (ut >= 0) up[r] = g.E + (size_t)ut * d;
            }
        }
    }
    double acc[NC][RT], ss[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        ss[r] = 0.0;
#pragma unroll
        for (int j = 0; j < NC; ++j) acc[j][r] = 0.0;
    }
#pragma unroll 2
    for (int c = (kw * 64 + lane) * 4; c < g.K; c += KW * 256) {
        float4 wv[NC], gv = make_float4(1.f, 1.f, 1.f, 1.f);
        double x[RT][4];
#pragma unroll
        for (int j = 0; j < NC; ++j) wv[j] = *reinterpret_cast<const float4*>(w[j] + c);
        if (NORM) gv = *reinterpret_cast<const float4*>(g.gain + c);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if (MODE == kDraft) {
                const int d = g.K / 3, seg = c >= 2 * d ? 2 : c >= d ? 1 : 0;   // (d is a multiple of 8)
                x[r][0] = x[r][1] = x[r][2] = x[r][3] = 0.0;
                const float* e = seg == 1 ? left[r] : up[r];
                if (on[r] && seg == 0) {
                    const double2 u = *reinterpret_cast<const double2*>(a[r] + c), v = *reinterpret_cast<const double2*>(a[r] + c + 2);
                    x[r][0] = u.x; x[r][1] = u.y; x[r][2] = v.x; x[r][3] = v.y;
                } else if (on[r] && e) {
                    const float4 u = *reinterpret_cast<const float4*>(e + (c - seg * d));
                    x[r][0] = u.x; x[r][1] = u.y; x[r][2] = u.z; x[r][3] = u.w;
                }
            } else {
                const double2 u = *reinterpret_cast<const double2*>(a[r] + c), v = *reinterpret_cast<const double2*>(a[r] + c + 2);
                x[r][0] = u.x; x[r][1] = u.y; x[r][2] = v.x; x[r][3] = v.y;
            }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if (NORM) {
                ss[r] += x[r][0] * x[r][0] + x[r][1] * x[r][1] + x[r][2] * x[r][2] + x[r][3] * x[r][3];
                x[r][0] *= gv.x; x[r][1] *= gv.y; x[r][2] *= gv.z; x[r][3] *= gv.w;
            }
#pragma unroll
            for (int j = 0; j < NC; ++j)
                acc[j][r] += x[r][0] * wv[j].x + x[r][1] * wv[j].y + x[r][2] * wv[j].z + x[r][3] * wv[j].w;
        }
    }
    // lane (g, q NC + j) finishes column j of row 4 q + quad_of(g)
    constexpr int RQ = (RT + 3) / 4;
    const int sub = lane & 15, mq = sub / NC, mj = sub % NC, rr = 4 * mq + quad_of(lane >> 4);
    double mine = 0.0, other = 0.0, mss = 0.0;   // (other: kSwiglu, W3's columns)
#pragma unroll
    for (int q = 0; q < RQ; ++q) {
        auto quad = [&](const double (&v)[RT]) {
            return quad_total(v[4 * q], 4 * q + 1 < RT ? v[4 * q + 1 < RT ? 4 * q + 1 : 0] : 0.0, 4 * q + 2 < RT ? v[4 * q + 2 < RT ? 4 * q + 2 : 0] : 0.0,
                              4 * q + 3 < RT ? v[4 * q + 3 < RT ? 4 * q + 3 : 0] : 0.0);
        };
        if (NORM) {
            const double t = quad(ss);
            mss = mq == q ? t : mss;
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const double t = quad(acc[j]);
            if (j >= OUT) other = mq == q && mj == j - OUT ? t : other;
            else mine = mq == q && mj == j ? t : mine;
        }
    }
    if (KW > 1) {
        if (sub < RQ * NC) part[wave][rr * NC + mj] = mine;
        __syncthreads();
        if (kw != 0) return;
        if (sub < RQ * NC) {
#pragma unroll
            for (int w2 = 1; w2 < KW; ++w2) mine += part[wave + w2][rr * NC + mj];
        }
    }
    const int row = r0 + rr, col = n0 + mj;
    if (sub >= RQ * NC || rr >= RT || row >= g.M || col >= g.N || mj >= OUT) return;
    const double scale = NORM ? 1.0 / sqrt(mss / (double)g.K + g.eps) : 1.0;
    if (MODE == kSwiglu) {
        const double p = mine * scale, q = other * scale;
        g.Y[(size_t)row * g.ldy + col] = p / (1.0 + exp(-p)) * q;
    } else if (MODE == kLogits) g.logits[(size_t)row * g.ldy + col] = (float)(mine * scale);
    else if (MODE == kResidual) g.Y[(size_t)row * g.ldy + col] += mine;
    else g.Y[(size_t)row * g.ldy + col] = mine * scale;
}

template <int MODE, int RT, int NC, int KW> void launch_tile(hipStream_t stream, const Product& g) {
    const int cols = (4 / KW) * (MODE == kSwiglu ? NC / 2 : NC);
    product_kernel<MODE, RT, NC, KW><<<dim3((g.N + cols - 1) / cols, (g.M + RT - 1) / RT), 256, 0, stream>>>(g);
}
// Few rows are chains of launches near their latency: one result a wave (four where the columns are many, the output layer:
// the rows' activations, 2 KB each, would be drawn once per column of 1 KB), K over four waves where the columns are few.
template <int MODE, int NC, int KW> bool launch_few(hipStream_t stream, const Product& g) {
    if (g.M == 1) launch_tile<MODE, 1, NC, KW>(stream, g);
    else if (g.M == 2) launch_tile<MODE, 2, NC, KW>(stream, g);
    else if (g.M <= 4) launch_tile<MODE, 4, NC, KW>(stream, g);
    else if (g.M <= 6) launch_tile<MODE, 6, NC, KW>(stream, g);
    else return false;
    return true;
}
// More rows are bound by fp64 issue and by the activations' way through L1 (8 bytes a value against 4 of a weight): several
// columns share a row's sum of squares, its gain and its loads, once one column a wave would be more waves than the units
// hold a few of.  Microseconds of one column (one of W1|W3; K over four waves where it is long) -> of the choice: QKV of 256
// wide, 24 rows 4.3 -> 3.9, of 2048 wide, 400 rows 1419 -> 567 (N * rows / 8 = 2304, 307200; at 1536 3.75 and 3.81); W1|W3
// of 256 wide, 16 rows 4.5 -> 4.0, 2048 wide, 400 rows 1553 -> 1048 (1408 pairs of waves; at 880 3.7 and 4.1); Wo, W2 with K
// over four waves: two columns 768 wide, 16 rows 15.6 -> 7.6, 2048 wide, 16 rows 100 -> 43, and from 4096 waves on four columns
// without the split, 1024 wide, 64 rows 80.6 -> 24.1 (two 31.9; at 3072 19.5 and 14.7), 2048 wide, 400 rows 2225 -> 594.
void launch_normed(hipStream_t stream, const Product& g) {
    if (launch_few<kNormed, 1, 1>(stream, g)) return;
    if ((long)g.N * ((g.M + 7) / 8) > 1536) launch_tile<kNormed, 8, 4, 1>(stream, g);
    else launch_tile<kNormed, 8, 1, 1>(stream, g);
}
void launch_swiglu_product(hipStream_t stream, const Product& g) {
    if (launch_few<kSwiglu, 2, 1>(stream, g)) return;
    if ((long)g.N * ((g.M + 7) / 8) > 1280) launch_tile<kSwiglu, 8, 4, 1>(stream, g);
    else launch_tile<kSwiglu, 8, 2, 1>(stream, g);
}
void launch_residual(hipStream_t stream, const Product& g) {
    const bool split = g.K > 256;
    if (split ? launch_few<kResidual, 1, 4>(stream, g) : launch_few<kResidual, 1, 1>(stream, g)) return;
    if ((long)g.N * ((g.M + 7) / 8) > (split ? 4096 : 1280)) launch_tile<kResidual, 8, 4, 1>(stream, g);
    else if (split) launch_tile<kResidual, 8, 2, 4>(stream, g);
    else launch_tile<kResidual, 8, 1, 1>(stream, g);
}

// ------------------------------------------------------------------------------------------ attention

__global__ void rope_table_kernel(const double* inv_freq, double2* tab, int pairs, int positions) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= pairs * positions) return;
    double sn, cs;
    sincos((double)(i / pairs) * inv_freq[i % pairs], &sn, &cs);
    tab[i] = make_double2(cs, sn);
}

struct Attn {
    const double* qkv;     // [M][3 d] raw projections
    double *Kc, *Vc;       // the layer's cache: [sequence][head][position][HD]
    const double2* rope;   // [position][HD / 2]
    RowMap map;
    int d, H, Tmax;
    double* out;           // [M][d]
};

// One workgroup per (head, row): rotates its query and key, appends key and value to the cache, and attends the cached
// entries and the pass's own rows - those from the raw projections, whoever appends them - up to its own (tree rows:
// its ancestors and itself).  HD / 4 lanes share a position.
template <int HD>
__global__ __launch_bounds__(256) void attn_kernel(Attn a) {
    constexpr int LP = HD / 4, STEP = 256 / LP;   // lanes per position, positions per look of the workgroup
    extern __shared__ double sc[];                // [Tmax] scores
    __shared__ double sq[HD], part[256], red[4];
    const int R = blockIdx.y, h = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const RowMap& m = a.map;
    const int s = R / m.rows_per_seq, r = R - s * m.rows_per_seq, b = s % m.batch;
    int root = 0;   // entry of the pass's first row = number of cached ones
    if (m.mode != 0) {
        if (r > m.k_eff[b]) return;
        root = m.n_cond + m.n[b] - 1;
    }
    const bool tree = m.mode == 2;
    auto pos_of = [&](int row) { return root + (tree ? m.tree_depth[row] : row); };
    const unsigned long long sees = tree ? m.tree_anc[r] | (1ull << r) : ~0ull;
    const size_t base = ((size_t)s * a.H + h) * a.Tmax * HD;
    const double* own = a.qkv + (size_t)R * 3 * a.d + (size_t)h * HD;
    if (tid < HD / 2) {
        const double2 t = a.rope[(size_t)pos_of(r) * (HD / 2) + tid], q = reinterpret_cast<const double2*>(own)[tid];
        sq[2 * tid] = q.x * t.x - q.y * t.y;
        sq[2 * tid + 1] = q.x * t.y + q.y * t.x;
    } else if (tid >= 64 && tid < 64 + HD / 2) {
        const int p = tid - 64;
        const double2 t = a.rope[(size_t)pos_of(r) * (HD / 2) + p], k = reinterpret_cast<const double2*>(own + a.d)[p];
        *reinterpret_cast<double2*>(a.Kc + base + (size_t)(root + r) * HD + 2 * p) = make_double2(k.x * t.x - k.y * t.y, k.x * t.y + k.y * t.x);
    } else if (tid >= 128 && tid < 128 + HD / 2) {
        const int p = tid - 128;
        *reinterpret_cast<double2*>(a.Vc + base + (size_t)(root + r) * HD + 2 * p) = reinterpret_cast<const double2*>(own + 2 * a.d)[p];
    }
    __syncthreads();
    const int dg = tid % LP, T = root + r + 1;
    const double scale = 1.0 / sqrt((double)HD);
    double q[4], mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = sq[dg * 4 + e];
    auto score = [&](int t, double2 k0, double2 k1, bool seen) {
        double v = group_sum<LP>(q[0] * k0.x + q[1] * k0.y + q[2] * k1.x + q[3] * k1.y) * scale;
        v = seen ? v : -INFINITY;
        if (dg == 0) sc[t] = v;
        mx = v > mx ? v : mx;
    };
    int t = tid / LP;
    for (; t < root; t += 4 * STEP) {   // four looks' keys requested together (past the cached ones: the last again)
        double2 k[4][2];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double2* src = reinterpret_cast<const double2*>(a.Kc + base + (size_t)min(t + u * STEP, root - 1) * HD + dg * 4);
            k[u][0] = src[0];
            k[u][1] = src[1];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (t + u * STEP < root) score(t + u * STEP, k[u][0], k[u][1], true);
    }
    t = root + tid / LP;
    const double* rows = a.qkv + (size_t)(R - r) * 3 * a.d + (size_t)h * HD;
    for (; t < T; t += STEP) {   // the pass's own rows
        const int row = t - root;
        const double2* k = reinterpret_cast<const double2*>(rows + (size_t)row * 3 * a.d + a.d + dg * 4);
        const double2* tab = a.rope + (size_t)pos_of(row) * (HD / 2) + dg * 2;
        const double2 k0 = k[0], k1 = k[1], t0 = tab[0], t1 = tab[1];
        score(t, make_double2(k0.x * t0.x - k0.y * t0.y, k0.x * t0.y + k0.y * t0.x),
              make_double2(k1.x * t1.x - k1.y * t1.y, k1.x * t1.y + k1.y * t1.x), !tree || ((sees >> row) & 1ull));
    }
#pragma unroll
    for (int o = 32; o >= LP; o >>= 1) { const double v = __shfl_xor(mx, o); mx = v > mx ? v : mx; }
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = red[0] > red[1] ? red[0] : red[1];
    mx = red[2] > mx ? red[2] : mx;
    mx = red[3] > mx ? red[3] : mx;
    double den = 0.0;
    for (int p = tid; p < T; p += 256) {
        const double e = exp(sc[p] - mx);
        sc[p] = e;
        den += e;
    }
    den = wave_total(den);
    __syncthreads();
    if (lane == 0) red[wave] = den;
    __syncthreads();
    den = (red[0] + red[1]) + (red[2] + red[3]);
    constexpr int NS = 256 / HD;
    const int f = tid % HD;
    int p = tid / HD;
    double acc = 0.0;
#pragma unroll 4
    for (; p < root; p += NS) acc += sc[p] * a.Vc[base + (size_t)p * HD + f];
    for (; p < T; p += NS) {   // (a row that is not seen has weight 0; its value must not reach the sum)
        const int row = p - root;
        if (!tree || ((sees >> row) & 1ull)) acc += sc[p] * rows[(size_t)row * 3 * a.d + 2 * a.d + f];
    }
    part[tid] = acc;
    __syncthreads();
    if (tid < HD) {
        double o = 0.0;
#pragma unroll
        for (int q2 = 0; q2 < NS; ++q2) o += part[q2 * HD + tid];
        a.out[(size_t)R * a.d + (size_t)h * HD + tid] = o / den;
    }
}

const float* w32(hawk_ctx* c, size_t off) { return reinterpret_cast<const float*>(c->ws + c->off.blob + off); }

Product normed(hawk_ctx* c, size_t off_x, size_t lda, size_t gain, size_t W, int N, int M) {
    Product g;
    memset(&g, 0, sizeof g);
    g.A = wsp<double>(c, off_x); g.lda = lda; g.W = w32(c, W); g.N = N; g.K = c->d; g.M = M; g.gain = w32(c, gain); g.eps = c->cfg.rms_eps;
    return g;
}
void add_product(hawk_ctx* c, size_t off_a, int K, size_t W, int M) {   // x += A W^T
    Product g;
    memset(&g, 0, sizeof g);
    g.A = wsp<double>(c, off_a); g.lda = K; g.W = w32(c, W); g.N = c->d; g.K = K; g.M = M; g.Y = wsp<double>(c, c->off.x); g.ldy = c->d;
    launch_residual(c->stream, g);
}

}  // namespace

int f32_fill_rope(hawk_ctx* c) {
    const int n = c->Tmax * (c->hd / 2);
    rope_table_kernel<<<(n + 255) / 256, 256, 0, c->stream>>>(wsp<double>(c, c->off.inv_freq), wsp<double2>(c, c->off.rtab), c->hd / 2, c->Tmax);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// All decoder layers over M rows held in x (residual stream, updated in place).
void f32_layers(hawk_ctx* c, const RowMap& map, int M) {
    const int d = c->d, m = c->m;
    for (int l = 0; l < c->L; ++l) {
        Product g = normed(c, c->off.x, d, c->w.g1[l], c->w.Wqkv[l], 3 * d, M);
        g.Y = wsp<double>(c, c->off.qkv); g.ldy = 3 * d;
        launch_normed(c->stream, g);

        if (c->hd == 32 || c->hd == 64 || c->hd == 128) {
            Attn a;
            const size_t layer = (size_t)l * c->Smax * c->Tmax * d;
            a.qkv = wsp<double>(c, c->off.qkv); a.Kc = wsp<double>(c, c->off.kc) + layer; a.Vc = wsp<double>(c, c->off.vc) + layer;
            a.rope = wsp<double2>(c, c->off.rtab); a.map = map; a.d = d; a.H = c->H; a.Tmax = c->Tmax; a.out = wsp<double>(c, c->off.o);
            auto k = c->hd == 32 ? attn_kernel<32> : c->hd == 64 ? attn_kernel<64> : attn_kernel<128>;
            k<<<dim3(c->H, M), 256, (size_t)c->Tmax * sizeof(double), c->stream>>>(a);
        } else {
            launch_rope_append(c, map, l, M);
            launch_attention(c, map, l, M);
        }
        add_product(c, c->off.o, d, c->w.Wo[l], M);

        g = normed(c, c->off.x, d, c->w.g2[l], c->w.W13[l], m, M);
        g.Y = wsp<double>(c, c->off.u); g.ldy = m;
        launch_swiglu_product(c->stream, g);
        add_product(c, c->off.u, m, c->w.W2[l], M);
    }
}

// Final norm and output layer over M rows, `stride` values apart.
void f32_output_layer(hawk_ctx* c, size_t off_x, size_t stride, size_t off_logits, int M) {
    Product g = normed(c, off_x, stride, c->w.g_f, c->w.W_out + (size_t)c->cfg.samp_lo * c->d * c->esz, c->Vs, M);
    g.logits = wsp<float>(c, off_logits); g.ldy = c->Vs;
    if (!launch_few<kLogits, 4, 1>(c->stream, g)) launch_tile<kLogits, 8, 4, 1>(c->stream, g);
}

// Draft micro-step i up to its logits: head output to off_out ([S][d]), reading the previous one from off_prev.
void f32_draft_pass(hawk_ctx* c, int i, size_t off_prev, size_t off_out) {
    Product g;
    memset(&g, 0, sizeof g);
    g.A = wsp<double>(c, off_prev); g.lda = c->d; g.W = w32(c, c->w.W_d); g.N = c->d; g.K = 3 * c->d; g.M = c->S;
    g.Y = wsp<double>(c, off_out); g.ldy = c->d;
    g.E = w32(c, c->w.E); g.n = wsp<int32_t>(c, c->off.n); g.k_eff = wsp<int32_t>(c, c->off.k_eff); g.grid = wsp<int32_t>(c, c->off.grid);
    g.draft = wsp<int32_t>(c, c->off.draft); g.i = i; g.B = c->B; g.cells = c->N; g.IW = c->gw; g.kstride = c->kmax + 1;
    if (!launch_few<kDraft, 1, 4>(c->stream, g)) launch_tile<kDraft, 8, 1, 4>(c->stream, g);
    f32_output_layer(c, off_out, c->d, c->off.dlogit_s, c->S);
}

}  // namespace hawk
