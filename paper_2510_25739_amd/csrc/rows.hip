// The target pass and the draft head over many rows (several prompts, guidance, the prompt pass, large
// candidate trees) for bf16 weights: five launches per decoder layer.
//
// Activations travel between the kernels as "planes": a value v is held as bf16 hi + bf16 lo (about 16 bits,
// two MFMAs per weight tile), and a plane is stored in MFMA operand order - 16 rows x 32 features are one
// contiguous kilobyte (plane_at) - so that every request of a wave is a whole kilobyte, like those for
// the tile-major weights.  Whoever produces a vector writes its planes; no launch only converts or copies.
//
// RMSNorm costs no launch either: the producer of the residual stream x writes the planes of x * gain and,
// per row, partial sums of squares of x; the product that reads the planes multiplies its results by the
// row's 1 / rms (a row's factor commutes with the product).
#include <string.h>

#include <algorithm>

#include "hawk_internal.h"

namespace hawk {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// Resource over `bytes` bytes from a wave-uniform address: requests past the end return zeros and move nothing.
__device__ __forceinline__ rsrc_t bounded(const void* base, unsigned bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    const uint64_t u = ((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32)) << 32) |
                       (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}

// Tile-major copy of W[N][K] (N % 16 == 0, K % 32 == 0): tile (strip s, k-tile kt) is the 1 KB
// block number s * (K / 32) + kt; inside it lane l of a wave owns bytes 16 l .. 16 l + 15 = row
// s * 16 + l % 16, columns kt * 32 + (l / 16) * 8 .. + 7: one MFMA A operand per tile.
// pairs > 0 (W1|W3, pairs = m): strip s holds W1 rows 8 s .. 8 s + 7 and the matching W3 rows
// interleaved (row 2 j = W1 row 8 s + j, row 2 j + 1 = W3 row 8 s + j), so that an MFMA result lane
// holds both halves of a SwiGLU pair.  Hidden features come in whole k-tiles: rows of W1|W3 and columns of W2 from m up
// to the next multiple of 32 are zeros, and so are the features between them.  cols: columns of W (m for W2, else K).
__global__ void pack_tiles_kernel(const uint16_t* W, int K, int cols, v4u* dst, size_t total, int pairs) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int lane = (int)(i & 63), r = lane & 15;
    const size_t tile = i >> 6, kts = (size_t)K / 32, s = tile / kts, kt = tile - s * kts;
    const size_t row = pairs ? (size_t)(r & 1) * pairs + s * 8 + (r >> 1) : s * 16 + r;
    const size_t col = kt * 32 + (lane >> 4) * 8;
    const bool inside = col < (size_t)cols && (!pairs || s * 8 + (r >> 1) < (size_t)pairs);
    dst[i] = inside ? *reinterpret_cast<const v4u*>(W + row * (size_t)cols + col) : (v4u){0u, 0u, 0u, 0u};
}

// Sum over the wave's 64 lanes, the same value in every lane.
template <int CTRL> __device__ __forceinline__ float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_value(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }
__device__ __forceinline__ float wave_total(float v) {
    v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);   // row_half_mirror
    v += dpp_move<0x140>(v);   // row_mirror
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Lane ^ 16 and lane ^ 32 by lane swaps (a shuffle goes through the LDS crossbar).
#define HAWK_SWAP(NAME, WIDTH, OP)                                                                                       \
    __device__ __forceinline__ float NAME(float v) {                                                                    \
        const auto r = __builtin_amdgcn_permlane##WIDTH##_swap(__float_as_uint(v), __float_as_uint(v), false, false);   \
        return OP(__uint_as_float(r[0]), __uint_as_float(r[1]));                                                        \
    }
__device__ __forceinline__ float addf(float a, float b) { return a + b; }
HAWK_SWAP(sum16, 16, addf)
HAWK_SWAP(sum32, 32, addf)
HAWK_SWAP(max16, 16, fmaxf)
HAWK_SWAP(max32, 32, fmaxf)
#undef HAWK_SWAP

// Four consecutive features f .. f + 3 (f % 4 == 0) of a row into the two planes.
__device__ __forceinline__ void store_planes4(uint16_t* hi, uint16_t* lo, int row, int f, int kts, f32x4 v) {
    unsigned h0, h1, h2, h3, l0, l1, l2, l3;
    bf16_split(v[0], h0, l0);
    bf16_split(v[1], h1, l1);
    bf16_split(v[2], h2, l2);
    bf16_split(v[3], h3, l3);
    const size_t at = plane_at(row, f, kts);
    *reinterpret_cast<uint2*>(hi + at) = make_uint2(h0 | (h1 << 16), h2 | (h3 << 16));
    *reinterpret_cast<uint2*>(lo + at) = make_uint2(l0 | (l1 << 16), l2 | (l3 << 16));
}
__device__ __forceinline__ f32x4 gains4(const uint16_t* g) {
    const uint2 w = *reinterpret_cast<const uint2*>(g);
    return (f32x4){__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16),
                   __uint_as_float(w.y & 0xFFFF0000u)};
}

// ------------------------------------------------------------------------------------------ products

// Lane's share of a row's partial sums of squares: the four it loaded before, and those past the first 256 (d > 4096).
__device__ __forceinline__ float ssq_share(const RowsGemm& g, int row, int lane, f32x4 first) {
    float v = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) v += lane * 4 + e < g.ssq_n ? first[e] : 0.f;
    for (int p = 256 + lane; p < g.ssq_n; p += 64) v += g.ssq[(size_t)row * g.ssq_ld + p];
    return v;
}

// A workgroup past a launch's own: brings its share of what the next launches read into the L2 it will be read from.  Their
// workgroup i runs on XCD i % 8 and so do strip group i % 8, + 8, .. of its weights; so do the workgroups here.
// (Kernels have an instance without this: the parameters and the look at them cost 0.2 us a launch.)
__device__ __forceinline__ void bring_ahead(const Ahead& a, int wave, int waves, int lane) {
    const int x = blockIdx.x & 7, all = (a.extra >> 3) * waves, mine = (((int)blockIdx.x - a.grid) >> 3) * waves + wave;
    for (int i = 0; i < a.n; ++i) {
        const int kb = a.of[i].kb, share = max(0, (a.of[i].groups - x + 7) >> 3) * kb;
        const rsrc_t r = bounded(a.of[i].W, (unsigned)a.of[i].total_kb * 1024u);
        for (int u = mine; u < share; u += 8 * all) {
            v4u v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = u + j * all, g = k / kb;
                const unsigned at = k < share ? (unsigned)(((g << 3) + x) * kb + (k - g * kb)) * 1024u + (unsigned)lane * 16u : 0x80000000u;
                v[j] = __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) asm volatile("" ::"v"(v[j]));
        }
    }
}

// What follows a product, for one result lane: features f .. f + 3 of a row (lane group kg of the strip).
template <int MODE>
__device__ __forceinline__ void gemm_epilogue(const RowsGemm& g, f32x4 v, int row, int f, bool strip_ok, int kg, float scale) {
    const bool live = row < g.M && strip_ok;
    if (g.ssq_n > 0) v *= scale;
    if (MODE == kGemmSwiglu) {   // pair-interleaved W1|W3 rows: (a0, b0, a1, b1) -> hidden features f / 2, f / 2 + 1
        if (live) {
            const float h0 = v[0] / (1.0f + expf(-v[0])) * v[1], h1 = v[2] / (1.0f + expf(-v[2])) * v[3];
            unsigned a0, b0, a1, b1;
            bf16_split(h0, a0, b0);
            bf16_split(h1, a1, b1);
            const size_t at = plane_at(row, f / 2, g.okts);
            *reinterpret_cast<unsigned*>(g.ohi + at) = a0 | (a1 << 16);
            *reinterpret_cast<unsigned*>(g.olo + at) = b0 | (b1 << 16);
        }
        return;
    }
    if (MODE == kGemmHeads) {   // square blocks of K features (draft heads): g = a + silu(y), row (row * blocks + block)
        if (live) {
            const int j = f / g.K, fb = f - j * g.K, orow = row * g.blocks + j;
            const float4 a = *reinterpret_cast<const float4*>(g.resid + (size_t)row * g.K + fb);
            v = (f32x4){a.x + v[0] / (1.0f + expf(-v[0])), a.y + v[1] / (1.0f + expf(-v[1])), a.z + v[2] / (1.0f + expf(-v[2])),
                        a.w + v[3] / (1.0f + expf(-v[3]))};
            if (g.Y) *reinterpret_cast<float4*>(g.Y + (size_t)orow * g.K + fb) = make_float4(v[0], v[1], v[2], v[3]);
            store_planes4(g.ohi, g.olo, orow, fb, g.okts, v);
        }
        return;
    }
    float* dst = g.Y + (size_t)row * g.ldy + f;
    if (live) {
        if (MODE == kGemmResidual) {
            const float4 old = *reinterpret_cast<const float4*>(dst);
            v += (f32x4){old.x, old.y, old.z, old.w};
        }
        *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
        if (g.ohi) store_planes4(g.ohi, g.olo, row, f, g.okts, v * gains4(g.gain + f));
    }
    if (g.ossq) {   // the strip's share of the row's sum of squares
        float p = (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
        p = sum32(sum16(p));
        if (live && kg == 0) g.ossq[(size_t)row * g.ossq_ld + (f >> 4)] = p;
    }
}

// Y = A W^T and what follows it, A as planes.  A workgroup owns SR strips of 16 features and CT tiles of 16
// rows; its KW waves split K and work alone - weight tiles and plane tiles straight into registers in operand
// order, D k-steps of 32 in flight, no LDS and no barrier in the loop - and add their partial results
// through LDS at the end, where each takes its share of the tiles through the epilogue.
// A k-step draws SR + 2 CT kilobytes for SR CT tiles of 2 MFMAs, every byte fetched once per workgroup; the tile is chosen per
// shape (pick_kernel).  Workgroups that share weights follow each other on one XCD, so that the second finds them in its L2.
// Bound by the weights' way from memory: 64 groups of strips by 4 of rows take in 60 to 115 KB a microsecond and unit over a
// k-step (79 with (7, 3) tiles, 2.8 TB/s of weights), 110 to 150 when the weights are in L2 already, and one workgroup alone
// 130 to 240; so the tile with the fewest bytes for a unit's share of the output is the fastest.  Eight waves rather than four
// shorten what comes before and after (W1|W3 of 192 rows at the XL widths: two (4, 3) workgroups to a unit 17.2 us, (7, 3) of
// four waves 17.1 us, of eight 15.1 us).
template <int SR, int CT, int D, int KW, bool PACKED, int MODE>
__device__ __forceinline__ void rows_gemm(const RowsGemm& g) {
    constexpr int PW = KW * SR * CT > 128 ? KW / 2 : KW;   // waves whose partial results LDS holds at a time
    __shared__ f32x4 part[PW][SR * CT][64];
    __shared__ float rscale[16 * CT];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4;
    // workgroup i runs on XCD i % 8: the row groups of a strip group follow each other on the same XCD
    const int strips = g.N / 16, tiles = (g.M + 15) / 16, groups = (tiles + CT - 1) / CT, i8 = blockIdx.x >> 3;
    const int s_first = ((i8 / groups) * 8 + (blockIdx.x & 7)) * SR, t_first = (i8 % groups) * CT;
    if (s_first >= strips) return;
    const int nk = g.K / 32, k0 = wave * nk / KW, n = (wave + 1) * nk / KW - k0;

    // rows' sums of squares first: their requests come back before everything else
    constexpr int RPW = (16 * CT + KW - 1) / KW;   // rows per wave
    f32x4 sq[RPW];
    if (g.ssq_n > 0) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            // straight-line: a loop per row would wait for each row in turn
            const int r = min(t_first * 16 + wave + i * KW, g.M - 1);
            sq[i] = *reinterpret_cast<const f32x4*>(g.ssq + (size_t)r * g.ssq_ld + min(lane * 4, g.ssq_ld - 4));
        }
    }
    rsrc_t rw[SR], rh[CT], rl[CT];
    const unsigned wl = (unsigned)(r16 * g.K + k0 * 32 + kg * 8) * 2u;   // row-major: the lane's first piece in a strip
#pragma unroll
    for (int s = 0; s < SR; ++s) {
        const int strip = min(s_first + s, strips - 1);   // strips past the end repeat the last (never stored)
        rw[s] = PACKED ? bounded(g.W + ((size_t)strip * nk + k0) * 512, n * 1024) : bounded(g.W + (size_t)strip * 16 * g.K, (unsigned)g.K * 32u);
    }
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const int tile = min(t_first + t, tiles - 1);
        rh[t] = bounded(g.hi + ((size_t)tile * nk + k0) * 512, n * 1024);
        rl[t] = bounded(g.lo + ((size_t)tile * nk + k0) * 512, n * 1024);
    }
    struct Step { v4u w[SR], h[CT], l[CT]; };
    auto load = [&](int s, Step& st) {
        const unsigned at = (unsigned)lane * 16u + (unsigned)s * 1024u;
#pragma unroll
        for (int i = 0; i < SR; ++i) {
            st.w[i] = __builtin_amdgcn_raw_buffer_load_b128(rw[i], PACKED ? at : s < n ? wl + (unsigned)s * 64u : 0x80000000u, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < CT; ++i) {
            st.h[i] = __builtin_amdgcn_raw_buffer_load_b128(rh[i], at, 0, 0);
            st.l[i] = __builtin_amdgcn_raw_buffer_load_b128(rl[i], at, 0, 0);
        }
    };
    f32x4 acc[SR][CT];
#pragma unroll
    for (int s = 0; s < SR; ++s)
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[s][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto fma_step = [&](const Step& st) {
#pragma unroll
        for (int s = 0; s < SR; ++s)
#pragma unroll
            for (int t = 0; t < CT; ++t)
                acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, st.w[s]), __builtin_bit_cast(bf16x8, st.h[t]), acc[s][t], 0, 0, 0);
#pragma unroll
        for (int s = 0; s < SR; ++s)
#pragma unroll
            for (int t = 0; t < CT; ++t)
                acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, st.w[s]), __builtin_bit_cast(bf16x8, st.l[t]), acc[s][t], 0, 0, 0);
    };
    Step ring[D];
#pragma unroll
    for (int j = 0; j < D; ++j) load(j, ring[j]);
    if (g.ssq_n > 0) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const float v = wave_total(ssq_share(g, min(t_first * 16 + wave + i * KW, g.M - 1), lane, sq[i]));
            if (lane == 0 && wave + i * KW < 16 * CT) rscale[wave + i * KW] = 1.0f / sqrtf(v / g.norm_d + g.eps);
        }
    }
    for (int s = 0; s < n; s += D) {   // steps past the end multiply zeros
#pragma unroll
        for (int j = 0; j < D; ++j) {
            fma_step(ring[j]);
            load(s + j + D, ring[j]);
        }
    }
    if (PW < KW) {   // the upper waves' first, added by the lower ones
        if (wave >= PW) {
#pragma unroll
            for (int s = 0; s < SR; ++s)
#pragma unroll
                for (int t = 0; t < CT; ++t) part[wave - PW][s * CT + t][lane] = acc[s][t];
        }
        __syncthreads();
        if (wave < PW) {
#pragma unroll
            for (int s = 0; s < SR; ++s)
#pragma unroll
                for (int t = 0; t < CT; ++t) acc[s][t] += part[wave][s * CT + t][lane];
        }
    }
    if (wave < PW) {
#pragma unroll
        for (int s = 0; s < SR; ++s)
#pragma unroll
            for (int t = 0; t < CT; ++t) part[wave][s * CT + t][lane] = acc[s][t];
    }
    __syncthreads();
    // lane holds features 16 (s_first + s) + 4 kg .. + 3 of row 16 (t_first + t) + r16
    for (int q = wave; q < SR * CT; q += KW) {
        const int s = q / CT, t = q - s * CT, strip = s_first + s, row = (t_first + t) * 16 + r16, f = strip * 16 + 4 * kg;
        f32x4 v = part[0][q][lane];
#pragma unroll
        for (int w = 1; w < PW; ++w) v += part[w][q][lane];
        gemm_epilogue<MODE>(g, v, row, f, strip < strips, kg, rscale[t * 16 + r16]);
    }
}

template <int SR, int CT, int D, int KW, bool PACKED, int MODE>
__global__ __launch_bounds__(64 * KW) void rows_gemm_kernel(RowsGemm g) { rows_gemm<SR, CT, D, KW, PACKED, MODE>(g); }
template <int SR, int CT, int D, int KW, int MODE>
__global__ __launch_bounds__(64 * KW) void rows_gemm_ahead_kernel(RowsGemm g, Ahead a) {
    if ((int)blockIdx.x >= a.grid) bring_ahead(a, __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), KW, threadIdx.x & 63);
    else rows_gemm<SR, CT, D, KW, true, MODE>(g);
}

// The same product where the rows are many enough to be a contraction (the prompt pass): a workgroup of WN x WM
// waves owns (WN SR) strips x (WM CT) row tiles; weight and plane tiles of a k-step go to LDS - whole tiles of 1 KB
// in operand order, moved by the load unit itself (no registers, no address arithmetic, no bank conflicts) - S
// stages deep, and every wave reads the SR + 2 CT tiles of its part for 2 SR CT MFMAs.  A k-step of a 20 x 12 tile is
// 1920 cycles of MFMA, 44 KB from L2 and 136 KB out of LDS.  Measured at 3840 rows of 3840 x 1280 (73 us): matrix cores
// 41 % busy, 11 bytes per cycle from L2, no bank conflicts; with one workgroup to a unit its waves meet at a
// barrier per k-step and nothing else runs meanwhile.  The k-steps' loads are counted by hand (inline assembly): hipcc would wait for all of them
// before every read of LDS.  The load reads M0 one wait state after it was written at the earliest; the compiler
// does not look into the block, so the s_nop is ours, and M0 is named as changed.
__device__ __forceinline__ void tile_to_lds(const uint16_t* src, const uint16_t* dst) {   // src per lane, dst wave-uniform
    const unsigned at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const uint16_t*)dst;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // M0 is never allocated, only written before an instruction that reads it
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(__builtin_amdgcn_readfirstlane((int)at)), "v"(src)
                 : "memory", "m0");
#pragma clang diagnostic pop
}
template <int WN, int WM, int SR, int CT, int S, bool PACKED, int MODE>
__global__ __launch_bounds__(64 * WN * WM) void rows_gemm_staged_kernel(RowsGemm g) {
    constexpr int NWV = WN * WM, BS = WN * SR, BT = WM * CT, NTL = BS + 2 * BT, LPW = (NTL + NWV - 1) / NWV;
    extern __shared__ __attribute__((aligned(1024))) uint16_t stage[];   // [S][NTL][512]
    __shared__ float rscale[16 * BT];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4, wn = wave / WM, wm = wave - wn * WM;
    const int strips = g.N / 16, tiles = (g.M + 15) / 16, nk = g.K / 32;
    // Workgroup i runs on XCD i % 8: an XCD takes a contiguous piece of the list (row groups outer, strip groups
    // inner), so that the row groups it works on at a time stay in its L2.
    const int sg = (strips + BS - 1) / BS, total = sg * ((tiles + BT - 1) / BT);
    const int per = (total + 7) / 8, id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || id >= total) return;
    const int s_first = (id % sg) * BS, t_first = (id / sg) * BT;

    // this wave's tiles of a stage: numbers wave, wave + NWV, .. (past the end: the first ones again, same bytes)
    const uint16_t* src[LPW];
    int slot[LPW], step[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        int q = wave + i * NWV;
        if (q >= NTL) q -= NTL;
        slot[i] = q * 512;
        const int strip = min(s_first + q, strips - 1), tile = min(t_first + (q < BS + BT ? q - BS : q - BS - BT), tiles - 1);
        src[i] = (q < BS ? g.W + (size_t)strip * nk * 512 : (q < BS + BT ? g.hi : g.lo) + (size_t)tile * nk * 512) + lane * 8;
        step[i] = 512;
        if (!PACKED && q < BS) {   // row-major: the lane's own row of the strip
            src[i] = g.W + (size_t)(strip * 16 + r16) * g.K + kg * 8;
            step[i] = 32;
        }
    }
    auto request = [&](int k) {   // k-steps past the end: the last one again, into a stage nobody reads any more
        const int kc = min(k, nk - 1), buf = (k % S) * NTL * 512;
#pragma unroll
        for (int i = 0; i < LPW; ++i) tile_to_lds(src[i] + (size_t)kc * step[i], stage + buf + slot[i]);
    };
    if (g.ssq_n > 0) {
        constexpr int RPW = 16 * BT / NWV;
        f32x4 sq[RPW];
#pragma unroll
        for (int i = 0; i < RPW; ++i)
            sq[i] = *reinterpret_cast<const f32x4*>(g.ssq + (size_t)min(t_first * 16 + wave * RPW + i, g.M - 1) * g.ssq_ld + min(lane * 4, g.ssq_ld - 4));
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const float v = wave_total(ssq_share(g, min(t_first * 16 + wave * RPW + i, g.M - 1), lane, sq[i]));
            if (lane == 0) rscale[wave * RPW + i] = 1.0f / sqrtf(v / g.norm_d + g.eps);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // written before the first barrier below, the only one where K is 32
    }
#pragma unroll
    for (int k = 0; k < S - 1; ++k) request(k);
    f32x4 acc[SR][CT];
#pragma unroll
    for (int s = 0; s < SR; ++s)
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[s][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < nk; ++k) {
        // own requests of stage k are done when at most those of the S - 2 younger stages are outstanding; behind the
        // barrier everyone's are, and nobody reads stage k - 1 any more, whose place the next request takes
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((S - 2) * LPW) : "memory");
        request(k + S - 1);
        const uint16_t* st = stage + (k % S) * NTL * 512 + lane * 8;
        bf16x8 w[SR], h[2], l[2];
        const uint16_t *sh = st + (BS + wm * CT) * 512, *sl = sh + BT * 512;
        h[0] = *reinterpret_cast<const bf16x8*>(sh);
#pragma unroll
        for (int s = 0; s < SR; ++s) w[s] = *reinterpret_cast<const bf16x8*>(st + (wn * SR + s) * 512);
        l[0] = *reinterpret_cast<const bf16x8*>(sl);
#pragma unroll
        for (int t = 0; t < CT; ++t) {   // the next row tile's planes are on their way while this one's are multiplied
            if (t + 1 < CT) {
                h[(t + 1) & 1] = *reinterpret_cast<const bf16x8*>(sh + (t + 1) * 512);
                l[(t + 1) & 1] = *reinterpret_cast<const bf16x8*>(sl + (t + 1) * 512);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < SR; ++s) acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], h[t & 1], acc[s][t], 0, 0, 0);
#pragma unroll
            for (int s = 0; s < SR; ++s) acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], l[t & 1], acc[s][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage's reads are done before the next barrier lets it be overwritten
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < SR; ++s)
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            const int strip = s_first + wn * SR + s, tr = wm * CT + t;
            gemm_epilogue<MODE>(g, acc[s][t], (t_first + tr) * 16 + r16, strip * 16 + 4 * kg, strip < strips, kg, g.ssq_n > 0 ? rscale[tr * 16 + r16] : 1.f);
        }
}

// The same with tile-major weights that go straight into registers, two k-steps ahead (three sets: the compiler waits for a
// set as if no plane tiles were in flight behind it, so for what was requested up to a k-step before), and only the planes
// through LDS, three stages deep.  Of a k-step of a 20 x 12 tile 24 KB are written to LDS and 96 KB read instead of 44 and 136,
// 1.0 us of LDS time beside 0.9 us of MFMA time at 1.95 GHz; and tiles that LDS has no stages for become possible, such as 18 x 12 on twelve
// waves (three to a SIMD cover each other's barriers) and 16 x 16.  3840 rows at the XL widths: W1|W3 148.4 us staged (20, 12),
// 140.1 this way, 129.8 with (18, 12), whose rounds are full; QKV 74.7 and 71.6.  Weight tiles that several waves share come
// from L1; the smaller (8, 8) and (10, 8) tiles stay staged, where a wave's weights would be most of its requests (Wo of 3200
// rows 30.2 and 30.7 us).
template <int WN, int WM, int SR, int CT, int MODE>
__global__ __launch_bounds__(64 * WN * WM) void rows_gemm_wide_kernel(RowsGemm g) {
    constexpr int S = 3, NWV = WN * WM, BS = WN * SR, BT = WM * CT, NTL = 2 * BT, LPW = (NTL + NWV - 1) / NWV;
    extern __shared__ __attribute__((aligned(1024))) uint16_t stage[];   // [S][NTL][512]
    __shared__ float rscale[16 * BT];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4, wn = wave / WM, wm = wave - wn * WM;
    const int strips = g.N / 16, tiles = (g.M + 15) / 16, nk = g.K / 32;
    const int sg = (strips + BS - 1) / BS, total = sg * ((tiles + BT - 1) / BT);
    const int per = (total + 7) / 8, id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || id >= total) return;
    const int s_first = (id % sg) * BS, t_first = (id / sg) * BT;
    const uint16_t* src[LPW];
    int slot[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        int q = wave + i * NWV;
        if (q >= NTL) q -= NTL;   // (past the end: the first ones again, same bytes)
        const int tile = min(t_first + (q < BT ? q : q - BT), tiles - 1);
        slot[i] = q * 512;
        src[i] = (q < BT ? g.hi : g.lo) + (size_t)tile * nk * 512 + lane * 8;
    }
    auto request = [&](int k) {   // k-steps past the end: the last one again, into a stage nobody reads any more
        const int kc = min(k, nk - 1), buf = (k % S) * NTL * 512;
#pragma unroll
        for (int i = 0; i < LPW; ++i) tile_to_lds(src[i] + (size_t)kc * 512, stage + buf + slot[i]);
    };
    const rsrc_t rw = bounded(g.W, (unsigned)strips * (unsigned)nk * 1024u);
    unsigned first[SR];
#pragma unroll
    for (int s = 0; s < SR; ++s) first[s] = (unsigned)min(s_first + wn * SR + s, strips - 1) * (unsigned)nk * 1024u;
    auto load = [&](int k, v4u (&w)[SR]) {
        const unsigned at = (unsigned)min(k, nk - 1) * 1024u;
#pragma unroll
        for (int s = 0; s < SR; ++s) w[s] = __builtin_amdgcn_raw_buffer_load_b128(rw, (unsigned)lane * 16u, first[s] + at, 0);
    };
    if (g.ssq_n > 0) {
        constexpr int RPW = 16 * BT / NWV;
        f32x4 sq[RPW];
#pragma unroll
        for (int i = 0; i < RPW; ++i)
            sq[i] = *reinterpret_cast<const f32x4*>(g.ssq + (size_t)min(t_first * 16 + wave * RPW + i, g.M - 1) * g.ssq_ld + min(lane * 4, g.ssq_ld - 4));
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const float v = wave_total(ssq_share(g, min(t_first * 16 + wave * RPW + i, g.M - 1), lane, sq[i]));
            if (lane == 0) rscale[wave * RPW + i] = 1.0f / sqrtf(v / g.norm_d + g.eps);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // written before the first barrier below, the only one where K is 32
    }
    v4u w[3][SR];
    load(0, w[0]);
    request(0);
    load(1, w[1]);
    request(1);
    f32x4 acc[SR][CT];
#pragma unroll
    for (int s = 0; s < SR; ++s)
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[s][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto step = [&](int k, int j) {   // j = k % 3
        // own requests of k-step k are done when at most those of the next one are outstanding
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(SR + LPW) : "memory");
        load(k + 2, w[(j + 2) % 3]);
        request(k + 2);
        const uint16_t* sh = stage + j * NTL * 512 + wm * CT * 512 + lane * 8;
        const uint16_t* sl = sh + BT * 512;
        bf16x8 h[2], l[2];
        h[0] = *reinterpret_cast<const bf16x8*>(sh);
        l[0] = *reinterpret_cast<const bf16x8*>(sl);
#pragma unroll
        for (int t = 0; t < CT; ++t) {   // the next row tile's planes are on their way while this one's are multiplied
            if (t + 1 < CT) {
                h[(t + 1) & 1] = *reinterpret_cast<const bf16x8*>(sh + (t + 1) * 512);
                l[(t + 1) & 1] = *reinterpret_cast<const bf16x8*>(sl + (t + 1) * 512);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < SR; ++s) acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[j][s]), h[t & 1], acc[s][t], 0, 0, 0);
#pragma unroll
            for (int s = 0; s < SR; ++s) acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[j][s]), l[t & 1], acc[s][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage's reads are done before the next barrier lets it be overwritten
    };
    int k = 0;
    for (; k + 3 <= nk; k += 3) {
        step(k, 0);
        step(k + 1, 1);
        step(k + 2, 2);
    }
    if (k < nk) step(k, 0);
    if (k + 1 < nk) step(k + 1, 1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < SR; ++s)
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            const int strip = s_first + wn * SR + s, tr = wm * CT + t;
            gemm_epilogue<MODE>(g, acc[s][t], (t_first + tr) * 16 + r16, strip * 16 + 4 * kg, strip < strips, kg, g.ssq_n > 0 ? rscale[tr * 16 + r16] : 1.f);
        }
}

// ------------------------------------------------------------------------------------------ rows in

// One row per workgroup: x (fp32), the planes of x * gain and the row's sum of squares (one partial sum).
__device__ __forceinline__ void emit_row(const float* src32, const uint16_t* src16, int row, int d, const uint16_t* gain, float* x,
                                         uint16_t* hi, uint16_t* lo, float* ssq, int ssq_ld) {
    __shared__ float red[4];
    float ss = 0.f;
    for (int f = threadIdx.x * 4; f < d; f += 1024) {
        f32x4 v;
        if (src32) {
            const float4 a = *reinterpret_cast<const float4*>(src32 + f);
            v = (f32x4){a.x, a.y, a.z, a.w};
        } else {
            v = gains4(src16 + f);   // four bf16 values
        }
        if (x) *reinterpret_cast<float4*>(x + (size_t)row * d + f) = make_float4(v[0], v[1], v[2], v[3]);
        store_planes4(hi, lo, row, f, d / 32, v * gains4(gain + f));
        ss += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
    }
    ss = wave_total(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) ssq[(size_t)row * ssq_ld] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Step and tree rows: the embedding of the row's token - row 0 of a sequence the last committed token, row
// r > 0 draft r - 1.
__global__ __launch_bounds__(256) void rows_embed_kernel(float* X, const uint16_t* E, RowMap map, const int32_t* grid, const int32_t* draft,
                                                         int N, int kstride, int d, const uint16_t* gain, uint16_t* hi, uint16_t* lo,
                                                         float* ssq, int ssq_ld) {
    const int s = blockIdx.x / map.rows_per_seq, r = blockIdx.x - s * map.rows_per_seq, b = s % map.batch;
    int tok = 0;
    if (r <= map.k_eff[b]) tok = r == 0 ? grid[(size_t)b * N + map.n[b] - 1] : draft[b * kstride + r - 1];
    if (tok < 0) tok = 0;
    emit_row(nullptr, E + (size_t)tok * d, blockIdx.x, d, gain, X, hi, lo, ssq, ssq_ld);
}

// Prompt rows: the condition vectors.
__global__ __launch_bounds__(256) void rows_cond_kernel(float* X, const float* cond, int d, const uint16_t* gain, uint16_t* hi, uint16_t* lo,
                                                        float* ssq, int ssq_ld) {
    emit_row(cond + (size_t)blockIdx.x * d, nullptr, blockIdx.x, d, gain, X, hi, lo, ssq, ssq_ld);
}

// Rows r * stride of X (the last condition row of every sequence) as planes for the output layer.
__global__ __launch_bounds__(256) void rows_pick_kernel(const float* X, size_t stride, int d, const uint16_t* gain, uint16_t* hi,
                                                        uint16_t* lo, float* ssq, int ssq_ld) {
    emit_row(X + (size_t)blockIdx.x * stride, nullptr, blockIdx.x, d, gain, nullptr, hi, lo, ssq, ssq_ld);
}

// Draft i (1-based) of every sequence: planes of [previous head output (the target's hidden state for the
// first draft) | E[left] | E[up]].  Block (part, sequence).
__global__ __launch_bounds__(256) void rows_draft_input_kernel(const float* prev, const uint16_t* E, const int32_t* n_arr,
                                                               const int32_t* k_eff, const int32_t* grid, const int32_t* draft, int i,
                                                               int B, int N, int IW, int kstride, int d, uint16_t* hi, uint16_t* lo) {
    const int part = blockIdx.x, s = blockIdx.y, b = s % B;
    const bool on = i <= k_eff[b];
    const uint16_t* e = nullptr;
    if (on && part > 0) {
        const int n = n_arr[b], t = n - 1 + i;
        const int tok = part == 1 ? (i == 1 ? grid[(size_t)b * N + n - 1] : draft[b * kstride + i - 2])
                                  : (t >= IW ? grid[(size_t)b * N + t - IW] : -1);
        if (tok >= 0) e = E + (size_t)tok * d;
    }
    for (int f = threadIdx.x * 4; f < d; f += 1024) {
        f32x4 v = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (part == 0 && on) {
            const float4 a = *reinterpret_cast<const float4*>(prev + (size_t)s * d + f);
            v = (f32x4){a.x, a.y, a.z, a.w};
        } else if (e) {
            v = gains4(e + f);
        }
        store_planes4(hi, lo, s, part * d + f, 3 * d / 32, v);
    }
}

// Planes of the rows of A as they are.  Block (row, 1024 features).
__global__ __launch_bounds__(256) void rows_split_kernel(const float* A, int lda, int K, uint16_t* hi, uint16_t* lo) {
    const int f = blockIdx.y * 1024 + threadIdx.x * 4;
    if (f >= K) return;
    const float4 a = *reinterpret_cast<const float4*>(A + (size_t)blockIdx.x * lda + f);
    store_planes4(hi, lo, blockIdx.x, f, K / 32, (f32x4){a.x, a.y, a.z, a.w});
}

__global__ void rope_table_kernel(const double* inv_freq, float2* tab, int pairs, int positions) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= pairs * positions) return;
    double sn, cs;
    sincos((double)(i / pairs) * inv_freq[i % pairs], &sn, &cs);
    tab[i] = make_float2((float)cs, (float)sn);
}

// ------------------------------------------------------------------------------------------ attention
//
// A tile of 16 keys is the A operand of the score product (lane (key, g): features 32 ks + 8 g .. + 7, straight
// from the fp16 rows), the 16 query rows - scaled, split into an fp16 hi and lo half - the B operand; the result
// lane (row, g) holds the scores of keys 4 g .. + 3, which is the B operand of v_mfma_f32_16x16x16_f16 for the
// weighted sum of the values (weights split hi / lo as well).  Its A operand is the transposed value tile,
// which ds_read_b64_tr_b16 forms from row-major LDS: lane i of a group of 16 names 4 features of row
// i / 4, and receives column i of the four rows.
//
// A pair of halves holds a fp32 value to one unit in its last place unless the low one is subnormal, so both are moved
// up by powers of two first: a query row by its own (largest feature in [2^14, 2^15)), weights by 2^14.  Error of
// the output against float64 on the same cache, before it becomes planes (2-norm; prompt / step rows): 32 sequences of
// 120 + 6 rows, heads of 64: scalar fp32 1.9e-7 / 2.3e-7, here 1.2e-7 / 1.5e-7; heads of 128: 2.6e-7 / 2.9e-7, here
// 1.3e-7 / 1.8e-7 (pairs without the powers of two: 3.8e-6 / 9.7e-6, and queries beyond 65504 were NaN).
constexpr float kWeightScale = 16384.f;

template <int HD> struct QRow { h8 hi[HD / 32], lo[HD / 32]; float back; };   // back: what undoes the row's power of two

// Eight consecutive features of a raw projection row, and after the rotary step (pairs (2 j, 2 j + 1)).
struct Raw8 { float4 a, b, c, d; };
__device__ __forceinline__ Raw8 load_raw8(const float* src, const float2* tab) {
    return {*reinterpret_cast<const float4*>(src), *reinterpret_cast<const float4*>(src + 4), *reinterpret_cast<const float4*>(tab),
            *reinterpret_cast<const float4*>(tab + 2)};
}
__device__ __forceinline__ void rope8(const Raw8& r, float (&o)[8]) {
    const float4 a = r.a, b = r.b, c = r.c, d = r.d;
    o[0] = a.x * c.x - a.y * c.y; o[1] = a.x * c.y + a.y * c.x;
    o[2] = a.z * c.z - a.w * c.w; o[3] = a.z * c.w + a.w * c.z;
    o[4] = b.x * d.x - b.y * d.y; o[5] = b.x * d.y + b.y * d.x;
    o[6] = b.z * d.z - b.w * d.w; o[7] = b.z * d.w + b.w * d.z;
}
__device__ __forceinline__ float row_max4(float v) {   // over the four lanes that share a row
    v = max16(v);
    return max32(v);
}
__device__ __forceinline__ float row_sum4(float v) {
    v = sum16(v);
    return sum32(v);
}
template <int HD>
__device__ __forceinline__ void load_query(const float* row, const float2* tab, int kg, Raw8 (&raw)[HD / 32]) {
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks) raw[ks] = load_raw8(row + ks * 32 + kg * 8, tab + ks * 16 + kg * 4);
}
template <int HD>
__device__ __forceinline__ void split_query(const Raw8 (&raw)[HD / 32], bool on, float scale, QRow<HD>& q) {
    float v[HD / 32][8], top = 0.f;
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks) {
        rope8(raw[ks], v[ks]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[ks][e] = on ? v[ks][e] * scale : 0.f;
            top = fmaxf(top, fabsf(v[ks][e]));
        }
    }
    // exponent of the largest feature; zero and subnormal rows move by 2^126, infinite ones as if they were finite
    const int ex = (int)(__float_as_uint(row_max4(top)) >> 23);
    const int shift = max(-113, min(126, 14 + 127 - ex));
    const float up = __uint_as_float((unsigned)(127 + shift) << 23);
    q.back = __uint_as_float((unsigned)(127 - shift) << 23);
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float x = v[ks][e] * up;
            q.hi[ks][e] = (_Float16)x;
            q.lo[ks][e] = (_Float16)(x - (float)q.hi[ks][e]);
        }
}
template <int HD> __device__ __forceinline__ f32x4 score_tile(const h8 (&k)[HD / 32], const QRow<HD>& q) {
    f32x4 s = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks) s = __builtin_amdgcn_mfma_f32_16x16x32_f16(k[ks], q.lo[ks], s, 0, 0, 0);
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks) s = __builtin_amdgcn_mfma_f32_16x16x32_f16(k[ks], q.hi[ks], s, 0, 0, 0);
    return s * q.back;
}
// o += 2^14 V^T P for one tile of 16 keys whose values sit row-major in LDS (row stride vs halves).
template <int HD>
__device__ __forceinline__ void value_tile(const _Float16* v, int vs, f32x4 p, int r16, int kg, f32x4 (&o)[HD / 16]) {
    h4 ph, pl;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float w = p[e] * kWeightScale;
        ph[e] = (_Float16)w;
        pl[e] = (_Float16)(w - (float)ph[e]);
    }
    const _Float16* at = v + (size_t)(4 * kg + (r16 >> 2)) * vs + (r16 & 3) * 4;
#pragma unroll
    for (int ft = 0; ft < HD / 16; ++ft) {
        const s4 raw = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s4*)const_cast<_Float16*>(at + ft * 16));
        const h4 a = __builtin_bit_cast(h4, raw);
        o[ft] = __builtin_amdgcn_mfma_f32_16x16x16f16(a, pl, o[ft], 0, 0, 0);
        o[ft] = __builtin_amdgcn_mfma_f32_16x16x16f16(a, ph, o[ft], 0, 0, 0);
    }
}
// A value of the rows in flight that is infinite or NaN as a half goes to LDS as zero: in the product its weight of zero
// would make NaN of rows that do not see it.  The rows that do get their NaN at the end (poison).
__device__ __forceinline__ bool finite_half(float x) { return fabsf(x) < 65520.f; }
__device__ __forceinline__ bool clear_not_finite(h8& v) {   // true: something was cleared
    const v4u b = __builtin_bit_cast(v4u, v);
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) bad = bad || (b[i] & 0x7C00u) == 0x7C00u || (b[i] & 0x7C000000u) == 0x7C000000u;
    if (bad) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = finite_half((float)v[e]) ? v[e] : (_Float16)0.f;
    }
    return bad;
}
__device__ __forceinline__ void poison(f32x4& o, const float* v) {   // v: the four features of a row that is seen
    const float4 x = *reinterpret_cast<const float4*>(v);
    const float nan = __uint_as_float(0x7FC00000u);
    o = (f32x4){finite_half(x.x) ? o[0] : nan, finite_half(x.y) ? o[1] : nan, finite_half(x.z) ? o[2] : nan, finite_half(x.w) ? o[3] : nan};
}

// v / d with r = 1 / d: the product's rounding is taken back once.
__device__ __forceinline__ f32x4 divided(f32x4 v, float d, float r) {
    f32x4 q = v * r;
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = fmaf(fmaf(-q[e], d, v[e]), r, q[e]);
    return q;
}

struct AttnArgs {
    const float* qkv;      // [M][3 d] raw projections
    _Float16 *Kc, *Vc;     // the layer's cache: [sequence][head][position][HD]
    const float2* rope;    // [position][HD / 2]
    RowMap map;
    int d, H, Tmax;
    uint16_t *hi, *lo;     // planes of the output rows
};

// Prompt rows: block (64-row group, head, sequence), wave w owns rows 16 w .. + 15 of the group.  Keys and
// values come 64 at a time from the raw projections (rotated here, so the prompt needs no rotary launch),
// shared by the four waves through LDS; the group on the diagonal also appends its rows to the cache.
template <int HD>
__global__ __launch_bounds__(256) void attn_prompt_kernel(AttnArgs a) {
    constexpr int KST = HD + 8, VST = HD + 16;
    __shared__ __attribute__((aligned(16))) _Float16 ks_[64 * KST], vs_[64 * VST];
    __shared__ int cleared[4];   // per wave: values that are not finite, in the block on the diagonal
    const int rg = blockIdx.x, h = blockIdx.y, s = blockIdx.z, C = a.map.rows_per_seq;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r16 = lane & 15, kg = lane >> 4;
    const int row = rg * 64 + wave * 16 + r16;
    const size_t base = (size_t)s * C;
    const float scale = 1.f / sqrtf((float)HD);
    QRow<HD> q;
    {
        Raw8 raw[HD / 32];
        load_query<HD>(a.qkv + (base + min(row, C - 1)) * 3 * a.d + (size_t)h * HD, a.rope + (size_t)min(row, C - 1) * (HD / 2), kg, raw);
        split_query<HD>(raw, row < C, scale, q);
    }
    f32x4 o[HD / 16];
#pragma unroll
    for (int ft = 0; ft < HD / 16; ++ft) o[ft] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float mx = -INFINITY, den = 0.f;
    const size_t cbase = ((size_t)s * a.H + h) * a.Tmax * HD;
    for (int kb = 0; kb <= rg; ++kb) {
        {   // thread (key, quarter of the head): HD / 4 features of the key's k and v
            const int key = threadIdx.x >> 2, f0 = (threadIdx.x & 3) * (HD / 4), pos = kb * 64 + key;
            const int pc = min(pos, C - 1);
            const float* kr = a.qkv + (base + pc) * 3 * a.d + a.d + (size_t)h * HD + f0;
            const float2* tab = a.rope + (size_t)pc * (HD / 2) + f0 / 2;
            bool bad = false;
#pragma unroll
            for (int c = 0; c < HD / 32; ++c) {
                float k[8];
                rope8(load_raw8(kr + c * 8, tab + c * 4), k);
                const float4 v0 = *reinterpret_cast<const float4*>(kr + a.d + c * 8), v1 = *reinterpret_cast<const float4*>(kr + a.d + c * 8 + 4);
                h8 kk, vv;
#pragma unroll
                for (int e = 0; e < 8; ++e) kk[e] = (_Float16)k[e];
                vv[0] = (_Float16)v0.x; vv[1] = (_Float16)v0.y; vv[2] = (_Float16)v0.z; vv[3] = (_Float16)v0.w;
                vv[4] = (_Float16)v1.x; vv[5] = (_Float16)v1.y; vv[6] = (_Float16)v1.z; vv[7] = (_Float16)v1.w;
                *reinterpret_cast<h8*>(ks_ + key * KST + f0 + c * 8) = kk;
                if (kb == rg) {
                    if (pos < C) {
                        *reinterpret_cast<h8*>(a.Kc + cbase + (size_t)pos * HD + f0 + c * 8) = kk;
                        *reinterpret_cast<h8*>(a.Vc + cbase + (size_t)pos * HD + f0 + c * 8) = vv;
                    }
                    bad |= clear_not_finite(vv);
                }
                *reinterpret_cast<h8*>(vs_ + key * VST + f0 + c * 8) = vv;
            }
            if (kb == rg) {
                const int any = __any(bad);
                if (lane == 0) cleared[wave] = any;
            }
        }
        __syncthreads();
        f32x4 sc[4];
        float m = mx;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
            h8 k[HD / 32];
#pragma unroll
            for (int c = 0; c < HD / 32; ++c) k[c] = *reinterpret_cast<const h8*>(ks_ + (kt * 16 + r16) * KST + c * 32 + kg * 8);
            sc[kt] = score_tile<HD>(k, q);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sc[kt][e] = kb * 64 + kt * 16 + 4 * kg + e <= row ? sc[kt][e] : -INFINITY;
                m = fmaxf(m, sc[kt][e]);
            }
        }
        m = row_max4(m);   // finite: key 0 is visible to every row
        const float alpha = expf(mx - m);
        mx = m;
        den *= alpha;
#pragma unroll
        for (int ft = 0; ft < HD / 16; ++ft) o[ft] *= alpha;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
            f32x4 p;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p[e] = expf(sc[kt][e] - m);
                den += p[e];
            }
            value_tile<HD>(vs_ + kt * 16 * VST, VST, p, r16, kg, o);
        }
        __syncthreads();
    }
    den = row_sum4(den);
    if (row < C) {
        den *= kWeightScale;
        const float rden = 1.f / den;
#pragma unroll
        for (int ft = 0; ft < HD / 16; ++ft) o[ft] = divided(o[ft], den, rden);
        if (cleared[0] | cleared[1] | cleared[2] | cleared[3])
            for (int key = rg * 64; key <= row; ++key) {
                const float* v = a.qkv + (base + key) * 3 * a.d + 2 * a.d + (size_t)h * HD + 4 * kg;
#pragma unroll
                for (int ft = 0; ft < HD / 16; ++ft) poison(o[ft], v + ft * 16);
            }
#pragma unroll
        for (int ft = 0; ft < HD / 16; ++ft) store_planes4(a.hi, a.lo, (int)base + row, h * HD + ft * 16 + 4 * kg, a.d / 32, o[ft]);
    }
}

// Step and tree rows: block (sequence, head, tile of 16 rows), NWV waves.  Wave w takes key tiles w, w + NWV, ..
// of the cached positions - keys and values of up to T tiles requested together, one pass with a running
// maximum - and the last waves the tiles of the pass's own rows, which come rotated from the raw projections
// and are appended to the cache by the workgroup of the same row tile.  The waves meet once, at the end.
// Bound by memory latency: one dependent chain (projection rows, then the merge), all cache requests in flight
// beside it.  Eight waves while every workgroup has a compute unit to itself, which they fill (157 registers); four, of
// which three workgroups fit a unit, from 256 workgroups on (32 sequences of 20 heads, 190 cached positions: 12.0 us, with
// eight 17.4) - counted with their row tiles: 16 layers of ten XL sequences of 34 rows, 600 workgroups, 1399 us a pass with
// four waves and 1495 with eight.  Below that eight are 10 % of a pass ahead at 4000 cached positions, four 1 to 4 % at up to 500.
// The query is asked for ahead of the cached tiles, so that its rotation does not wait for them, and sums over the lanes
// go by lane swaps, not through LDS (13.2 -> 12.0 us there, three sequences of 20 heads on eight waves 8.6 -> 7.9).
struct Nothing {};
// W: Ahead, or Nothing and a grid of sequences x heads x row tiles.
template <int HD, int NWV, class W>
__global__ __launch_bounds__(64 * NWV) void attn_step_kernel(AttnArgs a, W ahead) {
    constexpr int VST = HD + 16, T = HD == 64 ? 3 : 2, CH = HD / 32;   // CH: 16-byte chunks per lane of a value tile
    __shared__ __attribute__((aligned(16))) _Float16 vbuf[NWV][16 * VST];
    __shared__ float om[NWV][16][HD + 4], ml[NWV][2][16];
    __shared__ int cleared[NWV];
    int s = blockIdx.x, h = blockIdx.y, rt = blockIdx.z;
    const int R = a.map.rows_per_seq;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, r16 = lane & 15, kg = lane >> 4;
    if constexpr (sizeof(W) == sizeof(Ahead)) {
        if ((int)blockIdx.x >= ahead.grid) {
            bring_ahead(ahead, wave, NWV, lane);
            return;
        }
        const int rest = blockIdx.x / a.map.n_seq;
        s = (int)blockIdx.x - rest * a.map.n_seq; rt = rest / a.H; h = rest - rt * a.H;
    }
    const int b = s % a.map.batch, ke = a.map.k_eff[b];
    const int R0 = s * R, row = rt * 16 + r16;
    if (ke < rt * 16) {   // no row of this tile is in flight: defined planes, nothing else reads them
        for (int i = threadIdx.x; i < 16 * (HD / 4); i += 64 * NWV) {
            const int r = rt * 16 + i / (HD / 4), f = (i % (HD / 4)) * 4;
            if (r < R) store_planes4(a.hi, a.lo, R0 + r, h * HD + f, a.d / 32, (f32x4){0.f, 0.f, 0.f, 0.f});
        }
        return;
    }
    const bool tree = a.map.mode == 2;
    const int nrows = min(ke + 1, R);                     // rows of the sequence in flight
    const int pos0 = a.map.n_cond + a.map.n[b] - 1;       // first new entry = number of cached ones
    const size_t cbase = ((size_t)s * a.H + h) * a.Tmax * HD;
    const _Float16 *Kh = a.Kc + cbase, *Vh = a.Vc + cbase;
    const int ntile = (pos0 + 15) / 16;
    const rsrc_t rk = bounded(Kh, (unsigned)pos0 * HD * 2), rv = bounded(Vh, (unsigned)pos0 * HD * 2);
    struct Tile { h8 k[HD / 32]; v4u v[CH]; };
    auto request = [&](int tile, Tile& t) {   // tiles past the end: zeros, no traffic
#pragma unroll
        for (int c = 0; c < HD / 32; ++c)
            t.k[c] = __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(rk, (unsigned)((tile * 16 + r16) * HD + c * 32 + kg * 8) * 2u, 0, 0));
#pragma unroll
        for (int c = 0; c < CH; ++c) t.v[c] = __builtin_amdgcn_raw_buffer_load_b128(rv, (unsigned)(tile * 16 * HD) * 2u + (unsigned)(c * 64 + lane) * 16u, 0, 0);
    };
    // Requested in the order of need, since a unit answers in order: the query, without which no tile can be used, ahead of
    // the cached tiles.
    const int qpos = pos0 + (tree ? a.map.tree_depth[min(row, R - 1)] : row);
    Raw8 qraw[HD / 32];
    load_query<HD>(a.qkv + (size_t)(R0 + min(row, R - 1)) * 3 * a.d + (size_t)h * HD, a.rope + (size_t)min(qpos, a.Tmax - 1) * (HD / 2), kg, qraw);
    struct Own { Raw8 k; float4 v0, v1; };
    auto load_own = [&](int nt, Own (&t)[HD / 32]) {
        const int krc = min(nt * 16 + r16, nrows - 1);    // this lane's key row (A operand)
        const float* src = a.qkv + (size_t)(R0 + krc) * 3 * a.d + a.d + (size_t)h * HD + kg * 8;
        const float2* tab = a.rope + (size_t)(pos0 + (tree ? a.map.tree_depth[krc] : krc)) * (HD / 2) + kg * 4;
#pragma unroll
        for (int c = 0; c < HD / 32; ++c) {
            t[c].k = load_raw8(src + c * 32, tab + c * 16);
            t[c].v0 = *reinterpret_cast<const float4*>(src + a.d + c * 32);
            t[c].v1 = *reinterpret_cast<const float4*>(src + a.d + c * 32 + 4);
        }
    };
    Own own[HD / 32];
    int nt = NWV - 1 - wave;                              // own tile of this wave: the last waves have the first ones
    Tile ring[T];
#pragma unroll
    for (int j = 0; j < T; ++j) request(wave + j * NWV, ring[j]);
    QRow<HD> q;
    split_query<HD>(qraw, row < nrows, 1.f / sqrtf((float)HD), q);
    // The own keys and values come in behind the cached ones.  Not where workgroups should share a unit, nor with wide heads:
    // it takes 40 registers (14.1 us instead of 13.4 with four waves, since two workgroups fit a unit instead of three).
    constexpr bool EARLY = HD == 64 && NWV == 8;
    if (EARLY && nt * 16 < nrows) load_own(nt, own);
    // which of the pass's own entries the row attends, one bit each: its ancestors or the rows before it, and itself
    auto visible = [&](int r) { return tree ? a.map.tree_anc[r] | (1ull << r) : (2ull << r) - 1ull; };
    const unsigned long long sees = row < nrows ? visible(row) : 0ull;
    bool bad = false;   // values that are not finite among the pass's own
    f32x4 o[HD / 16];
#pragma unroll
    for (int ft = 0; ft < HD / 16; ++ft) o[ft] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float mx = -INFINITY, den = 0.f;
    _Float16* vb = vbuf[wave];
    // scores of one tile are in sc (-inf where masked), its values in vb
    auto absorb = [&](const f32x4& sc) {
        const float m = row_max4(fmaxf(mx, fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]))));
        const float ms = m == -INFINITY ? 0.f : m;        // nothing visible yet: all weights are zero
        const float alpha = expf(mx - ms);
        mx = m;
        den *= alpha;
        f32x4 p;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = expf(sc[e] - ms);
            den += p[e];
        }
#pragma unroll
        for (int ft = 0; ft < HD / 16; ++ft) o[ft] *= alpha;
        value_tile<HD>(vb, VST, p, r16, kg, o);
    };
    for (int i0 = wave; i0 < ntile; i0 += NWV * T) {
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const int tile = i0 + j * NWV;
            if (tile < ntile) {
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const int at = (c * 64 + lane) * 8;
                    *reinterpret_cast<v4u*>(vb + (at / HD) * VST + at % HD) = ring[j].v[c];
                }
                f32x4 sc = score_tile<HD>(ring[j].k, q);
#pragma unroll
                for (int e = 0; e < 4; ++e) sc[e] = tile * 16 + 4 * kg + e < pos0 ? sc[e] : -INFINITY;
                absorb(sc);
            }
            request(tile + NWV * T, ring[j]);
        }
    }
    // the pass's own entries: tile nt of 16 rows for wave NWV - 1 - nt % NWV
    for (; nt * 16 < nrows; nt += NWV) {
        const int kr = nt * 16 + r16;
        const size_t entry = cbase + (size_t)(pos0 + kr) * HD;
        if (!EARLY || nt >= NWV) load_own(nt, own);
        h8 k[HD / 32];
#pragma unroll
        for (int c = 0; c < HD / 32; ++c) {
            const int f = c * 32 + kg * 8;
            float v[8];
            rope8(own[c].k, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) k[c][e] = (_Float16)v[e];
            const float4 v0 = own[c].v0, v1 = own[c].v1;
            h8 vv;
            vv[0] = (_Float16)v0.x; vv[1] = (_Float16)v0.y; vv[2] = (_Float16)v0.z; vv[3] = (_Float16)v0.w;
            vv[4] = (_Float16)v1.x; vv[5] = (_Float16)v1.y; vv[6] = (_Float16)v1.z; vv[7] = (_Float16)v1.w;
            if (nt == rt && kr < nrows) {
                *reinterpret_cast<h8*>(a.Kc + entry + f) = k[c];
                *reinterpret_cast<h8*>(a.Vc + entry + f) = vv;
            }
            bad |= clear_not_finite(vv);
            *reinterpret_cast<h8*>(vb + r16 * VST + f) = vv;
        }
        f32x4 sc = score_tile<HD>(k, q);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // (a select, and not a branch around the assignment: hipcc lost the latter for vector elements)
            sc[e] = ((sees >> (nt * 16 + 4 * kg + e)) & 1ull) ? sc[e] : -INFINITY;
        }
        absorb(sc);
    }
    // merge: every wave's maximum, sum and weighted values
    den = row_sum4(den);
    const int any = __any(bad);
    if (lane == 0) cleared[wave] = any;
    if (kg == 0) {
        ml[wave][0][r16] = mx;
        ml[wave][1][r16] = den;
    }
#pragma unroll
    for (int ft = 0; ft < HD / 16; ++ft) *reinterpret_cast<f32x4*>(&om[wave][r16][ft * 16 + 4 * kg]) = o[ft];
    __syncthreads();
    int poisoned = 0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) poisoned |= cleared[w];
    for (int i = threadIdx.x; i < 16 * (HD / 4); i += 64 * NWV) {
        const int r = i / (HD / 4), f = (i % (HD / 4)) * 4, rr = rt * 16 + r;
        if (rr >= R) continue;
        f32x4 v = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (rr < nrows) {
            float m = ml[0][0][r], t = 0.f;
#pragma unroll
            for (int w = 1; w < NWV; ++w) m = fmaxf(m, ml[w][0][r]);
#pragma unroll
            for (int w = 0; w < NWV; ++w) {
                const float e = expf(ml[w][0][r] - m);    // a wave without visible keys: exp(-inf) = 0
                t += e * ml[w][1][r];
                v += *reinterpret_cast<const f32x4*>(&om[w][r][f]) * e;
            }
            v /= t * kWeightScale;
            if (poisoned)
                for (int key = 0; key < nrows; ++key)
                    if ((visible(rr) >> key) & 1ull) poison(v, a.qkv + (size_t)(R0 + key) * 3 * a.d + 2 * a.d + (size_t)h * HD + f);
        }
        store_planes4(a.hi, a.lo, R0 + rr, h * HD + f, a.d / 32, v);
    }
}

}  // namespace

// ------------------------------------------------------------------------------------------ launchers

// The kernels a product with tile-major weights can take.  A round of workgroups takes fixed + step microseconds per k-step
// of 32, and an XCD's compute units take its workgroups (see the kernels' mapping) 32 at a time, the small (4, 3) kernel's
// 64.  Smaller tiles draw fewer bytes into a unit, so the smallest that covers the output in one round wins; the staged
// ones once the rows are a contraction.  Fitted to 3900 times of these kernels (17 products of the B, XL and 7B widths, 2 to
// 512 rows, weights from memory): the choice is 0.9 % behind the fastest on average.  Counting workgroups over the whole
// chip, with a time per k-step alone, was 9.3 % behind: W1|W3 of 48 rows at the XL widths (2, 2) 14.5 us, (4, 2) 9.8 us, QKV
// of 72 rows 13.3 and 9.1 us; 384 rows of W2 (4, 2) 26.0 us, since two XCDs had 36 workgroups, (4, 3) 17.6 us.
// From 200 rows on the entries behind (10, 8) are fitted to 372 products of the same widths, 70 to 4100 rows: the choice is 1.1 %
// behind the fastest of these kernels on average and 3.6 % ahead of the choice among the staged forms alone (5.3 % behind); it is
// slower than that one for four sizes, by 5 % at most (W1|W3 of 1000 rows at the 7B widths, 330 us instead of 314; the whole prompt pass
// of 1000 rows, three layers, 3.39 -> 3.35 ms).
struct RowsKernel { int SR, CT; float fixed, step; int slots; bool staged; };
static const RowsKernel kRowsKernels[] = {
    {1, 1, 0.9f, 0.038f, 32, false}, {2, 1, 1.5f, 0.049f, 32, false}, {4, 1, 1.8f, 0.09f, 32, false},   {2, 2, 1.2f, 0.080f, 32, false},
    {3, 2, 1.9f, 0.093f, 32, false}, {4, 2, 1.5f, 0.116f, 32, false}, {6, 2, 2.5f, 0.143f, 32, false},  {4, 3, 2.6f, 0.129f, 32, false},
    {4, 3, 3.9f, 0.243f, 64, false}, {4, 4, 3.3f, 0.146f, 32, false}, {7, 3, 3.9f, 0.179f, 32, false},  {8, 8, 7.5f, 0.398f, 32, true},
    {10, 8, 7.9f, 0.481f, 32, true}, {16, 8, 12.0f, 0.674f, 32, true}, {20, 12, 18.3f, 1.135f, 32, true},
    {16, 12, 16.6f, 0.927f, 32, true}, {18, 12, 15.9f, 0.987f, 32, true}, {16, 16, 21.3f, 1.19f, 32, true}, {8, 12, 11.3f, 0.539f, 32, true}};
static int pick_kernel(const RowsGemm& g) {
    const int strips = g.N / 16, tiles = (g.M + 15) / 16;
    int best = 0;
    float cost = 1e30f;
    for (int i = 0; i < (int)(sizeof kRowsKernels / sizeof kRowsKernels[0]); ++i) {
        const RowsKernel& t = kRowsKernels[i];
        if (t.staged && tiles < 4) continue;
        const long sg = (strips + t.SR - 1) / t.SR, tg = (tiles + t.CT - 1) / t.CT;
        const long per_xcd = t.staged ? (sg * tg + 7) / 8 : (sg + 7) / 8 * tg;
        const float us = (float)((per_xcd + t.slots - 1) / t.slots) * (t.fixed + t.step * (float)(g.K / 32));
        if (us < cost) { cost = us; best = i; }
    }
    return best;
}

extern "C" int hawk_rows_kernel(int M, int N, int K) {
    RowsGemm g;
    memset(&g, 0, sizeof g);
    g.M = M; g.N = N; g.K = K;
    return pick_kernel(g);
}
// The tile of that product's kernel, strips * 100 + row tiles.
extern "C" int hawk_rows_tile(int M, int N, int K) {
    RowsGemm g;
    memset(&g, 0, sizeof g);
    g.M = M; g.N = N; g.K = K;
    const RowsKernel& t = kRowsKernels[pick_kernel(g)];
    return t.SR * 100 + t.CT;
}

// Row-major weights (the dual-direction heads, contexts without the tile-major copy) come as 64-byte pieces of 16 rows: a
// round of 256 workgroups takes fixed + step microseconds per k-step, whether a unit holds one of them or two, and
// kernels that draw the weights once for all rows win early.  Fitted to 45 products (K 768, 1280, 4096; 1 to 2048 rows;
// weights in the last-level cache and not): the choice is the fastest of these nine for 44 of them and 5 % behind for one.
// With the costs of the tile-major kernels, weights not in cache: 44 rows of 8192 x 4096 (4, 1) 50 us, (4, 3) here 35 us;
// one row of 8192 x 4096 (2, 1) of eight waves 27 us, of four waves 17.6 us; 1024 rows of 16384 x 1280 (4, 4) 245 us,
// (16, 8) 96 us.
struct RowMajorKernel { int SR, CT; float fixed, step; };
static const RowMajorKernel kRowMajorKernels[] = {{1, 1, 1.2f, 0.059f}, {2, 1, 1.5f, 0.094f}, {4, 1, 1.5f, 0.169f}, {2, 2, 1.9f, 0.11f}, {4, 3, 2.4f, 0.205f},
                                                  {4, 4, 5.3f, 0.202f}, {8, 8, 5.5f, 0.462f}, {16, 8, 8.9f, 0.802f}, {20, 12, 14.2f, 1.278f}};
static int pick_row_major(const RowsGemm& g) {
    const int strips = g.N / 16, tiles = (g.M + 15) / 16;
    int best = 0;
    float cost = 1e30f;
    for (int i = 0; i < (int)(sizeof kRowMajorKernels / sizeof kRowMajorKernels[0]); ++i) {
        const RowMajorKernel& t = kRowMajorKernels[i];
        const long wgs = (long)((strips + t.SR - 1) / t.SR) * ((tiles + t.CT - 1) / t.CT);
        const float us = (float)((wgs + 255) / 256) * (t.fixed + t.step * (float)(g.K / 32));
        if (us < cost) { cost = us; best = i; }
    }
    return best;
}

template <int WN, int WM, int SR, int CT, int S, bool PACKED, int MODE> static void launch_staged(hipStream_t stream, const RowsGemm& g) {
    constexpr int BS = WN * SR, BT = WM * CT, lds = S * (BS + 2 * BT) * 1024;
    const int strips = g.N / 16, tiles = (g.M + 15) / 16, total = ((strips + BS - 1) / BS) * ((tiles + BT - 1) / BT);
    auto k = rows_gemm_staged_kernel<WN, WM, SR, CT, S, PACKED, MODE>;
    // per launch: the attribute belongs to the current device; a failure shows as a failed launch
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    k<<<(total + 7) / 8 * 8, 64 * WN * WM, lds, stream>>>(g);
}
template <int WN, int WM, int SR, int CT, int MODE> static void launch_wide(hipStream_t stream, const RowsGemm& g) {
    constexpr int BS = WN * SR, BT = WM * CT, lds = 3 * 2 * BT * 1024;
    const int strips = g.N / 16, tiles = (g.M + 15) / 16, total = ((strips + BS - 1) / BS) * ((tiles + BT - 1) / BT);
    auto k = rows_gemm_wide_kernel<WN, WM, SR, CT, MODE>;
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    k<<<(total + 7) / 8 * 8, 64 * WN * WM, lds, stream>>>(g);
}
template <int SR, int CT, int D, int KW, bool PACKED, int MODE> static void launch_direct(hipStream_t stream, const RowsGemm& g, const Ahead* ahead = nullptr) {
    const int strips = g.N / 16, tiles = (g.M + 15) / 16;
    const int grid = ((strips + SR - 1) / SR + 7) / 8 * 8 * ((tiles + CT - 1) / CT);
    if constexpr (PACKED && MODE == kGemmResidual)
        if (ahead) {
            rows_gemm_ahead_kernel<SR, CT, D, KW, MODE><<<grid + ahead->extra, 64 * KW, 0, stream>>>(g, *ahead);
            return;
        }
    rows_gemm_kernel<SR, CT, D, KW, PACKED, MODE><<<grid, 64 * KW, 0, stream>>>(g);
}
template <int MODE> static void launch_packed(hipStream_t stream, const RowsGemm& g, const Ahead* ahead) {
    switch (pick_kernel(g)) {
        case 0: return launch_direct<1, 1, 8, 4, true, MODE>(stream, g, ahead);
        case 1: return launch_direct<2, 1, 5, 8, true, MODE>(stream, g, ahead);
        case 2: return launch_direct<4, 1, 4, 8, true, MODE>(stream, g, ahead);
        case 3: return launch_direct<2, 2, 6, 4, true, MODE>(stream, g, ahead);
        case 4: return launch_direct<3, 2, 6, 4, true, MODE>(stream, g, ahead);
        case 5: return launch_direct<4, 2, 3, 8, true, MODE>(stream, g, ahead);
        case 6: return launch_direct<6, 2, 4, 4, true, MODE>(stream, g, ahead);
        case 7: return launch_direct<4, 3, 2, 8, true, MODE>(stream, g, ahead);
        case 8: return launch_direct<4, 3, 3, 4, true, MODE>(stream, g, ahead);
        case 9: return launch_direct<4, 4, 2, 8, true, MODE>(stream, g, ahead);
        case 10: return launch_direct<7, 3, 2, 8, true, MODE>(stream, g, ahead);
        case 11: return launch_staged<2, 4, 4, 2, 4, true, MODE>(stream, g);
        case 12: return launch_staged<2, 4, 5, 2, 4, true, MODE>(stream, g);
        case 13: return launch_wide<4, 2, 4, 4, MODE>(stream, g);
        case 14: return launch_wide<4, 2, 5, 6, MODE>(stream, g);
        case 15: return launch_wide<4, 2, 4, 6, MODE>(stream, g);
        case 16: return launch_wide<6, 2, 3, 6, MODE>(stream, g);
        case 17: return launch_wide<4, 2, 4, 8, MODE>(stream, g);
        default: return launch_wide<2, 4, 4, 3, MODE>(stream, g);
    }
}
template <int MODE> static void launch_row_major(hipStream_t stream, const RowsGemm& g) {
    switch (pick_row_major(g)) {
        case 0: return launch_direct<1, 1, 6, 4, false, MODE>(stream, g);
        case 1: return launch_direct<2, 1, 4, 4, false, MODE>(stream, g);
        case 2: return launch_direct<4, 1, 3, 4, false, MODE>(stream, g);
        case 3: return launch_direct<2, 2, 4, 4, false, MODE>(stream, g);
        case 4: return launch_direct<4, 3, 3, 4, false, MODE>(stream, g);
        case 5: return launch_direct<4, 4, 2, 8, false, MODE>(stream, g);
        case 6: return launch_staged<2, 4, 4, 2, 4, false, MODE>(stream, g);
        case 7: return launch_staged<4, 2, 4, 4, 4, false, MODE>(stream, g);
        default: return launch_staged<4, 2, 5, 6, 3, false, MODE>(stream, g);
    }
}

// Waves of a step attention workgroup: see the kernel.
extern "C" int hawk_rows_attn_waves(int sequences, int heads, int rows) { return sequences * heads * ((rows + 15) / 16) >= 256 ? 4 : 8; }

void launch_rows_gemm(hipStream_t stream, const RowsGemm& g, const Ahead* ahead) {
    if (g.packed) {
        switch (g.mode) {
            case kGemmPlain: launch_packed<kGemmPlain>(stream, g, nullptr); return;
            case kGemmResidual: launch_packed<kGemmResidual>(stream, g, ahead); return;
            default: launch_packed<kGemmSwiglu>(stream, g, nullptr); return;
        }
    }
    if (g.mode == kGemmHeads) launch_row_major<kGemmHeads>(stream, g);
    else if (g.mode == kGemmResidual) launch_row_major<kGemmResidual>(stream, g);
    else launch_row_major<kGemmPlain>(stream, g);
}

int gemm_pack_weights(hawk_ctx* c) {
    if (!c->off.gpack) return 0;
    for (int i = 0; i < c->n_gpk; ++i) {
        const auto& e = c->gpk[i];
        const size_t total = (size_t)e.N * e.K / 8;   // 16-byte chunks
        pack_tiles_kernel<<<(unsigned)((total + 255) / 256), 256, 0, c->stream>>>(
            reinterpret_cast<const uint16_t*>(c->ws + c->off.blob + e.blob_off), e.K, e.cols,
            reinterpret_cast<v4u*>(c->ws + c->off.gpack + e.pack_off), total, e.pairs);
    }
    if (hipGetLastError() != hipSuccess) return -1;
    return hipStreamSynchronize(c->stream) == hipSuccess ? 0 : -1;
}

void launch_rows_split(hipStream_t stream, const float* A, int lda, int M, int K, uint16_t* hi, uint16_t* lo) {
    rows_split_kernel<<<dim3(M, (K + 1023) / 1024), 256, 0, stream>>>(A, lda, K, hi, lo);
}

// Contexts that take this path: those with the tile-major copy of their weights (bf16, d a multiple of 32).
bool rows_ok(const hawk_ctx* c) { return c->off.gpack != 0; }

int rows_fill_rope(hawk_ctx* c) {
    if (!c->off.rtab) return 0;
    const int n = c->Tmax * (c->hd / 2);
    rope_table_kernel<<<(n + 255) / 256, 256, 0, c->stream>>>(wsp<double>(c, c->off.inv_freq), wsp<float2>(c, c->off.rtab), c->hd / 2, c->Tmax);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

namespace {

struct PlanePtr { uint16_t *hi, *lo; };
PlanePtr plane_pair(hawk_ctx* c, size_t off, int M, int K) {
    PlanePtr p;
    p.hi = wsp<uint16_t>(c, off);
    p.lo = p.hi + plane_halves(M, K);
    return p;
}
const uint16_t* packed_weights(hawk_ctx* c, int i) { return reinterpret_cast<const uint16_t*>(c->ws + c->off.gpack + c->gpk[i].pack_off); }
const uint16_t* blob16(hawk_ctx* c, size_t off) { return reinterpret_cast<const uint16_t*>(c->ws + c->off.blob + off); }
int ssq_ld(const hawk_ctx* c) { return (c->d / 16 + 3) & ~3; }

RowsGemm product(hawk_ctx* c, const PlanePtr& in, int M, int K, int pack, int mode) {
    RowsGemm g;
    memset(&g, 0, sizeof g);
    g.hi = in.hi; g.lo = in.lo; g.W = packed_weights(c, pack); g.packed = 1; g.mode = mode;
    g.N = c->gpk[pack].N; g.K = K; g.M = M; g.norm_d = (float)c->d; g.eps = c->cfg.rms_eps;
    return g;
}
void scaled_by_rms(hawk_ctx* c, RowsGemm& g, int partials) {
    g.ssq = wsp<float>(c, c->off.ssq); g.ssq_ld = ssq_ld(c); g.ssq_n = partials;
}

}  // namespace

// The output layer over the rows of x (`stride` values apart), whose planes (of x * g_f) and sums of squares are current.
static void rows_output_layer(hawk_ctx* c, int M, int partials, size_t off_x, size_t stride, size_t off_logits) {
    if (c->Vs % 16) {   // no whole strips: row by row
        launch_rmsnorm(c, off_x, stride, c->w.g_f, c->off.a, M);
        launch_gemm(c, c->off.a, c->d, c->w.W_out + (size_t)c->cfg.samp_lo * c->d * c->esz, c->Vs, c->d, off_logits, c->Vs, M, false, true);
        return;
    }
    RowsGemm g = product(c, plane_pair(c, c->off.split, M, c->d), M, c->d, 4 * c->L + 1, kGemmPlain);
    scaled_by_rms(c, g, partials);
    g.Y = wsp<float>(c, off_logits); g.ldy = c->Vs;
    launch_rows_gemm(c->stream, g);
}

// Units a launch leaves idle bring the weights of a launch behind it into the L2s they will be read from (bring_ahead): an
// attention launch those of Wo and W1|W3, which it has time for, Wo's those of W2, W2's those of the next QKV.  A launch of
// few rows starts with its first weights a memory latency away and ends before the memory system is at its rate; from L2
// QKV of 18 rows at the XL widths takes 5.1 us instead of 6.6, Wo and W2 12.8 instead of 15.3, W1|W3 7.8 instead of 9.7 and
// the attention, with the transfer beside it, 9.6 instead of 7.7 (over images of three prompts: 126.4 -> 116.9 ms); 192 rows,
// where only the attention has units to spare, W1|W3 13.0 instead of 15.0 and the attention, at about 415 cached positions, 19.2
// instead of 17.7 (images 211.2 -> 206.5 ms).
// Not where a workgroup would have more to bring than the launch lasts (16 units for W2 of 192 rows 222 -> 246 ms, for QKV 240),
// nor for weights that do not fit: a matrix is brought whole or not at all, so passes at the 7B widths, where Wo alone has 32 MB,
// bring nothing.  Nor for prompt rows (B shape, 91 rows: 475 -> 482 us, XL shape, 80 rows: the same).  Where all layers' weights stay
// in the last-level cache (B shape, 170 MB) the line is at 64 rows: steps of 64 to 96 rows (18 calls, at 40 and 600 cached
// positions) take 1.8 % less to 0.7 % more with it, 0.6 % less on average; of 40 to 60 rows 1.8 % less to 0.2 % more; of 18 to 32
// rows up to 1.8 % more at 40 positions (18 rows 445 -> 453 us) and 1 to 4 % less at 600 (528 -> 509).
constexpr int kL2Kb = 24 * 1024;   // of the eight L2s' 32 MB: the rows' own data has the rest
static Ahead plan_ahead(hawk_ctx* c, int M, int grid, int idle, int kb_each, const int* packs, int n) {
    Ahead a;
    memset(&a, 0, sizeof a);
    a.grid = grid;
    a.extra = std::max(idle, 0) / 8 * 8;
    int kb = 0;
    for (int i = 0; i < n; ++i) {
        RowsGemm g;
        memset(&g, 0, sizeof g);
        g.M = M; g.N = c->gpk[packs[i]].N; g.K = c->gpk[packs[i]].K;
        const RowsKernel& t = kRowsKernels[pick_kernel(g)];
        kb += g.N / 16 * (g.K / 32);
        if (t.staged || kb > kL2Kb || kb > a.extra * kb_each) break;   // (the staged kernels take strips in another order)
        a.of[a.n].kb = t.SR * (g.K / 32); a.of[a.n].groups = (g.N / 16 + t.SR - 1) / t.SR; a.of[a.n].total_kb = g.N / 16 * (g.K / 32);
        a.n += 1;
    }
    return a;
}
// ... beside the product with matrix `pack`
static Ahead product_ahead(hawk_ctx* c, int M, int pack, int next) {
    RowsGemm g;
    memset(&g, 0, sizeof g);
    g.M = M; g.N = c->gpk[pack].N; g.K = c->gpk[pack].K;
    const RowsKernel& t = kRowsKernels[pick_kernel(g)];
    const int grid = ((g.N / 16 + t.SR - 1) / t.SR + 7) / 8 * 8 * (((M + 15) / 16 + t.CT - 1) / t.CT);
    return plan_ahead(c, M, grid, t.staged ? 0 : kNWG - grid, 128, &next, 1);
}

// All decoder layers over M rows (mode 0: condition rows, 1: step rows, 2: tree rows), from their embedding or
// condition vectors; leaves x and, for the output layer, the planes of x * g_f with the sums of squares.
static void rows_layers(hawk_ctx* c, const RowMap& map, int M) {
    const int d = c->d, m = (c->m + 31) & ~31;   // hidden features as the tile-major copies have them
    const PlanePtr pa = plane_pair(c, c->off.split, M, d), po = plane_pair(c, c->off.split + 2 * sizeof(uint16_t) * plane_halves(M, d), M, d),
                   pu = plane_pair(c, c->off.split2, M, m);
    float *x = wsp<float>(c, c->off.x), *ssq = wsp<float>(c, c->off.ssq);
    if (map.mode == 0)
        rows_cond_kernel<<<M, 256, 0, c->stream>>>(x, wsp<float>(c, c->off.cond), d, blob16(c, c->w.g1[0]), pa.hi, pa.lo, ssq, ssq_ld(c));
    else
        rows_embed_kernel<<<M, 256, 0, c->stream>>>(x, blob16(c, c->w.E), map, wsp<int32_t>(c, c->off.grid), wsp<int32_t>(c, c->off.draft),
                                                    c->N, c->kmax + 1, d, blob16(c, c->w.g1[0]), pa.hi, pa.lo, ssq, ssq_ld(c));
    const int R = map.rows_per_seq, nw = hawk_rows_attn_waves(c->S, c->H, R), attn_grid = c->S * c->H * ((R + 15) / 16), packs[2] = {1, 2};
    const bool step = map.mode != 0 && (c->hd == 64 || c->hd == 128), bring = step && (M >= 64 || c->L * (4.0 * d + 3.0 * m) * d * 2 > 256e6);
    // eight waves fill a unit; of four three workgroups fit, two with heads of 128
    const int idle = bring ? std::min(kNWG * (nw == 8 ? 1 : c->hd == 64 ? 3 : 2) - attn_grid, 192) : 0;
    Ahead attn = plan_ahead(c, M, attn_grid, idle, 192, packs, 2), after_o = attn, after_2 = attn;
    after_o.n = after_2.n = 0;
    if (bring) {
        after_o = product_ahead(c, M, 1, 3);
        after_2 = product_ahead(c, M, 3, 0);
    }
    for (int l = 0; l < c->L; ++l) {
        RowsGemm g = product(c, pa, M, d, 4 * l, kGemmPlain);
        scaled_by_rms(c, g, l == 0 ? 1 : d / 16);
        g.Y = wsp<float>(c, c->off.qkv); g.ldy = 3 * d;
        launch_rows_gemm(c->stream, g);

        AttnArgs a;
        const size_t layer = (size_t)l * c->Smax * c->Tmax * d;
        a.qkv = wsp<float>(c, c->off.qkv); a.Kc = wsp<_Float16>(c, c->off.kc) + layer; a.Vc = wsp<_Float16>(c, c->off.vc) + layer;
        a.rope = wsp<float2>(c, c->off.rtab); a.map = map; a.d = d; a.H = c->H; a.Tmax = c->Tmax; a.hi = po.hi; a.lo = po.lo;
        if (c->hd != 64 && c->hd != 128) {   // heads that the kernels above have no tiles for
            launch_rope_append(c, map, l, M);
            launch_attention(c, map, l, M);
            launch_rows_split(c->stream, wsp<float>(c, c->off.o), d, M, d, po.hi, po.lo);
        } else if (map.mode == 0) {
            auto k = c->hd == 64 ? attn_prompt_kernel<64> : attn_prompt_kernel<128>;
            k<<<dim3((R + 63) / 64, c->H, c->S), 256, 0, c->stream>>>(a);
        } else {
            if (attn.n) {
                for (int i = 0; i < attn.n; ++i) attn.of[i].W = packed_weights(c, 4 * l + packs[i]);
                auto k = c->hd == 64 ? (nw == 4 ? attn_step_kernel<64, 4, Ahead> : attn_step_kernel<64, 8, Ahead>)
                                     : (nw == 4 ? attn_step_kernel<128, 4, Ahead> : attn_step_kernel<128, 8, Ahead>);
                k<<<attn.grid + attn.extra, 64 * nw, 0, c->stream>>>(a, attn);
            } else {
                auto k = c->hd == 64 ? (nw == 4 ? attn_step_kernel<64, 4, Nothing> : attn_step_kernel<64, 8, Nothing>)
                                     : (nw == 4 ? attn_step_kernel<128, 4, Nothing> : attn_step_kernel<128, 8, Nothing>);
                k<<<dim3(c->S, c->H, (R + 15) / 16), 64 * nw, 0, c->stream>>>(a, Nothing());
            }
        }

        g = product(c, po, M, d, 4 * l + 1, kGemmResidual);
        g.Y = x; g.ldy = d; g.ohi = pa.hi; g.olo = pa.lo; g.okts = d / 32; g.gain = blob16(c, c->w.g2[l]);
        g.ossq = ssq; g.ossq_ld = ssq_ld(c);
        after_o.of[0].W = packed_weights(c, 4 * l + 3);
        launch_rows_gemm(c->stream, g, after_o.n ? &after_o : nullptr);

        g = product(c, pa, M, d, 4 * l + 2, kGemmSwiglu);
        scaled_by_rms(c, g, d / 16);
        g.ohi = pu.hi; g.olo = pu.lo; g.okts = m / 32;
        launch_rows_gemm(c->stream, g);

        g = product(c, pu, M, m, 4 * l + 3, kGemmResidual);
        g.Y = x; g.ldy = d; g.ohi = pa.hi; g.olo = pa.lo; g.okts = d / 32;
        g.gain = blob16(c, l + 1 < c->L ? c->w.g1[l + 1] : c->w.g_f);
        g.ossq = ssq; g.ossq_ld = ssq_ld(c);
        const bool more = l + 1 < c->L;
        after_2.of[0].W = packed_weights(c, more ? 4 * l + 4 : 0);
        launch_rows_gemm(c->stream, g, more && after_2.n ? &after_2 : nullptr);
    }
}

void rows_step_pass(hawk_ctx* c, const RowMap& map, int M) {
    rows_layers(c, map, M);
    rows_output_layer(c, M, c->d / 16, c->off.x, c->d, c->off.logit_s);
}

// Condition rows; logits of the last one of every sequence.
void rows_prompt_pass(hawk_ctx* c, const RowMap& map, int M) {
    rows_layers(c, map, M);
    const PlanePtr p = plane_pair(c, c->off.split, c->S, c->d);
    const size_t last = c->off.x + (size_t)(c->C - 1) * c->d * sizeof(float), stride = (size_t)c->C * c->d;
    rows_pick_kernel<<<c->S, 256, 0, c->stream>>>(wsp<float>(c, last), stride, c->d, blob16(c, c->w.g_f), p.hi, p.lo,
                                                  wsp<float>(c, c->off.ssq), ssq_ld(c));
    rows_output_layer(c, c->S, 1, last, stride, c->off.logit_s);
}

// Draft micro-step i up to its logits: head output to off_out ([S][d] fp32), reading the previous one from off_prev.
void rows_draft_pass(hawk_ctx* c, int i, size_t off_prev, size_t off_out) {
    const int d = c->d, S = c->S;
    const PlanePtr pin = plane_pair(c, c->off.split2, S, 3 * d), pa = plane_pair(c, c->off.split, S, d);
    rows_draft_input_kernel<<<dim3(3, S), 256, 0, c->stream>>>(wsp<float>(c, off_prev), blob16(c, c->w.E), wsp<int32_t>(c, c->off.n),
                                                               wsp<int32_t>(c, c->off.k_eff), wsp<int32_t>(c, c->off.grid),
                                                               wsp<int32_t>(c, c->off.draft), i, c->B, c->N, c->gw, c->kmax + 1, d, pin.hi, pin.lo);
    RowsGemm g = product(c, pin, S, 3 * d, 4 * c->L, kGemmPlain);
    g.Y = wsp<float>(c, off_out); g.ldy = d; g.ohi = pa.hi; g.olo = pa.lo; g.okts = d / 32; g.gain = blob16(c, c->w.g_f);
    g.ossq = wsp<float>(c, c->off.ssq); g.ossq_ld = ssq_ld(c);
    launch_rows_gemm(c->stream, g);
    rows_output_layer(c, S, d / 16, off_out, d, c->off.dlogit_s);
}

}  // namespace hawk
