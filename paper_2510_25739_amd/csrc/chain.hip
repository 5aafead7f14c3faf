// The whole draft chain of a step - k micro-steps of head, output projection and draw - as ONE launch of 256 workgroups,
// one per compute unit, of 16 waves.
//
// What bounds it: five micro-steps as launches of their own (a product kernel and a draw each) took 27 us apiece, 52 MB of
// weights drawn from memory every time at the XL shape and ten launches in a row.  W_d and the output layer's slice are
// 42 + 10 MB there and the chip's registers hold 128 MB, so a workgroup loads its strips of both once (40 + 12 registers of
// a lane) and keeps them for all micro-steps; what is left is a chain of exchanges:
//
//   W      a strip of W_d's column block of the previous state or of the upper neighbour -> memory
//   A      all workgroups have stored theirs (arrival counters, one per XCD, and release words)
//   LM     every workgroup adds both blocks' products and the left neighbour's, normalises, multiplies its strips of the
//          output layer -> memory
//   B      as A; only the workgroups that draw wait for it
//   draw   one workgroup a prompt (sample_rows.h), whose token all workgroups wait for
//
// Only the left neighbour is the token just drawn, so its block's products with every embedding of the slice are a table
// made once, when the weights are loaded (left_table_kernel; 84 MB at the XL shape): the token's row is read where its
// embedding, a product and a barrier came before.  (A committed token from outside the slice, which only forcing brings, has
// no row: in the first micro-step the workgroups of that block's strips, which have nothing to do otherwise, make its
// products as the other blocks' are made.)  The other blocks' products of micro-step i + 1 are made while micro-step
// i is drawn.  So A and B count on sets of their own: a workgroup may arrive at A(i + 1) before
// another one has arrived at B(i).  It cannot arrive at A(i + 1) before all have arrived at A(i), which it waits for, nor at
// B(i + 1) before all have arrived at B(i), since it waits for A(i + 1) and they arrive there later.
//
// Coherence: what one workgroup writes and another reads in this launch goes through to memory (agent-scope stores) and is
// read either by device-scope loads (logits, tokens, barrier words) or, the partials, by ordinary loads from addresses that
// no cache has seen since the launch began: every micro-step has its own.
//
// Every wait is bounded; one that runs out raises the error word, and the kernel ends without waiting again (accesses stay
// in bounds: a token that never came is the slice's first).
#include "exchange.h"
#include "sample_rows.h"
#include "chain.h"

namespace hawk {

namespace {

constexpr int kGroups = 8, kReplicas = 8;       // one group of arrivals per XCD; copies of the release words
constexpr unsigned kSpinLimit = 1u << 21;
constexpr int kTokReplicas = 32;                // copies of the tokens
constexpr int kRowsMax = kChainRows;
constexpr int kNone = -1, kOutside = -2;        // left neighbours without a row: no draft there; a token from outside the slice
// 4 KB pages of the chain's barrier memory (kChainBarBytes): counters and release words of A, of B, tokens
constexpr int kPageA = 0, kPageRelA = 8, kPageB = 16, kPageRelB = 24, kPageTok = 25;

struct Sync {
    unsigned* mem;
    unsigned* err;
    bool dead;
    __device__ __forceinline__ unsigned* page(int i) const { return mem + (size_t)i * 1024; }
    // One lane of the workgroup; its stores have been acknowledged.
    __device__ void arrive(int cnt_page, int rel_page, int replicas, unsigned id) {
        const unsigned g = blockIdx.x % kGroups;
        const unsigned prev = __hip_atomic_fetch_add(page(cnt_page + (int)g), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev + 1u == id * (unsigned)(kNWG / kGroups))
            for (int r = 0; r < replicas; ++r) st_u32(page(rel_page + r) + g, id);
    }
    // Whole wave: until all groups' words of one copy say `id`.
    __device__ void wait(int rel_page, unsigned id) {
        if (dead) return;
        const unsigned l = threadIdx.x & 63u;
        const unsigned* rel = page(rel_page) + (l < (unsigned)kGroups ? l : 0u);
        for (unsigned spins = 0; spins < kSpinLimit; ++spins) {
            const unsigned v = __hip_atomic_load(rel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__all((int)(v - id) >= 0)) { compiler_fence(); return; }
            if (given_up(spins)) break;
        }
        give_up();
    }
    // Whole wave: the token of prompt b, published under `id`; `none` if it does not come.
    __device__ int token(int b, unsigned id, int none) {
        if (dead) return none;
        const u64* at = reinterpret_cast<const u64*>(page(kPageTok) + (blockIdx.x % kTokReplicas) * 32) + b;
        for (unsigned spins = 0; spins < kSpinLimit; ++spins) {
            const u64 v = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__all((unsigned)(v >> 32) == id)) return __builtin_amdgcn_readfirstlane((int)(unsigned)v);
            if (given_up(spins)) break;
        }
        give_up();
        return none;
    }
    __device__ bool given_up(unsigned spins) {
        return (spins & 255u) == 255u && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
    }
    __device__ void give_up() {
        dead = true;
        st_u32(err, 1u);
    }
};

// The draws' row: written through to memory by the launch's other workgroups, so read by device-scope loads.
template <int E>
__device__ __forceinline__ void load_fresh_row(const float* lc, const float* lu, float scale, float inv_t, float* out, int n, float (&z)[E]) {
    const int th = (int)threadIdx.x;
    const float nan = __uint_as_float(0x7FC00000u);
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(lc), 0, n * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(lu ? lu : lc), 0, n * 4, 0x00020000);
    v4u a[E / 4], u[E / 4];
#pragma unroll
    for (int q = 0; q < E / 4; ++q) a[q] = __builtin_amdgcn_raw_buffer_load_b128(rc, entry<E>(4 * q, th) * 4, 0, 16);
    if (lu) {
#pragma unroll
        for (int q = 0; q < E / 4; ++q) u[q] = __builtin_amdgcn_raw_buffer_load_b128(ru, entry<E>(4 * q, th) * 4, 0, 16);
    }
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
        const int j = entry<E>(4 * q, th);   // n is a multiple of 16: all four or none of a thread's entries exist
        f32x4 l = __builtin_bit_cast(f32x4, a[q]);
        if (lu) {
            const f32x4 w = __builtin_bit_cast(f32x4, u[q]);
#pragma unroll
            for (int e = 0; e < 4; ++e) l[e] = fmaf(scale, l[e] - w[e], w[e]);
            if (j < n) *reinterpret_cast<f32x4*>(out + j) = l;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) z[4 * q + e] = j < n ? l[e] * inv_t : nan;
    }
}

// A draw from one row (index within the slice; statistics to *stat).  guided: logits of the prompt's conditional row, the
// unconditional one `shift` further on, combined to `row`; null: `row` holds them.  u < 0: `forced` is taken instead.
// Out of line: inlined in the micro-steps' loop, its constants and addresses are kept across the loop, which spills them (266
// registers).  What the XL kernel with 16 entries still spills: 16 registers, four tiles of weights, that a workgroup which draws
// saves around the call, seven address pairs, two of which a micro-step reads back, and scalars that go to lanes of two registers.
template <int E>
__device__ __noinline__ int draw(const float* guided, size_t shift, float* row, WarpStat* stat, float u, int forced, int point_mass,
                                 int n, int top_k, int greedy, float inv_t, float cfg_scale) {
    __shared__ FastShared fs;
    __shared__ CompactList L;
    float z[E];
    if (guided) load_fresh_row<E>(guided, guided + shift, cfg_scale, inv_t, row, n, z);
    else load_fresh_row<E>(row, nullptr, 1.f, inv_t, nullptr, n, z);
    int drawn = 0;
    WarpStat st = warp_and_draw<E>(z, n, top_k, greedy, fs, L, u < 0.f ? nullptr : &u, &drawn);
    if (u < 0.f) {
        drawn = forced;
        if (point_mass) { st.onehot = forced; st.total = 1.0; }
    }
    if (threadIdx.x == 0) *stat = st;
    return drawn;
}

// TPS: k-tiles of a quarter of d (d = 128 TPS); E: entries per thread of a draw.
template <int TPS, int E>
__global__ __launch_bounds__(NT, 1) void draft_chain_kernel(ChainP p) {
    constexpr int D = 128 * TPS, KT = 4 * TPS, WT = (KT + NW - 1) / NW;
    constexpr int CH = D / 256;             // pieces of a row, fp32: one wave's request of 4 values a lane
    constexpr int EH = (D + 511) / 512;     // pieces of an embedding row, bf16
    constexpr int Kp = D + 8;
    extern __shared__ uint4 smem[];
    __shared__ float ssp[kRowsMax][8];      // sums of squares of a row's pieces
    __shared__ int s_n[kRowsMax], s_ke[kRowsMax], s_left[2][kRowsMax];   // s_left: table row of a micro-step's left neighbour, kNone or kOutside
    uint16_t* const hi = reinterpret_cast<uint16_t*>(smem);
    uint16_t* const lo = hi + (size_t)p.S * Kp;
    f32x4* const red = reinterpret_cast<f32x4*>(lo + (size_t)p.S * Kp);   // [16 waves][64]

    const int wave = wave_id(), wg = blockIdx.x, S = p.S, B = p.B;
    int lane = threadIdx.x & 63;
    Sync sync = {p.bar, p.err, false};

    // this workgroup's strips: one of W_d (or none), up to four of the output layer, a quarter of whose k-tiles is a wave's
    const int32_t* const ew = p.tab_wd + (size_t)wg * 4;
    const int wstrip = ew[1] > 0 ? ew[2] & 0xFFFF : D / 16, blk = wstrip / (D / 16), wcol = (wstrip - blk * (D / 16)) * 16;
    const bool has_w = blk != 1;   // (the left neighbour's block is in the table)
    v4u wd[WT];
    {
        const v4u* src = reinterpret_cast<const v4u*>(p.wpack + (p.wd_base + (u64)(unsigned)ew[0]) * 64) + lane;
#pragma unroll
        for (int j = 0; j < WT; ++j) {
            wd[j] = (v4u){0u, 0u, 0u, 0u};
            if (has_w && wave + j * NW < KT) wd[j] = __builtin_nontemporal_load(src + (size_t)(wave + j * NW) * 64);
        }
    }
    int strip = -1;
    v4u wl[TPS];
    const v4u* lm_src = nullptr;
    {
        const int s = wave >> 2, q = wave & 3;
        const int32_t* e = p.tab_lm + (size_t)wg * 4;
        const int n0 = e[1];
        int si = s;
        if (s >= n0) { e += (size_t)kNWG * 4; si = s - n0; }
        const int ns = s < n0 ? n0 : p.lm_rounds > 1 ? e[1] : 0;
        if (si < ns) {
            strip = si == 0 ? e[2] & 0xFFFF : si == 1 ? (e[2] >> 16) & 0xFFFF : e[3];
            lm_src = reinterpret_cast<const v4u*>(p.wpack + (p.lm_base + (u64)(unsigned)e[0] + (u64)(q * ns + si) * TPS) * 64) + lane;
        }
    }
    auto load_lm = [&]() {
        unsigned long long at = reinterpret_cast<unsigned long long>(lm_src);
        asm volatile("" : "+v"(at));   // (one address, not one for each tile kept across the draw)
        const v4u* src = (const v4u*)(const __attribute__((address_space(1))) v4u*)at;
#pragma unroll
        for (int t = 0; t < TPS; ++t) wl[t] = strip >= 0 ? __builtin_nontemporal_load(src + (size_t)t * 64) : (v4u){0u, 0u, 0u, 0u};
    };
    load_lm();

    // the step's plan: drafts in flight of every prompt (-1: finished)
    const int step = *static_cast<const volatile int32_t*>(static_cast<int32_t*>(p.step)) + 1;
    if (threadIdx.x < (unsigned)B) {
        const int n = p.n[threadIdx.x], ke = n < p.N ? min(p.k, p.N - n - 1) : -1;
        s_n[threadIdx.x] = n;
        s_ke[threadIdx.x] = ke;
        if (wg == 0) p.k_eff[threadIdx.x] = ke;
    }
    __syncthreads();
    int most = -1;
    for (int b = 0; b < B; ++b) most = max(most, s_ke[b]);
    most = __builtin_amdgcn_readfirstlane(most);
    if (wave == NW - 1 && lane < B) {   // the first left neighbours, read in LM(1) behind W's barriers or the one below
        int left = kNone;
        if (s_ke[lane] > 0) {
            left = p.grid[(size_t)lane * p.N + s_n[lane] - 1] - p.sp.samp_lo;
            if (left < 0 || left >= p.sp.Vs) left = kOutside;
        }
        s_left[1][lane] = left;
    }
    int least_left = kNone;
    if (!has_w) {
        __syncthreads();
        for (int b = 0; b < B; ++b) least_left = min(least_left, s_left[1][b]);
    }
    if (ew[1] > 0 && __builtin_amdgcn_readfirstlane(least_left) == kOutside) {   // tokens that the table has no row of
        const uint16_t* const Emb = p.blob + p.E_off / 2;
        for (int it = wave; it < S * EH; it += NW) {
            const int c = it / EH, j = (it - c * EH) * 512 + lane * 8, b = c % B;
            const bool there = s_left[1][b] == kOutside;
            const int tok = there ? p.grid[(size_t)b * p.N + s_n[b] - 1] : 0;
            if (j < D) *reinterpret_cast<v4u*>(hi + (size_t)c * Kp + j) = there ? *reinterpret_cast<const v4u*>(Emb + (size_t)tok * D + j) : (v4u){0u, 0u, 0u, 0u};
        }
        __syncthreads();
        const int col = lane & 15, kg = lane >> 4;
        const v4u* src = reinterpret_cast<const v4u*>(p.wpack + (p.wd_base + (u64)(unsigned)ew[0]) * 64) + lane;
        const uint16_t* from = hi + (size_t)(col < S ? col : 0) * Kp + kg * 8;
        f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int kt = wave; kt < KT; kt += NW)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, src[(size_t)kt * 64]), *reinterpret_cast<const bf16x8*>(from + kt * 32), acc, 0, 0, 0);
        red[wave * 64 + lane] = acc;
        __syncthreads();
        if (wave == 0) {   // (which arrives at A(1) with these stores done)
            f32x4 v = red[lane];
#pragma unroll 1
            for (int w = 1; w < NW; ++w) v += red[w * 64 + lane];
            if (col < S) st_f32x4(p.outside + (size_t)col * D + wcol + 4 * kg, v);
            __builtin_amdgcn_s_waitcnt(0);
        }
    }
    const int mine = kNWG - 1 - wg;   // the prompt this workgroup draws for, if there is one

    auto kp = (const __attribute__((address_space(4))) ChainP*)__builtin_amdgcn_kernarg_segment_ptr();
    auto part_of = [&](int i) {   // products of micro-step i: [2][S][D]
        return global_of(kp->part) + (u64)((i - 1) / kp->per_slot) * kp->slot_floats + (u64)((i - 1) % kp->per_slot) * kp->part_floats;
    };
    auto left_product = [&](int left, int c, int j) {
        if (left == kNone) return (f32x4){0.f, 0.f, 0.f, 0.f};
        const float* q = left == kOutside ? global_of(kp->outside) + (size_t)c * D : global_of(kp->left) + (size_t)left * D;
        return *reinterpret_cast<const f32x4*>(q + j);
    };
    auto other_products = [&](int i, int c, int j, f32x4& x, f32x4& y) {
        const float* q = part_of(i) + (size_t)c * D + j;
        x = *reinterpret_cast<const f32x4*>(q);
        y = *reinterpret_cast<const f32x4*>(q + (size_t)S * D);
    };

    for (int i = 1; i <= kp->k; ++i) {
        const unsigned id = kp->epoch0 + (unsigned)i;
        asm volatile("" : "+v"(lane), "+s"(kp));   // addresses and parameters are made anew in every micro-step: kept across them most would spill
        const int col = lane & 15, kg = lane >> 4;
        const size_t frag = (size_t)(col < S ? col : 0) * Kp + kg * 8;   // columns past the rows repeat row 0; their results are not stored
        if (i > most) {   // nothing left to draft: only the counts go on
            if (wave == 0) {
                if (lane == 0) sync.arrive(kPageA, kPageRelA, kReplicas, id);
                sync.wait(kPageRelA + (int)(wg % kReplicas), id);
                if (lane == 0) sync.arrive(kPageB, kPageRelB, 1, id);
            }
            continue;
        }
        // ---- W
        if (has_w) {
            if (blk == 0) {
                for (int it = wave; it < S * CH; it += NW) {
                    const int c = it / CH, j = (it - c * CH) * 256 + lane * 4;
                    f32x4 v = (f32x4){0.f, 0.f, 0.f, 0.f}, y;
                    if (i <= s_ke[c % B]) {
                        if (i == 1) {
                            v = *reinterpret_cast<const f32x4*>(global_of(kp->hprev) + (size_t)c * D + j);
                        } else {   // g of the micro-step before
                            other_products(i - 1, c, j, v, y);
                            v = (v + left_product(s_left[(i - 1) & 1][c % B], c, j)) + y;
                        }
                    }
                    put_split(make_float4(v[0], v[1], v[2], v[3]), hi + (size_t)c * Kp + j, lo + (size_t)c * Kp + j);
                }
            } else {
                const uint16_t* const Emb = global_of(kp->blob) + kp->E_off / 2;
                for (int it = wave; it < S * EH; it += NW) {
                    const int c = it / EH, j = (it - c * EH) * 512 + lane * 8, b = c % B, n = s_n[b];
                    const int tok = i <= s_ke[b] && n - 1 + i >= kp->IW ? global_of(kp->grid)[(size_t)b * kp->N + n - 1 + i - kp->IW] : -1;
                    if (j < D) *reinterpret_cast<v4u*>(hi + (size_t)c * Kp + j) =
                        tok >= 0 ? *reinterpret_cast<const v4u*>(Emb + (size_t)tok * D + j) : (v4u){0u, 0u, 0u, 0u};
                }
            }
            __syncthreads();
            f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f}, acl = acc;
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                const int kt = min(wave + j * NW, KT - 1);   // (a tile past the strip is zero)
                const bf16x8 a = __builtin_bit_cast(bf16x8, wd[j]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, *reinterpret_cast<const bf16x8*>(hi + frag + kt * 32), acc, 0, 0, 0);
                if (blk == 0)   // (an embedding is its own hi part)
                    acl = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, *reinterpret_cast<const bf16x8*>(lo + frag + kt * 32), acl, 0, 0, 0);
            }
            red[wave * 64 + lane] = acc + acl;
            __syncthreads();
            if (wave == 0) {
                f32x4 v = red[lane];
#pragma unroll
                for (int w = 1; w < NW; ++w) v += red[w * 64 + lane];
                if (col < S) st_f32x4(part_of(i) + ((size_t)(blk >> 1) * S + col) * D + wcol + 4 * kg, v);
                __builtin_amdgcn_s_waitcnt(0);
                if (lane == 0) sync.arrive(kPageA, kPageRelA, kReplicas, id);
            }
        } else if (wave == 0) {
            if (lane == 0) sync.arrive(kPageA, kPageRelA, kReplicas, id);
        }
        // ---- LM
        if (wave < S * CH) sync.wait(kPageRelA + (int)(wg % kReplicas), id);
        for (int it = wave; it < S * CH; it += NW) {
            const int c = it / CH, ch = it - c * CH, j = ch * 256 + lane * 4;
            const int b = c % B;
            int left = i == 1 ? s_left[1][b] : kNone;
            f32x4 x, y;
            other_products(i, c, j, x, y);   // (asked for ahead of the token)
            const uint2 gn = *reinterpret_cast<const uint2*>(global_of(kp->blob) + kp->gf_off / 2 + j);
            if (i > 1 && i <= s_ke[b]) left = sync.token(b, id - 1u, kp->sp.samp_lo) - kp->sp.samp_lo;
            if (i > 1 && lane == 0) s_left[i & 1][b] = left;
            const f32x4 g = (x + left_product(left, c, j)) + y;
            float ss = (g[0] * g[0] + g[1] * g[1]) + (g[2] * g[2] + g[3] * g[3]);
            ss = wave_sum_f(ss);
            if (lane == 0) ssp[c][ch] = ss;
            put_split(make_float4(g[0] * bf16_f32(gn.x & 0xFFFFu), g[1] * bf16_f32(gn.x >> 16), g[2] * bf16_f32(gn.y & 0xFFFFu),
                                  g[3] * bf16_f32(gn.y >> 16)),
                      hi + (size_t)c * Kp + j, lo + (size_t)c * Kp + j);
        }
        __syncthreads();
        if (strip >= 0) {
            const uint16_t *bh = hi + frag + (size_t)(wave & 3) * TPS * 32, *bl = lo + frag + (size_t)(wave & 3) * TPS * 32;
            f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f}, acl = acc;
#pragma unroll
            for (int t = 0; t < TPS; ++t) {
                const bf16x8 a = __builtin_bit_cast(bf16x8, wl[t]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, *reinterpret_cast<const bf16x8*>(bh + t * 32), acc, 0, 0, 0);
                acl = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, *reinterpret_cast<const bf16x8*>(bl + t * 32), acl, 0, 0, 0);
            }
            red[wave * 64 + lane] = acc + acl;
        }
        __syncthreads();
        if ((wave & 3) == 0 && strip >= 0 && col < S && i <= s_ke[col % B]) {
            float ss = 0.f;
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) ss += ssp[col][ch];
            const float r = 1.0f / sqrtf(ss / (float)D + kp->eps);
            f32x4 v = red[wave * 64 + lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) v += red[(wave + w) * 64 + lane];
            float* row = kp->sp.use_cfg ? global_of(kp->logit_s) + (size_t)col * kp->sp.Vs : global_of(kp->dlogit_b) + ((size_t)col * kp->sp.kstride + (i - 1)) * kp->sp.Vs;
            st_f32x4(row + strip * 16 + 4 * kg, v * r);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0) sync.arrive(kPageB, kPageRelB, 1, id);
        // ---- draw
        if (mine < B && i <= s_ke[mine]) {
            const int b = mine;
            sync.wait(kPageRelB, id);
            asm volatile("" : "+s"(kp));
            const size_t at = (size_t)b * kp->sp.kstride + (i - 1);
            const float u = kp->fs_table.at ? -1.f
                            : kp->us.use_gen ? gen_uniform(kp->us.seed, (uint32_t)b, (uint32_t)step, (uint32_t)(kSlotDraft + (i - 1)))
                                           : global_of(kp->us_draft)[b * kp->k + (i - 1)];
            const int forced = kp->fs_table.at ? global_of(kp->fs_table)[(size_t)b * kp->fs.stride + (kp->fs.relative ? s_n[b] : 0) + (i - 1)] - kp->sp.samp_lo : -1;
            const int tok = kp->sp.samp_lo + draw<E>(kp->sp.use_cfg ? global_of(kp->logit_s) + (size_t)b * kp->sp.Vs : nullptr, (size_t)B * kp->sp.Vs, global_of(kp->dlogit_b) + at * kp->sp.Vs,
                                                   global_of(kp->qstat) + at, u, forced, kp->fs.point_mass, kp->sp.Vs, kp->sp.top_k, kp->sp.greedy, kp->sp.inv_t, kp->sp.cfg_scale);
            if (threadIdx.x < (unsigned)kTokReplicas)
                st_u64(reinterpret_cast<u64*>(sync.page(kPageTok) + threadIdx.x * 32) + b, (unsigned)tok, id);
            if (threadIdx.x == 0) global_of(kp->draft)[at] = tok;
            // A draw needs the registers of the weights: this workgroup asks for them again while the others go on.
#pragma unroll
            for (int j = 0; j < WT; ++j) wd[j] = (v4u){0u, 0u, 0u, 0u};   // (workgroups that draw have no strip of W_d: the last sixteen)
            load_lm();
        }
    }
    if (mine < B)   // the drafts that are not there
        for (int i = max(s_ke[mine], 0) + (int)threadIdx.x; i < p.sp.kstride; i += NT) p.draft[mine * p.sp.kstride + i] = -1;
    if (wg == 0 && threadIdx.x == 0) {   // every workgroup has read the counter: all have arrived at A(1)
        p.step[0] = step;
        if (most >= 0) p.counters[3] += 1ull;   // lock-step iterations that still had work
    }
}

// left[v] = W_d's column block of the left neighbour times the embedding of token samp_lo + v: a wave per 16 tokens and strip.
template <int TPS>
__global__ __launch_bounds__(256) void left_table_kernel(const uint4* tiles, const int32_t* tab_wd, const uint16_t* Emb, float* left, int Vs) {
    constexpr int D = 128 * TPS;
    const int lane = threadIdx.x & 63, s = blockIdx.x, v0 = ((int)blockIdx.y * 4 + ((int)threadIdx.x >> 6)) * 16;
    if (v0 >= Vs) return;
    const int v = v0 + (lane & 15);   // (Vs is a multiple of 16)
    // strip D / 16 + s of the three blocks' strips is workgroup D / 16 + s's
    const v4u* w = reinterpret_cast<const v4u*>(tiles + (u64)(unsigned)tab_wd[(D / 16 + s) * 4] * 64) + lane;
    const uint16_t* e = Emb + (size_t)v * D + (lane >> 4) * 8;
    f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int kt = 0; kt < 4 * TPS; ++kt)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[(size_t)kt * 64]), *reinterpret_cast<const bf16x8*>(e + kt * 32), acc, 0, 0, 0);
    *reinterpret_cast<f32x4*>(left + (size_t)v * D + s * 16 + (lane >> 4) * 4) = acc;
}

}  // namespace

void launch_left_table(hipStream_t stream, int d, const uint4* tiles, const int32_t* tab_wd, const uint16_t* Emb, float* left, int Vs) {
    (d == 1280 ? left_table_kernel<10> : left_table_kernel<6>)<<<dim3(d / 16, (Vs + 63) / 64), 256, 0, stream>>>(tiles, tab_wd, Emb, left, Vs);
}

size_t chain_lds_bytes(int S, int d) {
    const size_t need = (size_t)S * (d + 8) * 4 + (size_t)NW * 64 * 16;
    return need > 64 * 1024 ? need : 64 * 1024;   // with the static part more than half of a unit's LDS: one workgroup to a unit
}

int chain_entries(int n) { return n <= 4 * NT ? 4 : n <= 8 * NT ? 8 : n <= 16 * NT ? 16 : 0; }

const void* chain_kernel(int d, int n) {
    const int E = chain_entries(n);
#define CHAIN(TPS) (E == 4 ? reinterpret_cast<const void*>(draft_chain_kernel<TPS, 4>)   \
                  : E == 8 ? reinterpret_cast<const void*>(draft_chain_kernel<TPS, 8>)   \
                           : reinterpret_cast<const void*>(draft_chain_kernel<TPS, 16>))
    return d == 1280 ? CHAIN(10) : CHAIN(6);
#undef CHAIN
}

}  // namespace hawk
