// The draft chain's launch: parameters (chain.hip has the kernel, stream.hip plans and launches it).
#pragma once

#include "hawk_internal.h"

namespace hawk {

constexpr int kChainRows = 16;                 // sequences of a launch
constexpr size_t kChainBarBytes = 26 * 4096;   // counters, release words and tokens (cleared once per context)

// A pointer of the parameter block, which the kernel reads anew in every micro-step: read from memory, the compiler cannot
// know that it is to global memory (an integer: a cast of a generic pointer to global and back is folded away).
template <class T>
struct Global {
    uintptr_t at;
    Global& operator=(T* q) { at = reinterpret_cast<uintptr_t>(q); return *this; }
    __host__ __device__ __forceinline__ operator T*() const { return (T*)(__attribute__((address_space(1))) T*)at; }
};

template <class T>
__device__ __forceinline__ T* global_of(const __attribute__((address_space(4))) Global<T>& g) { return (T*)(__attribute__((address_space(1))) T*)g.at; }

struct ChainP {
    Global<const uint4> wpack;                 // the streaming kernels' packed weights and their job tables
    unsigned long long lm_base, wd_base;
    Global<const int32_t> tab_lm, tab_wd;
    Global<const uint16_t> blob;
    unsigned long long E_off, gf_off;
    Global<float> part;                        // partial products: per_slot micro-steps of part_floats each in every exchange slot
    unsigned long long slot_floats, part_floats;
    Global<const float> left;                  // [Vs][d]: products of W_d's left-neighbour block with the slice's embeddings
    Global<float> outside;                     // [S][d]: the same with committed tokens from outside the slice
    Global<const float> hprev;                 // [S][d]
    Global<const int32_t> grid, n;
    Global<int32_t> k_eff, draft, step;
    Global<unsigned long long> counters;
    Global<float> logit_s, dlogit_b;          // [S][Vs] (guidance), [B][kstride][Vs]
    Global<WarpStat> qstat;
    Global<unsigned> bar, err;
    unsigned epoch0;                    // micro-steps of all launches before
    int32_t lm_rounds, per_slot, S, B, N, IW, k;
    float eps;
    SampParams sp;
    UniformSrc us;
    ForcedSrc fs;
    Global<const float> us_draft;       // us.draft, fs.table
    Global<const int32_t> fs_table;
};

// stream.hip
bool chain_ok(const hawk_ctx*, int k);          // can the k micro-steps of a step run as one launch?
int launch_draft_chain(hawk_ctx*, int k, const SampParams&, const UniformSrc&, const ForcedSrc&);   // 0 = enqueued
// chain.hip
void launch_left_table(hipStream_t, int d, const uint4* wd_tiles, const int32_t* tab_wd, const uint16_t* slice_embeddings, float* left, int Vs);
size_t chain_lds_bytes(int S, int d);
int chain_entries(int n);                       // entries per thread of a draw from n logits (0: too many)
const void* chain_kernel(int d, int n);

}  // namespace hawk
