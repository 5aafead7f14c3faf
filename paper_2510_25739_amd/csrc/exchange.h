// What the persistent kernels exchange data with: write-through stores, and vectors split into bf16 hi and lo.
#pragma once

#include "hawk_internal.h"

namespace hawk {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// Exchange data is written once per launch, with stores that go through to memory, into a slot
// that no cache has seen in this launch; after the barrier ordinary cached loads return it and
// the 32 workgroups of an XCD share one L2 fill.
__device__ __forceinline__ void st_u32(void* p, unsigned v) {
    __hip_atomic_store(reinterpret_cast<unsigned*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_u64(void* p, unsigned lo, unsigned hi) {
    __hip_atomic_store(reinterpret_cast<u64*>(p), (u64)lo | ((u64)hi << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_f32(float* p, float v) { st_u32(p, __float_as_uint(v)); }
__device__ __forceinline__ void st_f32x2(float* p, float a, float b) { st_u64(p, __float_as_uint(a), __float_as_uint(b)); }
__device__ __forceinline__ void st_f32x4(float* p, f32x4 v) {
    st_f32x2(p, v[0], v[1]);
    st_f32x2(p + 2, v[2], v[3]);
}
__device__ __forceinline__ void compiler_fence() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }

__device__ __forceinline__ unsigned bf16_rne(float f) {
    unsigned u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ float bf16_f32(unsigned b) { return __uint_as_float(b << 16); }

// Writes four consecutive elements of a split vector: bf16 hi and lo halves, 8 bytes each.
__device__ __forceinline__ void st_split4(uint16_t* hi, uint16_t* lo, f32x4 v) {
    const unsigned h0 = bf16_rne(v[0]), h1 = bf16_rne(v[1]), h2 = bf16_rne(v[2]), h3 = bf16_rne(v[3]);
    const unsigned l0 = bf16_rne(v[0] - bf16_f32(h0)), l1 = bf16_rne(v[1] - bf16_f32(h1));
    const unsigned l2 = bf16_rne(v[2] - bf16_f32(h2)), l3 = bf16_rne(v[3] - bf16_f32(h3));
    st_u64(hi, h0 | (h1 << 16), h2 | (h3 << 16));
    st_u64(lo, l0 | (l1 << 16), l2 | (l3 << 16));
}
__device__ __forceinline__ void put_split(float4 v, uint16_t* hi, uint16_t* lo) {  // LDS destination
    const unsigned h0 = bf16_rne(v.x), h1 = bf16_rne(v.y), h2 = bf16_rne(v.z), h3 = bf16_rne(v.w);
    const unsigned l0 = bf16_rne(v.x - bf16_f32(h0)), l1 = bf16_rne(v.y - bf16_f32(h1));
    const unsigned l2 = bf16_rne(v.z - bf16_f32(h2)), l3 = bf16_rne(v.w - bf16_f32(h3));
    *reinterpret_cast<uint2*>(hi) = make_uint2(h0 | (h1 << 16), h2 | (h3 << 16));
    *reinterpret_cast<uint2*>(lo) = make_uint2(l0 | (l1 << 16), l2 | (l3 << 16));
}

}  // namespace

}  // namespace hawk
