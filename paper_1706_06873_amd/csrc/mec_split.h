// fp32 values as three bf16 values each, for products on the bf16 matrix cores
// (mec_gemm_tile.hip says why and how exact that is). Device code only.
#pragma once

#include "mec_mfma.h"

namespace mec {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// and, subtract and v_perm only, which the matrix cores' instructions hide (6
// fit beside each; v_cvt_pk_bf16_f32 takes two slots and v_dot2_f32_bf16 does
// not overlap them)
__device__ inline float top(float x) {
    return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & 0xffff0000u);
}
__device__ inline uint32_t pack_top(float a, float b) {
    return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, b), __builtin_bit_cast(uint32_t, a), 0x07060302u);
}
// 8 fp32 values -> their hi, mid and lo parts, 8 bf16 each. lost collects what lo
// leaves: its low half is nonzero only where bits fall below bf16's smallest
// subnormal.
__device__ inline void split8(const float* x, u32x4& h, u32x4& m, u32x4& l, uint32_t& lost) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = x[2 * i], b = x[2 * i + 1];
        const float ra = a - top(a), rb = b - top(b);
        const float qa = ra - top(ra), qb = rb - top(rb);
        h[i] = pack_top(a, b);
        m[i] = pack_top(ra, rb);
        l[i] = pack_top(qa, qb);
        lost |= __builtin_bit_cast(uint32_t, qa) | __builtin_bit_cast(uint32_t, qb);
    }
}

// 8 consecutive floats at a 4-byte boundary
__device__ inline void load8(__amdgpu_buffer_rsrc_t rsrc, uint32_t off, float* x) {
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    const f32x4 a = __builtin_bit_cast(f32x4, (v4)__builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
    const f32x4 b = __builtin_bit_cast(f32x4, (v4)__builtin_amdgcn_raw_buffer_load_b128(rsrc, off + 16u, 0, 0));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[e] = a[e];
        x[4 + e] = b[e];
    }
}

// byte offset of granule g (8 bf16 values) of a row of 32: granules permuted so
// that any 8 or 16 consecutive rows of one granule fall on different banks
__device__ inline uint32_t swz(uint32_t row, uint32_t g) {
    return row * 64u + ((g ^ (((row >> 1) ^ (row >> 3)) & 3u)) << 4);
}

__device__ inline __amdgpu_buffer_rsrc_t buffer(const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00027000);
}

// a value that is the same in every lane, in scalar registers
__device__ inline uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ inline const char* uniform(const char* x) {
    const uint64_t v = (uint64_t)x;
    return (const char*)((uint64_t)uniform((uint32_t)(v >> 32)) << 32 | uniform((uint32_t)v));
}

// What a wave whose values the split does not hold computes instead: a 32 x 32 block's
// products on the fp32 matrix instruction (TraitsF32), added to acc, `steps` times 16
// k. a(s, x) and b(s, x) fetch this lane's 8 k of step s, k 16 s + 8 (lane / 32).., of
// its row and of its column, zeros past the reduction; straight from memory, without
// staging. With every value a NaN, 58x58x64 -> 64 3x3 at batch 32 takes 171 us forward,
// 238 for dK and 192 for dI (ordinary values 57, 64 and 88; one serial sum per output
// took 3440, 9130 and 3470; the fixed fp32 kernels take 68 to 107 on any values).
template <class A, class B>
__device__ inline void plain_products(floatx16& acc, uint32_t steps, A a, B b) {
#pragma clang loop unroll(disable)
    for (uint32_t s = 0; s < steps; ++s) {
        float x[8], y[8];
        a(s, x);
        b(s, y);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], y[e], acc, 0, 0, 0);
    }
}

}  // namespace mec
