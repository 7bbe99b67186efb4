// fp32 values as three bf16 values each, for products on the bf16 matrix cores
// (mec_gemm_tile.hip says why and how exact that is), after Henry, Tang and Heinecke,
// "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision
// Computations", ARITH 2019. Device code only.
#pragma once

#include "mec_mfma.h"

namespace mec {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// two values rounded to the nearest bf16, and the values of such a pair
__device__ inline uint32_t rounded(float a, float b) {
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{a, b}), bf16x2));
}
__device__ inline float lower(uint32_t x) { return __builtin_bit_cast(float, x << 16); }
__device__ inline float upper(uint32_t x) { return __builtin_bit_cast(float, x & 0xffff0000u); }
// 8 fp32 values -> their hi, mid and lo parts, 8 bf16 each. hi and mid are rounded to
// nearest: they leave at most 16 and 8 significant bits, of either sign, so lo holds the
// rest exactly and what the six products leave out averages out. lost collects what lo
// leaves: its low half is nonzero only where bits fall below bf16's smallest subnormal.
// An infinity or NaN, or a value that rounds past bf16's range, leaves a NaN in lo.
// 12 vector instructions a pair, as many as cutting the parts off took (resnet_mid's
// shape 58.7 us cut off, 57.8 so, 61.1 with the rounding as integer additions; the cut
// parts' products leave out up to 2^-21, all of one sign).
__device__ inline void split8(const float* x, u32x4& h, u32x4& m, u32x4& l, uint32_t& lost) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[i] = rounded(x[2 * i], x[2 * i + 1]);
        const float ra = x[2 * i] - lower(h[i]), rb = x[2 * i + 1] - upper(h[i]);
        m[i] = rounded(ra, rb);
        const uint32_t qa = __builtin_bit_cast(uint32_t, ra - lower(m[i])), qb = __builtin_bit_cast(uint32_t, rb - upper(m[i]));
        l[i] = __builtin_amdgcn_perm(qb, qa, 0x07060302u);
        lost |= qa | qb;
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
