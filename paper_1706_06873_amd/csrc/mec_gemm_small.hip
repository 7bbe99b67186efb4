// Slab products of few outputs and a long reduction, from L or from I.
//
// Tiles of 64 and more rows leave such a shape on a handful of workgroups, each with
// the whole reduction as a serial chain of staged chunks (1 to 2 us per 32 k). Here a
// workgroup takes 16 x 16 outputs only and its up to 16 waves share the reduction:
// each reads its fragments straight from memory into registers, up to four steps in flight,
// with neither staging nor barriers, and the waves' sums are added once, in a fixed
// order, through LDS. What bounds it is the latency of a wave's few rounds of loads;
// every value is read once per 16 outputs, which the caches serve. 14x14x256 -> 256 3x3
// in fp32, one image: 27.4 -> 8.5 us; 7x7x482 -> 276 1x1 in bf16, batch 3: 74 -> 5.6.
#include <type_traits>

#include "mec_split.h"

namespace mec {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

struct SmallParams {
    const void* A;  // L or I
    const void* K;
    float* O;
    uint32_t M;
    int32_t N, n_tiles;
    FastDiv div_v, div_u, div_seg;       // row = (n * U + u) * V + v, as in mec_gemm_tile.hip
    uint32_t a_n, a_u, a_v, xstride;     // source elements
    int64_t o_n, o_u, o_v;               // output elements
    uint32_t kd;
    int32_t steps, a_bytes, k_bytes;
};

constexpr int kSmWaves = 16;

// VEC: runs are whole groups of a lane's consecutive k, at 4-byte boundaries. U: steps
// in flight.
template <typename T, bool VEC, int U>
__global__ __launch_bounds__(64 * kSmWaves) void small_gemm_kernel(SmallParams p) {
    constexpr int ES = sizeof(T), EL = 16 / ES, KS = 4 * EL;  // k per lane and step, k per step
    __shared__ float part[kSmWaves][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = (int)(blockDim.x >> 6);
    const uint32_t mt = blockIdx.x / (uint32_t)p.n_tiles, m0 = mt * 16u;
    const int n0 = (int)(blockIdx.x - mt * (uint32_t)p.n_tiles) * 16;
    auto place = [&](uint32_t row, uint32_t& n, uint32_t& u, uint32_t& v) {
        const uint32_t nu = p.div_v.div(row);
        v = row - nu * p.div_v.d;
        n = p.div_u.div(nu);
        u = nu - n * p.div_u.d;
    };
    uint32_t n, u, v;
    const uint32_t row = m0 + (uint32_t)(lane & 15);
    place(row < p.M ? row : p.M - 1, n, u, v);  // rows past the last are not stored
    const uint32_t base = n * p.a_n + u * p.a_u + v * p.a_v;
    const int col = n0 + (lane & 15);
    const __amdgpu_buffer_rsrc_t ars = buffer(p.A, p.a_bytes), krs = buffer(p.K, p.k_bytes);

    const int begin = wave * p.steps / waves, end = (wave + 1) * p.steps / waves;
    const uint32_t k_end = (uint32_t)end * KS < p.kd ? (uint32_t)end * KS : p.kd;  // this wave's; past it zeros
    floatx4 acc = {};
    for (int st = begin; st < end; st += U) {
        u32x4 a[U], b[U];
        uint32_t x[U][EL], y[U][EL];
        auto load = [&](__amdgpu_buffer_rsrc_t rs, uint32_t off) -> uint32_t {
            if constexpr (ES == 4) return __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
            else return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
        };
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint32_t k = (uint32_t)(st + i) * KS + (uint32_t)(lane >> 4) * EL;
            if constexpr (VEC) {
                const uint32_t seg = p.div_seg.div(k), off = (base + seg * p.xstride + (k - seg * p.div_seg.d)) * ES;
                a[i] = __builtin_amdgcn_raw_buffer_load_b128(ars, k < k_end ? off : 0x80000000u, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < EL; ++e) {
                const uint32_t ke = k + e;
                if constexpr (!VEC) {
                    const uint32_t seg = p.div_seg.div(ke), off = (base + seg * p.xstride + (ke - seg * p.div_seg.d)) * ES;
                    x[i][e] = load(ars, ke < k_end ? off : 0x80000000u);
                }
                y[i][e] = load(krs, ke < k_end && col < p.N ? (ke * (uint32_t)p.N + (uint32_t)col) * ES : 0x80000000u);
            }
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (ES == 4) {
                    if constexpr (!VEC) a[i][e] = x[i][e];
                    b[i][e] = y[i][e];
                } else {
                    if constexpr (!VEC) a[i][e] = x[i][2 * e] | x[i][2 * e + 1] << 16;
                    b[i][e] = y[i][2 * e] | y[i][2 * e + 1] << 16;
                }
            }
            if constexpr (ES == 4) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, (uint32_t)a[i][e]),
                                                               __builtin_bit_cast(float, (uint32_t)b[i][e]), acc, 0, 0, 0);
            } else {
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i]),
                                                              __builtin_bit_cast(bf16x8, b[i]), acc, 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) part[wave][e * 64 + lane] = acc[e];
    __syncthreads();
    for (int t = tid; t < 256; t += 64 * waves) {
        float sum = part[0][t];
        for (int w = 1; w < waves; ++w) sum += part[w][t];
        const uint32_t r = m0 + (uint32_t)(4 * ((t & 63) >> 4) + (t >> 6));
        const int c = n0 + (t & 15);
        if (r < p.M && c < p.N) {
            uint32_t on, ou, ov;
            place(r, on, ou, ov);
            p.O[(int64_t)on * p.o_n + (int64_t)ou * p.o_u + (int64_t)ov * p.o_v + c] = sum;
        }
    }
}

}  // namespace

// Its 32-bit offsets hold the shape.
bool gemm_small_holds(const Shape& s, int dtype, bool fused) {
    const int64_t M = s.i_n * s.o_h * s.o_w, kd = s.k_h * s.R, es = dtype == 0 ? 4 : 2, lim = int64_t(1) << 31;
    const int64_t src = fused ? s.i_n * s.i_h * s.i_w * s.i_c : s.i_n * s.o_w * s.i_h * s.R;
    return src * es < lim && kd * s.k_c * es < lim && M < (int64_t(1) << 26);
}

// Taken over reductions of at least 64 (below, the time is the call's) where it holds
// the shape, up to so many 16 x 16 tiles as measured, other
// kernels / here with four steps in flight always, from I, in us:
// * fp32 to 512 (two workgroups per compute unit): 14x14x256 -> 256 3x3, one image,
//   144 tiles, 27.4 / 9.8; 7x7x512 -> 512 48 / 16.6; 28x28x128 344 tiles 18.1 / 10.0;
//   16x16x512 416 tiles 51 / 28; 510 tiles over 864 16.9 / 8.7; past it 732 tiles
//   over 576 13.3 / 11.2, 1152 over 2304 35 / 37; reductions under 128 only to 256
//   (208 tiles over 64 4.3 / 3.3, 784 4.4 / 5.3);
// * bf16 to 256: 7x7 over 130 to 27 channels, 2 tiles, 370 / 29; 14x14x256 11.8 / 7.8;
//   224 tiles over 4608 19.3 / 14.6; 416 over 4608 22.4 / 24.4, 576 over 2304 14.9 /
//   20.5;
// * 1x1 kernels in bf16 to 1024: 7x7x2048 -> 512, batch 8, 800 tiles, 78 / 21; 784
//   tiles over 64 9.1 / 4.4.
bool gemm_small_preferred(const Shape& s, int dtype, bool fused) {
    if (!gemm_small_holds(s, dtype, fused)) return false;
    const int64_t M = s.i_n * s.o_h * s.o_w, kd = s.k_h * s.R;
    const int64_t tiles = ((M + 15) / 16) * ((s.k_c + 15) / 16);
    if (kd < 64) return false;
    return tiles <= (dtype == 0 ? (kd < 128 ? 256 : 512) : s.k_h == 1 ? 1024 : 256);
}

hipError_t launch_gemm_small(const Shape& s, const void* A, const void* K, float* O, int dtype, bool fused,
                             hipStream_t stream) {
    SmallParams p{};
    p.A = A;
    p.K = K;
    p.O = O;
    p.M = (uint32_t)(s.i_n * s.o_h * s.o_w);
    p.N = (int32_t)s.k_c;
    p.n_tiles = (p.N + 15) / 16;
    const int es = dtype == 0 ? 4 : 2, el = 16 / es;
    p.o_n = s.o_h * s.o_w * s.k_c;
    int64_t seglen, src;
    if (fused) {  // (n, h, w)
        p.div_u = FastDiv((uint32_t)s.o_h);
        p.div_v = FastDiv((uint32_t)s.o_w);
        p.a_n = (uint32_t)(s.i_h * s.i_w * s.i_c);
        p.a_u = (uint32_t)(s.s_h * s.i_w * s.i_c);
        p.a_v = (uint32_t)(s.s_w * s.i_c);
        p.o_u = s.o_w * s.k_c;
        p.o_v = s.k_c;
        seglen = s.R;
        p.xstride = (uint32_t)(s.i_w * s.i_c);
        src = s.i_n * s.i_h * s.i_w * s.i_c;
    } else {  // (n, w, h)
        p.div_u = FastDiv((uint32_t)s.o_w);
        p.div_v = FastDiv((uint32_t)s.o_h);
        p.a_n = (uint32_t)(s.o_w * s.i_h * s.R);
        p.a_u = (uint32_t)(s.i_h * s.R);
        p.a_v = (uint32_t)(s.s_h * s.R);
        p.o_u = s.k_c;
        p.o_v = s.o_w * s.k_c;
        seglen = s.k_h * s.R;
        src = s.i_n * s.o_w * s.i_h * s.R;
    }
    p.div_seg = FastDiv((uint32_t)seglen);
    p.kd = (uint32_t)(s.k_h * s.R);
    p.steps = (int32_t)((p.kd + 4 * el - 1) / (4 * el));
    p.a_bytes = (int32_t)(src * es);
    p.k_bytes = (int32_t)((int64_t)p.kd * p.N * es);
    // every window at a 4-byte boundary
    const bool even = dtype == 0 || (!((uintptr_t)A & 3u) && !((p.a_n | p.a_u | p.a_v | p.xstride) & 1u));
    const bool vec = seglen % el == 0 && even;
    const uint32_t tiles = (uint32_t)(((int64_t)p.M + 15) / 16 * p.n_tiles);
    const int waves = p.steps < kSmWaves ? p.steps : kSmWaves;
    // Steps in flight: loads past a wave's share cost as much as real ones, so the
    // count of 4, 3 or fewer that leaves the fewest of them (4 always,
    // against this: 7x7x482 -> 276 1x1 in bf16, batch 3, 8.3 / 5.6 us, 7x7x512 -> 128,
    // batch 32, 17.3 / 8.0, 14x14x256 3x3 in fp32 9.8 / 8.5; 8 or 6 at a time 12.4).
    const int each = (p.steps + waves - 1) / waves;
    int unroll = 4;
    for (int u = 3; u >= 1; --u)
        if ((each + u - 1) / u * u < (each + unroll - 1) / unroll * unroll && (u > 2 || each <= u)) unroll = u;
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(tiles), dim3(64 * waves), 0, stream, p);
        return hipGetLastError();
    };
    auto pick = [&](auto u) {
        constexpr int U = decltype(u)::value;
        if (dtype == 0) return vec ? launch(small_gemm_kernel<float, true, U>) : launch(small_gemm_kernel<float, false, U>);
        return vec ? launch(small_gemm_kernel<uint16_t, true, U>) : launch(small_gemm_kernel<uint16_t, false, U>);
    };
    switch (unroll) {
        case 1: return pick(std::integral_constant<int, 1>{});
        case 2: return pick(std::integral_constant<int, 2>{});
        case 3: return pick(std::integral_constant<int, 3>{});
        default: return pick(std::integral_constant<int, 4>{});
    }
}

}  // namespace mec
