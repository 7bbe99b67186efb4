// dL = dloss/dL on the bf16 matrix cores, fp32 as six bf16 products
// (mec_gemm_tile.hip says how and how exactly).
//
// Row x of pair (n, w) of dL receives G[n, h, w, :] K[a]^T for every (h, a) with
// h*s_h + a = x. The rows of one class x % s_h = rho take the same taps
// a = rho + s_h*j, and with x = rho + s_h*y the output row is h = y - j: each class
// is one implicit product whose rows are (n, w, y), whose reduction runs over the
// taps j and the k_c channels of G, and whose columns are the R columns (b, c). G
// rows outside 0 .. o_h - 1 read as zeros. Both operands have the channels along
// memory, so both are staged as they lie, 8 channels per load, split on their way
// to LDS. 128 rows x 64 columns per workgroup, two stages, two workgroups per
// compute unit. Rows of dL that no tap reaches (s_h > k_h) come out as zeros.
// Like the other split tiles it is bound by splitting and writing to LDS. dI (with
// the fold) against the fp32 kernel: 57x57x64 -> 128 3x3 stride 2, batch 16, 66 -> 36
// us; 24x24x96 -> 256 5x5, batch 32, 416 -> 161; 29x31x37 -> 61 5x5, batch 16, 86 -> 34;
// 227x227x3 -> 96 11x11 stride 4, batch 128, 2387 -> 600.
#include "mec_split.h"

namespace mec {
namespace {

constexpr int kMaxClasses = 8;

struct DgradTileParams {
    const float* G;
    const float* K;
    float* dL;
    int32_t i_h, o_h, k_h, s_h, k_c, R;
    uint32_t pairs;
    FastDiv div_ow;
    uint32_t first[kMaxClasses + 1];  // row tiles of the classes before each
    int32_t rows[kMaxClasses];        // y per pair: ceil((i_h - rho) / s_h)
    FastDiv div_y[kMaxClasses];
    int32_t n_tiles;
    uint32_t ntiles;
    int32_t g_bytes, k_bytes;
};

constexpr int kDtM = 128, kDtN = 64, kDtThreads = 256;
constexpr int kDtA = kDtM * 64, kDtB = kDtN * 64;  // bytes of one part's plane
constexpr int kDtStage = 3 * (kDtA + kDtB);

// VEC: k_c is a multiple of 8.
template <bool VEC>
__global__ __launch_bounds__(kDtThreads, 2) void dgrad_tile_kernel(DgradTileParams p) {
    __shared__ __align__(16) char lds[2 * kDtStage];
    __shared__ __align__(16) uint32_t ooff_s[kDtM];  // bytes of dL from the tile's first pair, 2^31 past the last row
    __shared__ uint32_t lost_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t t = xcd_remap(blockIdx.x, p.ntiles);
    const uint32_t rt = t / (uint32_t)p.n_tiles;
    const int n0 = (int)(t - rt * (uint32_t)p.n_tiles) * kDtN;
    int rho = 0;
    while (rho + 1 < p.s_h && rt >= p.first[rho + 1]) ++rho;
    const uint32_t m0 = (rt - p.first[rho]) * kDtM;
    const uint32_t Y = (uint32_t)p.rows[rho], M = p.pairs * Y;
    const FastDiv div_y = p.div_y[rho];
    const int taps = rho < p.k_h ? (p.k_h - rho + p.s_h - 1) / p.s_h : 0;
    const uint32_t pair0 = div_y.div(m0);
    constexpr uint32_t kNone = 0x80000000u;
    if (tid == 0) lost_s = 0;

    for (int r = tid; r < kDtM; r += kDtThreads) {
        const uint32_t row = m0 + (uint32_t)r, pair = div_y.div(row), y = row - pair * Y;
        ooff_s[r] = row < M ? 4u * ((pair - pair0) * (uint32_t)p.i_h + (uint32_t)rho + y * (uint32_t)p.s_h) * (uint32_t)p.R : kNone;
    }
    // staging: A rows tid / 4 and + 64, channels 8 (tid % 4).. of the chunk; B column
    // tid / 4, the same channels
    const uint32_t g = (uint32_t)tid & 3u, ar = (uint32_t)tid >> 2;
    uint32_t aoff[2];  // bytes of G at tap 0
    int ay[2];         // output row at tap 0
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        uint32_t row = m0 + ar + 64u * i;
        if (row >= M) row = M - 1;
        const uint32_t pair = div_y.div(row), y = row - pair * Y;
        const uint32_t n = p.div_ow.div(pair), w = pair - n * p.div_ow.d;
        aoff[i] = 4u * (((n * (uint32_t)p.o_h + y) * p.div_ow.d + w) * (uint32_t)p.k_c + g * 8u);
        ay[i] = (int)y;
    }
    const uint32_t col = n0 + (int)ar < p.R ? (uint32_t)n0 + ar : (uint32_t)p.R - 1u;
    const uint32_t koff = 4u * (((uint32_t)rho * (uint32_t)p.R + col) * (uint32_t)p.k_c + g * 8u);
    const uint32_t g_tap = 4u * p.div_ow.d * (uint32_t)p.k_c;                            // per tap, backwards
    const uint32_t k_tap = 4u * (uint32_t)p.s_h * (uint32_t)p.R * (uint32_t)p.k_c;
    const __amdgpu_buffer_rsrc_t grs = buffer(p.G, p.g_bytes), krs = buffer(p.K, p.k_bytes);

    struct Regs {
        float a[2][8], b[8];
    };
    int tap = 0, c0 = 0;  // the next chunk: its tap and first channel
    auto load = [&](Regs& r) {
        const int cnt = tap < taps ? p.k_c - c0 - 8 * (int)g : 0;  // channels left
        const uint32_t back = (uint32_t)tap * g_tap - 4u * (uint32_t)c0;
        uint32_t off[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) off[i] = cnt > 0 && (uint32_t)(ay[i] - tap) < (uint32_t)p.o_h ? aoff[i] - back : kNone;
        const uint32_t ko = cnt > 0 ? koff + (uint32_t)tap * k_tap + 4u * (uint32_t)c0 : kNone;
        if (VEC || cnt >= 8 || cnt <= 0) {
#pragma unroll
            for (int i = 0; i < 2; ++i) load8(grs, off[i], r.a[i]);
            load8(krs, ko, r.b);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t past = (uint32_t)((cnt - 1 - e) >> 31) & kNone;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    r.a[i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(grs, (off[i] + 4u * e) | past, 0, 0));
                r.b[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(krs, (ko + 4u * e) | past, 0, 0));
            }
        }
        c0 += 32;
        const int wrap = ~((c0 - p.k_c) >> 31);  // ~0 past the channels: the next tap
        c0 &= ~wrap;
        tap -= wrap;
    };
    uint32_t lost = 0;
    auto stage = [&](const Regs& r, char* __restrict__ to) {
        u32x4 h, m, l;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            char* at = to + swz(ar + 64u * i, g);
            split8(r.a[i], h, m, l, lost);
            *reinterpret_cast<u32x4*>(at) = h;
            *reinterpret_cast<u32x4*>(at + kDtA) = m;
            *reinterpret_cast<u32x4*>(at + 2 * kDtA) = l;
        }
        char* at = to + 3 * kDtA + swz(ar, g);
        split8(r.b, h, m, l, lost);
        *reinterpret_cast<u32x4*>(at) = h;
        *reinterpret_cast<u32x4*>(at + kDtB) = m;
        *reinterpret_cast<u32x4*>(at + 2 * kDtB) = l;
    };
    struct Frags {
        bf16x8 a[3], b[2][3];
    };
    auto read = [&](Frags& f, const char* __restrict__ from, int kk) {
        const uint32_t gg = (uint32_t)(2 * kk + (lane >> 5));
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            f.a[q] = *reinterpret_cast<const bf16x8*>(from + q * kDtA + swz((uint32_t)(wave * 32 + (lane & 31)), gg));
#pragma unroll
            for (int j = 0; j < 2; ++j)
                f.b[j][q] = *reinterpret_cast<const bf16x8*>(from + 3 * kDtA + q * kDtB + swz((uint32_t)(j * 32 + (lane & 31)), gg));
        }
    };
    floatx16 acc[2] = {}, low[2] = {};
    auto products = [&](const Frags& f) {
#define MEC_MM(X, Y, ACC)                            \
    _Pragma("unroll") for (int j = 0; j < 2; ++j)    \
        ACC[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[X], f.b[j][Y], ACC[j], 0, 0, 0);
        MEC_MM(0, 0, acc)
        MEC_MM(1, 0, low)
        MEC_MM(0, 1, low)
        MEC_MM(1, 1, low)
        MEC_MM(2, 0, low)
        MEC_MM(0, 2, low)
#undef MEC_MM
    };
    // as in mec_wgrad_tile.hip: one chunk from LDS, the next being split into the
    // other stage, two on their way; chunks past the last tap read as zeros
    Frags f0, f1;
    auto step = [&](Regs& r, const char* __restrict__ cur, char* __restrict__ nxt) {
        read(f0, cur, 0);
        read(f1, cur, 1);
        __builtin_amdgcn_sched_barrier(0);
        stage(r, nxt);
        products(f0);
#pragma unroll
        for (int n = 0; n < 12; ++n) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 10, 0);  // VALU
            __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   // LDS write
        }
        __builtin_amdgcn_sched_barrier(0);
        load(r);
        products(f1);
        __syncthreads();
    };
    Regs ra, rb;
    load(ra);
    load(rb);
    stage(ra, lds);
    load(ra);
    __syncthreads();
    const int chunks = taps * ((p.k_c + 31) / 32);
    for (int c = 0; c < chunks; c += 2) {
        step(rb, lds, lds + kDtStage);
        step(ra, lds + kDtStage, lds);
    }

    // results the split cannot have got right, as in mec_gemm_tile.hip
    uint32_t most = 0;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float x = acc[j][v] + low[j][v];
            acc[j][v] = x;
            const uint32_t bits = __builtin_bit_cast(uint32_t, x) & 0x7fffffffu;
            most = bits > most ? bits : most;
        }
    const bool bad = most >= 0x7f800000u;
    if (lost & 0xffffu) lost_s = 1;
    __syncthreads();
    float* const out = p.dL + (int64_t)pair0 * p.i_h * p.R;
    if (lost_s || __any(bad)) {
        uint32_t row = m0 + (uint32_t)(wave * 32 + (lane & 31));
        if (row >= M) row = M - 1;
        const uint32_t pair = div_y.div(row), y = row - pair * Y, n = p.div_ow.div(pair), w = pair - n * p.div_ow.d;
        const uint32_t go = 4u * ((n * (uint32_t)p.o_h + y) * p.div_ow.d + w) * (uint32_t)p.k_c;
        // 8 channels from `at` on, zeros past the last or where !on
        auto fetch = [&](__amdgpu_buffer_rsrc_t rs, uint32_t at, bool on, uint32_t st, float* x) {
            const int c = (int)(st * 16u) + 8 * (lane >> 5);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                x[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                    rs, on && c + e < p.k_c ? at + 4u * (uint32_t)(c + e) : kNone, 0, 0));
        };
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int c = n0 + j * 32 + (lane & 31);
            const uint32_t co = 4u * ((uint32_t)rho * (uint32_t)p.R + (uint32_t)(c < p.R ? c : p.R - 1)) * (uint32_t)p.k_c;
            acc[j] = floatx16{};
            for (uint32_t t = 0; t < (uint32_t)taps; ++t) {
                floatx16 sum = acc[j];
                plain_products(
                    sum, (uint32_t)(p.k_c + 15) / 16u,
                    [&](uint32_t st, float* x) { fetch(grs, go - t * g_tap, y - t < (uint32_t)p.o_h, st, x); },
                    [&](uint32_t st, float* x) { fetch(krs, co + t * k_tap, true, st, x); });
                // rows that this tap does not reach keep their sums: zeros of G may have
                // met infinities of K
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const uint32_t r = m0 + (uint32_t)(wave * 32 + acc_row(v, lane));
                    if (r - div_y.div(r) * Y - t < (uint32_t)p.o_h) acc[j][v] = sum[v];
                }
            }
        }
    }
    const __amdgpu_buffer_rsrc_t ors = buffer(out, 0x40000000);
    uint32_t coff[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int n = n0 + j * 32 + (lane & 31);
        coff[j] = n < p.R ? 4u * (uint32_t)n : 0x40000000u;
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const u32x4 ro = *reinterpret_cast<const u32x4*>(&ooff_s[wave * 32 + acc_row(4 * w, lane)]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float x = acc[j][4 * w + e];
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), ors, ro[e] + coff[j], 0, 0);
            }
    }
}

}  // namespace

// Its 32-bit offsets hold G, K and a tile's rows of dL, and the strides are at most
// kMaxClasses.
bool dgrad_tile_holds(const Shape& s) {
    const int64_t lim = int64_t(1) << 29;
    if (s.s_h > kMaxClasses || s.i_n * s.o_h * s.o_w * s.k_c >= lim || s.k_h * s.R * s.k_c >= lim) return false;
    const int64_t Y = s.i_h / s.s_h > 0 ? s.i_h / s.s_h : 1;
    return (128 / Y + 2) * s.i_h * s.R < (int64_t(1) << 28) && s.pairs * s.i_h < (int64_t(1) << 30);
}

// Taken where it holds the shape and there is work for tiles of 128 x 64 over chunks of
// 32 channels.
bool dgrad_tile_preferred(const Shape& s) {
    if (!dgrad_tile_holds(s)) return false;
    return s.k_c >= 16 && s.R >= 24 && s.pairs * s.i_h >= 512;
}

hipError_t launch_dgrad_tile(const Shape& s, const float* G, const float* K, float* dL, hipStream_t stream) {
    DgradTileParams p{};
    p.G = G;
    p.K = K;
    p.dL = dL;
    p.i_h = (int32_t)s.i_h; p.o_h = (int32_t)s.o_h; p.k_h = (int32_t)s.k_h; p.s_h = (int32_t)s.s_h;
    p.k_c = (int32_t)s.k_c; p.R = (int32_t)s.R;
    p.pairs = (uint32_t)s.pairs;
    p.div_ow = FastDiv((uint32_t)s.o_w);
    p.n_tiles = (p.R + kDtN - 1) / kDtN;
    int64_t tiles = 0;
    for (int rho = 0; rho < p.s_h; ++rho) {
        p.first[rho] = (uint32_t)tiles;
        p.rows[rho] = p.i_h > rho ? (p.i_h - rho + p.s_h - 1) / p.s_h : 0;
        if (p.rows[rho]) {
            p.div_y[rho] = FastDiv((uint32_t)p.rows[rho]);
            tiles += (s.pairs * p.rows[rho] + kDtM - 1) / kDtM;
        }
    }
    p.first[p.s_h] = (uint32_t)tiles;
    if (tiles * p.n_tiles > 0x7fffffff) return hipErrorInvalidValue;
    p.ntiles = (uint32_t)(tiles * p.n_tiles);
    p.g_bytes = (int32_t)(s.i_n * s.o_h * s.o_w * s.k_c * 4);
    p.k_bytes = (int32_t)(s.k_h * s.R * s.k_c * 4);
    auto kern = s.k_c % 8 == 0 ? dgrad_tile_kernel<true> : dgrad_tile_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(p.ntiles), dim3(kDtThreads), 0, stream, p);
    return hipGetLastError();
}

}  // namespace mec
