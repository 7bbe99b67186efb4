// The slab products as one implicit matrix product on the bf16 matrix cores,
// for any kernel height, width, stride and channel count, from L or from I.
//
// Row p of the product is output pixel (n, h, w); its reduction runs over nseg
// runs of seglen consecutive elements of the source, xstride apart:
//   from L  one run, the window L[n, w][s_h*R*h : s_h*R*h + k_h*R] (Section 3.2),
//   from I  k_h runs of R = k_w*i_c elements, one per kernel row,
// so the same code reads either, in the same order: elements j = 0 .. k_h*R - 1 of
// the window, in chunks of 32.
//
// fp32 on bf16 matrix cores. Each fp32 value x is split without loss into three
// bf16 values, x = hi + mid + lo (x rounded to 8 significant bits, what that leaves
// rounded to 8, and the rest; mec_split.h), and a product is the six bf16 products
//   hi*hi + (hi*mid + mid*hi) + (hi*lo + mid*mid + lo*hi),
// each exact in fp32. The three left out (mid*lo, lo*mid, lo*lo) come to at most
// 2^-24 of the product, 2^-28 on average, of either sign. v_mfma_f32_32x32x16_bf16 does
// 16 times the multiply-adds of v_mfma_f32_32x32x2_f32 in half its cycles per
// instruction, so six of them still run 2.6 times as many fp32 products. The
// matrix cores cut sums off at about 2^-24 of the largest addend where the fp32
// instruction rounds each of its steps, so the five small products go to
// accumulators of their own, added once at the end. Measured against 64 bits
// (reductions of 32 to 32768 terms; signed, non-negative and constant values): 0.2-0.5
// of the fp32 instruction's error, and less on constants.
// Not finite or very small values: an infinity or NaN in a window, and a sum
// that leaves fp32's range, leave infinities or NaNs in the accumulators, and
// values below 2^-110 lose bits of lo below bf16's smallest subnormal, which the
// split notes (below 2^-133 nothing is left of them, and a result of 0 may be such a
// loss). A wave that finds the first in its outputs, and the waves of a workgroup
// that noted the second, compute their outputs again in plain fp32 (plain_block).
#include <type_traits>

#include "mec_split.h"

namespace mec {
namespace {

struct TileParams {
    const void* A;  // L or I
    const void* K;
    float* O;
    uint32_t M;     // output pixels
    int32_t N;      // output channels
    FastDiv div_v, div_u;      // row p = (n * U + u) * V + v
    int64_t a_n, a_u, a_v;     // source elements per step of n, u, v
    int64_t o_n, o_u, o_v, o_off;  // output elements, likewise
    int32_t nseg, seglen;
    int64_t xstride;
    FastDiv div_seg;           // by seglen
    uint32_t kd;               // nseg * seglen
    int32_t groups;            // of 8 of its elements
    int32_t nchunks, n_tiles;
    uint32_t ntiles;
};

// BM x BN 32x32 blocks per wave, WM x WN waves. RUN: every run is whole chunks
// (seglen a multiple of 32), so a chunk's addresses are uniform. ONE: one chunk at a time
// in registers, which the largest tile's accumulators leave no room beside, and the
// compiler's own schedule.
template <int BM, int BN, int WM, int WN, bool RUN, bool ONE>
struct TileCfg {
    static constexpr bool kOne = ONE;
    // waves per SIMD that the LDS admits, for the register allocation
    static constexpr int kWaves = BM * BN == 4 ? (WM * WN == 8 ? 2 : 1) : BM * BN == 2 ? 2 : 3;
    static constexpr int kBM = BM, kBN = BN, kWM = WM, kWN = WN;
    static constexpr bool kRun = RUN;
    static constexpr int KT = 32, G = KT / 8;
    static constexpr int TM = 32 * BM * WM, TN = 32 * BN * WN;
    static constexpr int THREADS = 64 * WM * WN;
    static constexpr int AI = TM * G / THREADS, BI = TN * G / THREADS;
    static constexpr int ROWB = KT * 2;                  // bytes per LDS row of a plane
    static constexpr int APL = TM * ROWB, BPL = TN * ROWB;  // bytes per plane
    static constexpr int STAGE = 3 * (APL + BPL);
    static_assert(TM * G % THREADS == 0 && TN * G % THREADS == 0 && THREADS % TN == 0 && TN % 64 == 0, "items");
    static_assert(2 * STAGE + 4 * TM + 16 <= 160 * 1024, "LDS");
};

// A 32 x 32 block in plain fp32: ro and co are the byte offsets of this lane's row of A,
// from Ab, and of its column of K. A function of its own and not inlined: inlined, the
// main loop of the 128 x 64 tile spills 17 to 34 registers.
__device__ __attribute__((noinline)) floatx16 plain_block(const char* Ab, const char* K, uint32_t ro, uint32_t co, uint32_t kd,
                                                          uint32_t N, uint32_t seglen, uint32_t xstride, uint64_t div_m,
                                                          uint32_t div_shift, int lane) {
    const __amdgpu_buffer_rsrc_t ars = buffer(uniform(Ab), 0x7fffffff), krs = buffer(uniform(K), (int)(uniform(kd) * uniform(N) * 4u));
    kd = uniform(kd), N = uniform(N);
    const uint32_t jump = 4u * (xstride - seglen);
    floatx16 sum = {};
    plain_products(
        sum, (kd + 15u) / 16u,
        [&](uint32_t s, float* x) {  // as load() below
            const uint32_t k = s * 16u + 8u * (uint32_t)(lane >> 5);
            const uint32_t a = (uint32_t)(k * div_m >> div_shift), r = k - a * seglen, cnt = seglen - r;
            const uint32_t off = ro + (a * xstride + r) * 4u;
            if (cnt >= 8 || k >= kd) {
                load8(ars, k < kd ? off : 0x80000000u, x);
            } else {
#pragma unroll
                for (uint32_t e = 0; e < 8; ++e)
                    x[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                        ars, k + e < kd ? off + 4u * e + (e >= cnt ? jump : 0u) : 0x80000000u, 0, 0));
            }
        },
        [&](uint32_t s, float* x) {  // rows past kd lie past the resource's end
            const uint32_t k = s * 16u + 8u * (uint32_t)(lane >> 5);
#pragma unroll
            for (uint32_t e = 0; e < 8; ++e)
                x[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(krs, (k + e) * N * 4u + co, 0, 0));
        });
    return sum;
}

template <class C>
__global__ __launch_bounds__(C::THREADS, C::kWaves) void tile_gemm_f32_kernel(TileParams p) {
    constexpr int BM = C::kBM, BN = C::kBN, G = C::G, TM = C::TM, TN = C::TN;
    constexpr int AI = C::AI, BI = C::BI, THREADS = C::THREADS;
    __shared__ __align__(16) char lds[2 * C::STAGE];
    __shared__ uint32_t lost_s;  // some thread's split left bits out
    __shared__ __align__(16) uint32_t ooff_s[TM];  // bytes of O from the tile's first image, 2^31 past the last row

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % C::kWM, wn = wave / C::kWM;
    const uint32_t t = xcd_remap(blockIdx.x, p.ntiles);
    const uint32_t mt = t / (uint32_t)p.n_tiles, nt = t - mt * (uint32_t)p.n_tiles;
    const uint32_t m0 = mt * TM;
    const int n0 = (int)nt * TN;

    // source element of row r of the tile (rows past the last use the last)
    auto a_base = [&](uint32_t r) -> int64_t {
        uint32_t row = m0 + r;
        if (row >= p.M) row = p.M - 1;
        const uint32_t q = p.div_v.div(row), v = row - q * p.div_v.d;
        const uint32_t n = p.div_u.div(q), u = q - n * p.div_u.d;
        return n * p.a_n + u * p.a_u + v * p.a_v;
    };
    if (tid == 0) lost_s = 0;  // (ordered by the first barriers)
    const uint32_t image0 = p.div_u.div(p.div_v.div(m0));
    for (int r = tid; r < TM; r += THREADS) {
        const uint32_t row = m0 + r;
        const uint32_t q = p.div_v.div(row), v = row - q * p.div_v.d;
        const uint32_t n = p.div_u.div(q), u = q - n * p.div_u.d;
        ooff_s[r] = row < p.M ? 4u * (uint32_t)((n - image0) * p.o_n + u * p.o_u + v * p.o_v) : 0x80000000u;
    }

    // staging items: A 8 elements of one row, B 8 k of one column
    const int ag = tid % G, ar = tid / G;  // A item i: row ar + i * THREADS / G
    const int bn = tid % TN;               // B item i: group bg + i * THREADS / TN
    const int bg = __builtin_amdgcn_readfirstlane(tid / TN);
    // A through a buffer resource based at the tile's first image: a row's offset
    // there in bytes, plus (RUN) this thread's place in a chunk
    uint32_t aoff[AI];
    const char* const Ab = static_cast<const char*>(p.A) + (int64_t)image0 * p.a_n * 4;
#pragma unroll
    for (int i = 0; i < AI; ++i)
        aoff[i] = (uint32_t)(a_base((uint32_t)(ar + i * (THREADS / G))) - (int64_t)image0 * p.a_n) * 4u + (C::kRun ? ag * 32u : 0u);
    const uint32_t col = (uint32_t)(n0 + bn < p.N ? n0 + bn : p.N - 1);

    // the registers of a chunk on its way to LDS
    struct Regs {
        float a[AI][8], b[BI][8];
    };
    // The next chunk's rows of K. Rows past K's end read as 0 by the resource's
    // range check, so chunks past the last contribute nothing.
    const char* run_b = reinterpret_cast<const char*>(p.K);
    int64_t run_left = (int64_t)p.kd * p.N * 4;  // bytes of K from run_b on
    uint32_t koff[BI][4];  // bytes of this thread's column in 4 rows of K (the next 4 through a second resource)
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            koff[i][e] = 4u * (col + (uint32_t)((bg + i * (THREADS / TN)) * 8 + e) * (uint32_t)p.N);
    // RUN: the next chunk's position in its run and source offset, uniform
    int run_r = 0;
    int64_t run_off = 0;
    // else: its first group of 8 elements of the reduction
    uint32_t next_g = 0;
    auto load = [&](Regs& rg) {
        if constexpr (C::kRun) {
            const __amdgpu_buffer_rsrc_t ars =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(Ab) + run_off * 4, 0, 0x7fffffff, 0x00027000);
#pragma unroll
            for (int i = 0; i < AI; ++i) load8(ars, aoff[i], rg.a[i]);
        } else {
            const __amdgpu_buffer_rsrc_t ars =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(Ab), 0, 0x7fffffff, 0x00027000);
            uint32_t gi = next_g + (uint32_t)ag;
            if (gi >= (uint32_t)p.groups) gi = (uint32_t)p.groups - 1;  // meets zeros of B
            const uint32_t a = p.div_seg.div(gi * 8u), r = gi * 8u - a * (uint32_t)p.seglen;
            const uint32_t off = (a * (uint32_t)p.xstride + r) * 4u;
            const uint32_t cnt = (uint32_t)p.seglen - r;  // elements left in the run
            if (cnt >= 8) {
#pragma unroll
                for (int i = 0; i < AI; ++i) load8(ars, aoff[i] + off, rg.a[i]);
            } else {
                // the group goes on in the next run (seglen >= 8), or ends past the
                // reduction: out of the resource's range, read as 0. Masks, not
                // branches, for the registers' sake.
                const uint32_t jump = 4u * ((uint32_t)p.xstride - (uint32_t)p.seglen);
#pragma unroll
                for (uint32_t e = 0; e < 8; ++e) {
                    const uint32_t next = (uint32_t)((int32_t)(cnt - 1u - e) >> 31);
                    const uint32_t past = (uint32_t)((int32_t)(p.kd - 1u - (gi * 8u + e)) >> 31);
                    const uint32_t oe = off + 4u * e + (jump & next);
#pragma unroll
                    for (int i = 0; i < AI; ++i)
                        rg.a[i][e] = __builtin_bit_cast(
                            float, __builtin_amdgcn_raw_buffer_load_b32(ars, (aoff[i] + oe) | (past & 0x80000000u), 0, 0));
                }
            }
            next_g += G;
        }
        const int left4 = (int)run_left - 16 * p.N;
        const __amdgpu_buffer_rsrc_t rsrc[2] = {
            __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(run_b), 0, (int)run_left, 0x00027000),
            __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(run_b) + (int64_t)16 * p.N, 0, left4 < 0 ? 0 : left4, 0x00027000)};
#pragma unroll
        for (int i = 0; i < BI; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                rg.b[i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc[e / 4], koff[i][e % 4], 0, 0));
        // masks instead of branches, so that the chunk stays one block of code
        const int64_t kstep = (int64_t)C::KT * 4 * p.N;
        const int64_t more = ((kstep - run_left) >> 63);                   // ~0 before the last chunk
        run_b += kstep & more;
        run_left = (run_left - kstep) & more;
        if constexpr (C::kRun) {
            const int64_t wrap = ((int64_t)(run_r + C::KT - p.seglen) >> 63);  // ~0 inside the run
            run_off += (C::KT + ((p.xstride - p.seglen) & ~wrap)) & more;
            run_r = (run_r + C::KT) & (int)wrap;
        }
    };
    uint32_t lost = 0;
    auto stage = [&](const Regs& r, char* __restrict__ to) {
        char* const ldsA = to;
        char* const ldsB = to + 3 * C::APL;
#pragma unroll
        for (int i = 0; i < AI; ++i) {
            u32x4 h, m, l;
            split8(r.a[i], h, m, l, lost);
            const uint32_t o = swz((uint32_t)(ar + i * (THREADS / G)), (uint32_t)ag);
            *reinterpret_cast<u32x4*>(ldsA + o) = h;
            *reinterpret_cast<u32x4*>(ldsA + C::APL + o) = m;
            *reinterpret_cast<u32x4*>(ldsA + 2 * C::APL + o) = l;
        }
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            u32x4 h, m, l;
            split8(r.b[i], h, m, l, lost);
            const uint32_t o = swz((uint32_t)bn, (uint32_t)(bg + i * (THREADS / TN)));
            *reinterpret_cast<u32x4*>(ldsB + o) = h;
            *reinterpret_cast<u32x4*>(ldsB + C::BPL + o) = m;
            *reinterpret_cast<u32x4*>(ldsB + 2 * C::BPL + o) = l;
        }
    };

    floatx16 acc[BM][BN] = {}, low[BM][BN] = {};
    struct Frags {
        bf16x8 a[BM][3], b[BN][3];
    };
    auto read = [&](Frags& f, const char* __restrict__ from, int kk) {
        const char* const ldsA = from;
        const char* const ldsB = from + 3 * C::APL;
        const uint32_t g = (uint32_t)(2 * kk + (lane >> 5));
#pragma unroll
        for (int q = 0; q < 3; ++q) {
#pragma unroll
            for (int i = 0; i < BM; ++i)
                f.a[i][q] = *reinterpret_cast<const bf16x8*>(
                    ldsA + q * C::APL + swz((uint32_t)((wm * BM + i) * 32 + (lane & 31)), g));
#pragma unroll
            for (int j = 0; j < BN; ++j)
                f.b[j][q] = *reinterpret_cast<const bf16x8*>(
                    ldsB + q * C::BPL + swz((uint32_t)((wn * BN + j) * 32 + (lane & 31)), g));
        }
    };
    auto products = [&](const Frags& f) {
#define MEC_MM(X, Y, ACC)                                       \
    _Pragma("unroll") for (int i = 0; i < BM; ++i)              \
        _Pragma("unroll") for (int j = 0; j < BN; ++j)          \
            ACC[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i][X], f.b[j][Y], ACC[i][j], 0, 0, 0);
        MEC_MM(0, 0, acc)
        MEC_MM(1, 0, low)
        MEC_MM(0, 1, low)
        MEC_MM(1, 1, low)
        MEC_MM(2, 0, low)
        MEC_MM(0, 2, low)
#undef MEC_MM
    };

    // One chunk, in two halves of 16 k. The first half's fragments are in
    // registers on entry; while its products run, the second half's are read and
    // the next chunk is split into the other stage. After the barrier the next
    // chunk's first fragments are read and the chunk after the one already on
    // its way is requested, under the second half's products. Chunks past the
    // last are zeros.
    Frags f0, f1;
    auto step = [&](Regs& now, const char* __restrict__ cur, char* __restrict__ nxt) {
        __builtin_amdgcn_sched_barrier(0);
        read(f1, cur, 1);
        __builtin_amdgcn_sched_barrier(0);
        stage(now, nxt);
        products(f0);
#pragma unroll
        for (int s = 0; s < 6 * BM * BN; ++s) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);  // VALU
            __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // LDS write
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        read(f0, nxt, 0);
        __builtin_amdgcn_sched_barrier(0);
        load(now);
        products(f1);
#pragma unroll
        for (int s = 0; s < 6 * BM * BN; ++s) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // VALU
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // global read
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (C::kOne) {
        Regs r;
        load(r);
        stage(r, lds);
        load(r);
        __syncthreads();
        auto one = [&](const char* __restrict__ cur, char* __restrict__ nxt) {
            read(f0, cur, 0);
            stage(r, nxt);
            products(f0);
            read(f0, cur, 1);
            load(r);
            products(f0);
            __syncthreads();
        };
        for (int c = 0; c < p.nchunks; c += 2) {
            one(lds, lds + C::STAGE);
            one(lds + C::STAGE, lds);
        }
    } else {
        Regs r0, r1;
        load(r0);
        load(r1);
        stage(r0, lds);
        load(r0);
        __syncthreads();
        read(f0, lds, 0);
        // r1 holds chunk c + 1, r0 chunk c + 2
        for (int c = 0; c < p.nchunks; c += 2) {
            step(r1, lds, lds + C::STAGE);
            step(r0, lds + C::STAGE, lds);
        }
    }

    // Values the split does not hold (see the top). Rows and columns past the last
    // are copies of the last, so all accumulators count.
    uint32_t most = 0;
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float x = acc[i][j][v] + low[i][j][v];  // (a bit cast of the vector's element takes element 0)
                acc[i][j][v] = x;
                const uint32_t bits = __builtin_bit_cast(uint32_t, x) & 0x7fffffffu;
                most = bits > most ? bits : most;
            }
    const bool bad = most >= 0x7f800000u;
    if (lost & 0xffffu) lost_s = 1;
    __syncthreads();
    // O through a buffer resource based at the tile's first image: rows past the
    // last and channels past N have offsets beyond its range and are dropped
    const __amdgpu_buffer_rsrc_t orsrc = __builtin_amdgcn_make_buffer_rsrc(
        p.O + p.o_off + (int64_t)image0 * p.o_n, 0, 0x40000000, 0x00027000);
    if (lost_s || __any(bad)) {
#pragma clang loop unroll(disable)
        for (int block = 0; block < BM * BN; ++block) {
            const int i = block / BN, n = n0 + (wn * BN + block % BN) * 32 + (lane & 31);
            const int64_t row = a_base((uint32_t)((wm * BM + i) * 32 + (lane & 31))) - (int64_t)image0 * p.a_n;
            const floatx16 sum = plain_block(Ab, static_cast<const char*>(p.K), (uint32_t)row * 4u, 4u * (uint32_t)(n < p.N ? n : p.N - 1),
                                             p.kd, (uint32_t)p.N, (uint32_t)p.seglen, (uint32_t)p.xstride, p.div_seg.m,
                                             p.div_seg.shift, lane);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float x = sum[v];
                const uint32_t at = ooff_s[(wm * BM + i) * 32 + acc_row(v, lane)] + (n < p.N ? 4u * (uint32_t)n : 0x40000000u);
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), orsrc, at, 0, 2);
            }
        }
        return;
    }
    uint32_t coff[BN];
#pragma unroll
    for (int j = 0; j < BN; ++j) {
        const int n = n0 + (wn * BN + j) * 32 + (lane & 31);
        coff[j] = n < p.N ? 4u * (uint32_t)n : 0x40000000u;
    }
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const u32x4 ro = *reinterpret_cast<const u32x4*>(&ooff_s[(wm * BM + i) * 32 + acc_row(4 * w, lane)]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < BN; ++j) {
                    const float x = acc[i][j][4 * w + e];
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), orsrc, ro[e] + coff[j], 0, 2);
                }
        }
}

template <int BM, int BN, int WM, int WN, bool ONE = false, bool ANY = true>
hipError_t run_tile(TileParams p, hipStream_t stream) {
    using CA = TileCfg<BM, BN, WM, WN, true, ONE>;
    using CR = TileCfg<BM, BN, WM, WN, false, ONE>;
    p.n_tiles = (p.N + CA::TN - 1) / CA::TN;
    const int64_t ntiles = ((int64_t)p.M + CA::TM - 1) / CA::TM * p.n_tiles;
    if (ntiles > 0x7fffffff) return hipErrorInvalidValue;
    p.ntiles = (uint32_t)ntiles;
    p.nchunks = (p.groups + CA::G - 1) / CA::G;
    if constexpr (ANY) {
        if (p.seglen % 32) {
            hipLaunchKernelGGL(tile_gemm_f32_kernel<CR>, dim3(p.ntiles), dim3(CR::THREADS), 0, stream, p);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL(tile_gemm_f32_kernel<CA>, dim3(p.ntiles), dim3(CA::THREADS), 0, stream, p);
    return hipGetLastError();
}

}  // namespace

// Which tile: 0 256x128 (8 waves, one workgroup per compute unit), 1 128x128
// (one), 2 128x64 (two), 3 64x64 (three). The busiest compute unit takes
// ceil(tiles / 256) of them, as many at a time as fit; a chunk costs the times
// below with 1, 2, 3 resident, a tile's start and end the last figure, all in us
// and measured on this GPU on long reductions over whole chunks. Of 14000 shapes past 15
// us the model gives 0.85 to 1.2 of the time there, down to 0.7 where runs are gathered
// and 0.6 below 400 terms; it has to order the tiles, not to time them.
// Runs that are not whole chunks leave out 128x128, whose gathering loads spill
// registers (11x11 over 3 channels at batch 32: 226 us, 70 in 256x128).
int pick_tile(int64_t M, int64_t N, int64_t nchunks, bool run) {
    struct Opt {
        int tm, tn, fit;
        double chunk[3], ends;
    };
    constexpr Opt opts[4] = {{256, 128, 1, {1.85, 0, 0}, 10.0},
                             {128, 128, 1, {1.25, 0, 0}, 4.0},
                             {128, 64, 2, {0.88, 1.45, 0}, 3.0},
                             {64, 64, 3, {0.61, 0.85, 1.2}, 2.5}};
    int best = 0;
    double best_t = 0.0;
    for (int i = 0; i < 4; ++i) {
        if (i == 1 && !run) continue;
        const Opt& o = opts[i];
        const int64_t tiles = ((M + o.tm - 1) / o.tm) * ((N + o.tn - 1) / o.tn);
        const int64_t busiest = (tiles + 255) / 256;
        const int64_t rounds = busiest / o.fit, rest = busiest % o.fit;
        double t = (double)rounds * ((double)nchunks * o.chunk[o.fit - 1] + o.ends);
        if (rest) t += (double)nchunks * o.chunk[rest - 1] + o.ends;
        if (i == 0 || t < best_t) {
            best = i;
            best_t = t;
        }
    }
    return best;
}

// The ring kernel's tall layers that are faster here from I, against the ring (11x11
// stride 4 and 9x9 over 3 channels, us, ring / here): 33 to 64 channels always (batch 1
// 19.6 / 12.8, 32 57.9 / 43.2, 128 181 / 156; 9x9 14.3 / 10.6 to 131 / 116), past 96,
// which the ring takes in two passes, always (100 channels: 143 / 74, 9x9 103 / 57),
// between them, where a fourth of a 128-channel tile is empty, with at most 160 tiles
// (batch 1 25.5 / 12.6, 4 26.8 / 17.4) or full rounds of them (batch 128 245 / 237): over
// the batches of two rounds and more the ring takes 1.02 to 1.08 of the time here where
// tiles fill at least 0.8 of their rounds, 0.95 where 0.5 to 0.75. One round of 161 to 256
// tiles lies near even (1.02 to 1.12). Up to 32 channels the ring leads from batch 16 on
// (120 / 147 at 128).
static bool tall_from_input(const Shape& s) {
    if (s.k_h < 9 || s.R < 24 || s.k_c <= 32 || s.k_c > 128) return false;
    if (s.k_c <= 64 || s.k_c > 96) return true;
    const int64_t tiles = (s.i_n * s.o_h * s.o_w + 255) / 256;
    return tiles <= 160 || 5 * tiles >= 4 * ((tiles + 255) / 256 * 256);
}

// Its 32-bit offsets hold the shape: rows, K, and the span of O from a tile's first
// image. Runs are at least the groups of 8 they are loaded in.
bool gemm_tile_holds(const Shape& s, bool fused, const OutLayout* layout) {
    const int64_t M = s.i_n * s.o_h * s.o_w, kd = s.k_h * s.R;
    const int64_t img = layout ? layout->img : s.o_h * s.o_w * s.k_c;
    const int64_t images = 256 / (s.o_h * s.o_w) + 2;  // that 256 rows can touch
    const int64_t src = fused ? s.i_h * s.i_w * s.i_c : s.o_w * s.i_h * s.R;  // elements of an image
    if ((images < s.i_n ? images : s.i_n) * src >= (int64_t(1) << 29)) return false;
    if (M >= (int64_t(1) << 31) || kd >= (int64_t(1) << 28) || s.k_c >= (int64_t(1) << 28) ||
        kd * s.k_c >= (int64_t(1) << 29) || (images < s.i_n ? images : s.i_n) * img >= (int64_t(1) << 28))
        return false;
    return (fused ? s.R : kd) >= 8;
}

// Taken where it holds the shape, except for
// * reductions of one chunk, whose time is the tile's start and end (1x1 over 16
//   and 32 channels: 24 against 19 us and 13.1 against 12.1 for the plain tiles),
// * what the fixed kernels' own tiles (32 pairs x 2 rows x 64 channels, vectors at
//   16-byte boundaries) do faster; times here / there, in us:
//   - 3x3 and 5x5 at stride 1 and 7x7 at stride 2, reductions past 640, up to 128 of
//     their tiles, each of which they give to two workgroups (7x7x512 -> 512 at batch 32
//     86 / 60; 67x67x288 -> 32 7x7 at batch 8 231 / 187; 32x32x320 -> 528 5x5 131 / 89;
//     the median of 1600 shapes 0.7 of the time here, past 128 tiles 1.05 to 1.3). Rows
//     that are no multiples of 16 go through registers there: past 1280 (7x7x420 -> 84
//     3x3, batch 109, 76 / 56; of 150 shapes 0.62 to 0.96, below 1280 to 1.45),
//   - 3x3 at stride 1, and 5x5 from I, whose runs are not whole chunks of 32, up to a
//     tile per compute unit (18x18x368 -> 192 3x3, batch 19, 66 / 52; of 300 shapes 0.83
//     to 1.0; 18x18x48 -> 160 5x5, batch 16, 26.3 / 25.1; of 136 shapes 0.88 to 0.99, from
//     L 1.03 to 1.22; with whole chunks 1.04 to 1.15),
//   - one-row kernels whose runs end in half a chunk of at most three, from 1600 tiles of
//     64 x 64 on, where memory bounds both (79x79x80 -> 496 1x1, batch 29, 201 / 169;
//     52x52x80 -> 224, batch 50, 73 / 66; over 48 channels even),
// * the ring kernel's layers (7x7 stride 2 over 3 channels 98 against 83 us, 3x3
//   over 3 channels 91 against 45; 11x11 over 3 channels to 96, batch 128, from L:
//   248 against 239), but for the tall kernels below from I.
bool gemm_tile_preferred(const Shape& s, const void* A, const void* K, bool fused, const OutLayout* layout) {
    if (!gemm_tile_holds(s, fused, layout)) return false;
    const int64_t M = s.i_n * s.o_h * s.o_w, kd = s.k_h * s.R, n64 = (s.k_c + 63) / 64;
    if (kd <= 32) return false;
    if (s.R % 4 == 0 && !(fused && s.i_c % 4) && s.k_c % 4 == 0 && !(((uintptr_t)A | (uintptr_t)K) & 15u)) {
        const int64_t t2 = (s.pairs + 31) / 32 * ((s.o_h + 1) / 2) * n64;  // their tiles
        const bool k3 = s.k_h == 3 && s.s_h == 1, k5 = s.k_h == 5 && s.s_h == 1, k7 = s.k_h == 7 && s.s_h == 2;
        const bool whole = (fused ? s.R : kd) % 32 == 0, r16 = s.R % 16 == 0;
        if ((k3 || k5 || k7) && kd > (r16 ? 640 : 1280) && t2 <= 128 && !layout) return false;
        if ((k3 || (k5 && fused && !layout)) && r16 && !whole && t2 <= 256) return false;
        if (r16 && s.k_h == 1 && s.s_h == 1 && !whole && s.R <= 96 && (M + 63) / 64 * n64 >= 1600) return false;
    }
    if (gemm_ring_taken(s, 0, fused, layout)) return fused && tall_from_input(s);
    return true;
}

bool gemm_tile_from_input(const Shape& s, const void* I, const void* K) {
    return gemm_ring_taken(s, 0, false, nullptr) && tall_from_input(s) && gemm_tile_preferred(s, I, K, true, nullptr);
}

hipError_t launch_gemm_tile(const Shape& s, const void* A, const void* K, float* O, bool fused,
                            hipStream_t stream, const OutLayout* layout) {
    TileParams p{};
    p.A = A;
    p.K = K;
    p.O = O;
    p.M = (uint32_t)(s.i_n * s.o_h * s.o_w);
    p.N = (int32_t)s.k_c;
    const OutLayout o = layout ? *layout : OutLayout{s.o_h * s.o_w * s.k_c, s.o_w * s.k_c, s.k_c, 0};
    p.o_n = o.img;
    p.o_off = o.off;
    if (fused) {  // (n, h, w): neighbouring rows read neighbouring pixels
        p.div_u = FastDiv((uint32_t)s.o_h);
        p.div_v = FastDiv((uint32_t)s.o_w);
        p.a_n = s.i_h * s.i_w * s.i_c;
        p.a_u = s.s_h * s.i_w * s.i_c;
        p.a_v = s.s_w * s.i_c;
        p.o_u = o.row;
        p.o_v = o.col;
        p.nseg = (int32_t)s.k_h;
        p.seglen = (int32_t)s.R;
        p.xstride = s.i_w * s.i_c;
    } else {  // (n, w, h): neighbouring rows read overlapping windows
        p.div_u = FastDiv((uint32_t)s.o_w);
        p.div_v = FastDiv((uint32_t)s.o_h);
        p.a_n = s.o_w * s.i_h * s.R;
        p.a_u = s.i_h * s.R;
        p.a_v = s.s_h * s.R;
        p.o_u = o.col;
        p.o_v = o.row;
        p.nseg = 1;
        p.seglen = (int32_t)(s.k_h * s.R);
        p.xstride = 0;
    }
    p.kd = (uint32_t)(p.nseg * p.seglen);
    p.groups = (int32_t)((p.kd + 7) / 8);
    p.div_seg = FastDiv((uint32_t)p.seglen);
    switch (pick_tile(p.M, p.N, (p.groups + 3) / 4, p.seglen % 32 == 0)) {
        case 0: return run_tile<2, 2, 4, 2, true>(p, stream);
        case 1: return run_tile<2, 2, 2, 2, false, false>(p, stream);
        case 2: return run_tile<1, 2, 4, 1>(p, stream);
        default: return run_tile<1, 1, 2, 2>(p, stream);
    }
}

}  // namespace mec
