// The weight gradient's products on the bf16 matrix cores, fp32 as six bf16
// products (mec_gemm_tile.hip says how and how exactly):
//   part[s][j][m] = sum over the pixels p of share s of A[p][j] * G[p][m],
// where p runs over output pixels (n, h, w) and A[p] is the window of pixel p in
// L, or the same k_h runs of R elements in I. Both operands have the reduction
// index in their rows, so they are staged as they lie in memory (16-byte loads of 8
// columns of one pixel, split on their way to LDS) and turned by the transposing
// LDS reads. A workgroup takes 128 rows j x 64 columns m of dK over one share, in
// chunks of 32 pixels through two stages of LDS, two workgroups per compute unit.
// What bounds it is splitting and writing 192 columns to LDS per chunk beside 24
// matrix instructions a wave. Against the fp32 kernels, whole gradient (products and
// the shares' sum), batch 32: 58x58x64 -> 64 101 -> 70 us, 112x112x64 -> 128 561 ->
// 417, 28x28x128 99 -> 58, 14x14x256 83 -> 52, 24x24x96 -> 256 5x5 181 -> 130,
// 224x224x64 -> 64 7x7 1695 -> 982; errors against 64 bits 0.35-0.55 of theirs, on
// operands of one sign to 0.8. The
// windows' offsets are worked out once per chunk by one wave (83 us on the first of
// these with every thread dividing for itself).
#include "mec_split.h"

namespace mec {
namespace {

struct WgradTileParams {
    const float* A;  // L or I
    const float* G;
    float* part;
    uint32_t P;      // output pixels
    int32_t KD, N;   // k_h * R, k_c
    int32_t seglen;  // of the window's runs, as in mec_gemm_tile.hip
    uint32_t xstride;
    uint32_t a_n, a_h, a_w; // source elements per step of n, h, w
    FastDiv div_ow, div_oh, div_seg;
    int64_t a_bytes;
    int32_t g_bytes;
    int32_t j_tiles, m_tiles, splits, chunks;  // chunks of 32 pixels in all
    uint32_t ntiles;
};

constexpr int kJ = 128, kM = 64, kPix = 32, kWgThreads = 256;
constexpr int kAPlane = kPix * kJ * 2, kBPlane = kPix * kM * 2;  // bytes of one part's plane
constexpr int kWgStage = 3 * (kAPlane + kBPlane);

// WHOLE: runs are whole groups of 8 columns.
template <bool WHOLE>
__global__ __launch_bounds__(kWgThreads, 2) void wgrad_tile_kernel(WgradTileParams p) {
    __shared__ __align__(16) char lds[2 * kWgStage];
    __shared__ uint32_t lost_s;
    __shared__ uint32_t pix_s[4][kPix];  // byte offsets of the windows of chunks c .. c + 3, by c % 4
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wj = wave & 1, wn = wave >> 1;  // 64 x 32 of the tile per wave

    const uint32_t t = xcd_remap(blockIdx.x, p.ntiles);
    const int jt = (int)(t % (uint32_t)p.j_tiles);
    const uint32_t rest = t / (uint32_t)p.j_tiles;
    const int mt = (int)(rest % (uint32_t)p.m_tiles), s = (int)(rest / (uint32_t)p.m_tiles);
    const int j0 = jt * kJ, m0 = mt * kM;
    const int c_begin = (int)((int64_t)s * p.chunks / p.splits), c_end = (int)((int64_t)(s + 1) * p.chunks / p.splits);
    if (tid == 0) lost_s = 0;

    // source element of pixel p's window, from the share's first image on
    const uint32_t image0 = p.div_oh.div(p.div_ow.div((uint32_t)c_begin * kPix));
    auto pixel = [&](uint32_t q) -> uint32_t {
        const uint32_t r = p.div_ow.div(q), w = q - r * p.div_ow.d;
        const uint32_t n = p.div_oh.div(r), h = r - n * p.div_oh.d;
        return (n - image0) * p.a_n + h * p.a_h + w * p.a_w;
    };
    // staging: A pixels tid / 16 and + 16, columns 8 (tid % 16)..; G pixel tid / 8,
    // columns 8 (tid % 8)..
    const uint32_t ag = (uint32_t)tid & 15u, ar = (uint32_t)tid >> 4;
    const uint32_t bg = (uint32_t)tid & 7u, br = (uint32_t)tid >> 3;
    const uint32_t j = (uint32_t)j0 + ag * 8u;
    const uint32_t seg = p.div_seg.div(j), r0 = j - seg * (uint32_t)p.seglen;
    const uint32_t jcol = (seg * p.xstride + r0) * 4u;
    const uint32_t run = (uint32_t)p.seglen - r0;        // elements left in the run
    const uint32_t jump = 4u * (p.xstride - (uint32_t)p.seglen);
    const int64_t a_first = (int64_t)image0 * p.a_n, a_left = p.a_bytes - a_first * 4;
    const __amdgpu_buffer_rsrc_t ars = buffer(p.A + a_first, a_left > 0x7fffffff ? 0x7fffffff : (int)a_left),
                                 grs = buffer(p.G, p.g_bytes);
    constexpr uint32_t kNone = 0x80000000u;  // past any range: read as 0
    const uint32_t none = j < (uint32_t)p.KD ? 0u : kNone;
    // the offsets of chunk c's pixels, worked out once by one wave
    auto locate = [&](int c) {
        if (tid < kPix) {
            const uint32_t q = (uint32_t)c * kPix + (uint32_t)tid;
            pix_s[c & 3][tid] = c < c_end && q < p.P ? pixel(q) * 4u : kNone;
        }
    };

    struct Regs {
        float a[2][8], b[8];
    };
    auto load = [&](Regs& r, int c) {
        uint32_t off[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) off[i] = (pix_s[c & 3][ar + 16 * i] + jcol) | none;
        if (WHOLE || run >= 8 || none) {
#pragma unroll
            for (int i = 0; i < 2; ++i) load8(ars, off[i], r.a[i]);
        } else {  // the columns go on in the next run (seglen >= 8), or end
#pragma unroll
            for (uint32_t e = 0; e < 8; ++e) {
                const uint32_t next = (uint32_t)((int32_t)(run - 1u - e) >> 31);
                const uint32_t past = (uint32_t)((int32_t)((uint32_t)p.KD - 1u - (j + e)) >> 31) & kNone;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    r.a[i][e] = __builtin_bit_cast(
                        float, __builtin_amdgcn_raw_buffer_load_b32(ars, (off[i] + 4u * e + (jump & next)) | past, 0, 0));
            }
        }
        const uint32_t q = (uint32_t)c * kPix + br;
        load8(grs, c < c_end && q < p.P ? (q * (uint32_t)p.N + (uint32_t)m0 + bg * 8u) * 4u : kNone, r.b);
    };
    // granules permuted so that the rows a transposing read takes fall on
    // different banks (16 granules a row of A, 8 a row of G)
    uint32_t lost = 0;
    auto stage = [&](const Regs& r, char* __restrict__ to) {
        u32x4 h, m, l;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t row = ar + 16u * i;
            char* at = to + row * 256u + ((ag ^ (2u * (row & 3u) | (row & 8u))) << 4);
            split8(r.a[i], h, m, l, lost);
            *reinterpret_cast<u32x4*>(at) = h;
            *reinterpret_cast<u32x4*>(at + kAPlane) = m;
            *reinterpret_cast<u32x4*>(at + 2 * kAPlane) = l;
        }
        char* at = to + 3 * kAPlane + br * 128u + ((bg ^ (2u * (br & 3u))) << 4);
        split8(r.b, h, m, l, lost);
        *reinterpret_cast<u32x4*>(at) = h;
        *reinterpret_cast<u32x4*>(at + kBPlane) = m;
        *reinterpret_cast<u32x4*>(at + 2 * kBPlane) = l;
    };

    // the transposing read (see mec_gemm_patch.hip): row and column of this lane's
    // address within 16 pixels x 32 columns
    const uint32_t tr = (uint32_t)((lane >> 5) * 8 + ((lane & 15) >> 2));
    const uint32_t tc = (uint32_t)(((lane >> 4) & 1) * 16 + (lane & 3) * 4);
    uint32_t aat[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t col = (uint32_t)(wj * 64 + i * 32) + tc;
        aat[i] = tr * 256u + (((col >> 3) ^ (2u * (tr & 3u) | (tr & 8u))) << 4) + ((col & 7u) << 1);
    }
    const uint32_t bcol = (uint32_t)(wn * 32) + tc;
    const uint32_t bat = 3 * kAPlane + tr * 128u + (((bcol >> 3) ^ (2u * (tr & 3u))) << 4) + ((bcol & 7u) << 1);
    struct Frags {
        bf16x8 a[2][3], b[3];
    };
    auto turn = [&](const char* at, uint32_t row4) {  // 8 pixels of a column: two reads, 4 rows apart
        typedef short short4v __attribute__((ext_vector_type(4)));
        typedef short short8v __attribute__((ext_vector_type(8)));
        typedef __attribute__((address_space(3))) short4v lds_short4v;
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)at);
        const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)(at + row4));
        const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, v);
    };
    auto read = [&](Frags& f, const char* __restrict__ from, int kk) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            f.b[q] = turn(from + bat + q * kBPlane + kk * 16 * 128, 4 * 128);
#pragma unroll
            for (int i = 0; i < 2; ++i) f.a[i][q] = turn(from + aat[i] + q * kAPlane + kk * 16 * 256, 4 * 256);
        }
    };
    floatx16 acc[2] = {}, low[2] = {};
    auto products = [&](const Frags& f) {
#define MEC_MM(X, Y, ACC)                            \
    _Pragma("unroll") for (int i = 0; i < 2; ++i)    \
        ACC[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i][X], f.b[Y], ACC[i], 0, 0, 0);
        MEC_MM(0, 0, acc)
        MEC_MM(1, 0, low)
        MEC_MM(0, 1, low)
        MEC_MM(1, 1, low)
        MEC_MM(2, 0, low)
        MEC_MM(0, 2, low)
#undef MEC_MM
    };

    // chunk c is multiplied from one stage while c + 1 is split into the other and
    // c + 3 is requested (c + 2 is on its way); chunks past the share read as zeros
    Frags f0, f1;
    auto step = [&](Regs& r, int c, const char* __restrict__ cur, char* __restrict__ nxt) {
        read(f0, cur, 0);
        read(f1, cur, 1);
        __builtin_amdgcn_sched_barrier(0);
        stage(r, nxt);
        products(f0);
#pragma unroll
        for (int n = 0; n < 12; ++n) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 10, 0);  // VALU
            __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // LDS write
        }
        __builtin_amdgcn_sched_barrier(0);
        load(r, c + 3);
        locate(c + 4);
        products(f1);
        __syncthreads();
    };
    Regs ra, rb;
    for (int i = 0; i < 4; ++i) locate(c_begin + i);
    __syncthreads();
    load(ra, c_begin);
    load(rb, c_begin + 1);
    stage(ra, lds);
    load(ra, c_begin + 2);
    __syncthreads();
    for (int c = c_begin; c < c_end; c += 2) {
        step(rb, c, lds, lds + kWgStage);
        step(ra, c + 1, lds + kWgStage, lds);
    }

    // results the split cannot have got right, as in mec_gemm_tile.hip
    const int m = m0 + wn * 32 + (lane & 31);
    uint32_t most = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float x = acc[i][v] + low[i][v];
            acc[i][v] = x;
            const uint32_t bits = __builtin_bit_cast(uint32_t, x) & 0x7fffffffu;
            most = bits > most ? bits : most;
        }
    const bool bad = most >= 0x7f800000u && m < p.N;
    if (lost & 0xffffu) lost_s = 1;
    __syncthreads();
    const uint32_t p_begin = (uint32_t)c_begin * kPix;
    const uint32_t p_end = (uint32_t)c_end * kPix < p.P ? (uint32_t)c_end * kPix : p.P;
    if (lost_s || __any(bad)) {
        const uint32_t gm = 4u * (uint32_t)(m < p.N ? m : p.N - 1);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t jj = (uint32_t)(j0 + wj * 64 + i * 32 + (lane & 31));
            const uint32_t jc = jj < (uint32_t)p.KD ? jj : (uint32_t)p.KD - 1u, sj = p.div_seg.div(jc);
            const uint32_t cj = 4u * (sj * p.xstride + (jc - sj * (uint32_t)p.seglen));  // of this lane's row of dK in a window
            acc[i] = floatx16{};
            plain_products(
                acc[i], (p_end - p_begin + 15u) / 16u,
                [&](uint32_t st, float* x) {
                    const uint32_t q = p_begin + st * 16u + 8u * (uint32_t)(lane >> 5);
#pragma unroll
                    for (uint32_t e = 0; e < 8; ++e)
                        x[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                            ars, q + e < p_end ? pixel(q + e) * 4u + cj : kNone, 0, 0));
                },
                [&](uint32_t st, float* x) {
                    const uint32_t q = p_begin + st * 16u + 8u * (uint32_t)(lane >> 5);
#pragma unroll
                    for (uint32_t e = 0; e < 8; ++e)
                        x[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                            grs, q + e < p_end ? (q + e) * (uint32_t)p.N * 4u + gm : kNone, 0, 0));
                });
        }
    }
    float* const out = p.part + (int64_t)s * p.KD * p.N;
    if (m < p.N) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int jj = j0 + wj * 64 + i * 32 + acc_row(v, lane);
                if (jj < p.KD) out[(int64_t)jj * p.N + m] = acc[i][v];
            }
    }
}

}  // namespace

// Its 32-bit offsets hold the shape: G, and the images that a share's windows lie in. From
// L and from I alike, since dK is the same bit for bit from either.
bool wgrad_tile_holds(const Shape& s) {
    const int64_t lim = int64_t(1) << 31, pixels = s.i_n * s.o_h * s.o_w;
    if (s.R < 8 || pixels * s.k_c * 4 >= lim || s.i_n * s.i_h * s.i_w * s.i_c * 4 >= lim) return false;
    const int64_t image = s.o_w * s.i_h * s.R * 4;
    if (s.i_n * image < lim) return true;
    const int64_t chunks = (pixels + kPix - 1) / kPix, splits = wgrad_tile_splits(s, wgrad_splits(s));
    return ((chunks / splits + 1) * kPix / (s.o_h * s.o_w) + 2) * image < lim;
}

// Shares: the count, at most the partial sums' room, that minimises the busiest
// compute unit's chunks (two workgroups at a time, 1.2 us a chunk for the two, 0.8
// alone, 6 us to start and end) plus the partial sums' write and read-back.
int64_t wgrad_tile_splits(const Shape& s, int64_t room) {
    const uint32_t chunks = (uint32_t)((s.i_n * s.o_h * s.o_w + kPix - 1) / kPix);  // the pixels fit 29 bits
    const int64_t tiles = ((s.k_h * s.R + kJ - 1) / kJ) * ((s.k_c + kM - 1) / kM);
    const double sums = 8.0 * (double)(s.k_h * s.R * s.k_c);
    uint32_t best = 1;
    double best_t = 0.0;
    for (uint32_t sp = 1; sp <= (uint32_t)room && sp <= chunks; ++sp) {  // (a loop per call: 32-bit divisions, no more than needed)
        const double sums_t = (double)sp * sums / 5.0e6;
        if (sp > 1 && sums_t >= best_t) break;  // it only grows
        const int64_t busiest = (tiles * sp + 255) / 256;
        const uint32_t each = (chunks + sp - 1) / sp;
        const double t = (double)(busiest / 2) * ((double)each * 1.2 + 6.0) + (double)(busiest % 2) * ((double)each * 0.8 + 6.0) + sums_t;
        if (sp == 1 || t < best_t) {
            best = sp;
            best_t = t;
        }
    }
    return best;
}

hipError_t launch_wgrad_tile(const Shape& s, const float* A, const float* G, float* part, int64_t splits,
                             hipStream_t stream, bool fused) {
    WgradTileParams p{};
    p.A = A;
    p.G = G;
    p.part = part;
    p.P = (uint32_t)(s.i_n * s.o_h * s.o_w);
    p.KD = (int32_t)(s.k_h * s.R);
    p.N = (int32_t)s.k_c;
    if (fused) {
        p.seglen = (int32_t)s.R;
        p.xstride = (uint32_t)(s.i_w * s.i_c);
        p.a_n = (uint32_t)(s.i_h * s.i_w * s.i_c);
        p.a_h = (uint32_t)(s.s_h * s.i_w * s.i_c);
        p.a_w = (uint32_t)(s.s_w * s.i_c);
        p.a_bytes = s.i_n * s.i_h * s.i_w * s.i_c * 4;
    } else {
        p.seglen = p.KD;
        p.xstride = 0;
        p.a_n = (uint32_t)(s.o_w * s.i_h * s.R);
        p.a_h = (uint32_t)(s.s_h * s.R);
        p.a_w = (uint32_t)(s.i_h * s.R);
        p.a_bytes = s.i_n * s.o_w * s.i_h * s.R * 4;
    }
    p.g_bytes = (int32_t)(s.i_n * s.o_h * s.o_w * s.k_c * 4);
    p.div_ow = FastDiv((uint32_t)s.o_w);
    p.div_oh = FastDiv((uint32_t)s.o_h);
    p.div_seg = FastDiv((uint32_t)p.seglen);
    p.j_tiles = (p.KD + kJ - 1) / kJ;
    p.m_tiles = (p.N + kM - 1) / kM;
    p.splits = (int32_t)splits;
    p.chunks = (int32_t)((p.P + kPix - 1) / kPix);
    p.ntiles = (uint32_t)((int64_t)p.j_tiles * p.m_tiles * splits);
    auto kern = p.seglen % 8 == 0 ? wgrad_tile_kernel<true> : wgrad_tile_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(p.ntiles), dim3(kWgThreads), 0, stream, p);
    return hipGetLastError();
}

}  // namespace mec
