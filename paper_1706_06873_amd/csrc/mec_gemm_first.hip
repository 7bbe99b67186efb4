// bf16 slab products over at most 4 input channels, from I: the first layers of
// networks.
//
// Their rows of L are short and start at odd elements (33 of them for 11x11 over 3
// channels), so the general tiles gather them element by element: 95 us for
// 227x227x3 -> 96 at stride 4, batch 32, whose input, output and products ask for 8.
// Here a pixel takes 4 channels (zeros past i_c) of LDS, 8 bytes, and a workgroup
// keeps K whole in LDS as the matrix instruction reads it: two neighbouring taps of
// a kernel row are 8 consecutive k, a kernel row is padded to whole pairs of taps,
// and a pair of a lane's pixel is 16 consecutive bytes of the patch. The workgroups
// are persistent: each stages K once, then takes tiles of 256 output pixels (see
// mec_gemm_patch.hip) in turn, the next tile's pixels on their way to registers
// under the current one's products. No barrier stands between a tile's products.
#include "mec_split.h"

namespace mec {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct FirstParams {
    const uint16_t* I;
    const uint16_t* K;
    float* O;
    int32_t G, o_h, o_w, i_h, i_w, i_c, k_h, k_w, N, s_h, s_w;
    int32_t TH, TW, PW, pixels, pairs, kw2;  // pairs of taps in all, per kernel row
    int32_t w_tiles, n_tiles, tiles;         // tiles: of output pixels
    FastDiv div_oh, div_TW, div_PW, div_kw2, div_wt;
    int64_t i_bytes;
};

constexpr int kMaxRows = 512;  // patch rows at most
constexpr int kFtM = 256, kFtThreads = 256, kFtPixels = 24;  // patch pixels per thread at most

// STREAM: O by streaming stores, where a pixel's channels are whole 128-byte lines (3%
// faster on outputs past 40 MB); lines that two pixels share have to meet in the cache
// (172x172x3 3x3 -> 60, batch 42: 108 us streaming, 56 through it, 83 the generic tiles;
// 154x154x1 -> 56, batch 61: 111, 62, 84).
template <int BN, bool STREAM>
__global__ __launch_bounds__(kFtThreads, BN == 2 ? 2 : 1) void first_gemm_kernel(FirstParams p) {
    constexpr int TN = 32 * BN, BM = 2;
    extern __shared__ __align__(16) char lds[];  // K, the patch, 16 bytes of zeros
    __shared__ __align__(16) uint32_t ooff_s[2][kFtM];  // by turns
    __shared__ uint32_t prow_s[kFtM];
    __shared__ uint32_t src_s[kMaxRows];  // patch row -> pixel of its first column, from the first image
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int steps = (p.pairs + 1) / 2;
    char* const ldsA = lds + steps * 2 * TN * 16;
    const int n0 = (int)(blockIdx.x % (uint32_t)p.n_tiles) * TN;

    // K: pair q of column n at (q * TN + n) * 16, channels past i_c and the tap past
    // an odd kernel row as zeros
    constexpr int kBatch = 6;  // items whose loads are in flight together
    const __amdgpu_buffer_rsrc_t krs = buffer(p.K, p.k_h * p.k_w * p.i_c * p.N * 2);
    for (int it0 = tid; it0 < steps * 2 * TN; it0 += kBatch * kFtThreads) {
        uint16_t x[kBatch][8];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int it = it0 + u * kFtThreads, q = it / TN, n = n0 + it - q * TN;
            const int a = (int)p.div_kw2.div((uint32_t)q), b = 2 * (q - a * p.kw2);
            const uint32_t row = (uint32_t)((a * p.k_w + b) * p.i_c);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool on = q < p.pairs && n < p.N && b + e / 4 < p.k_w && e % 4 < p.i_c;
                const uint32_t off = ((row + (uint32_t)(e / 4 * p.i_c + e % 4)) * (uint32_t)p.N + (uint32_t)n) * 2u;
                x[u][e] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(krs, on ? off : 0x80000000u, 0, 0);
            }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int it = it0 + u * kFtThreads;
            if (it >= steps * 2 * TN) break;
            u32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = x[u][2 * e] | (uint32_t)x[u][2 * e + 1] << 16;
            *reinterpret_cast<u32x4*>(lds + it * 16) = v;
        }
    }
    const uint32_t zeros = (uint32_t)p.pixels * 8u;  // in the patch's bytes
    if (tid < 4) *reinterpret_cast<uint32_t*>(ldsA + zeros + tid * 4) = 0;

    // the tables of a tile (as in mec_gemm_patch.hip) and its pixels' offsets in I
    uint32_t image0 = 0;
    int th = 0, w0 = 0, used = 0;
    int turn = 0;  // the table of the tile being multiplied
    auto open = [&](int tile, int to) {
        const uint32_t gt = p.div_wt.div((uint32_t)tile);
        w0 = (tile - (int)gt * p.w_tiles) * p.TW;
        const int g0 = (int)gt * p.TH;
        image0 = p.div_oh.div((uint32_t)g0);
        th = p.G - g0 < p.TH ? p.G - g0 : p.TH;
        if (tid < th) {
            const uint32_t g = (uint32_t)(g0 + tid), n = p.div_oh.div(g);
            const int h = (int)(g - n * (uint32_t)p.o_h), k = (int)(n - image0);
            const int first = (int)((image0 + 1) * (uint32_t)p.o_h) - g0;
            const int before = k == 0 ? 0 : (first - 1) * p.s_h + p.k_h + (k - 1) * ((p.o_h - 1) * p.s_h + p.k_h);
            prow_s[tid] = (uint32_t)(before + (h - (k == 0 ? g0 - (int)image0 * p.o_h : 0)) * p.s_h);
            // the input rows this output row is the first to bring: all k_h after a
            // new image, else the last s_h (s_h <= k_h)
            const int lo = tid == 0 || h == 0 ? 0 : p.k_h - p.s_h;
            for (int r = lo; r < p.k_h; ++r)
                src_s[prow_s[tid] + r] = (uint32_t)((k * p.i_h + h * p.s_h + r) * p.i_w);
        }
        for (int m = tid; m < kFtM; m += kFtThreads) {
            const int tt = (int)p.div_TW.div((uint32_t)m), x = m - tt * p.TW;
            uint32_t o = 0x80000000u;
            if (tt < th && w0 + x < p.o_w) {
                const uint32_t g = (uint32_t)(g0 + tt), n = p.div_oh.div(g), h = g - n * (uint32_t)p.o_h;
                o = 4u * ((((n - image0) * (uint32_t)p.o_h + h) * (uint32_t)p.o_w + (uint32_t)(w0 + x)) * (uint32_t)p.N);
            }
            ooff_s[to][m] = o;
        }
    };
    // byte offset of patch pixel q (past the patch: of some pixel)
    auto place = [&](int q, uint32_t odd_base) {
        uint32_t pr = p.div_PW.div((uint32_t)q);
        int pc = w0 * p.s_w + q - (int)pr * p.PW;
        if (pc >= p.i_w) pc = p.i_w - 1;  // read by outputs past o_w, and by the tap past an odd row, only
        if (pr >= (uint32_t)kMaxRows) pr = 0;
        return (src_s[pr] + (uint32_t)pc) * (uint32_t)p.i_c * 2u + odd_base;
    };
    u32x2 px[kFtPixels];
    uint32_t half = 0;  // bit i: pixel i starts in the upper half of its first word
    auto load_patch = [&]() {
        used = __builtin_amdgcn_readfirstlane(((int)prow_s[th - 1] + p.k_h) * p.PW);
        const int64_t base = (int64_t)image0 * p.i_h * p.i_w * p.i_c * 2;
        // (an image may start between two words)
        const char* const Ib = reinterpret_cast<const char*>(p.I) + (base & ~(int64_t)3);
        const int64_t rest = p.i_bytes - (base & ~(int64_t)3);
        const uint32_t left = (uint32_t)(rest > 0x7fffffff ? 0x7fffffff : rest), odd_base = (uint32_t)base & 2u;
        const __amdgpu_buffer_rsrc_t rs = buffer(Ib, (int)left);
        bool last = false;
        half = 0;
#pragma unroll
        for (int i = 0; i < kFtPixels; ++i) {  // nothing waits here: all loads go out together
            if (kFtThreads * i >= used) break;
            const int q = tid + kFtThreads * i;
            const uint32_t o = place(q, odd_base), at = o & ~3u;  // the two aligned words that hold the pixel
            half |= (o >> 1 & 1u) << i;
            px[i] = __builtin_amdgcn_raw_buffer_load_b64(rs, q < used ? at : 0x80000000u, 0, 0);
            last |= q < used && at + 8u > left;
        }
        if (last) {  // the tensor's last pixels, by element
#pragma unroll
            for (int i = 0; i < kFtPixels; ++i) {
                const int q = tid + kFtThreads * i;
                const uint32_t o = place(q, odd_base);
                if (q < used && (o & ~3u) + 8u > left) {
                    const uint16_t* e = reinterpret_cast<const uint16_t*>(Ib + o);
                    px[i] = u32x2{e[0] | (p.i_c > 1 ? (uint32_t)e[1] << 16 : 0u),
                                  p.i_c > 2 ? e[2] | (p.i_c > 3 ? (uint32_t)e[3] << 16 : 0u) : 0u};
                    half &= ~(1u << i);
                }
            }
        }
    };
    const uint32_t mask0 = p.i_c == 1 ? 0xffffu : ~0u, mask1 = p.i_c <= 2 ? 0u : p.i_c == 3 ? 0xffffu : ~0u;
    auto write_patch = [&]() {
#pragma unroll
        for (int i = 0; i < kFtPixels; ++i) {
            if (kFtThreads * i >= used) break;
            const int q = tid + kFtThreads * i;
            const u32x2 v = px[i];
            const bool up = half >> i & 1u;
            const u32x2 w = {(up ? (v[0] >> 16) | (v[1] << 16) : v[0]) & mask0, (up ? v[1] >> 16 : v[1]) & mask1};
            if (q < used) *reinterpret_cast<u32x2*>(ldsA + q * 8) = w;
        }
    };

    const int first_tile = (int)(blockIdx.x / (uint32_t)p.n_tiles), stride = (int)(gridDim.x / (uint32_t)p.n_tiles);
    if (first_tile < p.tiles) {
        open(first_tile, 0);
        __syncthreads();
        load_patch();
    }
    const uint32_t odd = (p.k_w & 1) ? 0u : ~0u;  // keeps the second tap of a row's last pair
    for (int tile = first_tile; tile < p.tiles; tile += stride) {
        write_patch();
        // this tile's place, before the tables go to the next one
        uint32_t apix[BM];
#pragma unroll
        for (int i = 0; i < BM; ++i) {
            const int m = (wave * BM + i) * 32 + (lane & 31);
            const int tt = (int)p.div_TW.div((uint32_t)m), x = m - tt * p.TW;
            apix[i] = tt < th ? (prow_s[tt] * (uint32_t)p.PW + (uint32_t)(x * p.s_w)) * 8u : 0u;
        }
        float* const O0 = p.O + (int64_t)image0 * p.o_h * p.o_w * p.N;
        __syncthreads();
        if (tile + stride < p.tiles) open(tile + stride, turn ^ 1);
        __syncthreads();
        if (tile + stride < p.tiles) load_patch();

        floatx16 acc[BM][BN] = {};
        // this half-wave's pair: taps (a, 2 pb) and (a, 2 pb + 1)
        int q = lane >> 5, pb = q % p.kw2, a = q / p.kw2;
        uint32_t off = (uint32_t)(a * p.PW + 2 * pb) * 8u;
        const char* kat = lds + ((lane >> 5) * TN + (lane & 31)) * 16;
        struct Frags {
            bf16x8 a[BM], b[BN];
        };
        auto read = [&](Frags& f) {  // the next step's fragments; past the last pair zeros
            const bool on = q < p.pairs;
            const uint32_t keep = pb + 1 == p.kw2 ? odd : ~0u;
#pragma unroll
            for (int j = 0; j < BN; ++j) f.b[j] = *reinterpret_cast<const bf16x8*>(kat + j * 512);
#pragma unroll
            for (int i = 0; i < BM; ++i) {
                const char* at = ldsA + (on ? apix[i] + off : zeros);
                const uint2 t0 = *reinterpret_cast<const uint2*>(at), t1 = *reinterpret_cast<const uint2*>(at + 8);
                f.a[i] = __builtin_bit_cast(bf16x8, u32x4{t0.x, t0.y, t1.x & keep, t1.y & keep});
            }
            kat += q + 2 < 2 * steps ? 2 * TN * 16 : 0;  // stays inside K
            q += 2;
            pb += 2;
            off += 32u;
#pragma unroll
            for (int r = 0; r < 2; ++r)  // kw2 is 1 or more
                if (pb >= p.kw2) {
                    pb -= p.kw2;
                    off += (uint32_t)(p.PW - 2 * p.kw2) * 8u;
                }
        };
        auto products = [&](const Frags& f) {
#pragma unroll
            for (int i = 0; i < BM; ++i)
#pragma unroll
                for (int j = 0; j < BN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
        };
        Frags f0, f1;
        read(f0);
        // Reads past the last step stay in LDS and are not multiplied: they are of real
        // weights, and an infinity there times a zero of A would be a NaN.
        for (int s = 0; s < steps; s += 2) {
            read(f1);
            __builtin_amdgcn_sched_barrier(0);
            products(f0);
            __builtin_amdgcn_sched_barrier(0);
            if (s + 1 == steps) break;
            read(f0);
            __builtin_amdgcn_sched_barrier(0);
            products(f1);
            __builtin_amdgcn_sched_barrier(0);
        }
        const __amdgpu_buffer_rsrc_t ors = buffer(O0, 0x40000000);
        uint32_t coff[BN];
#pragma unroll
        for (int j = 0; j < BN; ++j) {
            const int n = n0 + j * 32 + (lane & 31);
            coff[j] = n < p.N ? 4u * (uint32_t)n : 0x40000000u;
        }
#pragma unroll
        for (int i = 0; i < BM; ++i)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const u32x4 ro = *reinterpret_cast<const u32x4*>(&ooff_s[turn][(wave * BM + i) * 32 + acc_row(4 * w, lane)]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < BN; ++j) {
                        const float x = acc[i][j][4 * w + e];
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), ors, ro[e] + coff[j], 0, STREAM ? 2 : 0);
                    }
            }
        turn ^= 1;
        __syncthreads();  // every wave is done with the patch
    }
}

struct FirstTile {
    int32_t TH, TW, pixels;
    double use;
};
int64_t first_k_bytes(const Shape& s, int TN) {
    const int64_t pairs = s.k_h * ((s.k_w + 1) / 2);
    return (pairs + 1) / 2 * 2 * TN * 16;
}
FirstTile pick_first(const Shape& s, int TN) {
    FirstTile best{0, 0, 0, 0.0};
    const int64_t G = s.i_n * s.o_h, kb = first_k_bytes(s, TN);
    for (int64_t parts = 1; parts <= 16 && parts <= s.o_w; ++parts) {
        const int64_t TW = (uint32_t)(s.o_w + parts - 1) / (uint32_t)parts;
        if (TW > kFtM) continue;
        if ((double)(kFtM / (int32_t)TW * s.o_w) <= best.use * (double)(parts * kFtM)) continue;  // no better however many rows
        for (int64_t TH = kFtM / TW; TH >= 1; TH = TH > 4 ? TH - 1 : TH / 2) {
            const int64_t images = TH > 1 ? (TH - 2) / s.o_h + 2 : 1;
            const int64_t im = images < s.i_n ? images : s.i_n;
            if (TH < im) continue;
            // one pixel more per row for the tap past an odd kernel row
            const int64_t pixels = ((TH - im) * s.s_h + im * s.k_h) * ((TW - 1) * s.s_w + (s.k_w + 1) / 2 * 2);
            const int64_t rows = (TH - im) * s.s_h + im * s.k_h;
            if (rows > kMaxRows || pixels > (int64_t)kFtPixels * kFtThreads || kb + pixels * 8 + 16 + 3 * 4 * kFtM + 4 * kMaxRows > 160 * 1024) continue;
            const double use = (double)(G * s.o_w) / (double)(((G + TH - 1) / TH) * parts * kFtM);
            if (use > best.use + 1e-9) best = {(int32_t)TH, (int32_t)TW, (int32_t)pixels, use};
            break;  // the most rows that fit: a planning loop per call has to stay short
        }
    }
    return best;
}
int first_tn(const Shape& s) { return s.k_c <= 64 ? 64 : 96; }

}  // namespace

// Taken in bf16 over at most 4 channels where its offsets and LDS hold the shape;
// with a large K, whose staging every workgroup repeats (11x11: 101 KB), from a
// workgroup per compute unit on. From I, general tiles against this: 227x227x3 11x11
// stride 4 -> 96 batch 32 83 -> 37 us, batch 1 (49 tiles) 13 against 24; 7x7 stride 2 ->
// 64 batch 32 81 -> 31; 224x224x3 3x3 -> 64 batch 32 100 -> 81 (its 404 MB of output at
// 5 TB/s), batch 16 54 -> 44, batch 1 12.3 and 12.7.
static bool first_offsets_hold(const Shape& s, const void* I) {
    if (s.i_c > 4 || s.k_h * s.k_w < 2 || s.s_h > s.k_h || ((uintptr_t)I & 3u)) return false;
    if (s.i_n * s.o_h >= (int64_t(1) << 30) || s.k_h * s.R * s.k_c >= (int64_t(1) << 30)) return false;
    const int64_t images = 256 / s.o_h + 2;
    const int64_t im = images < s.i_n ? images : s.i_n;
    if (im * s.o_h * s.o_w * s.k_c >= (int64_t(1) << 28) || im * s.i_h * s.i_w * s.i_c >= (int64_t(1) << 29)) return false;
    return true;
}

bool gemm_first_holds(const Shape& s, const void* I) {
    return first_offsets_hold(s, I) && pick_first(s, first_tn(s)).TH != 0;
}

bool gemm_first_preferred(const Shape& s, const void* I) {
    if (!first_offsets_hold(s, I)) return false;
    const FirstTile t = pick_first(s, first_tn(s));
    if (!t.TH) return false;
    const int64_t tiles = ((s.i_n * s.o_h + t.TH - 1) / t.TH) * ((s.o_w + t.TW - 1) / t.TW);
    return first_k_bytes(s, first_tn(s)) <= 32 * 1024 || tiles >= 256;
}

hipError_t launch_gemm_first(const Shape& s, const void* I, const void* K, float* O, hipStream_t stream) {
    const int TN = first_tn(s);
    const FirstTile t = pick_first(s, TN);
    if (!t.TH) return hipErrorInvalidValue;
    FirstParams p{};
    p.I = static_cast<const uint16_t*>(I);
    p.K = static_cast<const uint16_t*>(K);
    p.O = O;
    p.G = (int32_t)(s.i_n * s.o_h);
    p.o_h = (int32_t)s.o_h; p.o_w = (int32_t)s.o_w; p.i_h = (int32_t)s.i_h; p.i_w = (int32_t)s.i_w;
    p.i_c = (int32_t)s.i_c; p.k_h = (int32_t)s.k_h; p.k_w = (int32_t)s.k_w; p.N = (int32_t)s.k_c;
    p.s_h = (int32_t)s.s_h; p.s_w = (int32_t)s.s_w;
    p.TH = t.TH;
    p.TW = t.TW;
    p.pixels = t.pixels;
    p.kw2 = (p.k_w + 1) / 2;
    p.pairs = p.k_h * p.kw2;
    p.PW = (t.TW - 1) * p.s_w + 2 * p.kw2;
    p.w_tiles = (p.o_w + t.TW - 1) / t.TW;
    p.n_tiles = (p.N + TN - 1) / TN;
    const int64_t tiles = ((int64_t)p.G + t.TH - 1) / t.TH * p.w_tiles;
    if (tiles * p.n_tiles > 0x7fffffff) return hipErrorInvalidValue;
    p.tiles = (int32_t)tiles;
    p.div_oh = FastDiv((uint32_t)p.o_h);
    p.div_TW = FastDiv((uint32_t)p.TW);
    p.div_PW = FastDiv((uint32_t)p.PW);
    p.div_kw2 = FastDiv((uint32_t)p.kw2);
    p.div_wt = FastDiv((uint32_t)p.w_tiles);
    p.i_bytes = s.i_n * s.i_h * s.i_w * s.i_c * 2;
    const size_t bytes = (size_t)first_k_bytes(s, TN) + (size_t)t.pixels * 8 + 16;
    // as many workgroups as stay resident on the 256 compute units: by LDS, at most two
    // each (registers); on a device of fewer the rest wait their turn
    const int64_t fit = bytes + 3 * 4 * kFtM + 4 * kMaxRows + 64 <= 80 * 1024 ? 2 : 1;
    int64_t groups = fit * 256 / p.n_tiles;  // workgroups per channel tile
    if (groups < 1) groups = 1;
    if (groups > tiles) groups = tiles;
    const bool lines = p.N % 32 == 0;
    auto kern = TN == 64 ? (lines ? first_gemm_kernel<2, true> : first_gemm_kernel<2, false>)
                         : (lines ? first_gemm_kernel<3, true> : first_gemm_kernel<3, false>);
    hipLaunchKernelGGL(kern, dim3((uint32_t)(groups * p.n_tiles)), dim3(kFtThreads), bytes, stream, p);
    return hipGetLastError();
}

}  // namespace mec
