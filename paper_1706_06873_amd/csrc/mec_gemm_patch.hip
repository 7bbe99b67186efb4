// bf16 slab products with every input value staged once for all taps of the
// kernel, from I.
//
// Staging bounds tiles that load each input value again for every tap: LDS takes
// writes at only ~80 bytes a clock. Here a workgroup takes TH x TW output pixels
// (TH consecutive output rows in the order of images and rows, TW columns; at most
// 256) x 64 channels. Per chunk of 32 input channels it stages the patch of input
// pixels they read, once; tap (a, b) of output pixel (t, x) then reads patch pixel
// (row of t + a, x*s_w + b). Only K is staged per tap, in its own order by 16-byte
// loads (2-byte loads of a transposed stage took 752 instead of 282 us below), and
// turned by the transposing LDS reads; four taps between barriers, double-buffered.
// The next chunk's patch waits in registers while the taps of the current one run.
// 224x224x64 -> 64, 7x7 stride 2, batch 32: 402 us in the plain tiles, 240-258 here (590
// to 635 TFLOP/s). What is left: reads and address work between 16 products per wave
// and tap, at one wave per SIMD.
#include "mec_split.h"

namespace mec {
namespace {

struct PatchParams {
    const void* I;
    const void* K;
    float* O;
    int32_t G;        // output rows: i_n * o_h
    int32_t o_h, o_w, i_h, i_w, i_c, k_h, k_w, N, s_h, s_w;
    int32_t TH, TW, PW;
    int32_t pixels;   // patch pixels at most: rows x PW
    int32_t w_tiles, n_tiles;
    uint32_t ntiles;
    FastDiv div_oh, div_TW, div_PW;
    int64_t i_bytes;  // of I
};

// 4 waves of 64 x 64; kItems: patch granules (8 channels of a pixel) per thread at
// most.
constexpr int kThreadsP = 256, kTM = 256, kTN = 64, kBM = 2, kBN = 2, kTaps = 4, kItems = 27;
constexpr int kMaxRows = 512;                   // patch rows at most
constexpr int kTapBytes = 32 * kTN * 2;         // K of one tap and chunk
constexpr int kStageBytes = kTaps * kTapBytes;  // one stage of K

__global__ __launch_bounds__(kThreadsP, 1) void patch_gemm_kernel(PatchParams p) {
    constexpr int ES = 2;
    extern __shared__ __align__(16) char lds[];  // 2 stages of K, then the patch
    __shared__ __align__(16) uint32_t ooff_s[kTM];
    __shared__ uint32_t prow_s[kTM];   // patch row of output row t's first input row
    __shared__ uint32_t src_s[kMaxRows];  // patch row -> I offset in bytes of its first column, from the tile's first image
    char* const ldsA = lds + 2 * kStageBytes;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t t = xcd_remap(blockIdx.x, p.ntiles);
    const uint32_t rest = t / (uint32_t)p.n_tiles;
    const int n0 = (int)(t - rest * (uint32_t)p.n_tiles) * kTN;
    const uint32_t gt = rest / (uint32_t)p.w_tiles;
    const int w0 = (int)(rest - gt * (uint32_t)p.w_tiles) * p.TW;
    const int g0 = (int)gt * p.TH;
    const uint32_t image0 = p.div_oh.div((uint32_t)g0);
    const int th = p.G - g0 < p.TH ? p.G - g0 : p.TH;
    const char* const Ib = static_cast<const char*>(p.I) + (int64_t)image0 * p.i_h * p.i_w * p.i_c * ES;

    // output row t of the tile: its image, its input row, and its patch row. Rows
    // of one image share their input rows; a new image starts a fresh patch row.
    if (tid < th) {
        const uint32_t g = (uint32_t)(g0 + tid), n = p.div_oh.div(g);
        const int h = (int)(g - n * (uint32_t)p.o_h);
        // patch rows before this image: the first image's, then whole images
        const int first = (int)((image0 + 1) * (uint32_t)p.o_h) - g0;  // rows of the first image from g0 on
        const int k = (int)(n - image0);
        const int before = k == 0 ? 0 : (first - 1) * p.s_h + p.k_h + (k - 1) * ((p.o_h - 1) * p.s_h + p.k_h);
        const int h_first = k == 0 ? g0 - (int)image0 * p.o_h : 0;
        prow_s[tid] = (uint32_t)(before + (h - h_first) * p.s_h);
        // the input rows this output row is the first to bring: all k_h after a new
        // image, else the last s_h (s_h <= k_h)
        const int lo = tid == 0 || h == 0 ? 0 : p.k_h - p.s_h;
        for (int r = lo; r < p.k_h; ++r)
            src_s[prow_s[tid] + r] = (uint32_t)((k * p.i_h + h * p.s_h + r) * p.i_w) * (uint32_t)(p.i_c * ES);
    }
    __syncthreads();
    for (int m = tid; m < kTM; m += kThreadsP) {
        const int tt = (int)p.div_TW.div((uint32_t)m), x = m - tt * p.TW;
        uint32_t o = 0x80000000u;
        if (tt < th && w0 + x < p.o_w) {
            const uint32_t g = (uint32_t)(g0 + tt), n = p.div_oh.div(g), h = g - n * (uint32_t)p.o_h;
            o = 4u * (uint32_t)(((int64_t)(n - image0) * p.o_h + h) * p.o_w * p.N + (int64_t)(w0 + x) * p.N);
        }
        ooff_s[m] = o;
    }

    // this thread's patch granules: pixel tid / 4 + 64 i, granule tid % 4
    const int prows = (int)prow_s[th - 1] + p.k_h, used = prows * p.PW;
    const uint32_t ag = tid & 3u;
    uint32_t aoff[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int q = (tid >> 2) + 64 * i;
        const int pr = (int)p.div_PW.div((uint32_t)q);
        int pc = w0 * p.s_w + q - pr * p.PW;
        if (pc >= p.i_w) pc = p.i_w - 1;  // read by outputs past o_w only
        const uint32_t src = q < used ? src_s[pr] + (uint32_t)(pc * p.i_c * ES) + ag * 8u * ES : 0u;
        aoff[i] = q < used ? src : 0x80000000u;  // past the patch: not loaded
    }
    const int64_t from0 = p.i_bytes - (int64_t)image0 * p.i_h * p.i_w * p.i_c * ES;
    const int i_left = from0 > 0x7fffffff ? 0x7fffffff : (int)from0;

    u32x4 ra[kItems];
    auto load_patch = [&](int c0) {
        const __amdgpu_buffer_rsrc_t rs = buffer(Ib + c0 * ES, i_left - c0 * ES);
#pragma unroll
        for (int i = 0; i < kItems; ++i) ra[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, aoff[i], 0, 0);
    };
    // c0 is the first channel of the patch in registers: what lies past i_c there
    // belongs to the next pixel, whose infinities and NaNs zeros of K would not stop
    auto write_patch = [&](int c0) {
        const int left = p.i_c - c0 - 8 * (int)ag;  // channels of this thread's granules, an even number
        const u32x4 keep = {left > 0 ? ~0u : 0u, left > 2 ? ~0u : 0u, left > 4 ? ~0u : 0u, left > 6 ? ~0u : 0u};
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const uint32_t q = (uint32_t)(tid >> 2) + 64u * i;
            if ((int)q < used) *reinterpret_cast<u32x4*>(ldsA + swz(q, ag)) = ra[i] & keep;
        }
    };

    // K: item i is tap kTaps*step + i, row tid / 8 of the chunk, columns 8 (tid % 8)..
    // in K's own order; the transposing LDS reads below turn it
    const int taps = p.k_h * p.k_w, steps = (taps + kTaps - 1) / kTaps;
    const int chunks = (p.i_c + 31) / 32;
    const uint32_t krow = (uint32_t)tid >> 3, kg = (uint32_t)tid & 7u;
    const uint32_t koff = ES * (krow * (uint32_t)p.N + (uint32_t)n0 + kg * 8u);
    const uint32_t kat = krow * 128u + ((kg ^ (2u * (krow & 3u))) << 4);
    struct KRegs {
        u32x4 v[kTaps];
    };
    int nc = 0, ns = 0;  // the next step of K to load
    auto load_k = [&](KRegs& r) {
#pragma unroll
        for (int i = 0; i < kTaps; ++i) {
            const int tap = ns * kTaps + i;
            // rows past i_c belong to the next tap, taps past the last to nothing:
            // the resource ends before them and they read as 0
            const bool on = tap < taps && nc < chunks;
            const int64_t base = ((int64_t)(on ? tap : 0) * p.i_c + (on ? nc * 32 : 0)) * p.N * ES;
            const __amdgpu_buffer_rsrc_t rs =
                buffer(static_cast<const char*>(p.K) + base, (on ? p.i_c - nc * 32 : 0) * p.N * ES);
            r.v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, koff, 0, 0);
        }
        if (++ns == steps) ns = 0, ++nc;
    };
    auto write_k = [&](const KRegs& r, char* __restrict__ to) {
#pragma unroll
        for (int i = 0; i < kTaps; ++i) *reinterpret_cast<u32x4*>(to + i * kTapBytes + kat) = r.v[i];
    };

    // patch pixel of this lane's rows at tap (0, 0); rows past the tile's pixels
    // read pixel 0
    uint32_t arow[kBM];
#pragma unroll
    for (int i = 0; i < kBM; ++i) {
        const int m = (wave * kBM + i) * 32 + (lane & 31);
        const int tt = (int)p.div_TW.div((uint32_t)m), x = m - tt * p.TW;
        arow[i] = tt < th ? prow_s[tt] * (uint32_t)p.PW + (uint32_t)(x * p.s_w) : 0u;
    }

    // the transposing read: in each 16 lanes, lane i addresses row i / 4 at columns
    // 4 (i % 4).. and receives column i of the four rows. Two of them give a lane its
    // 8 k of a column.
    const uint32_t br = (uint32_t)((lane >> 5) * 8 + ((lane & 15) >> 2));          // row within 16
    const uint32_t bc = (uint32_t)(((lane >> 4) & 1) * 16 + (lane & 3) * 4);       // column within 32
    uint32_t boff[kBN];
#pragma unroll
    for (int j = 0; j < kBN; ++j)
        boff[j] = br * 128u + ((((bc + j * 32u) >> 3) ^ (2u * (br & 3u))) << 4) + ((bc & 7u) << 1);

    floatx16 acc[kBM][kBN] = {};
    struct Frags {
        bf16x8 a[kBM], b[kBN];
    };
    uint32_t at0[kBM];  // LDS offset of the lane's granule in its patch pixels at the current tap
    auto to_tap = [&](int a, int b) {
        // taps past the last meet zeros of K at a pixel of zeros: one of the patch
        // may hold an infinity
        const uint32_t on = (uint32_t)((a - p.k_h) >> 31), shift = (uint32_t)(a * p.PW + b);
#pragma unroll
        for (int j = 0; j < kBM; ++j)
            at0[j] = swz(((arow[j] + shift) & on) | ((uint32_t)p.pixels & ~on), (uint32_t)(lane >> 5));
    };
    auto read = [&](Frags& f, const char* __restrict__ from, int i, int kk) {
        typedef short short4v __attribute__((ext_vector_type(4)));
        typedef short short8v __attribute__((ext_vector_type(8)));
        typedef __attribute__((address_space(3))) short4v lds_short4v;
#pragma unroll
        for (int j = 0; j < kBM; ++j)  // the second 16 channels: granules 2 and 3, bit 5 of the offset
            f.a[j] = *reinterpret_cast<const bf16x8*>(ldsA + (at0[j] ^ (kk ? 32u : 0u)));
#pragma unroll
        for (int j = 0; j < kBN; ++j) {
            const char* at = from + i * kTapBytes + kk * 16 * 128 + boff[j];
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)at);
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)(at + 4 * 128));
            const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            f.b[j] = __builtin_bit_cast(bf16x8, v);
        }
    };
    auto products = [&](const Frags& f) {
#pragma unroll
        for (int u = 0; u < kBM; ++u)
#pragma unroll
            for (int v = 0; v < kBN; ++v)
                acc[u][v] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[u], f.b[v], acc[u][v], 0, 0, 0);
    };

    // Step (c, s) multiplies kTaps taps of chunk c from one stage of K, with the
    // fragments of each 16 k read under the products of the 16 before, while the
    // next step's K is written to the other stage and the one three steps on is
    // requested. The next chunk's patch waits in registers.
    if (tid < 4) *reinterpret_cast<u32x4*>(ldsA + p.pixels * 64 + tid * 16) = u32x4{0, 0, 0, 0};
    int c = 0, s = 0, ta = 0, tb = 0;
    uint32_t cur = 0;
    Frags f[2];
    auto step = [&](KRegs& k) {
        if (s == 0) {
            if (c) {  // every wave is done with the patch: its last step ended in a barrier
                write_patch(c * 32);
                __syncthreads();
            }
            if (c + 1 < chunks) load_patch((c + 1) * 32);
            ta = tb = 0;
        }
        const char* __restrict__ from = lds + cur;
        char* __restrict__ to = lds + (kStageBytes - cur);
        to_tap(ta, tb);
        read(f[0], from, 0, 0);
#pragma unroll
        for (int i = 0; i < kTaps; ++i) {
            read(f[1], from, i, 1);
            __builtin_amdgcn_sched_barrier(0);
            if (i == 0) write_k(k, to);
            products(f[0]);
            __builtin_amdgcn_sched_barrier(0);
            if (++tb == p.k_w) {
                tb = 0;
                ++ta;
            }
            if (i + 1 < kTaps) {
                to_tap(ta, tb);
                read(f[0], from, i + 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 == kTaps) load_k(k);
            products(f[1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        cur = kStageBytes - cur;
        if (++s == steps) s = 0, ++c;
    };
    KRegs k0, k1;
    load_patch(0);
    load_k(k0);
    load_k(k1);
    write_patch(0);
    write_k(k0, lds);
    load_k(k0);
    __syncthreads();
    for (int n = chunks * steps; n > 0; n -= 2) {
        step(k1);
        if (n > 1) step(k0);
    }

    float* const O0 = p.O + (int64_t)image0 * p.o_h * p.o_w * p.N;
    const __amdgpu_buffer_rsrc_t orsrc = buffer(O0, 0x40000000);
    uint32_t coff[kBN];
#pragma unroll
    for (int j = 0; j < kBN; ++j) {
        const int n = n0 + j * 32 + (lane & 31);
        coff[j] = n < p.N ? 4u * (uint32_t)n : 0x40000000u;
    }
#pragma unroll
    for (int i = 0; i < kBM; ++i)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const u32x4 ro = *reinterpret_cast<const u32x4*>(&ooff_s[(wave * kBM + i) * 32 + acc_row(4 * w, lane)]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < kBN; ++j) {
                    const float x = acc[i][j][4 * w + e];
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), orsrc, ro[e] + coff[j], 0, 2);
                }
        }
}

// Tile heights and widths: the widest of 1 .. 8 equal column ranges whose patch
// fits, by the share of the tile's slots that hold output pixels.
struct PatchTile {
    int32_t TH, TW, pixels;
    double use;
};
PatchTile pick_patch(const Shape& s) {
    PatchTile best{0, 0, 0, 0.0};
    const int64_t G = s.i_n * s.o_h;
    for (int64_t parts = 1; parts <= 16 && parts <= s.o_w; ++parts) {
        const int64_t TW = (uint32_t)(s.o_w + parts - 1) / (uint32_t)parts;
        if (TW > kTM) continue;
        if ((double)(kTM / (int32_t)TW * s.o_w) <= best.use * (double)(parts * kTM)) continue;  // no better however many rows
        for (int64_t TH = kTM / TW; TH >= 1; TH = TH > 4 ? TH - 1 : TH / 2) {
            const int64_t images = TH > 1 ? (TH - 2) / s.o_h + 2 : 1;  // that TH rows can touch
            const int64_t im = images < s.i_n ? images : s.i_n;
            const int64_t rows = (TH - im) * s.s_h + im * s.k_h;
            const int64_t pixels = rows * ((TW - 1) * s.s_w + s.k_w);
            if (TH < im || rows > kMaxRows || pixels * 4 > (int64_t)kItems * kThreadsP) continue;
            if (2 * kStageBytes + (pixels + 1) * 64 + 2 * 4 * kTM + 4 * kMaxRows + 64 > 160 * 1024) continue;
            const double use = (double)(G * s.o_w) / (double)(((G + TH - 1) / TH) * parts * kTM);
            if (use > best.use + 1e-9) best = {(int32_t)TH, (int32_t)TW, (int32_t)pixels, use};
            break;  // the most rows that fit: a planning loop per call has to stay short
        }
    }
    return best;
}

hipError_t run_patch(const Shape& s, const void* I, const void* K, float* O, hipStream_t stream) {
    const PatchTile t = pick_patch(s);
    if (!t.TH) return hipErrorNotSupported;
    PatchParams p{};
    p.I = I;
    p.K = K;
    p.O = O;
    p.G = (int32_t)(s.i_n * s.o_h);
    p.o_h = (int32_t)s.o_h; p.o_w = (int32_t)s.o_w; p.i_h = (int32_t)s.i_h; p.i_w = (int32_t)s.i_w;
    p.i_c = (int32_t)s.i_c; p.k_h = (int32_t)s.k_h; p.k_w = (int32_t)s.k_w; p.N = (int32_t)s.k_c;
    p.s_h = (int32_t)s.s_h; p.s_w = (int32_t)s.s_w;
    p.TH = t.TH;
    p.TW = t.TW;
    p.PW = (t.TW - 1) * p.s_w + p.k_w;
    p.pixels = t.pixels;
    p.w_tiles = (p.o_w + t.TW - 1) / t.TW;
    p.n_tiles = (p.N + kTN - 1) / kTN;
    const int64_t ntiles = ((int64_t)p.G + t.TH - 1) / t.TH * p.w_tiles * p.n_tiles;
    if (ntiles > 0x7fffffff) return hipErrorInvalidValue;
    p.ntiles = (uint32_t)ntiles;
    p.div_oh = FastDiv((uint32_t)p.o_h);
    p.div_TW = FastDiv((uint32_t)p.TW);
    p.div_PW = FastDiv((uint32_t)p.PW);
    p.i_bytes = s.i_n * s.i_h * s.i_w * s.i_c * 2;
    const size_t bytes = 2 * (size_t)kStageBytes + (size_t)(t.pixels + 1) * 64;
    hipLaunchKernelGGL(patch_gemm_kernel, dim3(p.ntiles), dim3(kThreadsP), bytes, stream, p);
    return hipGetLastError();
}

}  // namespace

// Taken in bf16 where the kernel has several taps and
// * its offsets hold the shape (and rows of I and K start on 4-byte boundaries),
// * no tile of its own exists for the kernel with these channels (3x3, 5x5 and 1x1
//   at stride 1 keep theirs: 3x3 over 64 channels 19 against 46 us) and at least 0.4 of
//   the chunks' channels and the tiles' output channels exist (112x112, 3x3 over 18
//   channels to 30: 36 against 28 us for the generic tiles), or it is the 7x7 stride 2
//   one and takes longer by patch_beats_k7s2.
// Against the generic tiles, batch 8 to 64: 3x3 stride 2 over 64 channels 35 -> 26
// us, over 512 223 -> 90; 3x3 over 100, 90 and 300 channels 89 -> 24, 85 -> 22 and
// 257 -> 52; 5x5 over 90 186 -> 34; 7x7 stride 2 over 100 at batch 2 406 -> 70.
static bool patch_offsets_hold(const Shape& s, const void* I, const void* K) {
    if (s.k_h * s.k_w < 2 || s.s_h > s.k_h || s.i_n * s.o_h >= (int64_t(1) << 30)) return false;
    if (s.k_h * s.R * s.k_c >= (int64_t(1) << 30)) return false;
    const int64_t images = 256 / s.o_h + 2;
    const int64_t im = images < s.i_n ? images : s.i_n;
    if (im * s.o_h * s.o_w * s.k_c >= (int64_t(1) << 28) || im * s.i_h * s.i_w * s.i_c >= (int64_t(1) << 30)) return false;
    if (s.i_c % 2 || s.k_c % 2 || ((uintptr_t)I & 3u) || ((uintptr_t)K & 3u)) return false;
    return true;
}

bool gemm_patch_holds(const Shape& s, const void* I, const void* K) {
    return patch_offsets_hold(s, I, K) && pick_patch(s).TH != 0;
}

// Both kernels' times in us, rounds of workgroups over the compute units times what a
// round takes; measured on this GPU (they give 91 shapes of 7 to 600 us within 10%, and
// the faster kernel of each within 5%). Of the fixed tiles those over at most 64 channels
// are two to a compute unit. 224x224x64 -> 64 (patch / fixed): batch 1 38 / 31, 4 43 / 69,
// 32 252 / 402; 78x78x16 -> 112, batch 90, 88 / 55; 168x164x48 -> 72, batch 24, 195 / 159.
static bool patch_beats_k7s2(const Shape& s, const PatchTile& t) {
    auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    const int64_t tiles = up(s.i_n * s.o_h, t.TH) * up(s.o_w, t.TW) * up(s.k_c, kTN);
    const double patch = (double)up(tiles, 256) * (0.353 * (double)(s.k_h * s.k_w * up(s.i_c, 32)) + 5.0);
    const int64_t chunks = up(s.R, 16);
    if (s.k_c > 64)
        return patch < (double)up(up(s.pairs, 32) * up(s.o_h, 4) * up(s.k_c, 128), 256) * (1.34 * (double)chunks + 4.2);
    const int64_t each = up(up(s.pairs, 32) * up(s.o_h, 2), 256);
    return patch < (double)(each / 2) * (1.25 * (double)chunks + 3.0) + (double)(each % 2) * (1.03 * (double)chunks + 3.0);
}

bool gemm_patch_preferred(const Shape& s, const void* I, const void* K) {
    if (!patch_offsets_hold(s, I, K)) return false;
    const bool fixed = launch_gemm_fixed(s, I, K, nullptr, 1, true, nullptr, true) == hipSuccess;
    if (fixed && (s.k_h != 7 || s.s_h != 2)) return false;
    const PatchTile t = pick_patch(s);
    if (!t.TH) return false;
    if (fixed) return patch_beats_k7s2(s, t);
    return 5 * s.i_c * s.k_c >= 2 * ((s.i_c + 31) / 32 * 32) * ((s.k_c + 63) / 64 * 64);
}

hipError_t launch_gemm_patch(const Shape& s, const void* I, const void* K, float* O, hipStream_t stream) {
    return run_patch(s, I, K, O, stream);
}

}  // namespace mec
