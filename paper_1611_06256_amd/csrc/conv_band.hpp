// The 4x4, stride-2 convolution layer with 32 input channels and 32 or 64
// filters on maps of any size (the paper's larger-network family, Sec. 5, whose
// maps are 9 to 77 pixels wide): what its kernels share, and the forward pass
// with operands rounded to bfloat16 (at fp32 accuracy: conv_band_f32.hpp).
//
// A work item is a band of output rows of one frame, or several whole small frames
// (BandGeom, chosen on the host); a block walks over items and the next item
// travels from memory while the current one is multiplied.  Operands are rounded
// while they are staged.  LDS holds [pixel][channel], so one staging unit (8
// channels of a pixel: eight loads along planes, coalesced over pixels) leaves as
// one 16-byte store, and the 8 consecutive channels a lane feeds to an MFMA are
// one 16-byte read; with stride 2 the even and the odd columns of an input row
// are stored apart, so that consecutive output pixels read consecutive LDS
// pixels.  Filters come as ready-made fragments (band_filter_fragments_kernel,
// once per parameter copy).
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "conv1_bf16x3.hpp"
#include "dense_gemm_bf16x6.hpp"

namespace ga3c {

constexpr int BAND_LDS = 160 * 1024;          // of a compute unit
constexpr int BAND_HALF_LDS = BAND_LDS / 2;   // two blocks per compute unit: one stages while the other multiplies
constexpr int BAND_CUS = 256;
// staging units (8 channels of a pixel) per thread: bounds the registers of a band in flight
constexpr int BAND_MAXU = 10;

// Which outputs of a layer of 32 filters are positive: a byte for four pixels of a filter, four filters to a plane: the byte of
// pixels 4 q .. 4 q + 3, counted through all frames, and filter o lies at `at` + o / 4 * `plane` + 4 q + o % 4, bit i for pixel
// 4 q + i.  That is how a lane of the forward pass has them, and what a lane of the input gradient wants, a pixel and its right
// neighbour of four filters, are eight bytes in one place.  at == nullptr: none.
struct PositiveBits {
    uint8_t *at = nullptr;
    size_t plane = 0;
    static size_t plane_of(size_t pixels) { return (pixels + 15) / 16 * 16 + 16; }      // whole tiles, and the last pixels' neighbours
    static constexpr int PLANES = 8;
};

typedef float f32x4_dw __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2_dw __attribute__((ext_vector_type(2), aligned(4)));

// Where the items of a launch lie.  "Rows" are output rows for the forward pass, rows of the stride-phase grid
// (ceil(H / 2)) for the input gradient (conv_band_grads.hpp).
struct BandGeom {
    int H, W, OH, OW;
    int F, R;                // an item: R rows of each of F consecutive frames (F > 1 only with all rows)
    int nb, items;           // bands per frame; items in all
    int rows, cols;          // rows and columns of an item as the kernel counts pixels: R x cols per frame
    FastDiv dFR, dC;         // by R * cols and by cols
};

// LDS pixel pitch in bytes for C channels.
template <int C>
constexpr int band_pitch() { return 16 * lds_row_units(C / 8); }

// ---------------------------------------------------------------- fragments --

__device__ __forceinline__ u32x4 band_round8(const float (&r)[8]) {
    return u32x4{pack_bf16_rne(r[0], r[1]), pack_bf16_rne(r[2], r[3]), pack_bf16_rne(r[4], r[5]), pack_bf16_rne(r[6], r[7])};
}
// The largest bfloat16 for what would round to infinity and is none (the last 0.4 % of what an fp32 holds): the first term of such a
// weight.  Infinity would leave minus infinity for the second, and every product of the filter would be no number.
__device__ __forceinline__ float within_bf16(float x) {
    const float most = __uint_as_float(0x7f7f0000u);
    return fabsf(x) > most && fabsf(x) < __uint_as_float(0x7f800000u) ? copysignf(most, x) : x;
}

// One tensor's fragments: n threads write a vector for each term (three, or one where operands are rounded to bfloat16), at
// dst[(i / 64 * TERMS + term) * 64 + i % 64]; FRAG_F32: one vector of four weights each, at dst[i].
enum { FRAG_CONV = 0, FRAG_BYTES8 = 1, FRAG_DGRAD = 2, FRAG_F32 = 3 };
struct FragJob {
    const float *w;          // [OC][C][KS][KS]
    u32x4 *dst;
    int kind, C, OC, KS, n, first_block;
};
constexpr int MAX_FRAG_JOBS = 12;
struct FragJobs {
    FragJob job[MAX_FRAG_JOBS];
    int n;
};
template <int TERMS>
__device__ __forceinline__ void band_filter_fragments_block(const FragJobs &jobs, const int block) {
    int q = 0;
    while (q + 1 < jobs.n && block >= jobs.job[q + 1].first_block) ++q;
    const FragJob &j = jobs.job[q];
    const int i = (block - j.first_block) * 256 + threadIdx.x;
    if (i >= j.n) return;
    const int lane = i % 64, l16 = lane & 15, g = lane >> 4;
    int blk = i / 64;
    if (j.kind == FRAG_F32) {                // [filter tile][group of 16 taps]: row = filter, a lane's k = four taps of the group
        const int groups = j.C * j.KS * j.KS / 16;
        const f32x4_dw v = *(const f32x4_dw *)(j.w + ((size_t)(blk / groups * 16 + l16) * groups + blk % groups) * 16 + 4 * g);
        ((float4 *)j.dst)[i] = make_float4(v.x, v.y, v.z, v.w);
        return;
    }
    float f[8];
    if (j.kind == FRAG_CONV) {               // [filter tile][(u, v, 32 channels)]: row = filter, k = channel
        const int cgs = j.C / 32, kbs = j.KS * j.KS * cgs;
        const int kb = blk % kbs, ot = blk / kbs, tap = kb / cgs, c0 = (kb % cgs) * 32 + 8 * g;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = j.w[((size_t)(ot * 16 + l16) * j.C + c0 + e) * j.KS * j.KS + tap];
    } else if (j.kind == FRAG_DGRAD) {       // 4x4, stride 2: [channel tile][ry][rx][(a, e, 32 filters)]: row = channel, k = filter
        const int ogs = j.OC / 32, kb = blk % (4 * ogs), ph = blk / (4 * ogs), tap = kb / ogs, o0 = (kb % ogs) * 32 + 8 * g;
        const int u = (ph >> 1 & 1) + 2 * (tap >> 1), v = (ph & 1) + 2 * (tap & 1), c = (ph >> 2) * 16 + l16;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = j.w[((size_t)(o0 + e) * j.C + c) * 16 + u * 4 + v];
    } else {                                 // byte layer, 4 planes, 8x8: [filter tile][u]: row = filter, k = (v, plane)
        const int u = blk % 8, ot = blk / 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = j.w[((size_t)(ot * 16 + l16) * 4 + e % 4) * 64 + u * 8 + 2 * g + e / 4];
    }
    u32x4 *dst = j.dst + (size_t)(i / 64) * TERMS * 64 + lane;
    if constexpr (TERMS == 1) dst[0] = band_round8(f);
    else {
        float near[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) near[e] = within_bf16(f[e]);
        dst[0] = band_round8(near);
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] -= bf16_rne(near[e]);
        dst[64] = band_round8(f);
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] -= bf16_rne(f[e]);
        dst[128] = band_round8(f);
    }
}

template <int TERMS>
__global__ __launch_bounds__(256) void band_filter_fragments_kernel(const FragJobs jobs) {
    band_filter_fragments_block<TERMS>(jobs, blockIdx.x);
}

// ------------------------------------------------------------------ staging --

// Eight channels, `plane` floats apart, of one pixel; `off` counts bytes from the (uniform) base.
__device__ __forceinline__ void band_load8(const float *base, uint32_t off, int plane, float (&r)[8]) {
#pragma unroll
    for (int c = 0; c < 8; ++c) r[c] = *(const float *)((const char *)(base + (size_t)c * plane) + off);
}
// Floats left in a tensor of `total` behind `base`, less the eight planes a unit reads: the largest offset a unit may use.
__device__ __forceinline__ uint32_t band_limit(size_t total, size_t base, int plane) {
    const size_t left = total - base - (size_t)7 * plane - 1;
    return left > 0x3fffffff ? 0x3fffffffu : (uint32_t)left;
}

// ------------------------------------------------------------------ forward --
// y[oc][oy][ox] = max(0, b[oc] + sum W[oc][c][u][v] x[c][2 oy + u][2 ox + v]).
// Pixels are the rows of the products and filters the columns, so a lane ends up with four consecutive pixels of one
// filter.  Wavefront w keeps the fragments of filter tile w % (OC / 16) in registers (64 of them) and takes every
// (64 / OC)-th pixel tile, up to four at a time; the operands of the next k-block are read while the current one is
// multiplied.  640 frames of 26x26 19 us, of 77x77 181 (for 600 MB).
template <int C, int OC>
__global__ __launch_bounds__(256, 2) void conv_band_fwd_kernel(const float *__restrict__ x, const u32x4 *__restrict__ wfrag,
                                                               const float *__restrict__ bias, float *__restrict__ y,
                                                               int nframes, const BandGeom b) {
    constexpr int KS = 4, S = 2, KB = KS * KS * C / 32, OT = OC / 16, PG = 4 / OT;
    constexpr int PIT = band_pitch<C>(), MAXU = BAND_MAXU;
    static_assert(C == 32 && (OC == 32 || OC == 64), "32 channels in, 32 or 64 filters");
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int ot = wave % OT, pg = wave / OT;
    const int HW = b.H * b.W, NPIX = b.OH * b.OW;
    const int RI = (b.R - 1) * S + KS, WH = (b.W + 1) / 2, WP = 2 * WH;
    const int npx = b.F * RI * b.W, NU = npx * (C / 8);
    const size_t total = (size_t)nframes * C * HW;

    // staging units: byte offset from the item's first input row, and place in LDS
    uint32_t src[MAXU];
    int dst[MAXU];
#pragma unroll
    for (int i = 0; i < MAXU; ++i) {
        const int u = min(tid + 256 * i, NU - 1);
        const int cg = u / npx, px = u % npx, row = px / b.W, xc = px % b.W, f = row / RI, r = row % RI;
        src[i] = (uint32_t)((f * C + cg * 8) * HW + r * b.W + xc);
        dst[i] = tid + 256 * i < NU ? (row * WP + (xc & 1) * WH + (xc >> 1)) * PIT + 16 * cg : -1;
    }
    float pre[MAXU][8];
    auto fetch = [&](int item) {
        const size_t base = (size_t)(item / b.nb) * b.F * C * HW + (size_t)(item % b.nb) * b.R * S * b.W;
        const uint32_t lim = band_limit(total, base, HW);
#pragma unroll
        for (int i = 0; i < MAXU; ++i)
            if (256 * i < NU) band_load8(x + base, 4u * min(src[i], lim), HW, pre[i]);      // rows past the map feed no output
    };
    int item = blockIdx.x;
    fetch(min(item, b.items - 1));

    Bf16x8Bits wq[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) wq[kb].u = wfrag[(size_t)(ot * KB + kb) * 64 + lane];
    const float bv = bias[ot * 16 + l16];

    for (; item < b.items; item += gridDim.x) {
        __syncthreads();                                     // the last item's planes have been read
#pragma unroll
        for (int i = 0; i < MAXU; ++i)
            if (dst[i] >= 0) *(u32x4 *)(band_smem + dst[i]) = band_round8(pre[i]);
        __syncthreads();
        fetch(min(item + (int)gridDim.x, b.items - 1));
        __builtin_amdgcn_sched_barrier(0);
        const int f0 = (item / b.nb) * b.F, i0 = (item % b.nb) * b.R;
        const int fr = b.R * b.OW, cnt = b.F * fr, vpix = min(b.R, b.OH - i0) * b.OW;      // valid pixels of each frame
        const int ntile = (cnt + 15) / 16;
        auto pass = [&](auto nc, int t0) {
            constexpr int N = decltype(nc)::value;
            int base[N];
#pragma unroll
            for (int n = 0; n < N; ++n) {
                uint32_t p = (uint32_t)((t0 + n * PG) * 16 + l16), f, rem, i, j;
                if ((int)p >= cnt) p = 0;
                b.dFR.divmod(p, f, rem);
                b.dC.divmod(rem, i, j);
                base[n] = (((int)f * RI + (int)i * S) * WP + (int)j) * PIT + 16 * g;
            }
            floatx4 acc[N];
#pragma unroll
            for (int n = 0; n < N; ++n) acc[n] = floatx4{0.f, 0.f, 0.f, 0.f};
            Bf16x8Bits xv[2][N];
            auto read = [&](int kb, Bf16x8Bits (&d)[N]) {
                const int tap = kb / (C / 32), cg = kb % (C / 32), u = tap / KS, v = tap % KS;
                const int koff = (u * WP + (v & 1) * WH + (v >> 1)) * PIT + cg * 64;
#pragma unroll
                for (int n = 0; n < N; ++n) d[n].u = *(const u32x4 *)(band_smem + base[n] + koff);
            };
            read(0, xv[0]);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                if (kb + 1 < KB) read(kb + 1, xv[(kb + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int n = 0; n < N; ++n) acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[kb & 1][n].v, wq[kb].v, acc[n], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const uint32_t p0 = (uint32_t)((t0 + n * PG) * 16 + 4 * g);
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = acc[n][r] + bv;
                    v[r] = v[r] > 0.f ? v[r] : 0.f;
                }
                uint32_t f, rem;
                b.dFR.divmod(p0, f, rem);
                float *out = y + ((size_t)(f0 + (int)f) * OC + ot * 16 + l16) * NPIX + i0 * b.OW;
                if ((int)p0 < cnt && f0 + (int)f < nframes && (int)rem + 3 < vpix) {
                    *(f32x4_dw *)(out + rem) = f32x4_dw{v[0], v[1], v[2], v[3]};
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        b.dFR.divmod(p0 + r, f, rem);
                        if ((int)p0 + r < cnt && f0 + (int)f < nframes && (int)rem < vpix)
                            y[((size_t)(f0 + (int)f) * OC + ot * 16 + l16) * NPIX + i0 * b.OW + rem] = v[r];
                    }
                }
            }
        };
        int t = pg, left = (ntile - pg + PG - 1) / PG;
        for (; left >= 4; left -= 4, t += 4 * PG) pass(std::integral_constant<int, 4>{}, t);
        if (left == 3) pass(std::integral_constant<int, 3>{}, t);
        else if (left == 2) pass(std::integral_constant<int, 2>{}, t);
        else if (left == 1) pass(std::integral_constant<int, 1>{}, t);
    }
}

// ------------------------------------------------------------------- launch --

// The most rows per item for which `bytes(F, R)` fits a compute unit's LDS and `units(F, R)` the staging registers,
// then as many bands as give every compute unit an item, in equal shares; small maps go several frames to an item
// while there are items enough.  Returns false if not even one row fits.
template <class Bytes, class Units>
inline bool band_split(BandGeom &b, int nframes, int rows, int cols, Bytes bytes, Units units, int maxu, int want) {
    auto fits = [&](int F, int R) { return bytes(F, R) <= BAND_LDS - 2048 && units(F, R) <= 256 * maxu; };
    int rmax = 0;
    while (rmax < rows && fits(1, rmax + 1)) ++rmax;
    if (rmax < 1) return false;
    b.rows = rows; b.cols = cols; b.F = 1;
    int nb = (rows + rmax - 1) / rmax;
    if (nb == 1)
        while ((nframes + b.F) / (b.F + 1) >= 2 * want && fits(b.F + 1, rows)) ++b.F;
    if (nframes * nb < want)          // fewer items than blocks the chip holds: smaller ones, of at least two pixel tiles
        nb = std::max(nb, std::min(want / nframes, std::max(1, rows * cols / 32)));
    b.R = (rows + nb - 1) / nb;
    b.nb = (rows + b.R - 1) / b.R;
    b.items = (nframes + b.F - 1) / b.F * b.nb;
    b.dFR = FastDiv((uint32_t)(b.R * cols)); b.dC = FastDiv((uint32_t)cols);
    return true;
}

inline BandGeom band_geom(int H, int W) {
    BandGeom b{};
    b.H = H; b.W = W; b.OH = (H - 4) / 2 + 1; b.OW = (W - 4) / 2 + 1;
    return b;
}
inline int band_in_px(const BandGeom &b, int F, int R) { return F * ((R - 1) * 2 + 4) * 2 * ((b.W + 1) / 2); }

template <int C>
inline bool band_fwd_geom(BandGeom &b, int nframes) {
    return band_split(b, nframes, b.OH, b.OW, [&](int F, int R) { return 2 * band_in_px(b, F, R) * band_pitch<C>(); },
                      [&](int F, int R) { return F * ((R - 1) * 2 + 4) * b.W * (C / 8); }, BAND_MAXU, 2 * BAND_CUS);
}

template <class K>
inline hipError_t band_allow_lds(K kernel, bool &done) {
    if (done) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, BAND_LDS - 2048);
    done = e == hipSuccess;
    return e;
}

// Whether maps of H x W can be run at all (the smallest item fits).
template <int C>
inline bool band_ok(int H, int W) {
    BandGeom b = band_geom(H, W);
    return H >= 4 && W >= 4 && band_fwd_geom<C>(b, 1);
}

// x [n][32][H][W] -> y [n][OC][OH][OW]; wfrag: FRAG_CONV of the filters, one term.
template <int C, int OC>
inline hipError_t launch_conv_band_fwd(const float *x, const u32x4 *wfrag, const float *bias, float *y, int n, int H, int W, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    BandGeom b = band_geom(H, W);
    if (!band_fwd_geom<C>(b, n)) return hipErrorInvalidValue;
    static bool attr = false;
    const hipError_t e = band_allow_lds(conv_band_fwd_kernel<C, OC>, attr);
    if (e != hipSuccess) return e;
    ga3c::launch((conv_band_fwd_kernel<C, OC>), dim3(std::min(b.items, 2 * BAND_CUS)), dim3(256), band_in_px(b, b.F, b.R) * band_pitch<C>(), s, x, wfrag,
                 bias, y, n, b);
    return hipGetLastError();
}

}  // namespace ga3c
