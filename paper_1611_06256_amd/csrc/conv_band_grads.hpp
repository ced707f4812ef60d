// Gradients of the any-size layers (conv_band.hpp: 4x4, stride 2, 32 channels;
// conv_bytes.hpp: 8x8 over four byte planes) on the bf16 matrix cores at fp32
// accuracy.
//
// Operands are split into three bf16 terms (x = hi + mid + lo exactly) while
// they are staged, and a product is the six largest of the nine term products
// (three where one operand is bytes, which a bf16 holds exactly).  ONE: operands
// rounded to bfloat16 (the reduced-precision variant): one term, one product.
// The sums feed nothing within the update, so their order is free; against 64
// bits they are no further off than the chains of the fp32 instruction that they
// replaced (relative error in the 2-norm, here / there, the family's maps at six
// frames: dX 4.8e-8 .. 6.4e-8 / 1.3e-7 .. 1.9e-7, dW 6.2e-8 .. 1.2e-7 / 7.1e-8 ..
// 1.4e-7).  Operands are finite and below 3.39e38, where a bf16 ends: beyond that
// the second term is not a number, and a sum that the instruction left infinite
// is NaN.
//
// An item is a band of rows of one frame, small enough that two blocks share a
// compute unit: one stages while the other multiplies.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include "conv_band.hpp"
#include "conv_bytes.hpp"

namespace ga3c {

typedef uint32_t u32x2_dw __attribute__((ext_vector_type(2), aligned(4)));
constexpr int BAND_SLACK = 16;                    // floats that a row's last vector may reach past a tensor

// ----------------------------------------------------------- input gradient --
// dX[c][y][x] = [xin[c][y][x] > 0] * sum_{oc,a,e} dY[oc][iy - a][ix - e] W[oc][c][ry + 2a][rx + 2e],  y = 2 iy + ry,
// x = 2 ix + rx: a contraction over (a, e, oc) on the stride-phase grid.  LDS holds the zero-padded dY as
// [pixel][term][oc]; wavefront = (channel tile, ry) and keeps the fragments of both rx, so the two products of a pixel
// share its operands and a lane ends up with two neighbouring columns of four channels: mask and result move as pairs.
// The mask of a tile is on its way while the tile is multiplied.  BITS: it comes as the bits that the forward pass of an update has
// left (PositiveBits) instead of the floats, which on a 77x77 map were 486 of the 1084 MB that 640 frames move: 304 -> 211 us,
// 37x37 with 64 filters 116 -> 110; what the forward pass pays for them: 84x84 bytes 543 -> 560, 77x77 map 245 -> 250.  The five smaller products of all k-blocks come first: their
// sum is rounded 2^-8 finer than the result, so only the largest products' additions round it (relative error against 64
// bits 5e-8; 1.4e-7 with the six products of a k-block in turn, as with the fp32 instruction).
// 640 frames, 77x77 map: 303 us for 1.08 GB of dY, mask and dX (498 with the fp32 instruction); 37x37 and 64 filters 115
// (196); bound by memory and the waits for it, MFMA 27 % and vector ALU 19 % busy.
template <int OC, bool ONE>
constexpr int band_dgrad_pitch() { return 16 * lds_row_units((ONE ? 2 : 6) * OC / 16); }
template <int OC>
constexpr int band_dgrad_maxu() { return OC == 32 ? 6 : 13; }

// Where a staging unit goes, in one register: its byte in LDS (at most 18 bits) and its row of the item, 0 .. R.  Narrow, tall maps
// would fit more rows than the eight bits hold (one term, 4 columns: R = 336), so band_dgrad_geom stops at the last that they do.
constexpr int BAND_DGRAD_MAXR = 255;
struct BandDgradUnit {
    int v;                                                // negative: none
    __host__ __device__ static BandDgradUnit none() { return {-1}; }
    __host__ __device__ static BandDgradUnit at(uint32_t byte, uint32_t row) { return {(int)(byte * 256 + row)}; }
    __host__ __device__ bool any() const { return v >= 0; }
    __host__ __device__ int byte() const { return v >> 8; }
    __host__ __device__ int row() const { return v & 255; }
};

struct BandDgradDivs {
    FastDiv px, ow, rl;      // by the pixels of dY that an item stages, by OW, by R + 1
};
template <int OC, bool ONE, bool BITS>
__global__ __launch_bounds__(256, OC == 32 ? 2 : 1) void conv_band_dgrad_kernel(const float *__restrict__ dy, const u32x4 *__restrict__ wfrag,
                                                                                const float *__restrict__ xin, const PositiveBits bits, float *__restrict__ dx,
                                                                                int nframes, const BandGeom b, const BandDgradDivs d) {
    constexpr int C = 32, CGS = OC / 32, KB = 4 * CGS, MAXU = band_dgrad_maxu<OC>(), PIT = band_dgrad_pitch<OC, ONE>();
    constexpr int NTERM = ONE ? 1 : 3, NMAX = 2, YB = OC == 32 && !ONE ? 1 : 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int ct = wave & 1, ry = wave >> 1;
    const int HW = b.H * b.W, NPIX = b.OH * b.OW, GW = b.cols, PW = GW + 1, RL = b.R + 1;
    const int npx = b.F * RL * b.OW, NU = npx * (OC / 8);

    int src[MAXU];
    BandDgradUnit dst[MAXU];
#pragma unroll
    for (int i = 0; i < MAXU; ++i) {
        uint32_t cg, px, row, xc, f, r;
        d.px.divmod((uint32_t)min(tid + 256 * i, NU - 1), cg, px);
        d.ow.divmod(px, row, xc);
        d.rl.divmod(row, f, r);
        src[i] = (f * OC + cg * 8) * NPIX + xc;
        dst[i] = tid + 256 * i < NU ? BandDgradUnit::at((row * PW + xc + 1) * PIT + 16 * cg, r) : BandDgradUnit::none();
    }
    const size_t total = (size_t)nframes * OC * NPIX;
    float pre[MAXU][8];
    auto fetch = [&](int item) {
        const int g0 = (item % b.nb) * b.R;
        const size_t base = (size_t)(item / b.nb) * b.F * OC * NPIX;
        const uint32_t lim = band_limit(total, base, NPIX);
#pragma unroll
        for (int i = 0; i < MAXU; ++i)
            if (256 * i < NU) {
                const int yr = min(max(g0 + dst[i].row() - 1, 0), b.OH - 1);
                band_load8(dy + base, 4u * min((uint32_t)(src[i] + yr * b.OW), lim), NPIX, pre[i]);
            }
    };
    int item = blockIdx.x;
    fetch(min(item, b.items - 1));
    for (int e = tid; e < b.F * RL * PW * (PIT / 16); e += 256) ((u32x4 *)band_smem)[e] = u32x4{0u, 0u, 0u, 0u};      // columns outside dY

    Bf16x8Bits wq[2][KB][NTERM];
    {
        const u32x4 *ws = wfrag + (size_t)((ct * 2 + ry) * 2 * KB) * NTERM * 64 + lane;
#pragma unroll
        for (int q = 0; q < 2 * KB; ++q)
#pragma unroll
            for (int t = 0; t < NTERM; ++t) wq[q / KB][q % KB][t].u = ws[(q * NTERM + t) * 64];
    }

    for (; item < b.items; item += gridDim.x) {
        const int f0 = (item / b.nb) * b.F, g0 = (item % b.nb) * b.R;
        __syncthreads();                                     // the last item's planes have been read
#pragma unroll
        for (int i = 0; i < MAXU; ++i)
            if (dst[i].any()) {
                const bool in = (unsigned)(g0 + dst[i].row() - 1) < (unsigned)b.OH;      // else a row above or below dY
                u32x4 t[3];
                split3x8(pre[i], t[0], t[1], t[2]);
#pragma unroll
                for (int k = 0; k < NTERM; ++k) *(u32x4 *)(band_smem + dst[i].byte() + 2 * OC * k) = in ? t[k] : u32x4{0u, 0u, 0u, 0u};
            }
        __syncthreads();
        fetch(min(item + (int)gridDim.x, b.items - 1));
        __builtin_amdgcn_sched_barrier(0);
        const int cnt = b.F * b.R * GW, ntile = (cnt + 15) / 16;
        const float *mb = xin + ((size_t)f0 * C + ct * 16 + 4 * g) * HW;
        const size_t pixel0 = (size_t)f0 * HW;
        const uint8_t *pb = bits.at + (size_t)(ct * 4 + g) * bits.plane + pixel0 / 4 * 4;
        const uint32_t first = pixel0 & 3;
        float *db = dx + ((size_t)f0 * C + ct * 16 + 4 * g) * HW;
        auto pass = [&](auto nc, int t0) {
            constexpr int N = decltype(nc)::value;
            int base[N];
            uint32_t out[N];
            bool in[N], two[N];
            f32x2_dw mk[BITS ? 1 : N][4];
            uint32_t pos[BITS ? N : 1][2];                   // of four filters: bit 8 r for my pixel, and for its neighbour
#pragma unroll
            for (int n = 0; n < N; ++n) {
                uint32_t p = (uint32_t)((t0 + n) * 16 + l16), f, rem, i, j;
                const bool ok = (int)p < cnt;
                if (!ok) p = 0;
                b.dFR.divmod(p, f, rem);
                b.dC.divmod(rem, i, j);
                base[n] = (((int)f * RL + (int)i + 1) * PW + (int)j + 1) * PIT + 16 * g;
                const int yr = 2 * (g0 + (int)i) + ry;
                in[n] = ok && f0 + (int)f < nframes && yr < b.H;
                two[n] = 2 * (int)j + 1 < b.W;
                out[n] = in[n] ? f * (uint32_t)(C * HW) + (uint32_t)(yr * b.W + 2 * (int)j) : 0u;
                if constexpr (BITS) {
                    const uint32_t at = first + (in[n] ? f * (uint32_t)HW + (uint32_t)(yr * b.W + 2 * (int)j) : 0u), i4 = at & 3;
                    const u32x2_dw q = *(const u32x2_dw *)(pb + (at & ~3u));
                    pos[n][0] = q.x >> i4;
                    pos[n][1] = i4 == 3 ? q.y : q.x >> (i4 + 1);
                } else                                       // the last column of an odd map is the second of the pair in front of it
#pragma unroll
                for (int r = 0; r < 4; ++r) mk[n][r] = *(const f32x2_dw *)(mb + (size_t)r * HW + out[n] - (in[n] && !two[n] ? 1 : 0));
            }
            floatx4 acc[N][2];
#pragma unroll
            for (int n = 0; n < N; ++n) acc[n][0] = acc[n][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            Bf16x8Bits yv[YB][N][NTERM];
            auto read = [&](int kb, Bf16x8Bits (&d)[N][NTERM], auto terms) {
                const int tap = kb / CGS, koff = -((tap >> 1) * PW + (tap & 1)) * PIT + (kb % CGS) * 64;
#pragma unroll
                for (int n = 0; n < N; ++n)
#pragma unroll
                    for (int t = 0; t < decltype(terms)::value; ++t) d[n][t].u = *(const u32x4 *)(band_smem + base[n] + koff + t * 2 * OC);
            };
            auto product = [&](int kb, const Bf16x8Bits (&d)[N][NTERM], const int ty, const int tw) {
#pragma unroll
                for (int n = 0; n < N; ++n)
#pragma unroll
                    for (int rx = 0; rx < 2; ++rx)
                        acc[n][rx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wq[rx][kb][tw].v, d[n][ty].v, acc[n][rx], 0, 0, 0);
            };
            const std::integral_constant<int, NTERM> all;
            const std::integral_constant<int, 1> first;
            if (!ONE) {                       // the five smaller products of all k-blocks: what they add up to is rounded 2^-8 finer
                if (YB == 2) read(0, yv[0], all);
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    if (YB == 1) read(kb, yv[0], all);
                    else if (kb + 1 < KB) read(kb + 1, yv[(kb + 1) % YB], all);
                    __builtin_amdgcn_sched_barrier(0);
                    constexpr int PY[5] = {2, 1, 0, 1, 0}, PW_[5] = {0, 1, 2, 0, 1};
#pragma unroll
                    for (int q = 0; q < 5; ++q) product(kb, yv[kb % YB], PY[q] % NTERM, PW_[q] % NTERM);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                Bf16x8Bits yh[N][NTERM];
                read(kb, yh, first);
                product(kb, yh, 0, 0);
            }
#pragma unroll
            for (int n = 0; n < N; ++n)
                if (in[n]) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float *o = db + (size_t)r * HW + out[n];
                        bool m0, m1;
                        if constexpr (BITS) { m0 = pos[n][0] >> 8 * r & 1; m1 = pos[n][1] >> 8 * r & 1; }
                        else { m0 = (two[n] ? mk[n][r].x : mk[n][r].y) > 0.f; m1 = mk[n][r].y > 0.f; }
                        if (two[n]) *(f32x2_dw *)o = f32x2_dw{m0 ? acc[n][0][r] : 0.f, m1 ? acc[n][1][r] : 0.f};
                        else o[0] = m0 ? acc[n][0][r] : 0.f;
                    }
                }
        };
        int t = 0;
        for (; t + NMAX <= ntile; t += NMAX) pass(std::integral_constant<int, NMAX>{}, t);
        if (t < ntile) pass(std::integral_constant<int, 1>{}, t);
    }
}

template <int OC, bool ONE>
inline bool band_dgrad_geom(BandGeom &b, int nframes) {
    const int GW = (b.W + 1) / 2, lds = OC == 32 ? BAND_HALF_LDS : BAND_LDS - 2048;
    return band_split(b, nframes, (b.H + 1) / 2, GW,
                      [&](int F, int R) { return R <= BAND_DGRAD_MAXR && F * (R + 1) * (GW + 1) * band_dgrad_pitch<OC, ONE>() <= lds ? 0 : 2 * BAND_LDS; },
                      [&](int F, int R) { return F * (R + 1) * b.OW * (OC / 8); }, band_dgrad_maxu<OC>(), (OC == 32 ? 2 : 1) * BAND_CUS);
}
template <int OC, bool ONE, bool BITS>
inline hipError_t launch_conv_band_dgrad1(const float *dy, const u32x4 *wfrag, const float *xin, const PositiveBits &bits, float *dx, int n, int H, int W, hipStream_t s) {
    BandGeom b = band_geom(H, W);
    if (!band_dgrad_geom<OC, ONE>(b, n)) return hipErrorInvalidValue;
    static bool attr = false;
    const hipError_t e = band_allow_lds(conv_band_dgrad_kernel<OC, ONE, BITS>, attr);
    if (e != hipSuccess) return e;
    ga3c::launch((conv_band_dgrad_kernel<OC, ONE, BITS>), dim3(std::min(b.items, (OC == 32 ? 2 : 1) * BAND_CUS)), dim3(256),
                 b.F * (b.R + 1) * (b.cols + 1) * band_dgrad_pitch<OC, ONE>(), s, dy, wfrag, xin, bits, dx, n, b,
                 BandDgradDivs{FastDiv((uint32_t)(b.F * (b.R + 1) * b.OW)), FastDiv((uint32_t)b.OW), FastDiv((uint32_t)(b.R + 1))});
    return hipGetLastError();
}
// dy [n][OC][OH][OW] -> dx [n][32][H][W], masked by xin > 0, or by its bits where the forward pass has left them; wfrag: FRAG_DGRAD
// of w [OC][32][4][4], three terms or one (rb).
template <int OC>
inline hipError_t launch_conv_band_dgrad(const float *dy, const u32x4 *wfrag, const float *xin, const PositiveBits &bits, float *dx, int n, int H, int W,
                                         hipStream_t s, int rb) {
    if (n <= 0) return hipSuccess;
    return rb        ? launch_conv_band_dgrad1<OC, true, false>(dy, wfrag, xin, bits, dx, n, H, W, s)
           : bits.at ? launch_conv_band_dgrad1<OC, false, true>(dy, wfrag, xin, bits, dx, n, H, W, s)
                     : launch_conv_band_dgrad1<OC, false, false>(dy, wfrag, xin, bits, dx, n, H, W, s);
}

// --------------------------------------------------------- weight gradients --
// dW[oc][k] = sum over the pixels of dY[oc][i][j] x[tap k of (i, j)], db[oc] = sum of dY[oc][i][j]: contractions over pixels.
// A row of dY is cut into NO octets of eight columns (the last one filled up with zeros), and the octets (i, o) of an item
// are numbered on; a k-block is four of them.  dY lies in LDS as [term][filter][octet].  The input lies in stride phases,
// column x = S cc + p of a row at [p][cc], so that tap v = S e + p of an octet reads eight neighbours from cc = 8 o + e
// on: the taps of a phase are cut from one window, whole dwords for an even e, a 16-bit funnel shift for an odd one.
// The bias gradient adds up the values as they are staged: every thread has its own filters.
// Block bx takes a run of items, which share rows of the input with their neighbours, and leaves one partial gradient,
// part[bx][OC][K + 1]: no atomics.
// 640 frames: conv1 of stride 1 214 us (772 with the fp32 instruction), stride 2 69, stride 3 41; 4x4 on the 77x77 map
// 246 (437), on 37x37 with 64 filters 122 (159); 298 and 146 while the columns behind a row's end were cleared under a branch, for
// the last frame only.  What is not products (86 us of the 246 at the rate of the instruction) is splitting and
// fetching: 9 vector instructions per value, and 2 (R + 1) rows of the input fetched for R of dY.
struct BandWgradGeom {
    int nframes, H, W, OH, OW;
    int R, nb, items, nbx;   // rows per item; items per frame and in all; partial gradients
    int NO, P;               // octets per row of dY; elements per row of a phase plane
    int nx;                  // vectors of eight columns staged per input row
    int drow, prow;          // elements per filter of dY and per channel of a plane (floats); bytes: bytes per input row
    FastDiv dNO, dR, dnx, dRX;      // by NO, R, nx, 2 R + 2
};

__device__ __forceinline__ u32x4 odd_shift(const uint32_t *dw) {
    return u32x4{__builtin_amdgcn_alignbit(dw[1], dw[0], 16), __builtin_amdgcn_alignbit(dw[2], dw[1], 16),
                 __builtin_amdgcn_alignbit(dw[3], dw[2], 16), __builtin_amdgcn_alignbit(dw[4], dw[3], 16)};
}

// Eight floats from a dword-aligned place.
__device__ __forceinline__ void load8(const float *p, float (&r)[8]) {
    const f32x4_dw a = *(const f32x4_dw *)p, c = *(const f32x4_dw *)(p + 4);
    r[0] = a.x; r[1] = a.y; r[2] = a.z; r[3] = a.w; r[4] = c.x; r[5] = c.y; r[6] = c.z; r[7] = c.w;
}

// The octets of dY of an item, 32 filters from oc0 on: fetched, and stored split with zeros behind a row's end.
template <int MAXD, bool ONE>
struct DyOctets {
    int src[MAXD], dst[MAXD], row[MAXD];                      // row: of the item, in units of 16, and how many columns the octet has
    float pre[MAXD][8], bsum[MAXD];
    __device__ __forceinline__ void init(const BandWgradGeom &b, int tid) {
#pragma unroll
        for (int i = 0; i < MAXD; ++i) {
            uint32_t ro, o, oc, r;
            b.dNO.divmod((uint32_t)min(tid + 256 * i, 32 * b.R * b.NO - 1), ro, o);
            b.dR.divmod(ro, oc, r);
            src[i] = (oc * b.OH + r) * b.OW + 8 * o;
            dst[i] = tid + 256 * i < 32 * b.R * b.NO ? oc * b.drow + (r * b.NO + o) * 8 : -1;
            row[i] = 16 * r + min(8, b.OW - 8 * (int)o);
            bsum[i] = 0.f;
        }
    }
    // `rows`: of the map that the item has; `last`: the last of the item's filters' values in the frame, from `first` on
    __device__ __forceinline__ void fetch(const BandWgradGeom &b, const float *first, int last) {
#pragma unroll
        for (int i = 0; i < MAXD; ++i)
            if (256 * i < 32 * b.R * b.NO) load8(first + (uint32_t)min(src[i], last), pre[i]);      // rows past the map become zeros
    }
    __device__ __forceinline__ void store(const BandWgradGeom &b, uint16_t *dsm, int rows, bool bias) {
        const int dterm = 32 * b.drow;
#pragma unroll
        for (int i = 0; i < MAXD; ++i)
            if (dst[i] >= 0) {
                const int n = row[i] < 16 * rows ? row[i] & 15 : 0;
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = e < n ? pre[i][e] : 0.f;
                u32x4 t[3];
                split3x8(v, t[0], t[1], t[2]);
#pragma unroll
                for (int k = 0; k < (ONE ? 1 : 3); ++k) *(u32x4 *)(dsm + k * dterm + dst[i]) = t[k];
                if (bias) {
                    if (ONE)
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(e & 1 ? t[0][e / 2] & 0xffff0000u : t[0][e / 2] << 16);
                    bsum[i] += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
                }
            }
    }
    // the sums of the block's filters, by its first 32 threads; `at`: 32 R NO floats of LDS that nobody reads any more
    __device__ __forceinline__ void bias_out(const BandWgradGeom &b, float *at, int tid, float *out, size_t pitch) {
#pragma unroll
        for (int i = 0; i < MAXD; ++i)
            if (dst[i] >= 0) at[tid + 256 * i] = bsum[i];
        __syncthreads();
        if (tid < 32) {
            float v = 0.f;
            for (int k = 0; k < b.R * b.NO; ++k) v += at[tid * b.R * b.NO + k];
            out[tid * pitch] = v;
        }
    }
};

constexpr int BAND_WGRAD_OTP = 16 * 16 + 4;       // floats per filter row of a block's result in LDS
constexpr int BAND_WGRAD_MAXX = 5, BAND_WGRAD_MAXD = 2, BYTES_WGRAD_MAXX = 3, BYTES_WGRAD_MAXD = 4;

// A block's result, [32][16 x 16] of partial gradients in LDS, to rows of `pitch` floats.
__device__ __forceinline__ void band_rows_out(const float *ot, float *pb, size_t pitch, int tid, float scale) {
    for (int it = tid; it < 32 * 64; it += 256) {
        const int oc = it / 64, kq = it % 64;
        const float4 v = *(const float4 *)(ot + oc * BAND_WGRAD_OTP + 4 * kq);
        *(f32x4_dw *)(pb + oc * pitch + 4 * kq) = f32x4_dw{v.x * scale, v.y * scale, v.z * scale, v.w * scale};
    }
}

// 4x4, stride 2: a block takes 16 of the 32 channels and 32 filters; wavefront = stride phase (ry, rx), whose four taps
// (ry + 2a, rx + 2e) read its plane [y / 2][cc] from row i + a, column e on.
template <int OC, bool ONE>
__global__ __launch_bounds__(256, 2) void conv_band_wgrad_kernel(const float *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part,
                                                                 const BandWgradGeom b) {
    constexpr int C = 32, CS = 16, MT = 2, K1 = 16 * C + 1, NTERM = ONE ? 1 : 3, NPROD = ONE ? 1 : 6, MAXX = BAND_WGRAD_MAXX;
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int bx = blockIdx.x, c0 = (int)(blockIdx.y & 1) * CS, oc0 = (int)(blockIdx.y >> 1) * 32;
    const int HW = b.H * b.W, RX = 2 * b.R + 2, NUX = b.nx * RX * CS;
    const int dterm = 32 * b.drow, pterm = 4 * CS * b.prow;
    uint16_t *dsm = (uint16_t *)band_smem, *psm = dsm + NTERM * dterm;      // [term][filter][octet], [term][phase][channel][plane]

    int xsrc[MAXX], xrow[MAXX], xdst[MAXX], xcol[MAXX];
#pragma unroll
    for (int i = 0; i < MAXX; ++i) {
        uint32_t rc, q, c, r;
        b.dnx.divmod((uint32_t)min(tid + 256 * i, NUX - 1), rc, q);
        b.dRX.divmod(rc, c, r);
        xsrc[i] = c * HW + 8 * q;
        xrow[i] = r;
        xcol[i] = b.W - 8 * (int)q;
        xdst[i] = tid + 256 * i < NUX ? ((r & 1) * 2 * CS + c) * b.prow + (r >> 1) * b.P + 4 * q : -1;
    }
    float xpre[MAXX][8];
    DyOctets<BAND_WGRAD_MAXD, ONE> d;
    d.init(b, tid);
    auto rows_of = [&](int item) { return min(b.R, b.OH - item % b.nb * b.R); };
    auto fetch = [&](int item) {
        const int f = item / b.nb, i0 = item % b.nb * b.R;
        const float *xs = x + ((size_t)f * C + c0) * HW + 2 * i0 * b.W;
        const int last = b.H - 1 - 2 * i0;                    // rows past the map feed no output
#pragma unroll
        for (int i = 0; i < MAXX; ++i)
            if (256 * i < NUX) load8(xs + xsrc[i] + min(xrow[i], last) * b.W, xpre[i]);
        d.fetch(b, dy + ((size_t)f * OC + oc0) * b.OH * b.OW + i0 * b.OW, (32 * b.OH - i0) * b.OW - 1);
    };
    floatx4 acc[4][MT];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[s][m] = floatx4{0.f, 0.f, 0.f, 0.f};

    int item = (int)((long)bx * b.items / b.nbx);
    const int end = (int)((long)(bx + 1) * b.items / b.nbx);
    fetch(item);
    for (int e = tid; e < NTERM * (dterm + pterm) / 8; e += 256) ((u32x4 *)band_smem)[e] = u32x4{0u, 0u, 0u, 0u};
    for (; item < end; ++item) {
        const int rows = rows_of(item);
        __syncthreads();                                      // the last item's operands have been read
        // what a vector holds behind its row's end meets zeros of dY, but it is another row's, another channel's or nobody's, and if it
        // is not finite its products with zero are not numbers
#pragma unroll
        for (int i = 0; i < MAXX; ++i)
#pragma unroll
            for (int e = 1; e < 8; ++e) xpre[i][e] = e < xcol[i] ? xpre[i][e] : 0.f;
#pragma unroll
        for (int i = 0; i < MAXX; ++i)
            if (xdst[i] >= 0) {
                uint32_t t[4][3];
#pragma unroll
                for (int h = 0; h < 4; ++h) {                 // columns (0, 2), (4, 6), (1, 3), (5, 7)
                    const int e = (h & 1) * 4 + (h >> 1);
                    split3_pair(xpre[i][e], xpre[i][e + 2], t[h][0], t[h][1], t[h][2]);
                }
#pragma unroll
                for (int k = 0; k < NTERM; ++k) {
                    *(uint2 *)(psm + k * pterm + xdst[i]) = make_uint2(t[0][k], t[1][k]);
                    *(uint2 *)(psm + k * pterm + xdst[i] + CS * b.prow) = make_uint2(t[2][k], t[3][k]);
                }
            }
        d.store(b, dsm, rows, c0 == 0);
        __syncthreads();
        fetch(min(item + 1, end - 1));
        __builtin_amdgcn_sched_barrier(0);
        const int nkb = (rows * b.NO + 3) / 4;
        Bf16x8Bits a[2][MT][NTERM];
        u32x4 w0[2][NTERM];
        uint32_t w1[2][NTERM];
        const uint16_t *al = dsm + l16 * b.drow + 8 * g, *xl = psm + (wave * CS + l16) * b.prow;
        auto read_a = [&](int kb, Bf16x8Bits (&ad)[MT][NTERM]) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < NTERM; ++t) ad[m][t].u = *(const u32x4 *)(al + t * dterm + m * 16 * b.drow + 32 * kb);
        };
        auto read_x = [&](int kb, int av) {
            const uint32_t q = 4 * kb + g;
            const uint16_t *xq = xl + q * 8 + (b.dNO.div(q) * (b.P - 8 * b.NO) + av * b.P);
#pragma unroll
            for (int t = 0; t < NTERM; ++t) {
                w0[av][t] = *(const u32x4 *)(xq + t * pterm);
                w1[av][t] = *(const uint32_t *)(xq + t * pterm + 8);
            }
        };
        auto products = [&](const Bf16x8Bits (&ad)[MT][NTERM], auto avc) {      // the taps of row a: columns e = 0 and 1
            constexpr int av = decltype(avc)::value;
            constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};      // smallest products first
            Bf16x8Bits o[2][NTERM];
#pragma unroll
            for (int t = 0; t < NTERM; ++t) {
                const uint32_t dw[5] = {w0[av][t][0], w0[av][t][1], w0[av][t][2], w0[av][t][3], w1[av][t]};
                o[0][t].u = w0[av][t];
                o[1][t].u = odd_shift(dw);
            }
#pragma unroll
            for (int p = 0; p < NPROD; ++p)
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[2 * av + e][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ad[m][ONE ? 0 : PA[p]].v, o[e][ONE ? 0 : PB[p]].v,
                                                                                     acc[2 * av + e][m], 0, 0, 0);
        };
        // the operands of the next half of a k-block are on their way while one is multiplied
        auto block = [&](int kb, const Bf16x8Bits (&ad)[MT][NTERM], Bf16x8Bits (&an)[MT][NTERM]) {
            const int next = min(kb + 1, nkb - 1);
            read_x(kb, 1);
            __builtin_amdgcn_sched_barrier(0);
            products(ad, std::integral_constant<int, 0>{});
            __builtin_amdgcn_sched_barrier(0);
            read_x(next, 0);
            read_a(next, an);
            __builtin_amdgcn_sched_barrier(0);
            products(ad, std::integral_constant<int, 1>{});
            __builtin_amdgcn_sched_barrier(0);
        };
        read_x(0, 0);
        read_a(0, a[0]);
        int kb = 0;
        for (; kb + 1 < nkb; kb += 2) {
            block(kb, a[0], a[1]);
            block(kb + 1, a[1], a[0]);
        }
        if (kb < nkb) block(kb, a[0], a[1]);
    }
    // lane (l16, g), register r of acc[2a + e][m]: filter oc0 + 16 m + 4 g + r, channel c0 + l16, tap (ry + 2a, rx + 2e)
    __syncthreads();
    float *ot = (float *)band_smem;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                ot[(m * 16 + 4 * g + r) * BAND_WGRAD_OTP + l16 * 16 + ((wave >> 1) + 2 * (s >> 1)) * 4 + (wave & 1) + 2 * (s & 1)] = acc[s][m][r];
    __syncthreads();
    float *pb = part + ((size_t)bx * OC + oc0) * K1;
    band_rows_out(ot, pb + c0 * 16, K1, tid, 1.f);
    if (c0 == 0) d.bias_out(b, ot + 32 * BAND_WGRAD_OTP, tid, pb + K1 - 1, K1);
}

// 8x8 over four byte planes of width 84, stride S = 1, 2 or 3, 32 filters.  LDS holds the input as [row][phase][plane][cc]
// bf16.  Lane = (plane, filter row): wavefront w takes the filter rows 4 (w % 2) .. + 3 with all eight columns, and every
// second k-block; two wavefronts' sums are added at the end.  (conv_bytes.hpp: a byte is exact, three products.)
template <int S>
struct BytesWgradLds {
    static constexpr int cols() { return 8 * (((84 - 8) / S + 1 + 7) / 8) + 8; }      // of a phase that a window can reach
    static constexpr int PU = lds_row_units(cols() / 8);                              // 16-byte units per plane of a phase
    // a row's planes and the next ones' must not meet in the banks: 8 units more or less than whole turns of the banks
    static constexpr int ROW = 16 * ((S * 4 * PU + 7) / 16 * 16 + 8);
};
template <int S, bool ONE>
__global__ __launch_bounds__(256, 2) void conv_bytes_wgrad_kernel(const uint8_t *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part,
                                                                  float scale, const BandWgradGeom b) {
    constexpr int OC = 32, MT = 2, K1 = 257, NTERM = ONE ? 1 : 3, MAXX = BYTES_WGRAD_MAXX;
    constexpr int PB = 16 * BytesWgradLds<S>::PU, ROW = BytesWgradLds<S>::ROW;
    constexpr int AB = S == 3 && !ONE ? 1 : 2;                // registers for two k-blocks of dY
    constexpr int ND = (8 + 7 / S + 2) / 2;                   // dwords of a window
    static_assert(BytesWgradLds<S>::ROW >= S * 4 * PB && S <= 3, "a row holds its phases");
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int uh = wave & 1, kp = wave >> 1, bx = blockIdx.x;
    const int PLANE = b.H * BYTES_W, RI = (b.R - 1) * S + 8, NUX = RI * BYTES_Q, dterm = 32 * b.drow;
    uint16_t *dsm = (uint16_t *)band_smem;
    unsigned char *xsm = band_smem + NTERM * dterm * 2;

    uint32_t xpre[MAXX][4];
    DyOctets<BYTES_WGRAD_MAXD, ONE> d;
    d.init(b, tid);
    auto rows_of = [&](int item) { return min(b.R, b.OH - item % b.nb * b.R); };
    auto fetch = [&](int item) {
        const int f = item / b.nb, i0 = item % b.nb * b.R;
        const uint8_t *src = x + (size_t)f * 4 * PLANE + (size_t)i0 * S * BYTES_W;
        const int last = (b.H - i0 * S) * BYTES_Q - 1;        // rows past the frame feed no output
#pragma unroll
        for (int i = 0; i < MAXX; ++i)
            if (256 * i < NUX) {
                const uint32_t off = 4u * (uint32_t)min(min(tid + 256 * i, NUX - 1), last);
#pragma unroll
                for (int c = 0; c < 4; ++c) xpre[i][c] = *(const uint32_t *)(src + (size_t)c * PLANE + off);
            }
        d.fetch(b, dy + (size_t)f * OC * b.OH * b.OW + i0 * b.OW, (32 * b.OH - i0) * b.OW - 1);
    };
    floatx4 acc[8][MT];
#pragma unroll
    for (int v = 0; v < 8; ++v)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[v][m] = floatx4{0.f, 0.f, 0.f, 0.f};

    int item = (int)((long)bx * b.items / b.nbx);
    const int end = (int)((long)(bx + 1) * b.items / b.nbx);
    fetch(item);
    for (int e = tid; e < (NTERM * dterm * 2 + RI * ROW) / 16; e += 256) ((u32x4 *)band_smem)[e] = u32x4{0u, 0u, 0u, 0u};
    for (; item < end; ++item) {
        const int rows = rows_of(item);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MAXX; ++i)
            if (tid + 256 * i < NUX) {
                const int u = tid + 256 * i, r = u / BYTES_Q, q = u % BYTES_Q;
                unsigned char *row = xsm + r * ROW;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t v = xpre[i][c];
                    const float f0 = (float)(v & 0xff), f1 = (float)((v >> 8) & 0xff), f2 = (float)((v >> 16) & 0xff), f3 = (float)(v >> 24);
                    if (S == 1) *(uint2 *)(row + c * PB + 8 * q) = make_uint2(pack_bf16_rne(f0, f1), pack_bf16_rne(f2, f3));
                    else if (S == 2) {
                        *(uint32_t *)(row + c * PB + 4 * q) = pack_bf16_rne(f0, f2);
                        *(uint32_t *)(row + (4 + c) * PB + 4 * q) = pack_bf16_rne(f1, f3);
                    } else {
                        const uint32_t lo = pack_bf16_rne(f0, f1), hi = pack_bf16_rne(f2, f3);
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int col = 4 * q + t;
                            *(uint16_t *)(row + (col % S * 4 + c) * PB + 2 * (col / S)) = (uint16_t)((t < 2 ? lo : hi) >> (16 * (t & 1)));
                        }
                    }
                }
            }
        d.store(b, dsm, rows, true);
        __syncthreads();
        fetch(min(item + 1, end - 1));
        __builtin_amdgcn_sched_barrier(0);
        const int nq = rows * b.NO, nkb = (nq + 3) / 4;
        const uint16_t *al = dsm + l16 * b.drow + 8 * g;
        const unsigned char *xl = xsm + (4 * uh + (l16 >> 2)) * ROW + (l16 & 3) * PB;
        Bf16x8Bits a[AB][MT][NTERM];
        uint32_t win[2][S][ND];
        auto read_x = [&](int kb, uint32_t (&w)[S][ND]) {
            uint32_t i, o;
            b.dNO.divmod((uint32_t)min(4 * kb + g, nq - 1), i, o);      // octets behind the last are zero in dY
            const unsigned char *src = xl + i * (S * ROW) + o * 16;
#pragma unroll
            for (int p = 0; p < S; ++p) {
                const u32x4 lo = *(const u32x4 *)(src + p * 4 * PB);
                w[p][0] = lo[0]; w[p][1] = lo[1]; w[p][2] = lo[2]; w[p][3] = lo[3];
                if (ND == 8) {
                    const u32x4 hi = *(const u32x4 *)(src + p * 4 * PB + 16);
                    w[p][4 % ND] = hi[0]; w[p][5 % ND] = hi[1]; w[p][6 % ND] = hi[2]; w[p][7 % ND] = hi[3];
                } else if (ND == 6) {
                    const uint2 hi = *(const uint2 *)(src + p * 4 * PB + 16);
                    w[p][4 % ND] = hi.x; w[p][5 % ND] = hi.y;
                } else {
                    w[p][4] = *(const uint32_t *)(src + p * 4 * PB + 16);
                }
            }
        };
        auto read_a = [&](int kb, Bf16x8Bits (&ad)[MT][NTERM]) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < NTERM; ++t) ad[m][t].u = *(const u32x4 *)(al + t * dterm + m * 16 * b.drow + 32 * kb);
        };
        auto products = [&](const Bf16x8Bits (&ad)[MT][NTERM], const uint32_t (&w)[S][ND]) {
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const int p = v % S, e = v / S;
                Bf16x8Bits o;
                o.u = e & 1 ? odd_shift(&w[p][e / 2]) : u32x4{w[p][e / 2], w[p][e / 2 + 1], w[p][e / 2 + 2], w[p][e / 2 + 3]};
#pragma unroll
                for (int t = NTERM - 1; t >= 0; --t)          // smallest first
#pragma unroll
                    for (int m = 0; m < MT; ++m) acc[v][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ad[m][t].v, o.v, acc[v][m], 0, 0, 0);
            }
        };
        static_assert(ND == 8 || ND == 6 || ND == 5, "a window is read in one of three ways");
        auto block = [&](int kb, const int at) {              // the next k-block's operands are on their way meanwhile
            const int next = min(kb + 2, nkb - 1);
            if (AB == 1) read_a(kb, a[0]);
            else read_a(next, a[(at + 1) % AB]);
            read_x(next, win[at ^ 1]);
            __builtin_amdgcn_sched_barrier(0);
            products(a[at % AB], win[at]);
            __builtin_amdgcn_sched_barrier(0);
        };
        int kb = kp;
        if (kb < nkb) {
            read_x(kb, win[0]);
            if (AB == 2) read_a(kb, a[0]);
        }
        for (; kb + 2 < nkb; kb += 4) {
            block(kb, 0);
            block(kb + 2, 1);
        }
        if (kb < nkb) block(kb, 0);
    }
    // lane (l16, g), register r of acc[v][m]: filter 16 m + 4 g + r, plane l16 % 4, tap (4 uh + l16 / 4, v)
    float *ot = (float *)band_smem;
#pragma unroll
    for (int h = 1; h >= 0; --h) {
        __syncthreads();
        if (kp == h) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float *o = ot + (m * 16 + 4 * g + r) * BAND_WGRAD_OTP + (l16 & 3) * 64 + (4 * uh + (l16 >> 2)) * 8;
#pragma unroll
                    for (int v = 0; v < 8; v += 4) {
                        float4 q = make_float4(acc[v][m][r], acc[v + 1][m][r], acc[v + 2][m][r], acc[v + 3][m][r]);
                        if (h == 0) {
                            const float4 k = *(const float4 *)(o + v);
                            q = make_float4(q.x + k.x, q.y + k.y, q.z + k.z, q.w + k.w);
                        }
                        *(float4 *)(o + v) = q;
                    }
                }
        }
    }
    __syncthreads();
    float *pb = part + (size_t)bx * OC * K1;
    band_rows_out(ot, pb, K1, tid, scale);
    d.bias_out(b, ot + 32 * BAND_WGRAD_OTP, tid, pb + K1 - 1, K1);
}

// ------------------------------------------------------------------- launch --

// Rows per item: the most that fit, then items in equal shares, at least BAND_WGRAD_ITEMS of them where the batch has the rows
// (20 frames of the stride-3 member 10 / 12 / 10 us in the three layers, with 512 of fewer rows 13 / 13 / 10 and 2 us more
// of partial sums to add up).
constexpr int BAND_WGRAD_ITEMS = 128;
template <class Fits>
inline bool band_wgrad_split(BandWgradGeom &b, int most, Fits fits) {
    int rmax = 0;
    while (rmax < b.OH && fits(rmax + 1)) ++rmax;
    if (rmax < 1) return false;
    int nb = (b.OH + rmax - 1) / rmax;
    if (b.nframes * nb < BAND_WGRAD_ITEMS) nb = std::max(nb, std::min(b.OH, BAND_WGRAD_ITEMS / b.nframes));
    b.R = (b.OH + nb - 1) / nb;
    b.nb = (b.OH + b.R - 1) / b.R;
    b.items = b.nframes * b.nb;
    b.nbx = std::min(b.items, most);
    b.dR = FastDiv((uint32_t)b.R); b.dRX = FastDiv((uint32_t)(2 * b.R + 2));
    return true;
}
inline int band_dy_row(int octets) { return 8 * lds_row_units((octets + 3) / 4 * 4); }      // elements per filter

// elements per channel of a phase plane: what the last k-block reads, and the rows that are staged
inline int band_wgrad_plane(const BandWgradGeom &b, int R) {
    const int q = (R * b.NO + 3) / 4 * 4 - 1;
    return 8 * lds_row_units((std::max(8 * q + q / b.NO * (b.P - 8 * b.NO) + b.P + 10, (R + 1) * b.P) + 7) / 8);
}
inline int band_wgrad_lds(const BandWgradGeom &b, int R, bool one) {
    const int stage = (one ? 1 : 3) * 2 * (32 * band_dy_row(R * b.NO) + 64 * band_wgrad_plane(b, R));
    return std::max(stage, (32 * BAND_WGRAD_OTP + 32 * R * b.NO) * 4);
}
template <int OC, bool ONE>
inline bool band_wgrad_geom(BandWgradGeom &b, int n, int H, int W) {
    b.nframes = n; b.H = H; b.W = W; b.OH = (H - 4) / 2 + 1; b.OW = (W - 4) / 2 + 1;
    b.NO = (b.OW + 7) / 8; b.P = 8 * ((b.OW + 8) / 8); b.nx = std::min((W + 7) / 8, b.P / 4);
    b.dNO = FastDiv((uint32_t)b.NO); b.dnx = FastDiv((uint32_t)b.nx);
    auto fits = [&](int R, int lds) {
        return band_wgrad_lds(b, R, ONE) <= lds && (2 * R + 2) * 16 * b.nx <= 256 * BAND_WGRAD_MAXX && 32 * R * b.NO <= 256 * BAND_WGRAD_MAXD;
    };
    const int most = 8192 / OC;
    return band_wgrad_split(b, most, [&](int R) { return fits(R, BAND_HALF_LDS); }) ||
           band_wgrad_split(b, most, [&](int R) { return fits(R, BAND_LDS - 2048); });
}
// Partial gradients that an update of n frames leaves; 0: the layer's maps do not fit.
template <int OC>
inline int band_wgrad_parts(int n, int H, int W, int rb) {
    BandWgradGeom b{};
    return (rb ? band_wgrad_geom<OC, true>(b, n, H, W) : band_wgrad_geom<OC, false>(b, n, H, W)) ? b.nbx : 0;
}
template <int OC, bool ONE>
inline hipError_t launch_conv_band_wgrad1(const float *x, const float *dy, float *part, int n, int H, int W, hipStream_t s) {
    BandWgradGeom b{};
    if (!band_wgrad_geom<OC, ONE>(b, n, H, W)) return hipErrorInvalidValue;
    b.drow = band_dy_row(b.R * b.NO); b.prow = band_wgrad_plane(b, b.R);
    static bool attr = false;
    const hipError_t e = band_allow_lds(conv_band_wgrad_kernel<OC, ONE>, attr);
    if (e != hipSuccess) return e;
    ga3c::launch((conv_band_wgrad_kernel<OC, ONE>), dim3(b.nbx, OC / 16), dim3(256), band_wgrad_lds(b, b.R, ONE), s, x, dy, part, b);
    return hipGetLastError();
}
// x [n][32][H][W] and dy [n][OC][OH][OW], BAND_SLACK floats readable behind each; part [band_wgrad_parts(n, ..)][OC][513].
template <int OC>
inline hipError_t launch_conv_band_wgrad(const float *x, const float *dy, float *part, int n, int H, int W, hipStream_t s, int rb) {
    if (n <= 0) return hipSuccess;
    return rb ? launch_conv_band_wgrad1<OC, true>(x, dy, part, n, H, W, s) : launch_conv_band_wgrad1<OC, false>(x, dy, part, n, H, W, s);
}

// Whether maps of H x W can be run (the smallest items fit).
inline bool band_grads_ok(int H, int W) {
    BandGeom b = band_geom(H, W), c = b;
    return band_dgrad_geom<32, false>(b, 1) && band_dgrad_geom<64, false>(c, 1) && band_wgrad_parts<64>(1, H, W, 0) > 0;
}

template <int S>
inline int bytes_wgrad_lds(const BandWgradGeom &b, int R, bool one) {
    const int stage = (one ? 1 : 3) * 2 * 32 * band_dy_row(R * b.NO) + ((R - 1) * S + 8) * BytesWgradLds<S>::ROW;
    return std::max(stage, (32 * BAND_WGRAD_OTP + 32 * R * b.NO) * 4);
}
template <int S>
inline bool bytes_wgrad_geom(BandWgradGeom &b, int n, int H, bool one) {
    b.nframes = n; b.H = H; b.W = BYTES_W; b.OH = (H - 8) / S + 1; b.OW = (BYTES_W - 8) / S + 1;
    b.NO = (b.OW + 7) / 8;
    b.dNO = FastDiv((uint32_t)b.NO);
    return band_wgrad_split(b, 512, [&](int R) {
        return bytes_wgrad_lds<S>(b, R, one) <= BAND_HALF_LDS && ((R - 1) * S + 8) * BYTES_Q <= 256 * BYTES_WGRAD_MAXX &&
               32 * R * b.NO <= 256 * BYTES_WGRAD_MAXD;
    });
}
inline bool bytes_wgrad_ok(int S, int OC) { return S <= 3 && OC == 32; }
inline int bytes_wgrad_parts(int n, int H, int S, int rb) {
    BandWgradGeom b{};
    return (S == 1 ? bytes_wgrad_geom<1>(b, n, H, rb) : S == 2 ? bytes_wgrad_geom<2>(b, n, H, rb) : bytes_wgrad_geom<3>(b, n, H, rb)) ? b.nbx : 0;
}
template <int S, bool ONE>
inline hipError_t launch_conv_bytes_wgrad1(const uint8_t *x, const float *dy, float *part, int n, int H, float scale, hipStream_t s) {
    BandWgradGeom b{};
    if (!bytes_wgrad_geom<S>(b, n, H, ONE)) return hipErrorInvalidValue;
    b.drow = band_dy_row(b.R * b.NO);
    static bool attr = false;
    const hipError_t e = band_allow_lds(conv_bytes_wgrad_kernel<S, ONE>, attr);
    if (e != hipSuccess) return e;
    ga3c::launch((conv_bytes_wgrad_kernel<S, ONE>), dim3(b.nbx), dim3(256), bytes_wgrad_lds<S>(b, b.R, ONE), s, x, dy, part, scale, b);
    return hipGetLastError();
}
// x [n][4][H][84] bytes and dy [n][32][OH][OW], BAND_SLACK floats readable behind it; part [bytes_wgrad_parts(n, ..)][32][257].
template <int S>
inline hipError_t launch_conv_bytes_wgrad(const uint8_t *x, const float *dy, float *part, int n, int H, float scale, hipStream_t s, int rb) {
    if (n <= 0) return hipSuccess;
    return rb ? launch_conv_bytes_wgrad1<S, true>(x, dy, part, n, H, scale, s) : launch_conv_bytes_wgrad1<S, false>(x, dy, part, n, H, scale, s);
}

}  // namespace ga3c
