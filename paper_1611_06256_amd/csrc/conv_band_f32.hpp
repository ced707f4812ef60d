// The layers of conv_band.hpp and conv_bytes.hpp on the fp32 matrix instruction,
// for maps of any size (the 4x4 stride-2 layer on 32 channels, and the 8x8 byte
// layer of any stride): forward pass, input gradient and weight gradient.
//
// Every sum is formed by the same instructions in the same order as in
// gemm_mfma.hpp (v_mfma_f32_16x16x4_f32, product t of a group of 16 k sums
// k = 16 kb + 4 g + t over g, groups and t ascending), so activations and
// gradients are the same bits as those of the any-shape kernels.  In the forward
// pass of an update that matters: where a pre-activation lies within rounding of
// zero, another order of the sum can put it on the other side of the rectifier,
// and a map of millions of pixels has enough of those to move the gradient of a
// filter by 1e-4 of itself.  The gradients decide nothing: an input gradient's
// mask is the stored activation, and a weight gradient feeds nothing within the
// update.  Keeping their order of sums too buys equal bits, not accuracy, and
// costs the rate of the bf16 instruction.
//
// What bounds them is the instruction: 146 - 150 TFLOP/s on this chip.  With k
// in the filter's own order (c, u, v), the four k of a lane are four columns of
// one filter row: a 16-byte piece of a filter, and four neighbouring values (or
// bytes) of an input row.  So the input stays in LDS as it is in memory, without
// any re-laying or conversion, and one read of 16 bytes per lane feeds four
// instructions per filter tile.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include "conv_band.hpp"
#include "conv_bytes.hpp"

namespace ga3c {

constexpr int BAND_F32_LDS = 80 * 1024;           // two blocks per compute unit: one stages while the other multiplies
constexpr int BAND_F32_MAXK = 3;                  // values of a channel in flight per thread

// 4x4, stride 2, 32 channels; a block takes the pixel tiles of its item four wavefronts apart, all filters.
// RB: both operands rounded to bfloat16.
template <int C, int OC, bool RB>
__global__ __launch_bounds__(256, 2) void conv_band_f32_fwd_kernel(const float *__restrict__ x, const float *__restrict__ w,
                                                                   const float *__restrict__ bias, float *__restrict__ y, int nframes,
                                                                   const BandGeom b) {
    constexpr int OT = OC / 16, K = 16 * C, MAXK = BAND_F32_MAXK;
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    float *xs = (float *)band_smem;                   // [c][frame][row][W]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int HW = b.H * b.W, NPIX = b.OH * b.OW, RI = (b.R - 1) * 2 + 4;
    const int chunk = RI * b.W, plane = b.F * chunk;      // a frame's band of a channel is contiguous in memory
    const size_t total = (size_t)nframes * C * HW;

    // value k of a thread and channel: number tid + 256 k of the channel's part of the item
    uint32_t src[MAXK];
#pragma unroll
    for (int k = 0; k < MAXK; ++k) {
        const int e = min(tid + 256 * k, plane - 1);
        src[k] = (uint32_t)(e / chunk * C * HW + e % chunk);
    }
    float pre[C][MAXK];
    auto fetch = [&](int item) {
        const size_t base = (size_t)(item / b.nb) * b.F * C * HW + (size_t)(item % b.nb) * b.R * 2 * b.W;
        const size_t left = total - base - (size_t)(C - 1) * HW - 1;
        const uint32_t lim = left > 0x3fffffff ? 0x3fffffffu : (uint32_t)left;
#pragma unroll
        for (int k = 0; k < MAXK; ++k)
            if (256 * k < plane) {
                const uint32_t off = 4u * min(src[k], lim);          // rows past the map feed no output
#pragma unroll
                for (int c = 0; c < C; ++c) pre[c][k] = *(const float *)((const char *)(x + base + (size_t)c * HW) + off);
            }
    };
    int item = blockIdx.x;
    fetch(min(item, b.items - 1));
    float bv[OT];
#pragma unroll
    for (int m = 0; m < OT; ++m) bv[m] = bias[m * 16 + l16];
    const float *wl = w + (size_t)l16 * K + 4 * g;    // my four taps of channel 0 in filter l16

    int turn = 0;
    for (; item < b.items; item += gridDim.x, ++turn) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MAXK; ++k)
            if (tid + 256 * k < plane) {
#pragma unroll
                for (int c = 0; c < C; ++c) xs[c * plane + tid + 256 * k] = RB ? bf16_rne(pre[c][k]) : pre[c][k];
            }
        __syncthreads();
        fetch(min(item + (int)gridDim.x, b.items - 1));
        __builtin_amdgcn_sched_barrier(0);
        const int f0 = (item / b.nb) * b.F, i0 = (item % b.nb) * b.R;
        const int cnt = b.F * b.R * b.OW, vpix = min(b.R, b.OH - i0) * b.OW, ntile = (cnt + 15) / 16;
        auto pass = [&](auto nc, int t0) {
            constexpr int N = decltype(nc)::value;
            const float *base[N];
#pragma unroll
            for (int n = 0; n < N; ++n) {
                uint32_t p = (uint32_t)((t0 + 4 * n) * 16 + l16), f, rem, i, j;
                if ((int)p >= cnt) p = 0;
                b.dFR.divmod(p, f, rem);
                b.dC.divmod(rem, i, j);
                base[n] = xs + (int)f * chunk + (2 * (int)i + g) * b.W + 2 * (int)j;
            }
            floatx4 acc[N][OT];
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int m = 0; m < OT; ++m) acc[n][m] = floatx4{0.f, 0.f, 0.f, 0.f};
            float4 wv[2][OT];
            auto read_w = [&](int c, float4 (&d)[OT]) {
#pragma unroll
                for (int m = 0; m < OT; ++m) {
                    d[m] = *(const float4 *)(wl + (size_t)m * 16 * K + 16 * c);
                    if (RB) d[m] = bf16_rne(d[m]);
                }
            };
            float xv[2][N][4];
            auto read_x = [&](int c, float (&d)[N][4]) {
#pragma unroll
                for (int n = 0; n < N; ++n)
#pragma unroll
                    for (int e = 0; e < 4; ++e) d[n][e] = base[n][c * plane + e];
            };
            read_w(0, wv[0]);
            read_x(0, xv[0]);
#pragma unroll 2
            for (int c = 0; c < C; ++c) {
                const int cn = min(c + 1, C - 1);
                read_w(cn, wv[(c + 1) & 1]);
                read_x(cn, xv[(c + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int m = 0; m < OT; ++m) {
                        const float4 q = wv[c & 1][m];
                        const float we = e == 0 ? q.x : e == 1 ? q.y : e == 2 ? q.z : q.w;
#pragma unroll
                        for (int n = 0; n < N; ++n) acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[c & 1][n][e], we, acc[n][m], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const uint32_t p0 = (uint32_t)((t0 + 4 * n) * 16 + 4 * g);
                uint32_t f, rem;
                b.dFR.divmod(p0, f, rem);
                const bool whole = (int)p0 < cnt && f0 + (int)f < nframes && (int)rem + 3 < vpix;
#pragma unroll
                for (int m = 0; m < OT; ++m) {
                    float v[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        v[r] = acc[n][m][r] + bv[m];
                        v[r] = v[r] > 0.f ? v[r] : 0.f;
                    }
                    if (whole) {
                        *(f32x4_dw *)(y + ((size_t)(f0 + (int)f) * OC + m * 16 + l16) * NPIX + i0 * b.OW + rem) = f32x4_dw{v[0], v[1], v[2], v[3]};
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            uint32_t fe, re;
                            b.dFR.divmod(p0 + r, fe, re);
                            if ((int)p0 + r < cnt && f0 + (int)fe < nframes && (int)re < vpix)
                                y[((size_t)(f0 + (int)fe) * OC + m * 16 + l16) * NPIX + i0 * b.OW + re] = v[r];
                        }
                    }
                }
            }
        };
        constexpr int NMAX = OC == 32 ? 4 : 2;        // accumulators of a pass: NMAX x OC / 16
        const int wt = (wave + turn) & 3;             // who gets an odd tile more changes from item to item: the SIMDs share it
        int t = wt, left = (ntile - wt + 3) / 4;      // (640 frames of 77x77 402 -> 397 us)
        for (; left >= NMAX; left -= NMAX, t += 4 * NMAX) pass(std::integral_constant<int, NMAX>{}, t);
        if (NMAX > 2 && left == 3) pass(std::integral_constant<int, 3>{}, t);
        else if (NMAX > 2 && left == 2) pass(std::integral_constant<int, 2>{}, t);
        else if (left == 1) pass(std::integral_constant<int, 1>{}, t);
    }
}

// The byte layer: 8x8 filters over four planes of width 84.  A wavefront keeps all filters in registers (64 x OC / 16) and
// takes every fourth pixel tile; a lane's four bytes of a filter row come out of the two dwords they lie in.
template <int OC, bool RB>
__global__ __launch_bounds__(256, 2) void conv_bytes_f32_fwd_kernel(const uint8_t *__restrict__ x, const float *__restrict__ w,
                                                                    const float *__restrict__ bias, float *__restrict__ y, int nframes,
                                                                    float scale, const BytesGeom b) {
    constexpr int OT = OC / 16, KB = 16, MAXU = 7;
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];      // [plane][row][84] bytes, and a dword more
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int RI = (b.R - 1) * b.S + 8, NU = RI * BYTES_Q, PLANE = b.H * BYTES_W, NPIX = b.OH * b.OW;

    uint32_t pre[MAXU][4];
    auto fetch = [&](int item) {
        const int r0 = (item % b.nb) * b.R * b.S;
        const uint8_t *src = x + (size_t)(item / b.nb) * 4 * PLANE + (size_t)r0 * BYTES_W;
        const int last = (b.H - r0) * BYTES_Q - 1;            // rows past the frame feed no output
#pragma unroll
        for (int i = 0; i < MAXU; ++i)
            if (256 * i < NU) {
                const uint32_t off = 4u * (uint32_t)min(min(tid + 256 * i, NU - 1), last);
#pragma unroll
                for (int c = 0; c < 4; ++c) pre[i][c] = *(const uint32_t *)(src + (size_t)c * PLANE + off);
            }
    };
    int item = blockIdx.x;
    fetch(min(item, b.items - 1));
    // group kb of 16 taps: plane kb / 4, filter rows 2 (kb % 4) and the next; my four taps: row + g / 2, columns 4 (g % 2) ..
    float4 wq[KB][OT];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int m = 0; m < OT; ++m) {
            wq[kb][m] = *(const float4 *)(w + (size_t)(m * 16 + l16) * 256 + 16 * kb + 4 * g);
            if (RB) wq[kb][m] = bf16_rne(wq[kb][m]);
        }
    float bv[OT];
#pragma unroll
    for (int m = 0; m < OT; ++m) bv[m] = bias[m * 16 + l16];
    for (; item < b.items; item += gridDim.x) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MAXU; ++i)
            if (tid + 256 * i < NU) {
#pragma unroll
                for (int c = 0; c < 4; ++c) ((uint32_t *)band_smem)[c * NU + tid + 256 * i] = pre[i][c];
            }
        __syncthreads();
        fetch(min(item + (int)gridDim.x, b.items - 1));
        __builtin_amdgcn_sched_barrier(0);
        const int i0 = (item % b.nb) * b.R, cnt = min(b.R, b.OH - i0) * b.OW, ntile = (cnt + 15) / 16;
        float *yb = y + ((size_t)(item / b.nb) * OC + l16) * NPIX + i0 * b.OW;
        auto pass = [&](auto nc, int t0) {
            constexpr int N = decltype(nc)::value;
            const uint32_t *base[N];
            uint32_t sh[N];
#pragma unroll
            for (int n = 0; n < N; ++n) {
                uint32_t p = (uint32_t)((t0 + 4 * n) * 16 + l16), i, j;
                if ((int)p >= cnt) p = 0;
                b.dC.divmod(p, i, j);
                const int at = ((int)i * b.S + (g >> 1)) * BYTES_W + (int)j * b.S + 4 * (g & 1);
                base[n] = (const uint32_t *)band_smem + (at >> 2);
                sh[n] = (uint32_t)at & 3u;
            }
            floatx4 acc[N][OT];
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int m = 0; m < OT; ++m) acc[n][m] = floatx4{0.f, 0.f, 0.f, 0.f};
            uint32_t lo[2][N], hi[2][N];
            auto read = [&](int kb, uint32_t (&a)[N], uint32_t (&c)[N]) {
                const int off = (kb / 4) * NU + 2 * (kb % 4) * BYTES_Q;
#pragma unroll
                for (int n = 0; n < N; ++n) { a[n] = base[n][off]; c[n] = base[n][off + 1]; }
            };
            read(0, lo[0], hi[0]);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                if (kb + 1 < KB) read(kb + 1, lo[(kb + 1) & 1], hi[(kb + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                float xv[N][4];
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    const uint32_t v = __builtin_amdgcn_alignbyte(hi[kb & 1][n], lo[kb & 1][n], sh[n]);
                    xv[n][0] = (float)(v & 0xff); xv[n][1] = (float)((v >> 8) & 0xff);
                    xv[n][2] = (float)((v >> 16) & 0xff); xv[n][3] = (float)(v >> 24);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int m = 0; m < OT; ++m) {
                        const float4 q = wq[kb][m];
                        const float we = e == 0 ? q.x : e == 1 ? q.y : e == 2 ? q.z : q.w;
#pragma unroll
                        for (int n = 0; n < N; ++n) acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[n][e], we, acc[n][m], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const int p0 = (t0 + 4 * n) * 16 + 4 * g;
#pragma unroll
                for (int m = 0; m < OT; ++m) {
                    float v[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        v[r] = acc[n][m][r] * scale + bv[m];
                        v[r] = v[r] > 0.f ? v[r] : 0.f;
                    }
                    float *o = yb + (size_t)m * 16 * NPIX + p0;
                    if (p0 + 3 < cnt) *(f32x4_dw *)o = f32x4_dw{v[0], v[1], v[2], v[3]};
                    else {
#pragma unroll
                        for (int r = 0; r < 3; ++r)
                            if (p0 + r < cnt) o[r] = v[r];
                    }
                }
            }
        };
        int t = wave, left = (ntile - wave + 3) / 4;
        for (; left >= 4; left -= 4, t += 16) pass(std::integral_constant<int, 4>{}, t);
        if (left == 3) pass(std::integral_constant<int, 3>{}, t);
        else if (left == 2) pass(std::integral_constant<int, 2>{}, t);
        else if (left == 1) pass(std::integral_constant<int, 1>{}, t);
    }
}

// ----------------------------------------------------------- input gradient --
// dX[c][y][x] = [xin[c][y][x] > 0] * sum_{oc,a,e} dY[oc][iy - a][ix - e] W[oc][c][ry + 2a][rx + 2e],  y = 2 iy + ry,
// x = 2 ix + rx, with k in the order (oc, a, e): a group of 16 is four filters, the four products of a group are the four
// (a, e).  The zero-padded dY sits in LDS as it is in memory; the four phases (ry, rx) of 16 channels share one fetch of
// it, and a lane's 16 taps of (filter, channel) are 64 contiguous bytes of the weights.  Wavefront = (channel tile, half
// of the pixel tiles), two pixel tiles at a time.
// Bound by the instruction (28.7 GFLOP of conv2 at 640 frames of 77x77: 200 us at 144 TFLOP/s).
template <int OC>
constexpr int band_f32_dgrad_maxk() { return 64 / OC; }      // values of a filter's plane in flight per thread

template <int OC, bool RB>
__global__ __launch_bounds__(256, 2) void conv_band_f32_dgrad_kernel(const float *__restrict__ dy, const float *__restrict__ w,
                                                                     const float *__restrict__ xin, float *__restrict__ dx,
                                                                     int nframes, int pitch, const BandGeom b) {
    constexpr int C = 32, MAXK = band_f32_dgrad_maxk<OC>(), KB = OC / 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    float *ys = (float *)band_smem;                   // [oc][frame][row][PW], `pitch` floats per filter
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int ct = wave & 1, pg = wave >> 1;
    const int HW = b.H * b.W, NPIX = b.OH * b.OW, GW = b.cols, PW = GW + 1, RL = b.R + 1;
    const int chunk = RL * b.OW, plane = b.F * chunk;

    for (int e = tid; e < OC * pitch; e += 256) ys[e] = 0.f;      // columns outside dY stay zero

    int src[MAXK], dst[MAXK], urow[MAXK];
#pragma unroll
    for (int k = 0; k < MAXK; ++k) {
        const int e = min(tid + 256 * k, plane - 1), f = e / chunk, r = e % chunk / b.OW, xc = e % b.OW;
        src[k] = f * OC * NPIX + xc;
        urow[k] = r - 1;
        dst[k] = (f * RL + r) * PW + xc + 1;
    }
    const size_t total = (size_t)nframes * OC * NPIX;
    float pre[OC][MAXK];
    auto fetch = [&](int item) {
        const int f0 = (item / b.nb) * b.F, g0 = (item % b.nb) * b.R;
        const size_t base = (size_t)f0 * OC * NPIX;
        const size_t left = total - base - (size_t)(OC - 1) * NPIX - 1;
        const uint32_t lim = left > 0x3fffffff ? 0x3fffffffu : (uint32_t)left;
#pragma unroll
        for (int k = 0; k < MAXK; ++k)
            if (256 * k < plane) {
                const int yr = min(max(g0 + urow[k], 0), b.OH - 1);
                const uint32_t off = 4u * min((uint32_t)(src[k] + yr * b.OW), lim);
#pragma unroll
                for (int c = 0; c < OC; ++c) pre[c][k] = *(const float *)((const char *)(dy + base + (size_t)c * NPIX) + off);
            }
    };
    int item = blockIdx.x;
    fetch(min(item, b.items - 1));
    const float *wl = w + ((size_t)g * C + ct * 16 + l16) * 16;      // my taps of filter g

    for (; item < b.items; item += gridDim.x) {
        const int f0 = (item / b.nb) * b.F, g0 = (item % b.nb) * b.R;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MAXK; ++k)
            if (tid + 256 * k < plane) {
                const bool in = (unsigned)(g0 + urow[k]) < (unsigned)b.OH;      // else a row above or below dY
#pragma unroll
                for (int c = 0; c < OC; ++c) ys[c * pitch + dst[k]] = in ? (RB ? bf16_rne(pre[c][k]) : pre[c][k]) : 0.f;
            }
        __syncthreads();
        fetch(min(item + (int)gridDim.x, b.items - 1));
        __builtin_amdgcn_sched_barrier(0);
        const int cnt = b.F * b.R * GW, ntile = (cnt + 15) / 16;
        auto pass = [&](auto nc, int t0) {
            constexpr int N = decltype(nc)::value;
            const float *base[N];
            size_t out[N];
            bool in[N][2], two[N];
#pragma unroll
            for (int n = 0; n < N; ++n) {
                uint32_t p = (uint32_t)((t0 + 2 * n) * 16 + l16), f, rem, i, j;
                bool ok = (int)p < cnt;
                if (!ok) p = 0;
                b.dFR.divmod(p, f, rem);
                b.dC.divmod(rem, i, j);
                base[n] = ys + g * pitch + ((int)f * RL + (int)i + 1) * PW + (int)j + 1;
                const int yr = 2 * (g0 + (int)i);
                ok = ok && f0 + (int)f < nframes;
                in[n][0] = ok && yr < b.H;
                in[n][1] = ok && yr + 1 < b.H;
                two[n] = 2 * (int)j + 1 < b.W;
                out[n] = in[n][0] ? ((size_t)(f0 + (int)f) * C + ct * 16 + 4 * g) * HW + yr * b.W + 2 * (int)j : 0;
            }
            floatx4 acc[N][2][2];
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[n][q >> 1][q & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
            float4 wv[2][4];
            auto read_w = [&](int kb, float4 (&d)[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    d[u] = ((const float4 *)(wl + (size_t)kb * 4 * C * 16))[u];
                    if (RB) d[u] = bf16_rne(d[u]);
                }
            };
            float yv[2][N][4];
            auto read_y = [&](int kb, float (&d)[N][4]) {
#pragma unroll
                for (int n = 0; n < N; ++n)
#pragma unroll
                    for (int t = 0; t < 4; ++t) d[n][t] = base[n][kb * 4 * pitch - (t >> 1) * PW - (t & 1)];
            };
            read_w(0, wv[0]);
            read_y(0, yv[0]);
#pragma unroll 2
            for (int kb = 0; kb < KB; ++kb) {
                const int kn = min(kb + 1, KB - 1);
                read_w(kn, wv[(kb + 1) & 1]);
                read_y(kn, yv[(kb + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int ry = 0; ry < 2; ++ry) {
                        const float4 q = wv[kb & 1][ry + 2 * (t >> 1)];
#pragma unroll
                        for (int rx = 0; rx < 2; ++rx) {
                            const float we = t & 1 ? (rx ? q.w : q.z) : (rx ? q.y : q.x);
#pragma unroll
                            for (int n = 0; n < N; ++n)
                                acc[n][ry][rx] = __builtin_amdgcn_mfma_f32_16x16x4f32(we, yv[kb & 1][n][t], acc[n][ry][rx], 0, 0, 0);
                        }
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int n = 0; n < N; ++n) {
                f32x2_dw mk[2][4];
                // the last column of an odd map is the second of the pair in front of it
#pragma unroll
                for (int ry = 0; ry < 2; ++ry)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        mk[ry][r] = *(const f32x2_dw *)(xin + out[n] + (in[n][ry] ? ry * b.W : 0) + (size_t)r * HW - (in[n][0] && !two[n] ? 1 : 0));
#pragma unroll
                for (int ry = 0; ry < 2; ++ry)
                    if (in[n][ry]) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            float *o = dx + out[n] + ry * b.W + (size_t)r * HW;
                            const f32x2_dw m = mk[ry][r];
                            if (two[n]) *(f32x2_dw *)o = f32x2_dw{m.x > 0.f ? acc[n][ry][0][r] : 0.f, m.y > 0.f ? acc[n][ry][1][r] : 0.f};
                            else o[0] = m.y > 0.f ? acc[n][ry][0][r] : 0.f;
                        }
                    }
            }
        };
        int t = pg, left = (ntile - pg + 1) / 2;
        for (; left >= 2; left -= 2, t += 4) pass(std::integral_constant<int, 2>{}, t);
        if (left == 1) pass(std::integral_constant<int, 1>{}, t);
    }
}

// ---------------------------------------------------------- weight gradient --
// dW[oc][k] = scale * sum over the pixels P of all frames of dY[P][oc] x[P][tap k], db[oc] = sum of dY[P][oc], in the chunks of
// pixels and the order of problems.hpp's ConvWgradP: part[chunk][OC][K + 1].  TIn bytes: 8x8 filters over four
// planes, any stride; floats: 4x4, stride 2, 32 channels.
//
// A chunk is one long chain of sums, so the parallelism left is chunks x columns: a wavefront keeps one tile of 16 taps (a
// channel of the 4x4 filters, two rows of an 8x8 plane) of all filters.  The instruction adds its four products one after
// the other, so the column of the bias gradient, whose products are dY itself, is formed with plain additions in that order,
// by one wavefront of a chunk on the side (a wavefront of its own would end last: one chain of dependent instructions).
// The chunk goes by in steps of KT pixels, whose dY lies in LDS as [filter][pixel] and whose input rows as they are in memory:
// the rows that a frame's windows touch, numbered on from frame to frame (S (OH - 1) + KS to a frame), are contiguous for any
// run of pixels, also across frames, and a table gives each pixel's place in them.  The next step's values go from memory
// straight to the other half of the LDS buffers (no registers hold them).
// Bound by the instruction next to the address and byte-conversion instructions (8 per 8 products of 32 cycles), and by whole
// wavefronts per SIMD: conv1 at 640 frames of 84x84, stride 1, is 2736 tiles of 161 us on 1024 SIMDs (483 us; 776 measured,
// 4 ms for the gather kernel).
template <class TIn> constexpr int f32_wgrad_kt() { return sizeof(TIn) == 1 ? 128 : 64; }
struct F32WgradGeom {
    int nframes, C, H, W, S, OH, OW;
    int K, kchunk, nz;       // pixels in all, pixels per chunk, chunks
    int ny;                  // blocks per chunk
    int rows;                // input rows of a step in LDS, at most
    int RF, d;               // rows per frame in the numbering above; frame boundaries in a step, at most
    int stage;               // bytes of one half of the LDS buffers
    FastDiv dNPIX, dOW;
    float scale;
};
template <class TIn> constexpr int f32_wgrad_waves() { return sizeof(TIn) == 1 ? 4 : 8; }
template <class TIn> constexpr int f32_wgrad_maxx() { return 13; }      // dwords of input per thread and step

template <class TIn, int OC, bool RB>
__global__ __launch_bounds__(64 * f32_wgrad_waves<TIn>(), sizeof(TIn) == 1 ? 5 : 4) void conv_f32_wgrad_kernel(
    const TIn *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part, const F32WgradGeom b) {
    constexpr bool BYTE = sizeof(TIn) == 1;
    constexpr int OT = OC / 16, KS = BYTE ? 8 : 4, KT = f32_wgrad_kt<TIn>(), AP = KT + 4, NW = f32_wgrad_waves<TIn>(), NT = 64 * NW, MAXX = f32_wgrad_maxx<TIn>();
    constexpr int NG = KT / 16, ESZ = (int)sizeof(TIn);
    // each half: dY [OC][AP] floats, [KT] byte offsets of the pixels' windows, the input [row][channel][W]
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    constexpr int OTAB = OC * AP * 4, XS = OTAB + KT * 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int NPIX = b.OH * b.OW, HW = b.H * b.W, ncol = BYTE ? 16 : b.C;
    // an XCD takes every eighth chunk, the blocks of a chunk next to each other: its dY then comes from the L2
    const int local = (int)blockIdx.x / 8, by = local % b.ny, z = local / b.ny * 8 + (int)blockIdx.x % 8;
    if (z >= b.nz) return;
    const int q = by * NW + wave;
    // the channels this block's tiles need, in dwords
    const int c0 = BYTE ? 0 : by * NW, nch = BYTE ? 4 : NW;
    const int UW = b.W * ESZ / 4, UR = nch * UW, NU = b.rows * UR, ROW = nch * b.W * ESZ;      // dwords of a row of a channel and of all; bytes
    const int kbeg = z * b.kchunk, kend = min(b.K, kbeg + b.kchunk);

    uint32_t xoff[MAXX];
    int xrow[MAXX];
#pragma unroll
    for (int i = 0; i < MAXX; ++i) {
        const int u = min(tid + NT * i, NU - 1), rem = u % UR;
        xrow[i] = u / UR;
        xoff[i] = (uint32_t)((c0 * HW + rem / UW * HW + xrow[i] * b.W) * ESZ + 4 * (rem % UW));
    }
    const uint32_t jump = (uint32_t)((b.C * b.H - b.RF) * b.W * ESZ);         // over the rows between two frames' channels
    const size_t xbytes = (size_t)b.nframes * b.C * HW * ESZ;
    auto fetch = [&](int k0, unsigned char *half) {
        const uint32_t lds = lds_address(half);
        uint32_t f0, p0, f1, p1;
        b.dNPIX.divmod((uint32_t)k0, f0, p0);
        b.dNPIX.divmod((uint32_t)min(k0 + KT, kend) - 1, f1, p1);
        const int r0 = (int)b.dOW.div(p0) * b.S;
        const int rows = (int)(f1 - f0) * b.RF + (int)b.dOW.div(p1) * b.S + KS - r0;      // that this step's windows touch
        const int nu = rows * UR;
        const size_t xb = (size_t)f0 * b.C * HW * ESZ + (size_t)r0 * b.W * ESZ;
        const uint32_t lim = xbytes - xb > 0x7fffffff ? 0x7fffffffu : (uint32_t)(xbytes - xb) - 4u;
#pragma unroll
        for (int i = 0; i < MAXX; ++i)
            if (64 * wave + NT * i < nu) {
                uint32_t off = xoff[i] + (xrow[i] >= b.RF - r0 ? jump : 0u);
                if (b.d > 1)
                    for (int q = 2; q <= b.d; ++q) off += xrow[i] >= q * b.RF - r0 ? jump : 0u;
                load_dword_to_lds((const char *)x + xb, min(off, lim), lds + XS + (64 * wave + NT * i) * 4);
            }
        const float *src = dy + (size_t)f0 * OC * NPIX;
#pragma unroll
        for (int h = 0; h < KT; h += 64) {
            const int k = k0 + h + lane;
            uint32_t f, p, i, j;
            b.dNPIX.divmod((uint32_t)min(k, b.K - 1), f, p);
            const uint32_t off = 4u * ((f - f0) * (uint32_t)(OC * NPIX) + p);
#pragma unroll
            for (int m = 0; m < OC; m += NW)
                if (OC % NW == 0 || m + wave < OC) load_dword_to_lds(src + (size_t)(m + wave) * NPIX, off, lds + ((m + wave) * AP + h) * 4);
            if (wave == 0) {
                b.dOW.divmod(p, i, j);
                ((int *)(half + OTAB))[h + lane] = k < kend ? ((int)(f - f0) * b.RF + (int)i * b.S - r0) * ROW + (int)j * b.S * ESZ : 0;
            }
        }
    };
    fetch(kbeg, band_smem);

    floatx4 acc[OT];
    float bsum = 0.f;
#pragma unroll
    for (int m = 0; m < OT; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    // my tap's place behind a window's first value
    const int xl = BYTE ? (2 * (q % 4) + (l16 >> 3)) * ROW + (q / 4) * b.W + (l16 & 7)
                        : (l16 >> 2) * ROW + ((q - c0) * b.W + (l16 & 3)) * 4;
    int at = 0;
    for (int k0 = kbeg; k0 < kend; k0 += KT, at ^= 1) {
        unsigned char *half = band_smem + at * b.stage;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // my loads for this step have arrived in LDS
        __syncthreads();                                      // everybody's have, and the other half has been read
        if (k0 + KT < kend) fetch(k0 + KT, band_smem + (at ^ 1) * b.stage);
        else if (k0 + KT > kend) {                            // no pixels behind the chunk's last
            for (int oc = wave; oc < OC; oc += NW)
                for (int kk = lane; kk < KT; kk += 64)
                    if (k0 + kk >= kend) ((float *)half)[oc * AP + kk] = 0.f;
            __syncthreads();
        }
        const float *al = (const float *)half + l16 * AP + 4 * g;
        auto read_a = [&](int grp, float4 (&d)[OT]) {
#pragma unroll
            for (int m = 0; m < OT; ++m) {
                d[m] = *(const float4 *)(al + m * 16 * AP + 16 * grp);
                if (RB) d[m] = bf16_rne(d[m]);
            }
        };
        const int4 *ol = (const int4 *)(half + OTAB) + g;
        const unsigned char *xb = half + XS + xl;
        uint32_t xr[2][4];
        auto read_x = [&](const int4 o, uint32_t (&d)[4]) {
            if (BYTE) { d[0] = xb[o.x]; d[1] = xb[o.y]; d[2] = xb[o.z]; d[3] = xb[o.w]; }
            else {
                d[0] = *(const uint32_t *)(xb + o.x); d[1] = *(const uint32_t *)(xb + o.y);
                d[2] = *(const uint32_t *)(xb + o.z); d[3] = *(const uint32_t *)(xb + o.w);
            }
        };
        int4 o = ol[0];
        float4 av[2][OT];
        read_x(o, xr[0]);
        read_a(0, av[0]);
        o = ol[4];
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) {
            if (grp + 1 < NG) {
                read_x(o, xr[(grp + 1) & 1]);
                read_a(grp + 1, av[(grp + 1) & 1]);
                if (grp + 2 < NG) o = ol[4 * (grp + 2)];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint32_t v = xr[grp & 1][t];
                const float xv = BYTE ? (float)v : RB ? bf16_rne(__uint_as_float(v)) : __uint_as_float(v);
#pragma unroll
                for (int m = 0; m < OT; ++m) {
                    const float4 a = av[grp & 1][m];
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(t == 0 ? a.x : t == 1 ? a.y : t == 2 ? a.z : a.w, xv, acc[m], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (by == 0 && wave == (z & (NW - 1))) {      // the bias gradient, a filter per lane: the sums the instruction would form
            const float *bl = (const float *)half + min(lane, OC - 1) * AP;
#pragma unroll
            for (int grp = 0; grp < NG; ++grp) {
                float v[16];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float4 d = *(const float4 *)(bl + 16 * grp + 4 * e);
                    v[4 * e] = d.x; v[4 * e + 1] = d.y; v[4 * e + 2] = d.z; v[4 * e + 3] = d.w;
                }
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) bsum += RB ? bf16_rne(v[4 * e + t]) : v[4 * e + t];
            }
        }
    }
    const int K1 = 16 * ncol + 1;
    float *pb = part + (size_t)z * OC * K1;
#pragma unroll
    for (int m = 0; m < OT; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) pb[(size_t)(m * 16 + 4 * g + r) * K1 + 16 * q + l16] = acc[m][r] * b.scale;
    if (by == 0 && wave == (z & (NW - 1)) && lane < OC) pb[(size_t)lane * K1 + K1 - 1] = bsum;
}

template <int C>
inline bool band_f32_geom(BandGeom &b, int nframes) {
    auto px = [&](int F, int R) { return F * ((R - 1) * 2 + 4) * b.W; };
    return band_split(b, nframes, b.OH, b.OW, [&](int F, int R) { return px(F, R) * C * 4 <= BAND_F32_LDS ? 0 : 2 * BAND_LDS; },
                      [&](int F, int R) { return px(F, R) <= 256 * BAND_F32_MAXK ? 0 : 1 << 30; }, BAND_MAXU, 2 * BAND_CUS);
}

template <int C, int OC, bool RB>
inline hipError_t launch_conv_band_f32_fwd1(const float *x, const float *w, const float *bias, float *y, int n, int H, int W, hipStream_t s) {
    BandGeom b = band_geom(H, W);
    if (!band_f32_geom<C>(b, n)) return hipErrorInvalidValue;
    static bool attr = false;
    const hipError_t e = band_allow_lds(conv_band_f32_fwd_kernel<C, OC, RB>, attr);
    if (e != hipSuccess) return e;
    ga3c::launch((conv_band_f32_fwd_kernel<C, OC, RB>), dim3(std::min(b.items, 2 * BAND_CUS)), dim3(256),
                 b.F * ((b.R - 1) * 2 + 4) * b.W * C * 4, s, x, w, bias, y, n, b);
    return hipGetLastError();
}
// x [n][32][H][W] -> y [n][OC][OH][OW]; w [OC][32][4][4], 16-byte aligned.
template <int C, int OC>
inline hipError_t launch_conv_band_f32_fwd(const float *x, const float *w, const float *bias, float *y, int n, int H, int W, hipStream_t s, int rb) {
    if (n <= 0) return hipSuccess;
    return rb ? launch_conv_band_f32_fwd1<C, OC, true>(x, w, bias, y, n, H, W, s) : launch_conv_band_f32_fwd1<C, OC, false>(x, w, bias, y, n, H, W, s);
}

template <int OC, bool RB>
inline hipError_t launch_conv_bytes_f32_fwd1(const uint8_t *x, const float *w, const float *bias, float *y, int n, int H, int S, float scale, hipStream_t s) {
    const BytesGeom b = bytes_fwd_geom(H, S, n);
    static bool attr = false;
    const hipError_t e = band_allow_lds(conv_bytes_f32_fwd_kernel<OC, RB>, attr);
    if (e != hipSuccess) return e;
    const int RI = (b.R - 1) * b.S + 8;
    ga3c::launch((conv_bytes_f32_fwd_kernel<OC, RB>), dim3(std::min(b.items, 2 * BAND_CUS)), dim3(256), RI * BYTES_W * 4 + 16, s, x, w, bias, y, n, scale, b);
    return hipGetLastError();
}
// x [n][4][H][84] bytes -> y [n][OC][OH][OW]; w [OC][4][8][8], 16-byte aligned.
template <int OC>
inline hipError_t launch_conv_bytes_f32_fwd(const uint8_t *x, const float *w, const float *bias, float *y, int n, int H, int S, float scale, hipStream_t s,
                                            int rb) {
    if (n <= 0) return hipSuccess;
    return rb ? launch_conv_bytes_f32_fwd1<OC, true>(x, w, bias, y, n, H, S, scale, s) : launch_conv_bytes_f32_fwd1<OC, false>(x, w, bias, y, n, H, S, scale, s);
}

template <int OC>
inline int band_f32_dgrad_pitch(const BandGeom &b) {      // floats per filter: the four filters of a group on different banks
    const int n = b.F * (b.R + 1) * (b.cols + 1);
    return (n + 47) / 64 * 64 + 16;
}
template <int OC>
inline bool band_f32_dgrad_geom(BandGeom &b, int nframes) {
    const int GW = (b.W + 1) / 2;
    return band_split(b, nframes, (b.H + 1) / 2, GW,
                      [&](int F, int R) { return (F * (R + 1) * (GW + 1) + 63) * OC * 4 <= BAND_F32_LDS ? 0 : 2 * BAND_LDS; },
                      [&](int F, int R) { return F * (R + 1) * b.OW <= 256 * band_f32_dgrad_maxk<OC>() ? 0 : 1 << 30; }, BAND_MAXU,
                      2 * BAND_CUS);
}
template <int OC, bool RB>
inline hipError_t launch_conv_band_f32_dgrad1(const float *dy, const float *w, const float *xin, float *dx, int n, int H, int W, hipStream_t s) {
    BandGeom b = band_geom(H, W);
    if (!band_f32_dgrad_geom<OC>(b, n)) return hipErrorInvalidValue;
    static bool attr = false;
    const hipError_t e = band_allow_lds(conv_band_f32_dgrad_kernel<OC, RB>, attr);
    if (e != hipSuccess) return e;
    const int pitch = band_f32_dgrad_pitch<OC>(b);
    ga3c::launch((conv_band_f32_dgrad_kernel<OC, RB>), dim3(std::min(b.items, 2 * BAND_CUS)), dim3(256), OC * pitch * 4, s, dy, w, xin, dx, n,
                 pitch, b);
    return hipGetLastError();
}
// dy [n][OC][OH][OW] -> dx [n][32][H][W], masked by xin > 0; w [OC][32][4][4], 16-byte aligned.
template <int OC>
inline hipError_t launch_conv_band_f32_dgrad(const float *dy, const float *w, const float *xin, float *dx, int n, int H, int W, hipStream_t s, int rb) {
    if (n <= 0) return hipSuccess;
    return rb ? launch_conv_band_f32_dgrad1<OC, true>(dy, w, xin, dx, n, H, W, s) : launch_conv_band_f32_dgrad1<OC, false>(dy, w, xin, dx, n, H, W, s);
}

// Whether the forward pass and the input gradient can run maps of H x W.
template <int C>
inline bool band_f32_ok(int H, int W) {
    BandGeom b = band_geom(H, W), c = b, d = b;
    return band_f32_geom<C>(b, 1) && band_f32_dgrad_geom<32>(c, 1) && band_f32_dgrad_geom<64>(d, 1);
}

// b.rows: rows of input that a step can touch; it covers up to R output rows and d frame boundaries.
template <class TIn>
inline F32WgradGeom f32_wgrad_geom(int C, int H, int W, int S, int n, int kchunk, float scale) {
    constexpr int KS = sizeof(TIn) == 1 ? 8 : 4;
    F32WgradGeom b{};
    b.nframes = n; b.C = C; b.H = H; b.W = W; b.S = S; b.OH = (H - KS) / S + 1; b.OW = (W - KS) / S + 1;
    b.K = n * b.OH * b.OW; b.kchunk = kchunk; b.scale = scale;
    b.RF = S * (b.OH - 1) + KS;
    const int R = (f32_wgrad_kt<TIn>() - 2) / b.OW + 2;
    b.d = (R - 2) / b.OH + 1;
    b.rows = S * (R - 1) + KS + b.d * std::max(0, KS - S);
    b.dNPIX = FastDiv((uint32_t)(b.OH * b.OW)); b.dOW = FastDiv((uint32_t)b.OW);
    return b;
}
template <class TIn>
inline int f32_wgrad_stage(const F32WgradGeom &b, int OC) {      // the input's part rounded up to whole wavefronts
    const int x = (sizeof(TIn) == 1 ? 4 : f32_wgrad_waves<TIn>()) * b.rows * b.W * (int)sizeof(TIn);
    return (OC * (f32_wgrad_kt<TIn>() + 4) + f32_wgrad_kt<TIn>()) * 4 + (x + 255) / 256 * 256;
}
// Whether a step fits the threads and half of a compute unit's LDS.
template <class TIn>
inline bool f32_wgrad_ok(int C, int H, int W, int S, int OC) {
    const F32WgradGeom b = f32_wgrad_geom<TIn>(C, H, W, S, 1, f32_wgrad_kt<TIn>(), 1.f);
    const int nch = sizeof(TIn) == 1 ? 4 : f32_wgrad_waves<TIn>();
    return nch * b.rows * (W * (int)sizeof(TIn) / 4) <= 64 * f32_wgrad_waves<TIn>() * f32_wgrad_maxx<TIn>() &&
           2 * f32_wgrad_stage<TIn>(b, OC) <= BAND_F32_LDS;
}
// part [nz][OC][K + 1], nz chunks of kchunk pixels (a multiple of 16).
template <class TIn, int OC>
inline hipError_t launch_conv_f32_wgrad(const TIn *x, const float *dy, float *part, int n, int C, int H, int W, int S, int nz, int kchunk, float scale,
                                        hipStream_t s, int rb) {
    if (n <= 0) return hipSuccess;
    F32WgradGeom b = f32_wgrad_geom<TIn>(C, H, W, S, n, kchunk, scale);
    b.stage = f32_wgrad_stage<TIn>(b, OC);
    constexpr int NW = f32_wgrad_waves<TIn>();
    b.nz = nz; b.ny = (sizeof(TIn) == 1 ? 16 : C) / NW;
    const dim3 grid((nz + 7) / 8 * 8 * b.ny), block(64 * NW);
    const int lds = 2 * b.stage;
    static bool attr0 = false, attr1 = false;
    if (rb) {
        const hipError_t e = band_allow_lds(conv_f32_wgrad_kernel<TIn, OC, true>, attr1);
        if (e != hipSuccess) return e;
        ga3c::launch((conv_f32_wgrad_kernel<TIn, OC, true>), grid, block, lds, s, x, dy, part, b);
    } else {
        const hipError_t e = band_allow_lds(conv_f32_wgrad_kernel<TIn, OC, false>, attr0);
        if (e != hipSuccess) return e;
        ga3c::launch((conv_f32_wgrad_kernel<TIn, OC, false>), grid, block, lds, s, x, dy, part, b);
    }
    return hipGetLastError();
}

}  // namespace ga3c
