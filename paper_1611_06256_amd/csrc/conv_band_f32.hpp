// The layers of conv_band.hpp and conv_bytes.hpp on the fp32 matrix instruction,
// for maps of any size (the 4x4 stride-2 layer on 32 channels, and the 8x8 byte
// layer of any stride): forward pass, and the byte layer's weight gradient for
// the strides and filter counts that conv_band_grads.hpp does not take.
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
// update (conv_band_grads.hpp has them on the bf16 instruction).
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

// ---------------------------------------------------------- weight gradient --
// dW[oc][k] = scale * sum over the pixels P of all frames of dY[P][oc] x[P][tap k], db[oc] = sum of dY[P][oc], in the chunks of
// pixels and the order of problems.hpp's ConvWgradP: part[chunk][OC][K + 1].  8x8 filters over four planes of bytes, any
// stride.
//
// A chunk is one long chain of sums, so the parallelism left is chunks x columns: a wavefront keeps one tile of 16 taps (two
// rows of a plane's 8x8) of all filters.  The instruction adds its four products one after
// the other, so the column of the bias gradient, whose products are dY itself, is formed with plain additions in that order,
// by one wavefront of a chunk on the side (a wavefront of its own would end last: one chain of dependent instructions).
// The chunk goes by in steps of KT pixels, whose dY lies in LDS as [filter][pixel] and whose input rows as they are in memory:
// the rows that a frame's windows touch, numbered on from frame to frame (S (OH - 1) + KS to a frame), are contiguous for any
// run of pixels, also across frames, and a table gives each pixel's place in them.  The next step's values go from memory
// straight to the other half of the LDS buffers (no registers hold them).
// Bound by the instruction next to the address and byte-conversion instructions (8 per 8 products of 32 cycles), and by whole
// wavefronts per SIMD.
constexpr int F32_WGRAD_KT = 128, F32_WGRAD_WAVES = 4;
constexpr int F32_WGRAD_MAXX = 13;                // dwords of input per thread and step
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

template <int OC, bool RB>
__global__ __launch_bounds__(64 * F32_WGRAD_WAVES, 5) void conv_f32_wgrad_kernel(const uint8_t *__restrict__ x, const float *__restrict__ dy,
                                                                                 float *__restrict__ part, const F32WgradGeom b) {
    constexpr int OT = OC / 16, KS = 8, KT = F32_WGRAD_KT, AP = KT + 4, NW = F32_WGRAD_WAVES, NT = 64 * NW, MAXX = F32_WGRAD_MAXX;
    constexpr int NG = KT / 16;
    // each half: dY [OC][AP] floats, [KT] byte offsets of the pixels' windows, the input [row][channel][W]
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    constexpr int OTAB = OC * AP * 4, XS = OTAB + KT * 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int NPIX = b.OH * b.OW, HW = b.H * b.W;
    // an XCD takes every eighth chunk, the blocks of a chunk next to each other: its dY then comes from the L2
    const int local = (int)blockIdx.x / 8, by = local % b.ny, z = local / b.ny * 8 + (int)blockIdx.x % 8;
    if (z >= b.nz) return;
    const int q = by * NW + wave;
    const int UW = b.W / 4, UR = 4 * UW, NU = b.rows * UR, ROW = 4 * b.W;      // dwords of a row of a plane and of all; bytes
    const int kbeg = z * b.kchunk, kend = min(b.K, kbeg + b.kchunk);

    uint32_t xoff[MAXX];
    int xrow[MAXX];
#pragma unroll
    for (int i = 0; i < MAXX; ++i) {
        const int u = min(tid + NT * i, NU - 1), rem = u % UR;
        xrow[i] = u / UR;
        xoff[i] = (uint32_t)(rem / UW * HW + xrow[i] * b.W + 4 * (rem % UW));
    }
    const uint32_t jump = (uint32_t)((b.C * b.H - b.RF) * b.W);         // over the rows between two frames' channels
    const size_t xbytes = (size_t)b.nframes * b.C * HW;
    auto fetch = [&](int k0, unsigned char *half) {
        const uint32_t lds = lds_address(half);
        uint32_t f0, p0, f1, p1;
        b.dNPIX.divmod((uint32_t)k0, f0, p0);
        b.dNPIX.divmod((uint32_t)min(k0 + KT, kend) - 1, f1, p1);
        const int r0 = (int)b.dOW.div(p0) * b.S;
        const int rows = (int)(f1 - f0) * b.RF + (int)b.dOW.div(p1) * b.S + KS - r0;      // that this step's windows touch
        const int nu = rows * UR;
        const size_t xb = (size_t)f0 * b.C * HW + (size_t)r0 * b.W;
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
                ((int *)(half + OTAB))[h + lane] = k < kend ? ((int)(f - f0) * b.RF + (int)i * b.S - r0) * ROW + (int)j * b.S : 0;
            }
        }
    };
    fetch(kbeg, band_smem);

    floatx4 acc[OT];
    float bsum = 0.f;
#pragma unroll
    for (int m = 0; m < OT; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    // my tap's place behind a window's first value
    const int xl = (2 * (q % 4) + (l16 >> 3)) * ROW + (q / 4) * b.W + (l16 & 7);
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
        auto read_x = [&](const int4 o, uint32_t (&d)[4]) { d[0] = xb[o.x]; d[1] = xb[o.y]; d[2] = xb[o.z]; d[3] = xb[o.w]; };
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
                const float xv = (float)xr[grp & 1][t];
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
    constexpr int K1 = 257;
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

// Whether the forward pass can run maps of H x W.
template <int C>
inline bool band_f32_ok(int H, int W) {
    BandGeom b = band_geom(H, W);
    return band_f32_geom<C>(b, 1);
}

// b.rows: rows of input that a step can touch; it covers up to R output rows and d frame boundaries.
inline F32WgradGeom f32_wgrad_geom(int C, int H, int W, int S, int n, int kchunk, float scale) {
    constexpr int KS = 8;
    F32WgradGeom b{};
    b.nframes = n; b.C = C; b.H = H; b.W = W; b.S = S; b.OH = (H - KS) / S + 1; b.OW = (W - KS) / S + 1;
    b.K = n * b.OH * b.OW; b.kchunk = kchunk; b.scale = scale;
    b.RF = S * (b.OH - 1) + KS;
    const int R = (F32_WGRAD_KT - 2) / b.OW + 2;
    b.d = (R - 2) / b.OH + 1;
    b.rows = S * (R - 1) + KS + b.d * std::max(0, KS - S);
    b.dNPIX = FastDiv((uint32_t)(b.OH * b.OW)); b.dOW = FastDiv((uint32_t)b.OW);
    return b;
}
inline int f32_wgrad_stage(const F32WgradGeom &b, int OC) {      // the input's part rounded up to whole wavefronts
    return (OC * (F32_WGRAD_KT + 4) + F32_WGRAD_KT) * 4 + (4 * b.rows * b.W + 255) / 256 * 256;
}
// Whether a step fits the threads and half of a compute unit's LDS.
inline bool f32_wgrad_ok(int C, int H, int W, int S, int OC) {
    const F32WgradGeom b = f32_wgrad_geom(C, H, W, S, 1, F32_WGRAD_KT, 1.f);
    return b.rows * W <= 64 * F32_WGRAD_WAVES * F32_WGRAD_MAXX && 2 * f32_wgrad_stage(b, OC) <= BAND_F32_LDS;
}
// part [nz][OC][K + 1], nz chunks of kchunk pixels (a multiple of 16).
template <int OC>
inline hipError_t launch_conv_f32_wgrad(const uint8_t *x, const float *dy, float *part, int n, int C, int H, int W, int S, int nz, int kchunk, float scale,
                                        hipStream_t s, int rb) {
    if (n <= 0) return hipSuccess;
    F32WgradGeom b = f32_wgrad_geom(C, H, W, S, n, kchunk, scale);
    b.stage = f32_wgrad_stage(b, OC);
    b.nz = nz; b.ny = 16 / F32_WGRAD_WAVES;
    const dim3 grid((nz + 7) / 8 * 8 * b.ny), block(64 * F32_WGRAD_WAVES);
    const int lds = 2 * b.stage;
    static bool attr0 = false, attr1 = false;
    if (rb) {
        const hipError_t e = band_allow_lds(conv_f32_wgrad_kernel<OC, true>, attr1);
        if (e != hipSuccess) return e;
        ga3c::launch((conv_f32_wgrad_kernel<OC, true>), grid, block, lds, s, x, dy, part, b);
    } else {
        const hipError_t e = band_allow_lds(conv_f32_wgrad_kernel<OC, false>, attr0);
        if (e != hipSuccess) return e;
        ga3c::launch((conv_f32_wgrad_kernel<OC, false>), grid, block, lds, s, x, dy, part, b);
    }
    return hipGetLastError();
}

}  // namespace ga3c
