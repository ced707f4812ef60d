// Forward pass of the layers of conv_band.hpp and conv_bytes.hpp on the fp32
// matrix instruction, for maps of any size: the 4x4 stride-2 layer on 32
// channels, and the 8x8 byte layer of any stride.
//
// Every output is formed by the same instructions in the same order as in
// gemm_mfma.hpp (v_mfma_f32_16x16x4_f32, product t of a group of 16 k sums
// k = 16 kb + 4 g + t over g, groups and t ascending), so the activations are
// the same bits as those of the any-shape kernels.  That matters in training:
// where a pre-activation lies within rounding of zero, another order of the sum
// can put it on the other side of the rectifier, and a map of millions of
// pixels has enough of those to move the gradient of a filter by 1e-4 of itself.
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

    for (; item < b.items; item += gridDim.x) {
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
        int t = wave, left = (ntile - wave + 3) / 4;
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

}  // namespace ga3c
