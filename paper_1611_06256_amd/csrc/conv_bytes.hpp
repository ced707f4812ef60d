// First convolution layer (8x8 filters over four planes of bytes, any stride;
// the paper's larger-network family, Sec. 5, uses 4, 3, 2 and 1): forward
// pass of predictions on the bf16 matrix cores at fp32 accuracy, and of both
// calls with operands rounded to bfloat16 (ONE: one term).
//
// A byte is exact in bf16 and an fp32 weight or gradient is the exact sum of
// three bf16 terms, so a product is three bf16 products that are exact in the
// fp32 accumulator (conv1_bf16x3.hpp).
//
// LDS holds a band of the frame as [row][column][plane] bf16, 8 bytes per
// pixel.  The contraction index of the forward pass is ordered (u, v, plane):
// one k-block of 32 is one filter row, and the 8 values of a lane are two
// neighbouring pixels, 16 bytes at an 8-byte aligned place whatever the stride.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include "conv_band.hpp"

namespace ga3c {

// Bands of the byte layer: R output rows of one frame.
struct BytesGeom {
    int H, S, OH, OW, R, nb, items;
    FastDiv dC;              // by OW
};
constexpr int BYTES_W = 84;                       // pixels per row (a template of one: row offsets are immediates)
constexpr int BYTES_Q = BYTES_W / 4;              // dwords per row and plane
constexpr int BYTES_ROW = BYTES_W * 8;            // LDS bytes per row

// One dword of each plane (four pixels) -> 32 LDS bytes.
__device__ __forceinline__ void bytes_store4(unsigned char *dst, const uint32_t (&v)[4]) {
    u32x4 o[2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float f[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) f[c] = (float)((v[c] >> (8 * t)) & 0xff);
        o[t / 2][(t % 2) * 2] = pack_bf16_rne(f[0], f[1]);
        o[t / 2][(t % 2) * 2 + 1] = pack_bf16_rne(f[2], f[3]);
    }
    ((u32x4 *)dst)[0] = o[0];
    ((u32x4 *)dst)[1] = o[1];
}

// y[oc][i][j] = max(0, scale * sum W[oc][c][u][v] x[c][S i + u][S j + v] + b[oc]).  Wavefront w keeps the fragments of
// filter tile w % (OC / 16) in registers (96 of them) and takes every (64 / OC)-th pixel tile, four at a time; two blocks
// share a compute unit.
template <int OC, bool ONE>
__global__ __launch_bounds__(256, 2) void conv_bytes_fwd_kernel(const uint8_t *__restrict__ x, const u32x4 *__restrict__ wfrag,
                                                                const float *__restrict__ bias, float *__restrict__ y, int nframes,
                                                                float scale, const BytesGeom b) {
    constexpr int OT = OC / 16, PG = 4 / OT, NTERM = ONE ? 1 : 3, KB = 8, MAXU = 7;
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int ot = wave % OT, pg = wave / OT;
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
    Bf16x8Bits wq[KB][NTERM];
    {
        const u32x4 *ws = wfrag + (size_t)(ot * KB) * NTERM * 64 + lane;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int t = 0; t < NTERM; ++t) wq[kb][t].u = ws[(kb * NTERM + t) * 64];
    }
    const float bv = bias[ot * 16 + l16];
    for (; item < b.items; item += gridDim.x) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MAXU; ++i)
            if (tid + 256 * i < NU) bytes_store4(band_smem + (size_t)(tid + 256 * i) * 32, pre[i]);
        __syncthreads();
        fetch(min(item + (int)gridDim.x, b.items - 1));
        __builtin_amdgcn_sched_barrier(0);
        const int i0 = (item % b.nb) * b.R, cnt = min(b.R, b.OH - i0) * b.OW, ntile = (cnt + 15) / 16;
        float *yb = y + ((size_t)(item / b.nb) * OC + ot * 16 + l16) * NPIX + i0 * b.OW;
        auto pass = [&](auto nc, int t0) {
            constexpr int N = decltype(nc)::value;
            const unsigned char *base[N];
#pragma unroll
            for (int n = 0; n < N; ++n) {
                uint32_t p = (uint32_t)((t0 + n * PG) * 16 + l16), i, j;
                if ((int)p >= cnt) p = 0;
                b.dC.divmod(p, i, j);
                base[n] = band_smem + ((int)i * b.S * BYTES_W + (int)j * b.S + 2 * g) * 8;
            }
            floatx4 acc[N];
#pragma unroll
            for (int n = 0; n < N; ++n) acc[n] = floatx4{0.f, 0.f, 0.f, 0.f};
            Bf16x8Bits xv[2][N];
            auto read = [&](int kb, Bf16x8Bits (&d)[N]) {
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    const uint2 lo = *(const uint2 *)(base[n] + kb * BYTES_ROW), hi = *(const uint2 *)(base[n] + kb * BYTES_ROW + 8);
                    d[n].u = u32x4{lo.x, lo.y, hi.x, hi.y};
                }
            };
            read(0, xv[0]);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                if (kb + 1 < KB) read(kb + 1, xv[(kb + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = NTERM - 1; t >= 0; --t)
#pragma unroll
                    for (int n = 0; n < N; ++n)
                        acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[kb & 1][n].v, wq[kb][t].v, acc[n], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const int p0 = (t0 + n * PG) * 16 + 4 * g;
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = acc[n][r] * scale + bv;
                    v[r] = v[r] > 0.f ? v[r] : 0.f;
                }
                if (p0 + 3 < cnt) *(f32x4_dw *)(yb + p0) = f32x4_dw{v[0], v[1], v[2], v[3]};
                else {
#pragma unroll
                    for (int r = 0; r < 3; ++r)
                        if (p0 + r < cnt) yb[p0 + r] = v[r];
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

inline BytesGeom bytes_geom(int H, int S) {
    BytesGeom b{};
    b.H = H; b.S = S; b.OH = (H - 8) / S + 1; b.OW = (BYTES_W - 8) / S + 1;
    b.dC = FastDiv((uint32_t)b.OW);
    return b;
}
// rmax: rows an item may have; enough bands for `want` items where the batch has fewer frames, of at least two pixel tiles.
inline void bytes_split(BytesGeom &b, int nframes, int rmax, int want) {
    int nb = (b.OH + rmax - 1) / rmax;
    if (nframes * nb < want) nb = std::max(nb, std::min(want / nframes, std::max(1, b.OH * b.OW / 32)));
    b.R = (b.OH + nb - 1) / nb;
    b.nb = (b.OH + b.R - 1) / b.R;
    b.items = nframes * b.nb;
}
inline BytesGeom bytes_fwd_geom(int H, int S, int n) {
    BytesGeom b = bytes_geom(H, S);
    int r = 1;                                            // 80 KB per block and seven staging units per thread
    while (r < b.OH && (r * S + 8) * BYTES_ROW <= 80 * 1024 && (r * S + 8) * BYTES_Q <= 7 * 256) ++r;
    bytes_split(b, n, r, 2 * BAND_CUS);
    return b;
}
// Frames of H rows of 84 pixels, any stride.  A row of the map must fit an item.
inline bool bytes_ok(int H, int W, int S) {
    return W == BYTES_W && H >= 8 && S >= 1 && (BYTES_W - 8) / S + 1 <= 128;
}

template <int OC, bool ONE>
inline hipError_t launch_conv_bytes_fwd1(const uint8_t *x, const u32x4 *wfrag, const float *bias, float *y, int n, int H, int S, float scale, hipStream_t s) {
    const BytesGeom b = bytes_fwd_geom(H, S, n);
    static bool attr = false;
    const hipError_t e = band_allow_lds(conv_bytes_fwd_kernel<OC, ONE>, attr);
    if (e != hipSuccess) return e;
    const int RI = (b.R - 1) * S + 8, units = (RI * BYTES_Q + 255) / 256 * 256;
    ga3c::launch((conv_bytes_fwd_kernel<OC, ONE>), dim3(std::min(b.items, 2 * BAND_CUS)), dim3(256), units * 32, s, x, wfrag, bias, y, n, scale, b);
    return hipGetLastError();
}
template <int OC>
inline hipError_t launch_conv_bytes_fwd(const uint8_t *x, const u32x4 *wfrag, const float *bias, float *y, int n, int H, int S, float scale, hipStream_t s, int rb) {
    if (n <= 0) return hipSuccess;
    return rb ? launch_conv_bytes_fwd1<OC, true>(x, wfrag, bias, y, n, H, S, scale, s) : launch_conv_bytes_fwd1<OC, false>(x, wfrag, bias, y, n, H, S, scale, s);
}

}  // namespace ga3c
