// A convolution layer on the fp32 matrix instruction, inside a block that holds a frame's maps in LDS: what a kernel on two float16 terms
// (split_f16.hpp) turns to when filters hold weights that the terms do not (F16_WIDE), or channels of a map, by their filters and biases,
// are too far apart for one scale (F16_APART).  Products and sums are fp32's, whatever the sizes.
//
// A wavefront takes 16 filters and up to seven tiles of 16 pixels at a time.  Sixteen k of a filter are one vector a lane, its own group of
// four; the pixels' values come one by one from LDS.  Such a call takes the float16
// kernel's time as well.  us a call, by the kernels on three bfloat16 terms that had all of this work / by a thread per output / so: larger net
// 1 frame 25 / 1220 / 70, 256 frames 48 / 1280 / 83, 512: 70 / 2530 / 154; small net 128: 17 / 394 / 32, 1024: 37 / 1566 / 97; stride-4 member
// 128: 33 / 858 / 50, stride 3: 37 / 1320 / 82.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_mfma.hpp"

namespace ga3c {

// Pixel tiles a wavefront takes at a time, so that the one with the most work has the least.
constexpr int plain_conv_tiles(const int nt, const int ot, const int nw) {
    int best = 1, least = 1 << 30;
    for (int t = 1; t <= 7; ++t) {
        const int work = (ot * ((nt + t - 1) / t) + nw - 1) / nw * t;
        if (work <= least) { least = work; best = t; }
    }
    return best;
}

// y [OC][OH][OW] = max(0, b + sum w (scale x)) by the block's NW wavefronts; x in LDS, w 16-byte aligned in memory, y: in memory or in LDS.
template <class In, int C, int H, int OC, int KS, int S, int NW>
__device__ __forceinline__ void plain_conv_layer(const In *x, const float scale, const float *__restrict__ w, const float *__restrict__ b, float *y,
                                                 const int wave, const int lane) {
    constexpr int K = C * KS * KS, OH = (H - KS) / S + 1, NPIX = OH * OH, NT = (NPIX + 15) / 16, PT = plain_conv_tiles(NT, OC / 16, NW), GROUPS = (NT + PT - 1) / PT;
    static_assert(K % 16 == 0 && OC % 16 == 0, "whole vectors of k, whole tiles of filters");
    const int l16 = lane & 15, g = lane >> 4;
#pragma unroll 1
    for (int u = wave; u < OC / 16 * GROUPS; u += NW) {
        const int ot = u / GROUPS, first = u % GROUPS * PT;
        const float *f = w + (size_t)(ot * 16 + l16) * K + 4 * g;
        const In *from[PT];
        floatx4 acc[PT];
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int p = min((first + i) * 16 + l16, NPIX - 1);
            from[i] = x + (p / OH * H + p % OH) * S;
            acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll 4
        for (int kb = 0; kb < K / 16; ++kb) {
            const float4 wv = *(const float4 *)(f + 16 * kb);
            const float wk[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = 16 * kb + 4 * g + j, at = (k / (KS * KS) * H + k / KS % KS) * H + k % KS;
#pragma unroll
                for (int i = 0; i < PT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wk[j], (float)from[i][at] * scale, acc[i], 0, 0, 0);
            }
        }
        const float4 bias = *(const float4 *)(b + ot * 16 + 4 * g);
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int p = (first + i) * 16 + l16;
            if (p < NPIX) {
                float *to = y + (ot * 16 + 4 * g) * NPIX + p;
                to[0] = fmaxf(acc[i][0] + bias.x, 0.f);
                to[NPIX] = fmaxf(acc[i][1] + bias.y, 0.f);
                to[2 * NPIX] = fmaxf(acc[i][2] + bias.z, 0.f);
                to[3 * NPIX] = fmaxf(acc[i][3] + bias.w, 0.f);
            }
        }
    }
}

}  // namespace ga3c
