// A convolution layer as plain sums of fp32 products: what a kernel on two float16 terms (split_f16.hpp) turns to when filters hold weights
// that the terms do not (F16_WIDE), or channels of a map, by their filters and biases, are too far apart for one scale (F16_APART).  A thread per output, hundreds of times slower; nothing that initialisation or training makes of a filter
// comes here.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ga3c {

// y [OC][OH][OW] = max(0, b + sum w (scale x)) by `n` threads; x, y: in memory or in LDS.
template <class In>
__device__ __forceinline__ void plain_conv_layer(const In *x, const float scale, const float *__restrict__ w, const float *__restrict__ b, float *y,
                                                 const int C, const int H, const int W, const int OC, const int KS, const int S, const int tid, const int n) {
    const int OH = (H - KS) / S + 1, OW = (W - KS) / S + 1;
#pragma unroll 1
    for (int o = tid; o < OC * OH * OW; o += n) {
        const int oc = o / (OH * OW), p = o % (OH * OW);
        const In *from = x + (p / OW * S) * W + p % OW * S;
        const float *f = w + (size_t)oc * C * KS * KS;
        float sum = 0.f;
#pragma unroll 1
        for (int t = 0; t < C * KS; ++t)                   // (channel, row)
#pragma unroll 1
            for (int v = 0; v < KS; ++v) sum = fmaf(f[t * KS + v], (float)from[(t / KS * H + t % KS) * W + v] * scale, sum);
        y[o] = fmaxf(sum + b[oc], 0.f);
    }
}

}  // namespace ga3c
