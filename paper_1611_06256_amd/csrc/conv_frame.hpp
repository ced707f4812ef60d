// A convolution layer's shape as a type, for the kernels that are compiled for one geometry (the layers of the networks of Sec.
// 3.2, of the larger network of the workload list and of the paper's larger-network family).
#pragma once
#include <stdint.h>

#include "gemm_mfma.hpp"

namespace ga3c {

template <class TIn_, int C_, int H_, int W_, int OC_, int KS_, int S_>
struct ConvSpec {
    typedef TIn_ TIn;
    static constexpr int C = C_, H = H_, W = W_, OC = OC_, KS = KS_, S = S_;
    static constexpr int OH = (H - KS) / S + 1, OW = (W - KS) / S + 1;
    static constexpr int K = C * KS * KS, NPIX = OH * OW, CHW = C * H * W;
    static constexpr int NT = (NPIX + 15) / 16;      // pixel tiles per frame
    static constexpr int OT = OC / 16;               // filter tiles
    static_assert(OC % 16 == 0 && (OT == 1 || OT == 2 || OT == 4), "filter count must be 16, 32 or 64");
    static_assert(K % 16 == 0, "filter length must be a multiple of 16");
    // element offset inside a frame of filter tap k = (c, u, v)
    __host__ __device__ static constexpr int koff(int k) {
        return (k / (KS * KS)) * H * W + ((k / KS) % KS) * W + (k % KS);
    }
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

}  // namespace ga3c
