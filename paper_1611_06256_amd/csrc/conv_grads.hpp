// Both gradients of a 4x4 stride-2 convolution layer in one launch.  They read
// the same dY and neither needs the other.  The input gradient's blocks come
// first (the layer below waits for them); the weight gradient's take the compute
// units those leave idle, all of them at small batches, the end of the launch at
// large ones.  Two launches against one, us of an update: small net 5 frames 70.8 /
// 64.9, 40: 75.4 / 69.6, 640: 124.0 / 119.3, 2560: 270.2 / 265.9; larger net 5: 148.1 /
// 140.6, 640: 344.3 / 333.2, 1280: 505 / 508; stride-4 member 640: 243.1 / 236.9.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include <algorithm>

#include "conv_dgrad_bf16x6.hpp"
#include "conv_wgrad_f16.hpp"

namespace ga3c {

template <class SP, bool ONE, int OCB>
__global__ __launch_bounds__(256, 2) void conv_grads_kernel(const float *__restrict__ x, const float *__restrict__ dy,
                                                                   const float *__restrict__ w, const u32x4 *__restrict__ wfrag,
                                                                   float *__restrict__ dx, float *__restrict__ part, int nframes,
                                                                   int nbd, int nbw) {
    constexpr int SLICES = SP::C / 16;
    int b = blockIdx.x, slice = 0;
    if (b < nbd * SLICES) {
        for (; b >= nbd; b -= nbd) ++slice;
        conv_dgrad_bf16x6_block<SP, ONE>(dy, w, x, dx, nframes, wfrag, b, slice, nbd);
        return;
    }
    for (b -= nbd * SLICES; b >= nbw; b -= nbw) ++slice;
    conv_wgrad_f16_block<SP, ONE, OCB>(x, dy, part, nframes, 1.f, b, slice % SLICES, slice / SLICES, nbw);
}

// x [n][C][H][W] (the layer's input, and the ReLU mask of dx), dy [n][OC][OH][OW], w the filters, wfrag their fragments for the
// input gradient or nullptr; all 16-byte aligned.  part: [conv_wgrad_f16_blocks(n)][OC][K + 1].
template <class SP, int OCB = SP::OC>
inline hipError_t launch_conv_grads(const float *x, const float *dy, const float *w, const u32x4 *wfrag, float *dx, float *part,
                                           int nframes, hipStream_t s, int rb) {
    if (nframes <= 0) return hipSuccess;
    constexpr int SLICES = SP::C / 16;
    // As few blocks as take the same number of frames each at most: the weight gradient's start the earlier.  16 channels: half of the 512
    // places each, so that all blocks start at once; 32: the weight gradient's blocks (four to a partial sum) follow the input gradient's.
    // us an update by places / partial sums, small net 2560 frames 512 / 512: 235, 512 / 256: 238, 384 / 256: 236, 256 / 256: 220; 640: 103, 102,
    // 102, 98; larger net 1280 frames 512 / 256: 413, 512 / 128: 402, 384 / 128: 406; stride-4 member 640: 512 / 256: 189.9, 512 / 128: 188.8.
    constexpr int PLACES = SP::C == 16 ? 256 : 512;
    const int per = (nframes * SLICES + PLACES - 1) / PLACES, nbd = (nframes + per - 1) / per, nbw = conv_wgrad_f16_blocks<SP>(nframes);
    auto lds = [](bool one) { return std::max(ConvDgradBf16Geom<SP>::lds_bytes(one), ConvWgradGeom<SP, OCB>::lds_bytes(one)); };
    static bool attr_set = false;          // once per layer shape: let the kernels use more than 64 KB of LDS
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)conv_grads_kernel<SP, false, OCB>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds(false));
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)conv_grads_kernel<SP, true, OCB>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, lds(true));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const dim3 grid(nbd * SLICES + nbw * SLICES * (SP::OC / OCB));
    if (rb) ga3c::launch((conv_grads_kernel<SP, true, OCB>), grid, dim3(256), lds(true), s, x, dy, w, wfrag, dx, part, nframes, nbd, nbw);
    else ga3c::launch((conv_grads_kernel<SP, false, OCB>), grid, dim3(256), lds(false), s, x, dy, w, wfrag, dx, part, nframes, nbd, nbw);
    return hipGetLastError();
}

}  // namespace ga3c
