// Weight and bias gradient of a 4x4, stride-2 convolution layer on the 16-bit
// matrix cores at fp32 accuracy (backward pass of the network of Sec. 3.2; the
// layer is the second convolution of both networks):
//
//   dW[oc][c][u][v] = sum over frames and output pixels (i, j) of dY[oc][i][j] x[c][2i+u][2j+v]
//   db[oc]          = sum of dY[oc][i][j]
//
// The contraction runs over the output pixels of a frame.  The input falls
// into 2 x 2 stride phases P[ry][rx][c][y'][x'] = x[c][2y'+ry][2x'+rx], and
// with u = ry + 2a, v = rx + 2e the tap (u, v) meets P[ry][rx][c][i+a][j+e]:
// on the phase grid (GW = W / 2 wide) pixel (i, j) is index k = i GW + j, and
// the tap's operand is the phase plane read from index k + a GW + e on.  So
// dY goes to LDS as [oc][k] (column GW - 1 and the tail of the last group of
// 32 are zero) and every phase plane as [c][k]; both operands of an MFMA are
// eight consecutive k, and the four shifts (a, e) of a phase are cut from one
// 48-byte window of the plane: whole dwords for e = 0, a 16-bit funnel shift
// for e = 1.  Wavefront w owns phase w: 4 shifts x OC / 16 filter tiles of
// accumulators [16 filters] x [16 channels], kept over all frames of its block.
// The bias gradient is one more product, dY times a column of ones, which the
// wavefronts of channel slice 0 share by groups of 32 k.
//
// Both operands are split into two float16 terms while they are staged, three
// products a sum (split_f16.hpp); the two small ones have accumulators of their
// own.  Every channel and every filter has a scale, by the largest values that
// the block has met in it so far; where a frame brings larger ones, the sums so
// far are brought to the new scale.  So a value of 2^-15 of the largest one that
// goes into the same sums still has its 22 bits, and what is smaller an error of
// 2^-37 of that one.  The lanes that stage a channel or a filter are neighbours
// and find its largest value between themselves.  (One scale for all channels and
// one for all filters took the bits of those far smaller than another, and cost
// an exchange between the wavefronts: the same time.)  Three bfloat16 terms, six
// products, operands of the next group read ahead, against two, error of dW in the 2-norm: small net 40
// frames 1.45e-7 -> 1.34e-7, 2560: 1.8e-7 -> 1.1e-7, larger net 1280: 1.8e-7 -> 1.1e-7
// (with one accumulator 1.6e-7, 1.6e-7 and 1.9e-7).
//
// A block takes 16 input channels, 16 by .. (C / 16 slices), and
// OCB filters, OCB bz .. (all of them, or 32 where two blocks then fit
// a compute unit's LDS), of
// frames bx, + nbx, .. and writes its part of one partial gradient,
// part[bx][OC][K + 1] (K = 16 C; the last column is the bias gradient,
// written by the blocks of channel slice 0), which a second kernel adds up in
// block order: no atomics, the result does not depend on timing.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include "split_f16.hpp"

namespace ga3c {

// OCB: filters per block (a multiple of 16; bz takes the slices of OCB filters)
template <class SP, int OCB = SP::OC>
struct ConvWgradGeom {
    static constexpr int CS = 16;
    static constexpr int GH = SP::H / 2, GW = SP::W / 2;
    static constexpr int KTOT = SP::OH * GW;                       // k = i * GW + j
    static constexpr int NKB = (KTOT + 31) / 32;                   // groups of 32 k
    static constexpr int DROW = 8 * lds_row_units(NKB * 4);        // elements per filter row of dY
    static constexpr int WIN = 24;                                 // elements of a plane row a lane reads per group and term
    static constexpr int PROW = 8 * lds_row_units((NKB * 32 - 8 + WIN) / 8);      // and per channel row of a phase plane
    static constexpr int MT = OCB / 16;
    static constexpr int DTERM = OCB * DROW, PTERM = 4 * CS * PROW;         // elements per term
    static constexpr int OTP = CS * 16 + 4;                        // floats per filter row of the block's result in LDS
    __host__ __device__ static constexpr int lds_bytes(bool one) {
        const int stage = (one ? 1 : 2) * (DTERM + PTERM) * 2, out = OCB * OTP * 4;
        return stage > out ? stage : out;
    }
    static constexpr int PER_CU = 2 * lds_bytes(false) <= 160 * 1024 ? 2 : 1;
};

// ONE: operands rounded to bfloat16 (the reduced-precision variant): one term, one product.
template <class SP, bool ONE, int OCB = SP::OC>
__device__ __forceinline__ void conv_wgrad_f16_block(const float *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part,
                                                        int nframes, float scale, const int bx, const int by, const int bz, const int nbx) {
    typedef ConvWgradGeom<SP, OCB> G;
    static_assert(SP::OC % OCB == 0 && OCB % 16 == 0, "whole slices of filters");
    static_assert(SP::KS == 4 && SP::S == 2, "kernel must be 4x4 with stride 2");
    static_assert(SP::C % 16 == 0 && SP::OC % 16 == 0 && SP::OC <= 256, "channels and filters in groups of 16");
    static_assert(SP::H % 2 == 0 && SP::W % 4 == 0 && G::GW % 2 == 0, "rows are read four values at a time; shifts are whole dwords");
    static_assert(G::GW + 9 <= G::WIN, "the window must hold the largest shift plus eight elements");
    static_assert(SP::OW + 1 <= G::GW && SP::OH + 1 <= G::GH, "shifted pixels must stay on the phase grid");
    static_assert((G::DTERM % 8) == 0 && (G::PTERM % 8) == 0, "16-byte steps");
    constexpr int CS = G::CS, GW = G::GW, NKB = G::NKB, DROW = G::DROW, PROW = G::PROW, MT = G::MT;
    constexpr int DTERM = G::DTERM, PTERM = G::PTERM, OTP = G::OTP;
    constexpr int NTERM = ONE ? 1 : 2;
    typedef F16Rows<SP::H * SP::W, CS, 256> RX;        // staging: channels of the input slice, my filters' dY
    typedef F16Rows<SP::NPIX, OCB, 256> RD;
    constexpr int W4 = SP::W / 4, XPT = RX::PER, DPT = RD::PER;
    constexpr int K1 = SP::K + 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t *dsm = (uint16_t *)smem;                  // [term][oc][DROW]
    uint16_t *psm = dsm + NTERM * DTERM;                 // [term][phase][c][PROW]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int ry = wave / 2, rx = wave % 2;
    const int c0 = by * CS, oc0 = bz * OCB;

    for (int e = tid; e < NTERM * (DTERM + PTERM) / 8; e += 256) ((u32x4 *)smem)[e] = u32x4{0u, 0u, 0u, 0u};   // padding stays zero

    // staging descriptors.  Input: float4 item -> (c, y, x = 4q..4q+3): x, x+2 are neighbours in phase column 0 and
    // x+1, x+3 in phase column 1 of phase row y % 2.
    const int xrow = RX::row(tid), drow = RD::row(tid);
    int xdst[XPT];
#pragma unroll
    for (int i = 0; i < XPT; ++i) {
        const int y = RX::at(tid, i) / SP::W, q = RX::at(tid, i) % SP::W / 4;
        xdst[i] = ((y % 2) * 2 * CS + xrow) * PROW + (y / 2) * GW + 2 * q;
    }
    int ddst[DPT][4];
#pragma unroll
    for (int i = 0; i < DPT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int pix = RD::at(tid, i) + j;
            ddst[i][j] = drow * DROW + (pix / SP::OW) * GW + pix % SP::OW;
        }

    constexpr bool LOW = !ONE;                         // small products have sums of their own
    floatx4 acc[4][MT], low[4][LOW ? MT : 1];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[s][m] = low[s][LOW ? m : 0] = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4 bacc[MT];                                  // dY times ones: every column holds the row sums
#pragma unroll
    for (int m = 0; m < MT; ++m) bacc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    constexpr uint32_t ONES = ONE ? 0x3F803F80u : 0x3C003C00u;
    const u32x4 ones{ONES, ONES, ONES, ONES};
    // exponents of the scales (channels, then filters), and how they have changed with this frame
    __shared__ __attribute__((aligned(16))) int scales[CS + OCB], steps[CS + OCB];
    int xe = F16_NO_SCALE, de = F16_NO_SCALE;          // of the channel and the filter that I stage

    typedef float f32x4_dword_aligned __attribute__((ext_vector_type(4), aligned(4)));
    f32x4_dword_aligned xpre[XPT], dpre[DPT];
    auto fetch = [&](int f) {
        const float *xs = x + (size_t)f * SP::CHW + (size_t)(c0 + xrow) * (SP::H * SP::W);
#pragma unroll
        for (int i = 0; i < XPT; ++i) xpre[i] = *(const f32x4_dword_aligned *)(xs + RX::at(tid, i));
        const float *ds = dy + ((size_t)f * SP::OC + oc0 + drow) * SP::NPIX;
#pragma unroll
        for (int i = 0; i < DPT; ++i) dpre[i] = *(const f32x4_dword_aligned *)(ds + RD::at(tid, i));
    };
    int f = bx;
    fetch(min(f, nframes - 1));
    for (; f < nframes; f += nbx) {
        __syncthreads();                      // the last frame's operands have been read
        if constexpr (!ONE) {
            auto four = [](const f32x4_dword_aligned v, const auto &fold) { fold(v.x); fold(v.y); fold(v.z); fold(v.w); };
            const int nx = f16_row_exponent<RX::LANES>(xe, [&](const auto &fold) {
#pragma unroll
                for (int i = 0; i < XPT; ++i) four(xpre[i], fold);
            });
            const int nd = f16_row_exponent<RD::LANES>(de, [&](const auto &fold) {
#pragma unroll
                for (int i = 0; i < DPT; ++i) four(dpre[i], fold);
            });
            if (tid % RX::LANES == 0) { scales[xrow] = nx; steps[xrow] = nx - xe; }
            if (tid % RD::LANES == 0) { scales[CS + drow] = nd; steps[CS + drow] = nd - de; }
            xe = nx;
            de = nd;
        }
        const float xscale = f16_power(xe), dscale = f16_power(de);
#pragma unroll
        for (int i = 0; i < XPT; ++i)
            if (RX::there(tid, i)) {
                uint32_t t0[2], t1[2];
                split_terms<ONE>(xpre[i].x, xpre[i].z, xscale, t0);
                split_terms<ONE>(xpre[i].y, xpre[i].w, xscale, t1);
#pragma unroll
                for (int t = 0; t < NTERM; ++t) {
                    *(uint32_t *)(psm + t * PTERM + xdst[i]) = t0[t];
                    *(uint32_t *)(psm + t * PTERM + xdst[i] + CS * PROW) = t1[t];
                }
            }
#pragma unroll
        for (int i = 0; i < DPT; ++i)
            if (RD::there(tid, i)) {
                uint32_t t0[2], t1[2];
                split_terms<ONE>(dpre[i].x, dpre[i].y, dscale, t0);
                split_terms<ONE>(dpre[i].z, dpre[i].w, dscale, t1);
                uint16_t *dst = (uint16_t *)dsm;
#pragma unroll
                for (int t = 0; t < NTERM; ++t) {
                    dst[t * DTERM + ddst[i][0]] = (uint16_t)(t0[t] & 0xffffu);
                    dst[t * DTERM + ddst[i][1]] = (uint16_t)(t0[t] >> 16);
                    dst[t * DTERM + ddst[i][2]] = (uint16_t)(t1[t] & 0xffffu);
                    dst[t * DTERM + ddst[i][3]] = (uint16_t)(t1[t] >> 16);
                }
            }
        __syncthreads();
        fetch(min(f + nbx, nframes - 1));
        // the loads above go out before the products start (the compiler would otherwise sink them below the MFMAs)
        __builtin_amdgcn_sched_barrier(0);
        if (!ONE && f != bx) {                // the sums so far come to the scales of the largest values so far
            int4 sd[MT];
            const int sx = steps[l16];
            int any = sx;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                sd[m] = *(const int4 *)(steps + CS + 16 * m + 4 * g);
                any |= sd[m].x | sd[m].y | sd[m].z | sd[m].w;
            }
            if (__any(any != 0)) {
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    f16_ldexp4(bacc[m], sd[m], 0);
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        f16_ldexp4(acc[s][m], sd[m], sx);
                        if (LOW) f16_ldexp4(low[s][LOW ? m : 0], sd[m], sx);
                    }
                }
            }
        }
        u32x4 a[MT][NTERM], win[NTERM][3];
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < NTERM; ++t) a[m][t] = *(const u32x4 *)(dsm + t * DTERM + (m * 16 + l16) * DROW + 32 * kb + 8 * g);
#pragma unroll
            for (int t = 0; t < NTERM; ++t) {
                const u32x4 *src = (const u32x4 *)(psm + t * PTERM + (wave * CS + l16) * PROW + 32 * kb + 8 * g);
                win[t][0] = src[0]; win[t][1] = src[1]; win[t][2] = src[2];
            }
            u32x4 b[4][NTERM];
#pragma unroll
            for (int t = 0; t < NTERM; ++t) {
                const u32x4 w0 = win[t][0], w1 = win[t][1], w2 = win[t][2];
                const uint32_t dw[12] = {w0[0], w0[1], w0[2], w0[3], w1[0], w1[1], w1[2], w1[3], w2[0], w2[1], w2[2], w2[3]};
#pragma unroll
                for (int av = 0; av < 2; ++av) {
                    const int o = av * (GW / 2);          // a shift of a rows of the phase grid is GW / 2 dwords
                    b[2 * av][t] = u32x4{dw[o], dw[o + 1], dw[o + 2], dw[o + 3]};
                    b[2 * av + 1][t] = u32x4{__builtin_amdgcn_alignbit(dw[o + 1], dw[o], 16), __builtin_amdgcn_alignbit(dw[o + 2], dw[o + 1], 16),
                                             __builtin_amdgcn_alignbit(dw[o + 3], dw[o + 2], 16), __builtin_amdgcn_alignbit(dw[o + 4], dw[o + 3], 16)};
                }
            }
            if (by == 0 && kb % 4 == wave) {      // bias, smallest first
#pragma unroll
                for (int t = NTERM - 1; t >= 0; --t)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        bacc[m] = mfma_terms<ONE>(a[m][t], ones, bacc[m]);
            }
#pragma unroll
            for (int q = 0; q < F16_PRODUCTS<ONE>; ++q)
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        floatx4 &sum = LOW && q < 2 ? low[s][LOW ? m : 0] : acc[s][m];
                        sum = mfma_terms<ONE>(a[m][f16_a_term<ONE>(q)], b[s][f16_b_term<ONE>(q)], sum);
                    }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    }
    if constexpr (!ONE) {
        const int sx = 127 - scales[l16];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int4 e = *(const int4 *)(scales + CS + 16 * m + 4 * g), back{127 - e.x, 127 - e.y, 127 - e.z, 127 - e.w};
            f16_ldexp4(bacc[m], back, 0);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (LOW) acc[s][m] += low[s][LOW ? m : 0];
                f16_ldexp4(acc[s][m], back, sx);
            }
        }
    }
    // lane (l16, g), register r of acc[s = 2a + e][m]: filter 16 m + 4 g + r, channel c0 + l16, tap (ry + 2a, rx + 2e).
    // The block's result is put together in LDS and leaves in rows.
    __syncthreads();
    float *ot = (float *)smem;                         // [oc][OTP]
    __shared__ float bsh[4][OCB];                      // bias sums of the four wavefronts
    if (l16 == 0) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) bsh[wave][m * 16 + 4 * g + r] = bacc[m][r];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int u = ry + 2 * (s / 2), v = rx + 2 * (s % 2);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) ot[(m * 16 + 4 * g + r) * OTP + l16 * 16 + u * 4 + v] = acc[s][m][r];
    }
    __syncthreads();
    float *pb = part + ((size_t)bx * SP::OC + oc0) * K1 + c0 * 16;
    for (int it = tid; it < OCB * CS * 4; it += 256) {
        const int oc = it / (CS * 4), kq = it % (CS * 4);
        const float4 v = *(const float4 *)(ot + oc * OTP + 4 * kq);
        *(f32x4_dword_aligned *)(pb + (size_t)oc * K1 + 4 * kq) = f32x4_dword_aligned{v.x * scale, v.y * scale, v.z * scale, v.w * scale};
    }
    if (by == 0 && tid < OCB)
        part[((size_t)bx * SP::OC + oc0 + tid) * K1 + SP::K] = (bsh[0][tid] + bsh[1][tid]) + (bsh[2][tid] + bsh[3][tid]);
}
template <class SP, bool ONE, int OCB = SP::OC>
__global__ __launch_bounds__(256, (ConvWgradGeom<SP, OCB>::PER_CU)) void conv_wgrad_f16_kernel(const float *__restrict__ x,
                                                                                              const float *__restrict__ dy,
                                                                                              float *__restrict__ part,
                                                                                              int nframes, float scale) {
    conv_wgrad_f16_block<SP, ONE, OCB>(x, dy, part, nframes, scale, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.x);
}

// One partial dW per block.  They are written, read and added up again, so there are no more of them than it takes to fill the
// chip beside the input gradient's blocks (conv_grads.hpp).
template <class SP>
inline int conv_wgrad_f16_blocks(int nframes) {
    constexpr int LIMIT = SP::C == 16 ? 256 : 128;
    return nframes < LIMIT ? nframes : LIMIT;
}

// x: [n][C][H][W] and dy: [n][OC][OH][OW], both 16-byte aligned; part: [conv_wgrad_f16_blocks(n)][OC][K + 1].
template <class SP, int OCB = SP::OC>
inline hipError_t launch_conv_wgrad_f16(const float *x, const float *dy, float *part, int nframes, float scale,
                                           hipStream_t s, int rb = 0) {
    if (nframes <= 0) return hipSuccess;
    typedef ConvWgradGeom<SP, OCB> G;
    static bool attr_set = false;          // once per layer shape: let the kernels use more than 64 KB of LDS
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)conv_wgrad_f16_kernel<SP, false, OCB>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, G::lds_bytes(false));
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)conv_wgrad_f16_kernel<SP, true, OCB>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, G::lds_bytes(true));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const dim3 grid(conv_wgrad_f16_blocks<SP>(nframes), SP::C / 16, SP::OC / OCB);
    if (rb)
        ga3c::launch((conv_wgrad_f16_kernel<SP, true, OCB>), grid, dim3(256), G::lds_bytes(true), s, x, dy, part, nframes, scale);
    else
        ga3c::launch((conv_wgrad_f16_kernel<SP, false, OCB>), grid, dim3(256), G::lds_bytes(false), s, x, dy, part, nframes, scale);
    return hipGetLastError();
}

}  // namespace ga3c
