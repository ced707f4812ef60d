// Weight and bias gradient of a stride-1 convolution layer with 64 input
// channels (the third layer of the larger network) on the 16-bit matrix cores at
// fp32 accuracy:
//
//   dW[oc][c][u][v] = sum over frames and output pixels (i, j) of dY[oc][i][j] x[c][i+u][j+v]
//   db[oc]          = sum of dY[oc][i][j]
//
// The contraction runs over the output pixels of a frame, numbered on the
// input's grid: pixel (i, j) is k = i W + j, so that tap (u, v) meets the input
// plane read from index k + u W + v on.  dY goes to LDS as [oc][k] (columns OW
// .. W - 1 and the tail of the last group of 32 are zero) and the input as
// [c][k]; both operands of an MFMA are eight consecutive k, and all KS x KS
// shifts of a channel are cut from one 64-byte window of its plane: whole
// dwords for even shifts, a 16-bit funnel shift for odd ones.  Wavefront w owns
// the channels 16 w .. 16 w + 15: KS x KS taps x 2 filter tiles of accumulators
// [16 filters] x [16 channels], kept over all frames of its block.  The bias
// gradient is one more product, dY times a column of ones.  (With three bfloat16 terms, rows at the pitch of
// lds_row_units, and staging in 8-byte instead of 2-byte stores with one unaligned
// 16-byte load each gained nothing: 1280 frames 30.5 us, 31.1 with the latter.)
//
// Both operands are split into two float16 terms while they are staged, three
// products a sum, under scales for every channel and every filter, by the largest
// values that the block has met so far (split_f16.hpp, conv_wgrad_f16.hpp).  With three bfloat16 terms, six
// products, 1280 frames took 37.5 us instead of 29.7; error of dW in the 2-norm
// 1.27e-7 both (320 frames 1.42e-7 -> 1.40e-7).  There is no room for accumulators of the small products.
//
// A block takes 32 filters, 32 blockIdx.y .. (gridDim.y = OC / 32), of frames
// blockIdx.x, + gridDim.x, .. and writes its rows of one partial gradient,
// part[blockIdx.x][OC][K + 1] (the last column is the bias gradient), which a
// second kernel adds up in block order: no atomics, the result does not depend
// on timing.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include "split_f16.hpp"

namespace ga3c {

template <class SP>
struct ConvWgradS1Geom {
    static constexpr int MS = 2;                                   // filter tiles of 16 per block
    static constexpr int KTOT = (SP::OH - 1) * SP::W + SP::OW;     // k = i * W + j
    static constexpr int NKB = (KTOT + 31) / 32;                   // groups of 32 k
    static constexpr int DROW = NKB * 32 + 8;                      // elements per filter row of dY
    static constexpr int WIN = 32;                                 // elements of a plane row a lane reads per group and term
    static constexpr int SHIFT = (SP::KS - 1) * SP::W + SP::KS - 1;         // the largest shift
    static constexpr int PROW = ((NKB * 32 + WIN - 8) / 8) * 8 + 16;        // and per channel row of the input (52 dwords)
    static constexpr int DTERM = MS * 16 * DROW, PTERM = SP::C * PROW;      // elements per term
    static constexpr int OTP = SP::K + 4;                          // floats per filter row of a tile's result in LDS
    __host__ __device__ static constexpr int lds_bytes(bool one) {
        const int stage = (one ? 1 : 2) * (DTERM + PTERM) * 2, out = 16 * OTP * 4;
        return stage > out ? stage : out;
    }
};

// ONE: operands rounded to bfloat16 (the reduced-precision variant): one term, one product.
template <class SP, bool ONE>
__global__ __launch_bounds__(256, 2) void conv_wgrad_s1_f16_kernel(const float *__restrict__ x, const float *__restrict__ dy,
                                                                      float *__restrict__ part, int nframes, float scale) {
    typedef ConvWgradS1Geom<SP> G;
    static_assert(SP::S == 1 && SP::C == 64 && SP::OC % 32 == 0, "stride 1, 64 channels in (16 per wavefront), filters in groups of 32");
    static_assert(G::SHIFT + 8 <= G::WIN && G::NKB * 32 - 8 + G::WIN <= G::PROW, "the window holds every shift and stays in its row");
    static_assert(SP::H * SP::W <= G::PROW, "a plane fits its row");
    static_assert((G::DTERM % 8) == 0 && (G::PTERM % 8) == 0, "16-byte steps");
    static_assert((G::PROW / 2) % 8 == 4 && (G::DROW / 2) % 8 == 4, "rows of an odd number of 16-byte units");
    constexpr int MS = G::MS, NKB = G::NKB, DROW = G::DROW, PROW = G::PROW, KS = SP::KS, NTAP = KS * KS;
    constexpr int DTERM = G::DTERM, PTERM = G::PTERM, OTP = G::OTP, HW = SP::H * SP::W;
    constexpr int NTERM = ONE ? 1 : 2;
    typedef F16Rows<HW, SP::C, 256> RX;                                    // staging: channels of the input frame, my filters' dY
    typedef F16Rows<SP::NPIX, MS * 16, 256> RD;
    constexpr int XPT = RX::PER, DPT = RD::PER;
    constexpr int K1 = SP::K + 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t *dsm = (uint16_t *)smem;                  // [term][oc][DROW]
    uint16_t *psm = dsm + NTERM * DTERM;                 // [term][c][PROW]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int oc0 = blockIdx.y * MS * 16;

    for (int e = tid; e < NTERM * (DTERM + PTERM) / 8; e += 256) ((u32x4 *)smem)[e] = u32x4{0u, 0u, 0u, 0u};   // padding stays zero

    // staging descriptors: element -> its place in LDS (term 0)
    const int xrow = RX::row(tid), drow = RD::row(tid);
    int ddst[DPT][4];
#pragma unroll
    for (int i = 0; i < DPT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int pix = RD::at(tid, i) + j;
            ddst[i][j] = drow * DROW + (pix / SP::OW) * SP::W + pix % SP::OW;
        }

    floatx4 acc[NTAP][MS], bacc[MS];
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        bacc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NTAP; ++s) acc[s][m] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    constexpr uint32_t ONES = ONE ? 0x3F803F80u : 0x3C003C00u;
    const u32x4 ones{ONES, ONES, ONES, ONES};
    // exponents of the scales (channels, then filters), and how they have changed with this frame
    __shared__ __attribute__((aligned(16))) int scales[SP::C + MS * 16], steps[SP::C + MS * 16];
    int xe = F16_NO_SCALE, de = F16_NO_SCALE;          // of the channel and the filter that I stage

    typedef float f32x4_dword_aligned __attribute__((ext_vector_type(4), aligned(4)));
    f32x4_dword_aligned xpre[XPT], dpre[DPT];
    auto fetch = [&](int f) {
        const float *xs = x + (size_t)f * SP::CHW + xrow * HW;
#pragma unroll
        for (int i = 0; i < XPT; ++i) xpre[i] = *(const f32x4_dword_aligned *)(xs + RX::at(tid, i));
        const float *ds = dy + ((size_t)f * SP::OC + oc0 + drow) * SP::NPIX;
#pragma unroll
        for (int i = 0; i < DPT; ++i) dpre[i] = *(const f32x4_dword_aligned *)(ds + RD::at(tid, i));
    };
    auto stash4 = [&](const f32x4_dword_aligned v, float scale, uint16_t *base, int tstride, const int (&dst)[4]) {
        uint32_t t0[2], t1[2];
        split_terms<ONE>(v.x, v.y, scale, t0);
        split_terms<ONE>(v.z, v.w, scale, t1);
#pragma unroll
        for (int t = 0; t < NTERM; ++t) {
            base[t * tstride + dst[0]] = (uint16_t)(t0[t] & 0xffffu);
            base[t * tstride + dst[1]] = (uint16_t)(t0[t] >> 16);
            base[t * tstride + dst[2]] = (uint16_t)(t1[t] & 0xffffu);
            base[t * tstride + dst[3]] = (uint16_t)(t1[t] >> 16);
        }
    };
    int f = blockIdx.x;
    fetch(min(f, nframes - 1));
    for (; f < nframes; f += gridDim.x) {
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
            if (tid % RD::LANES == 0) { scales[SP::C + drow] = nd; steps[SP::C + drow] = nd - de; }
            xe = nx;
            de = nd;
        }
        const float xscale = f16_power(xe), dscale = f16_power(de);
#pragma unroll
        for (int i = 0; i < XPT; ++i)
            if (RX::there(tid, i)) {
                const int to = xrow * PROW + RX::at(tid, i);
                const int at[4] = {to, to + 1, to + 2, to + 3};
                stash4(xpre[i], xscale, psm, PTERM, at);
            }
#pragma unroll
        for (int i = 0; i < DPT; ++i)
            if (RD::there(tid, i)) stash4(dpre[i], dscale, dsm, DTERM, ddst[i]);
        __syncthreads();
        fetch(min(f + (int)gridDim.x, nframes - 1));
        // the loads above go out before the products start (the compiler would otherwise sink them below the MFMAs)
        __builtin_amdgcn_sched_barrier(0);
        if (!ONE && f != (int)blockIdx.x) {   // the sums so far come to the scales of the largest values so far
            int4 sd[MS];
            const int sx = steps[16 * wave + l16];
            int any = sx;
#pragma unroll
            for (int m = 0; m < MS; ++m) {
                sd[m] = *(const int4 *)(steps + SP::C + 16 * m + 4 * g);
                any |= sd[m].x | sd[m].y | sd[m].z | sd[m].w;
            }
            if (__any(any != 0)) {
#pragma unroll
                for (int m = 0; m < MS; ++m) {
                    f16_ldexp4(bacc[m], sd[m], 0);
#pragma unroll
                    for (int s = 0; s < NTAP; ++s) f16_ldexp4(acc[s][m], sd[m], sx);
                }
            }
        }
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            u32x4 a[MS][NTERM];
            uint32_t dw[NTERM][16];
#pragma unroll
            for (int m = 0; m < MS; ++m)
#pragma unroll
                for (int t = 0; t < NTERM; ++t)
                    a[m][t] = *(const u32x4 *)(dsm + t * DTERM + (m * 16 + l16) * DROW + 32 * kb + 8 * g);
#pragma unroll
            for (int t = 0; t < NTERM; ++t) {
                const u32x4 *src = (const u32x4 *)(psm + t * PTERM + (wave * 16 + l16) * PROW + 32 * kb + 8 * g);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u32x4 w = src[q];
                    dw[t][4 * q] = w[0]; dw[t][4 * q + 1] = w[1]; dw[t][4 * q + 2] = w[2]; dw[t][4 * q + 3] = w[3];
                }
            }
            if (kb % 4 == wave) {             // bias, smallest first
#pragma unroll
                for (int t = NTERM - 1; t >= 0; --t)
#pragma unroll
                    for (int m = 0; m < MS; ++m)
                        bacc[m] = mfma_terms<ONE>(a[m][t], ones, bacc[m]);
            }
            // one row of taps at a time: KS shifts x MS filter tiles of independent accumulators
#pragma unroll
            for (int u = 0; u < KS; ++u) {
                u32x4 b[KS][NTERM];
#pragma unroll
                for (int v = 0; v < KS; ++v) {
                    const int sh = u * SP::W + v, o = sh / 2;
#pragma unroll
                    for (int t = 0; t < NTERM; ++t) {
                        if (sh % 2 == 0)
                            b[v][t] = u32x4{dw[t][o], dw[t][o + 1], dw[t][o + 2], dw[t][o + 3]};
                        else
                            b[v][t] = u32x4{__builtin_amdgcn_alignbit(dw[t][o + 1], dw[t][o], 16), __builtin_amdgcn_alignbit(dw[t][o + 2], dw[t][o + 1], 16),
                                              __builtin_amdgcn_alignbit(dw[t][o + 3], dw[t][o + 2], 16), __builtin_amdgcn_alignbit(dw[t][o + 4], dw[t][o + 3], 16)};
                    }
                }
#pragma unroll
                for (int q = 0; q < F16_PRODUCTS<ONE>; ++q)
#pragma unroll
                    for (int v = 0; v < KS; ++v)
#pragma unroll
                        for (int m = 0; m < MS; ++m)
                            acc[u * KS + v][m] = mfma_terms<ONE>(a[m][f16_a_term<ONE>(q)], b[v][f16_b_term<ONE>(q)], acc[u * KS + v][m]);
            }
        }
        __builtin_amdgcn_s_setprio(0);
    }
    if constexpr (!ONE) {
        const int sx = 127 - scales[16 * wave + l16];
#pragma unroll
        for (int m = 0; m < MS; ++m) {
            const int4 e = *(const int4 *)(scales + SP::C + 16 * m + 4 * g), back{127 - e.x, 127 - e.y, 127 - e.z, 127 - e.w};
            f16_ldexp4(bacc[m], back, 0);
#pragma unroll
            for (int s = 0; s < NTAP; ++s) f16_ldexp4(acc[s][m], back, sx);
        }
    }
    // lane (l16, g), register r of acc[tap][m]: filter oc0 + 16 m + 4 g + r, channel 16 wave + l16.  One filter tile at a
    // time is put together in LDS and leaves in rows.
    __shared__ float bsh[4][MS * 16];                  // bias sums of the four wavefronts
    float *ot = (float *)smem;                         // [16 filters][OTP]
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        __syncthreads();
        if (l16 == 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) bsh[wave][m * 16 + 4 * g + r] = bacc[m][r];
        }
#pragma unroll
        for (int s = 0; s < NTAP; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r) ot[(4 * g + r) * OTP + (wave * 16 + l16) * NTAP + s] = acc[s][m][r];
        __syncthreads();
        float *pb = part + ((size_t)blockIdx.x * SP::OC + oc0 + m * 16) * K1;
        for (int it = tid; it < 16 * (SP::K / 4); it += 256) {
            const int oc = it / (SP::K / 4), kq = it % (SP::K / 4);
            const float4 v = *(const float4 *)(ot + oc * OTP + 4 * kq);
            *(f32x4_dword_aligned *)(pb + (size_t)oc * K1 + 4 * kq) = f32x4_dword_aligned{v.x * scale, v.y * scale, v.z * scale, v.w * scale};
        }
    }
    if (tid < MS * 16)
        part[((size_t)blockIdx.x * SP::OC + oc0 + tid) * K1 + SP::K] = (bsh[0][tid] + bsh[1][tid]) + (bsh[2][tid] + bsh[3][tid]);
}

// One partial dW per block: fewer blocks where a partial is large.
template <class SP>
inline int conv_wgrad_s1_f16_blocks(int nframes) {
    constexpr int LIMIT = SP::OC * (SP::K + 1) > 16384 ? 256 : 512;
    return nframes < LIMIT ? nframes : LIMIT;
}

// x: [n][C][H][W] and dy: [n][OC][OH][OW], both 16-byte aligned; part: [conv_wgrad_s1_f16_blocks(n)][OC][K + 1].
template <class SP>
inline hipError_t launch_conv_wgrad_s1_f16(const float *x, const float *dy, float *part, int nframes, float scale,
                                              hipStream_t s, int rb = 0) {
    if (nframes <= 0) return hipSuccess;
    typedef ConvWgradS1Geom<SP> G;
    static bool attr_set = false;          // once per layer shape: let the kernels use more than 64 KB of LDS
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)conv_wgrad_s1_f16_kernel<SP, false>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, G::lds_bytes(false));
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)conv_wgrad_s1_f16_kernel<SP, true>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, G::lds_bytes(true));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const dim3 grid(conv_wgrad_s1_f16_blocks<SP>(nframes), SP::OC / 32);
    if (rb)
        ga3c::launch((conv_wgrad_s1_f16_kernel<SP, true>), grid, dim3(256), G::lds_bytes(true), s, x, dy, part, nframes, scale);
    else
        ga3c::launch((conv_wgrad_s1_f16_kernel<SP, false>), grid, dim3(256), G::lds_bytes(false), s, x, dy, part, nframes, scale);
    return hipGetLastError();
}

}  // namespace ga3c
