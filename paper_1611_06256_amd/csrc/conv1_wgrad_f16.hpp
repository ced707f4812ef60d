// Weight and bias gradient of the first convolution layer (8x8 filters, stride 4, on 4x84x84 byte frames) on the 16-bit
// matrix cores at fp32 accuracy:
//   dW[oc][c][u][v] = sum_{i,j} dY[oc][i][j] x[c][4i+u][4j+v],   db[oc] = sum dY[oc][i][j]
// A byte is exact in float16, and dY is split into two float16 terms, every filter's under the scale of the largest values that the block
// has met in it so far (split_f16.hpp, conv_wgrad_f16.hpp): two products a sum.  Rounded operands (ONE) are one bfloat16 term, and the
// bytes bfloat16 as well.
//
// The contraction runs over output pixels, 8 consecutive pixels of a row per
// lane, so the frame is re-laid in LDS "space to depth": with u = 4a + u',
// v = 4b + v' the pixel x[c][4i+u][4j+v] is X[(c,u',v')][i+a][j+b], and 8
// consecutive j are 8 consecutive elements of a row of plane (c,u',v').  Plane
// index q = (c,u',v') is the column of the MFMA tile (a wavefront has a channel's
// 16 planes), the filters are the rows, and the four (a,b) are four
// accumulators per 16 filters.  Shift b = 1 is made from the b = 0 vector and one more dword.
// Rows of 20 pixels are padded to 24 = 3 blocks of 8 with zero dY.
// part: [gridDim.x][OCT][257]; the last column is the bias gradient.  A block takes OC of the layer's OCT filters
// (blockIdx.y): all 32 where a slice of 16 per block would not find a compute unit of its own.
// Vector instructions and LDS traffic of the staging, the LDS reads and the matrix instructions bound it, one after the other: one block
// fills a compute unit's LDS.  By kernel trace, with three bfloat16 terms of dY and a slice of 16 filters per block before: 2560 frames of
// 16 filters 40.2 -> 38.2 us, 40 frames 7.6 -> 7.0, 1280 frames of 32 filters 44.9 -> 35.3, rounded 35.1 -> 26.6.  dW is as far from
// 64 bits as before (2560 frames 1.27e-7 -> 1.16e-7, 1280 of 32 filters 1.35e-7 -> 1.28e-7).  The loop over pixel blocks is not
// unrolled: unrolled, 32 filters spill 50 registers.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include <type_traits>

#include "split_f16.hpp"

namespace ga3c {

template <int OCT, int OC, bool TABLE, bool ONE>
__global__ __launch_bounds__(1024) void conv1_wgrad_kernel(const uint8_t *__restrict__ x, const uint8_t *const *__restrict__ table,
                                                           const float *__restrict__ dy, float *__restrict__ part, int nframes, float scale) {
    // ONE: dY enters the products (and the bias sums) rounded to bfloat16
    constexpr int C = 4, H = 84, W = 84, OH = 20, NPIX = 400, K = 256, CHW = C * H * W;
    // 16-bit elements.  Blocks of 8 pixels are consecutive units of 16 bytes, in the planes as in dY; dY's filters lie at a pitch
    // of lds_row_units.  A plane (c, u', v') lies 4 u' + {0, 2, 8, 10}[v'] (mod 16) units behind a multiple of 256 bytes: even
    // places that differ within {0-3, 12-15} and within {4-11}, as lds_row_units wants them, and the four u' that a store
    // instruction meets are 64 bytes apart.
    constexpr int XROW = 24, XPLANE = 80 * 8, XALL = 64 * XPLANE + 16 * 8;
    constexpr int DROW = 24, DOC = 8 * lds_row_units(OH * 3);
    constexpr int NTERM = ONE ? 1 : 2, MT = OC / 16;
    constexpr int NPART = 4, NTHR = 256 * NPART;           // NPART wavefronts per SIMD, so that one's LDS and
                                                           // staging work fills another's MFMA waits
    constexpr int NITEM = 336 * 6, IPT = (NITEM + NTHR - 1) / NTHR;    // (frame row, group of 4 dwords)
    typedef F16Rows<NPIX, OC, NTHR> RD;                    // staging: my filters' dY
    constexpr int NDV = OC * NPIX / 4, DPT = RD::PER;      // float4 of dY per frame
    constexpr int NSTEP = OH * 3 / 4;                      // 60 blocks of 8 pixels, 4 per MFMA
    constexpr int XCH = (NPART - 1) * 4 * MT * 16 * 64;    // floats: sums that three of the four parts hand over
    static_assert(OCT % OC == 0 && OC % 16 == 0 && 16 * OC <= NTHR, "whole tiles of 16 filters, 16 lanes for each one's bias");
    constexpr int STAGE_BYTES = (XALL + NTERM * OC * DOC) * 2, SMEM = STAGE_BYTES > 4 * XCH ? STAGE_BYTES : 4 * XCH;
    __shared__ __attribute__((aligned(16))) uint16_t xp[SMEM / 2];
    __shared__ float bsh[NDV];
    // exponents of the filters' scales, and how they have changed with this frame
    __shared__ __attribute__((aligned(16))) int scales[OC], steps[OC];
    uint16_t *dp = xp + XALL;                              // [term][filter][DOC]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int oc0 = blockIdx.y * OC;                       // my slice of the filters

    for (int e = tid; e < STAGE_BYTES / 4; e += NTHR) ((uint32_t *)xp)[e] = 0u;     // padding stays zero

    // staging descriptors: where my dwords come from and where they go.  A row of 21 dwords is five groups of four
    // and a last group of one; that one is fetched as the last of the row's dwords 17..20, so that every fetch is one
    // 16-byte load (4-byte aligned) that stays inside the frame.
    int xsrc[IPT], xdst[IPT], xup[IPT], xcnt[IPT];       // xup: where v' = 2 lies, from v' = 0
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int it = min(tid + NTHR * i, NITEM - 1);
        const int row = it / 6, gq = it % 6;               // row = c*84 + r
        const int c = row / H, r = row % H;
        xsrc[i] = row * (W / 4) + (gq == 5 ? 17 : 4 * gq); // dword index in the frame
        xcnt[i] = (tid + NTHR * i < NITEM) ? (gq == 5 ? 1 : 4) : 0;
        xdst[i] = ((c * 4 + r % 4) * 4) * XPLANE + 4 * (r % 4) * 8 + (r / 4) * XROW + 4 * gq;   // plane (c, u'=r%4, v'=0)
        xup[i] = 2 * XPLANE + (r % 4 < 2 ? 64 : -64);
    }
    const int drow = RD::row(tid);
    int ddst[DPT];
#pragma unroll
    for (int i = 0; i < DPT; ++i) ddst[i] = drow * DOC + RD::at(tid, i) / OH * DROW + RD::at(tid, i) % OH;       // 5 float4 per row of 20

    floatx4 acc[MT][2][2];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[m][a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    int exponent = F16_NO_SCALE;                           // of the filter that I stage

    typedef uint32_t u32x4_dword_aligned __attribute__((ext_vector_type(4), aligned(4)));
    u32x4 xpre[IPT];
    float4 dpre[DPT];
    auto fetch = [&](const uint8_t *at, int ff) {
        const uint32_t *xs = (const uint32_t *)at;
#pragma unroll
        for (int i = 0; i < IPT; ++i) xpre[i] = *(const u32x4_dword_aligned *)(xs + xsrc[i]);
        const float *ds = dy + ((size_t)ff * OCT + oc0 + drow) * NPIX;
#pragma unroll
        for (int i = 0; i < DPT; ++i) dpre[i] = *(const float4 *)(ds + RD::at(tid, i));
    };
    int f = blockIdx.x;
    FramePointer<TABLE> next;
    next.ask(x, table, min(f, nframes - 1), CHW);
    fetch(next.get(), min(f, nframes - 1));
    if (TABLE) next.ask(x, table, min(f + (int)gridDim.x, nframes - 1), CHW);
    const int ch = wave & 3, prt = wave >> 2;        // wavefronts w, w + 4, ... share channel w and divide the pixel blocks
    const uint16_t *xq = xp + (ch * 16 + l16) * XPLANE + 8 * ((4 * (l16 >> 2) + (l16 & 1) * 2 + (l16 & 2) * 4) & 15);      // my plane
    for (; f < nframes; f += gridDim.x) {
        __syncthreads();                             // the last frame's operands have been read
        if constexpr (!ONE) {
            const int need = f16_row_exponent<RD::LANES>(exponent, [&](const auto &fold) {
#pragma unroll
                for (int i = 0; i < DPT; ++i) { fold(dpre[i].x); fold(dpre[i].y); fold(dpre[i].z); fold(dpre[i].w); }
            });
            if (tid % RD::LANES == 0) { scales[drow] = need; steps[drow] = need - exponent; }
            exponent = need;
        }
        const float dscale = f16_power(exponent);
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            if (xcnt[i] > 0) {
                // a last group holds its dword in the fourth place; the other three places become zero padding
                const u32x4 xv = xcnt[i] == 4 ? xpre[i] : u32x4{xpre[i][3], 0u, 0u, 0u};
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {             // plane v' = vq gets byte vq of each dword
                    uint2 o;
                    if constexpr (ONE) {
                        auto byte = [&](int t) { return (float)((xv[t] >> (8 * vq)) & 0xff); };
                        o = uint2{pack_bf16_rne(byte(0), byte(1)), pack_bf16_rne(byte(2), byte(3))};
                    } else {
                        const uint32_t sel = 0x0c040c00u + 0x00010001u * vq;
                        o = uint2{f16_pair_of_bytes(__builtin_amdgcn_perm(xv[1], xv[0], sel) | 0x64006400u), f16_pair_of_bytes(__builtin_amdgcn_perm(xv[3], xv[2], sel) | 0x64006400u)};
                    }
                    *(uint2 *)(xp + xdst[i] + (vq / 2) * xup[i] + (vq % 2) * (XPLANE + 16)) = o;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < DPT; ++i) {
            if (RD::there(tid, i)) {
                const float4 v = dpre[i];
                uint32_t t0[2], t1[2];
                split_terms<ONE>(v.x, v.y, dscale, t0);
                split_terms<ONE>(v.z, v.w, dscale, t1);
#pragma unroll
                for (int term = 0; term < NTERM; ++term) *(uint2 *)(dp + term * OC * DOC + ddst[i]) = uint2{t0[term], t1[term]};
                auto low = [](uint32_t u) { return __uint_as_float(u << 16); };
                auto high = [](uint32_t u) { return __uint_as_float(u & 0xffff0000u); };
                bsh[drow * (NPIX / 4) + RD::at(tid, i) / 4] = ONE ? (low(t0[0]) + high(t0[0])) + (low(t1[0]) + high(t1[0])) : (v.x + v.y) + (v.z + v.w);
            }
        }
        __syncthreads();
        if (!TABLE) next.ask(x, table, min(f + (int)gridDim.x, nframes - 1), CHW);
        fetch(next.get(), min(f + (int)gridDim.x, nframes - 1));
        if (TABLE) next.ask(x, table, min(f + 2 * (int)gridDim.x, nframes - 1), CHW);
        if (!ONE && f != (int)blockIdx.x) {          // the sums so far come to the scales of the largest values so far
            int4 sd[MT];
            int any = 0;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                sd[m] = *(const int4 *)(steps + 16 * m + 4 * g);
                any |= sd[m].x | sd[m].y | sd[m].z | sd[m].w;
            }
            if (__any(any != 0)) {
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int b = 0; b < 2; ++b) f16_ldexp4(acc[m][a][b], sd[m], 0);
            }
        }
        if (tid < 16 * OC) {   // bias: 16 lanes share a filter, 100 partial sums each
            const int oc = tid / 16, pt = tid % 16;
            float sum = 0.f;
            for (int m = pt; m < NPIX / 4; m += 16) sum += bsh[oc * (NPIX / 4) + m];
            sum += dpp_row_f32<0xB1>(sum); sum += dpp_row_f32<0x4E>(sum);
            sum += dpp_row_f32<0x141>(sum); sum += dpp_row_f32<0x140>(sum);
            bsum += sum;
        }
        auto step = [&](int st) {
            const int blk = 4 * st + g;                   // row blk / 3 of 24 pixels, block blk % 3 of it
            u32x4 d[MT][NTERM];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int term = 0; term < NTERM; ++term)
                    d[m][term] = *(const u32x4 *)(dp + (term * OC + 16 * m + l16) * DOC + 8 * blk);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const uint16_t *src = xq + 8 * blk + a * XROW;
                const u32x4 x0 = *(const u32x4 *)src;
                const uint32_t x4 = *(const uint32_t *)(src + 8);
                const u32x4 x1{__builtin_amdgcn_alignbit(x0[1], x0[0], 16), __builtin_amdgcn_alignbit(x0[2], x0[1], 16),
                               __builtin_amdgcn_alignbit(x0[3], x0[2], 16), __builtin_amdgcn_alignbit(x4, x0[3], 16)};
#pragma unroll
                for (int term = NTERM - 1; term >= 0; --term)
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        acc[m][a][0] = mfma_terms<ONE>(d[m][term], x0, acc[m][a][0]);
                        acc[m][a][1] = mfma_terms<ONE>(d[m][term], x1, acc[m][a][1]);
                    }
            }
        };
        const int st0 = prt * NSTEP / NPART, st1 = (prt + 1) * NSTEP / NPART;
#pragma unroll 1
        for (int st = st0; st < st1; ++st) step(st);
    }
    float *pb = part + ((size_t)blockIdx.x * OCT + oc0) * (K + 1);
    if (tid < 16 * OC && tid % 16 == 0) pb[(tid / 16) * (K + 1) + K] = bsum;
    // the parts of a channel's pixel blocks are added through LDS (the operands are no longer needed)
    __syncthreads();
    float *xch = (float *)xp;
    auto at = [&](int q, int m, int a, int b, int r) { return (((q * 4 + ch) * MT + m) * 16 + (a * 2 + b) * 4 + r) * 64 + lane; };
    if (prt > 0) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) xch[at(prt - 1, m, a, b, r)] = acc[m][a][b][r];
    }
    __syncthreads();
    if (prt > 0) return;
#pragma unroll
    for (int q = 0; q < NPART - 1; ++q)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[m][a][b][r] += xch[at(q, m, a, b, r)];
    // lane (l16, g), register r of acc[m][a][b]: filter 16 m + 4g + r, tap (c = wave, u = 4a + l16/4, v = 4b + l16%4)
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int4 e = ONE ? int4{127, 127, 127, 127} : *(const int4 *)(scales + 16 * m + 4 * g), back{127 - e.x, 127 - e.y, 127 - e.z, 127 - e.w};
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                if constexpr (!ONE) f16_ldexp4(acc[m][a][b], back, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    pb[(16 * m + 4 * g + r) * (K + 1) + ch * 64 + (4 * a + l16 / 4) * 8 + 4 * b + l16 % 4] = acc[m][a][b][r] * scale;
            }
    }
}

inline int conv1_wgrad_blocks(int nframes) { return nframes < 256 ? nframes : 256; }

template <int OCT>
inline hipError_t launch_conv1_wgrad(const uint8_t *x, const uint8_t *const *table, const float *dy, float *part, int nframes, float scale,
                                     hipStream_t s, int rb = 0) {
    if (nframes <= 0) return hipSuccess;
    auto go = [&](auto kernel, int slices) {
        ga3c::launch(kernel, dim3(conv1_wgrad_blocks(nframes), slices), dim3(1024), 0, s, x, table, dy, part, nframes, scale);
    };
    auto pick = [&](auto filters) {
        constexpr int OC = decltype(filters)::value, N = OCT / OC;
        if (table) rb ? go(conv1_wgrad_kernel<OCT, OC, true, true>, N) : go(conv1_wgrad_kernel<OCT, OC, true, false>, N);
        else rb ? go(conv1_wgrad_kernel<OCT, OC, false, true>, N) : go(conv1_wgrad_kernel<OCT, OC, false, false>, N);
    };
    // All filters in one block where slices of 16 would be more blocks than compute units (one fits each), and every frame staged twice.
    if (OCT / 16 * nframes > 256) pick(std::integral_constant<int, OCT>{});
    else pick(std::integral_constant<int, 16>{});
    return hipGetLastError();
}

}  // namespace ga3c
