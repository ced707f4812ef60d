// The three convolution layers of the larger network (32 8x8 stride 4 on the 4x84x84 byte frame, 64 4x4 stride 2, 64 3x3
// stride 1, each with its rectifier) in one kernel, for predictions: a block of eight wavefronts takes a frame from its
// bytes to the fc layer's input, and nothing in between leaves the compute unit.
//
// Operands are two float16 terms each (split_f16.hpp), bytes one.  Filters come scaled and split, in the order in which the
// lanes take them, from a buffer per parameter copy; an activation map is scaled by its own largest value, which the eight
// wavefronts find between a layer's products and its way to LDS (one barrier more than without).
//
//   layer 1  both filter tiles from one read of a pixel tile's bytes: wavefront w has tiles w, w + 8, w + 16 of the 25, and the last
//            one is shared by wavefronts 0 and 1, a filter tile each
//   layer 2  wavefront w has filter tile w % 4 and every other of the six pixel tiles; layer 3 likewise, of four
//
// LDS holds the frame as float16 (later layer 2's output) and layer 1's output in the layouts of conv_fwd_bf16x6.hpp.  Every
// wavefront keeps a layer's filters in registers, 64 to 144 of them; those of the next layer take the place of the ones that have been
// multiplied, k-block by k-block, so that no layer waits for its filters.
//
// Bound by one frame's chain through a compute unit: bytes in, three layers and six barriers.  us a call (with the fc layer and the heads
// behind it) against a kernel per layer on three bfloat16 terms: 1 frame 26.2 -> 21.6, 64: 28.8 -> 23.2, 128: 36.9 -> 25.6, 256: 47.4 ->
// 29.0, 512: 71.5 -> 45.5, 1024: 116 -> 80.  Error of the logits against 64 bits (2-norm, 256 frames) 5.1e-7 -> 4.3e-7.
//
// Updates keep the layers' own kernels: another rounding of a sum puts a pre-activation next to zero on the other side of the
// rectifier now and then, and a map's gradients with it.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include "conv_fwd_bf16x6.hpp"
#include "split_f16.hpp"

namespace ga3c {

// Filters of the three layers: [filter tile][k-block][term][lane] vectors of eight float16 each; then the reciprocals of
// the filters' scales, 32 + 64 + 64 floats.
struct Conv123Frags {
    static constexpr int KB1 = 8, KB2 = 16, KB3 = 18;
    static constexpr int F1 = 0, F2 = F1 + 2 * KB1 * 128, F3 = F2 + 4 * KB2 * 128, INV = F3 + 4 * KB3 * 128, VECS = INV + (32 + 64 + 64) / 4;
    static constexpr int BLOCKS = 2 * 2 + 4 * 4 + 4 * 5;       // of the kernel that writes them: four k-blocks of a filter tile each
};

// Block b of BLOCKS, 256 threads.  w1 [32][4][8][8], w2 [64][32][4][4], w3 [64][64][3][3], 16-byte aligned.
__device__ __forceinline__ void conv123_fragments_block(const float *__restrict__ w1, const float *__restrict__ w2, const float *__restrict__ w3,
                                                        u32x4 *__restrict__ frag, int b) {
    typedef Conv123Frags G;
    __shared__ float scales[16];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    int layer, ot, kb0, K, KB, at;
    const float *w;
    if (b < 4) { layer = 1; ot = b / 2; kb0 = b % 2 * 4; K = 256; KB = G::KB1; w = w1; at = G::F1; }
    else if (b < 20) { layer = 2; ot = (b - 4) / 4; kb0 = (b - 4) % 4 * 4; K = 512; KB = G::KB2; w = w2; at = G::F2; }
    else { layer = 3; ot = (b - 20) / 5; kb0 = (b - 20) % 5 * 4; K = 576; KB = G::KB3; w = w3; at = G::F3; }
    w += (size_t)ot * 16 * K;
    // everything is asked for at once: my eight values, and sixteen threads, which are a row of lanes, find a filter's largest one
    const int kb = kb0 + (tid >> 6);
    float v[8], m = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        int k;                                             // of the filter as it lies in memory: (channel, row, column)
        if (layer == 1) k = 32 * kb + 8 * g + j;
        else if (layer == 2) k = (8 * g + j) * 16 + kb;
        else k = (kb % 2 * 32 + 8 * g + j) * 9 + kb / 2;
        v[j] = w[(size_t)l16 * K + min(k, K - 1)];
    }
    float4 all[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) all[i] = *(const float4 *)(w + (size_t)(tid >> 4) * K + min(4 * (tid & 15) + 64 * i, K - 4));
#pragma unroll
    for (int i = 0; i < 9; ++i) m = fmaxf(fmaxf(fmaxf(m, fabsf(all[i].x)), fmaxf(fabsf(all[i].y), fabsf(all[i].z))), fabsf(all[i].w));
    m = fmaxf(m, dpp_row_f32<0xB1>(m)); m = fmaxf(m, dpp_row_f32<0x4E>(m));
    m = fmaxf(m, dpp_row_f32<0x141>(m)); m = fmaxf(m, dpp_row_f32<0x140>(m));
    if ((tid & 15) == 0) {
        float s, inv;
        f16_scale(m, s, inv);
        scales[tid >> 4] = s;
        if (kb0 == 0) ((float *)(frag + G::INV))[(layer == 1 ? 0 : layer == 2 ? 32 : 96) + ot * 16 + (tid >> 4)] = inv;
    }
    __syncthreads();
    if (kb >= KB) return;
    const float s = scales[l16];
    u32x4 hi, lo;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t h, l;
        split2_pair(v[2 * j], v[2 * j + 1], s, h, l);
        hi[j] = h; lo[j] = l;
    }
    u32x4 *dst = frag + at + (size_t)(ot * KB + kb) * 128 + lane;
    dst[0] = hi;
    dst[64] = lo;
}

template <class SP2, class SP3>
struct Conv123Geom {
    typedef ConvFwdBf16Geom<SP2> G2;
    typedef ConvFwdBf16Geom<SP3> G3;
    static constexpr int NV = 4 * 84 * 84 / 16;                                        // 16-byte vectors of a frame
    static constexpr int XS = 0, Y1 = NV * 32, Y2 = 0, LDS = Y1 + 2 * G2::PLANE;        // layer 2's output takes the frame's place
    static_assert(Y2 + 2 * G3::PLANE <= Y1 && LDS <= 160 * 1024 - 64, "LDS");
};

// x: [n][4][84][84] bytes, or table: where each frame lies; frag: Conv123Frags; b1 [32], b2, b3 [64]; y: [n][64][49].
template <class SP2, class SP3, bool TABLE>
__global__ __launch_bounds__(512, 1) void conv123_f16_kernel(const uint8_t *__restrict__ x, const uint8_t *const *__restrict__ table,
                                                             const u32x4 *__restrict__ frag, const float *__restrict__ b1,
                                                             const float *__restrict__ b2, const float *__restrict__ b3, float *__restrict__ y,
                                                             int nframes, float scale) {
    typedef Conv123Geom<SP2, SP3> G;
    typedef typename G::G2 G2;
    typedef typename G::G3 G3;
    typedef Conv123Frags R;
    constexpr int CHW = 4 * 84 * 84, NV = G::NV, VPT = (NV + 511) / 512;
    extern __shared__ __attribute__((aligned(16))) unsigned char c123_smem[];
    __shared__ float most[2][8];                           // largest values of layers 1 and 2, by wavefront
    __shared__ __attribute__((aligned(16))) float consts[2][160];       // by filter: reciprocal of its scale, bias
    _Float16 *xs = (_Float16 *)(c123_smem + G::XS);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    u32x4 pre[VPT];
    int f = blockIdx.x;
    FramePointer<TABLE> next;
    auto fetch = [&]() {
        const u32x4 *src = (const u32x4 *)next.get();
#pragma unroll
        for (int i = 0; i < VPT; ++i) pre[i] = src[min(tid + 512 * i, NV - 1)];
    };
    next.ask(x, table, min(f, nframes - 1), CHW);
    fetch();
    if (TABLE) next.ask(x, table, min(f + (int)gridDim.x, nframes - 1), CHW);

    // layer 1: w1[0] is filter tile `own`, w1[1] the other one
    const int own = wave & 1, ot = wave & 3, pg = wave >> 2;
    F16x8Bits w1[2][R::KB1][2], w2[R::KB2][2], w3[R::KB3][2];
    // A wavefront's place is added to the scalar address, a lane's is the same for all vectors.
    uint32_t again = 0;
    const uint32_t mine = 16 * lane;
    auto vec = [&](int at) { return *(const u32x4 *)((const char *)(frag + again + at) + mine); };
    auto load1 = [&](int kb) {
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int t = 0; t < 2; ++t) w1[o][kb][t].u = vec(R::F1 + (((own ^ o) * R::KB1 + kb) * 2 + t) * 64);
    };
    auto load2 = [&](int kb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) w2[kb][t].u = vec(R::F2 + ((ot * R::KB2 + kb) * 2 + t) * 64);
    };
    auto load3 = [&](int kb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) w3[kb][t].u = vec(R::F3 + ((ot * R::KB3 + kb) * 2 + t) * 64);
    };
    if (tid < 160) {
        consts[0][tid] = ((const float *)(frag + R::INV))[tid] * (tid < 32 ? scale : 1.f);
        consts[1][tid] = tid < 32 ? b1[tid] : tid < 96 ? b2[tid - 32] : b3[tid - 96];
    }

    // Largest value of all wavefronts, as a scale (behind a barrier).
    auto scale_of = [&](const float (&m)[8], float &s, float &si) {
        const float a = fmaxf(fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3])), fmaxf(fmaxf(m[4], m[5]), fmaxf(m[6], m[7])));
        f16_scale(__uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(a))), s, si);
    };
    auto wave_most = [&](float m) {
        m = fmaxf(m, dpp_row_f32<0xB1>(m)); m = fmaxf(m, dpp_row_f32<0x4E>(m));
        m = fmaxf(m, dpp_row_f32<0x141>(m)); m = fmaxf(m, dpp_row_f32<0x140>(m));
        const int u = __float_as_int(m);
        return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(u, 0)), __int_as_float(__builtin_amdgcn_readlane(u, 16))),
                     fmaxf(__int_as_float(__builtin_amdgcn_readlane(u, 32)), __int_as_float(__builtin_amdgcn_readlane(u, 48))));
    };
    for (; f < nframes; f += gridDim.x) {
        // what a frame does not change is read and worked out anew for each: there are no registers to keep it in
        int own_lane = lane;
        asm volatile("" : "+s"(again), "+v"(own_lane));
        const int l16 = own_lane & 15, g = own_lane >> 4;
        const float4 *inv = (const float4 *)consts[0] + g, *bias = (const float4 *)consts[1] + g;      // my four filters of tile t: [4 t]
#pragma unroll
        for (int kb = 0; kb < R::KB1; ++kb) load1(kb);
        __syncthreads();                                   // the last frame's layer-2 output has been read
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            const int v = tid + 512 * i;
            u32x4 a, b;
            bytes_to_f16(pre[i], a, b);
            if (v < NV) {
                u32x4 *dst = (u32x4 *)(xs + (size_t)v * 16);
                dst[0] = a; dst[1] = b;
            }
        }
        __syncthreads();
        if (!TABLE) next.ask(x, table, min(f + (int)gridDim.x, nframes - 1), CHW);
        fetch();
        if (TABLE) next.ask(x, table, min(f + 2 * (int)gridDim.x, nframes - 1), CHW);
        // four filters' values of a pixel (4 g .. of filter tile t), as terms
        auto store4 = [&](unsigned char *plane, int plane_bytes, int at, int t, const float (&v)[4], float s) {
            uint2 hi, lo;
            split2_pair(v[0], v[1], s, hi.x, lo.x);
            split2_pair(v[2], v[3], s, hi.y, lo.y);
            *(uint2 *)(plane + at + t * 32 + 8 * g) = hi;
            *(uint2 *)(plane + plane_bytes + at + t * 32 + 8 * g) = lo;
        };
        // ---- layer 1
        {
            auto base_of = [&](int t) {
                const int p = t * 16 + l16;
                return (p / 20 * 4 + g) * 84 + p % 20 * 4;
            };
            auto operand = [&](int base, int kb) {
                const _Float16 *src = xs + base + (kb / 2) * (84 * 84) + 4 * (kb % 2) * 84;      // 8-byte aligned
                const uint2 lo = *(const uint2 *)src, hi = *(const uint2 *)(src + 4);
                F16x8Bits v;
                v.u = u32x4{lo.x, lo.y, hi.x, hi.y};
                return v.v;
            };
            int base[3];
            floatx4 acc[3][2], accx = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                base[i] = base_of(wave + 8 * i);
                acc[i][0] = acc[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            if (wave < 2) {                                // before the filters go
                const int b24 = base_of(24);
#pragma unroll
                for (int kb = 0; kb < R::KB1; ++kb) {
                    const f16x8 v = operand(b24, kb);
#pragma unroll
                    for (int t = 1; t >= 0; --t) accx = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[0][kb][t].v, v, accx, 0, 0, 0);
                }
            }
            f16x8 xv[2][3];
#pragma unroll
            for (int i = 0; i < 3; ++i) xv[0][i] = operand(base[i], 0);
#pragma unroll
            for (int kb = 0; kb < R::KB1; ++kb) {
                if (kb + 1 < R::KB1) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) xv[(kb + 1) & 1][i] = operand(base[i], kb + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 1; t >= 0; --t)
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int o = 0; o < 2; ++o)
                            acc[i][o] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[o][kb][t].v, xv[kb & 1][i], acc[i][o], 0, 0, 0);
                load2(2 * kb);
                load2(2 * kb + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            float m = 0.f;
            const float4 iv[2] = {inv[4 * own], inv[4 * (own ^ 1)]}, bv[2] = {bias[4 * own], bias[4 * (own ^ 1)]};
            auto finish = [&](floatx4 &a, int o) {
                const float v[4] = {a[0] * iv[o].x + bv[o].x, a[1] * iv[o].y + bv[o].y, a[2] * iv[o].z + bv[o].z, a[3] * iv[o].w + bv[o].w};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    a[r] = v[r] > 0.f ? v[r] : 0.f;
                    m = fmaxf(m, a[r]);
                }
            };
#pragma unroll
            for (int i = 0; i < 3; ++i) { finish(acc[i][0], 0); finish(acc[i][1], 1); }
            if (wave < 2) finish(accx, 0);
            m = wave_most(m);
            if (lane == 0) most[0][wave] = m;
            __syncthreads();
            float s, si;
            scale_of(most[0], s, si);
            auto put = [&](const floatx4 a, int t, int o) {
                const int p = t * 16 + l16;
                const float v[4] = {a[0], a[1], a[2], a[3]};
                store4(c123_smem + G::Y1, G2::PLANE, G2::pixel(p / 20, p % 20), own ^ o, v, s);
            };
#pragma unroll
            for (int i = 0; i < 3; ++i) { put(acc[i][0], wave + 8 * i, 0); put(acc[i][1], wave + 8 * i, 1); }
            if (wave < 2) put(accx, 24, 0);
        }
        __syncthreads();
        // ---- layer 2
        {
            float s, si;
            scale_of(most[0], s, si);
            floatx4 acc[3];
            int pb[3], px[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int p = (pg + 2 * i) * 16 + l16, q = p < SP2::NPIX ? p : 0;
                px[i] = p < SP2::NPIX ? p : -1;
                pb[i] = G::Y1 + (q / SP2::OW) * 2 * G2::ROW + (q % SP2::OW) * G2::PIT + 16 * g;
                acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            F16x8Bits xv[2][3][2];
            auto read = [&](int kb) {
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        xv[kb & 1][i][t].u = *(const u32x4 *)(c123_smem + t * G2::PLANE + pb[i] + G2::pixel(kb / 4, kb % 4));
            };
            read(0);
#pragma unroll
            for (int kb = 0; kb < R::KB2; ++kb) {
                if (kb + 1 < R::KB2) read(kb + 1);
                __builtin_amdgcn_sched_barrier(0);
                constexpr int WT[3] = {1, 0, 0}, XT[3] = {0, 1, 0};      // smallest products first
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w2[kb][WT[q]].v, xv[kb & 1][i][XT[q]].v, acc[i], 0, 0, 0);
                load3(kb);
                if (kb >= R::KB2 - 2) load3(kb + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            float m = 0.f;
            const float4 iv = inv[4 * (2 + ot)], bv = bias[4 * (2 + ot)];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const float v[4] = {acc[i][0] * iv.x * si + bv.x, acc[i][1] * iv.y * si + bv.y, acc[i][2] * iv.z * si + bv.z, acc[i][3] * iv.w * si + bv.w};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    acc[i][r] = v[r] > 0.f ? v[r] : 0.f;
                    m = px[i] >= 0 ? fmaxf(m, acc[i][r]) : m;
                }
            }
            m = wave_most(m);
            if (lane == 0) most[1][wave] = m;
            __syncthreads();
            scale_of(most[1], s, si);
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (px[i] >= 0) {
                    const float v[4] = {acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
                    store4(c123_smem + G::Y2, G3::PLANE, G3::pixel(px[i] / SP3::W, px[i] % SP3::W), ot, v, s);
                }
        }
        __syncthreads();
        // ---- layer 3
        {
            float s, si;
            scale_of(most[1], s, si);
            floatx4 acc[2];
            int pb[2], px[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int p = (pg + 2 * i) * 16 + l16, q = p < SP3::NPIX ? p : 0;
                px[i] = p < SP3::NPIX ? p : -1;
                pb[i] = G::Y2 + (q / SP3::OW) * G3::ROW + (q % SP3::OW) * G3::PIT + 16 * g;
                acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            F16x8Bits xv[2][2][2];
            auto read = [&](int kb) {
                const int tap = kb / 2;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        xv[kb & 1][i][t].u = *(const u32x4 *)(c123_smem + t * G3::PLANE + pb[i] + G3::pixel(tap / 3, tap % 3) + kb % 2 * 64);
            };
            read(0);
#pragma unroll
            for (int kb = 0; kb < R::KB3; ++kb) {
                if (kb + 1 < R::KB3) read(kb + 1);
                __builtin_amdgcn_sched_barrier(0);
                constexpr int WT[3] = {1, 0, 0}, XT[3] = {0, 1, 0};
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w3[kb][WT[q]].v, xv[kb & 1][i][XT[q]].v, acc[i], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            float *yb = y + (size_t)f * SP3::OC * SP3::NPIX;
            const float4 iv = inv[4 * (6 + ot)], bv = bias[4 * (6 + ot)];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float v[4] = {acc[i][0] * iv.x * si + bv.x, acc[i][1] * iv.y * si + bv.y, acc[i][2] * iv.z * si + bv.z, acc[i][3] * iv.w * si + bv.w};
                if (px[i] >= 0) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) yb[(ot * 16 + 4 * g + r) * SP3::NPIX + px[i]] = v[r] > 0.f ? v[r] : 0.f;
                }
            }
        }
    }
}

template <class SP2, class SP3>
inline hipError_t launch_conv123_f16(const uint8_t *x, const uint8_t *const *table, const u32x4 *frag, const float *b1, const float *b2,
                                     const float *b3, float *y, int nframes, float scale, hipStream_t s) {
    if (nframes <= 0) return hipSuccess;
    constexpr int LDS = Conv123Geom<SP2, SP3>::LDS;
    static bool attr_set = false;
    if (!attr_set) {
        for (const void *k : {(const void *)conv123_f16_kernel<SP2, SP3, false>, (const void *)conv123_f16_kernel<SP2, SP3, true>}) {
            const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
            if (e != hipSuccess) return e;
        }
        attr_set = true;
    }
    const int grid = nframes < 256 ? nframes : 256;
    if (table) ga3c::launch((conv123_f16_kernel<SP2, SP3, true>), dim3(grid), dim3(512), LDS, s, x, table, frag, b1, b2, b3, y, nframes, scale);
    else ga3c::launch((conv123_f16_kernel<SP2, SP3, false>), dim3(grid), dim3(512), LDS, s, x, table, frag, b1, b2, b3, y, nframes, scale);
    return hipGetLastError();
}

}  // namespace ga3c
