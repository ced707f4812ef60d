// The two convolution layers of the small network (paper Sec. 3.2: 16 filters 8x8 stride 4 on the 4x84x84 byte frame, 32 filters
// 4x4 stride 2, each with its rectifier) in one kernel, for predictions of more frames than predict_small_kernel takes.
//
// Operands are two float16 terms each (split_f16.hpp), bytes one, as in conv123_f16.hpp; sums of small and of large terms have
// accumulators of their own.  A block takes a frame at a time, first layer 1, then layer 2, with its filters of both in registers for
// the whole launch.  Frames come to LDS as the bytes they are, the next one while this one is worked on.  Layer 1's map is scaled by
// the largest value that it can have with these filters (sum of a filter's positive weights and its bias; a byte is 1 at most), so nobody
// has to look for the one that it has: some bits of the scale are lost, of those to spare (F16_APART).
//
// The map: [term][pixel][16 channels], even and odd columns of a row apart; a k-block of layer 2 is two neighbouring taps of a
// filter row, one of layer 1 four rows of a plane.
//
// Bound by vector instructions next to the products (bytes to float16, splitting, rectifiers: 25 % and 18 % of the SIMD cycles at
// 1024 frames, and the two add up) and, with one frame a block, by its chain of latencies.  us a call, with the fc layer and the heads behind
// it, against conv12_fused.hpp's pipeline on three bfloat16 terms: 65 frames 17.2 -> 16.9, 128: 18.6 -> 18.2, 256: 20.5 -> 20.4, 512: 28.0 ->
// 26.5, 1024: 36.5 -> 33.2, 2048: 62.4 -> 56.6 (bytes as subnormal numbers, 1024 frames 31.5, are not exact enough: split_f16.hpp).  Error of
// the logits against 64 bits (2-norm, 130 frames) 3.1e-7 -> 2.8e-7; with one accumulator a tenth more.  Built and taken out:
// blocks of four wavefronts, two to a compute unit (1024 frames 35.1); one barrier per frame, layer 2 of the last frame beside layer 1 of
// this one (33.5); frames as float16 in LDS (34.8).
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include <type_traits>

#include "conv1_bf16x3.hpp"
#include "conv_plain.hpp"
#include "gemm_mfma.hpp"
#include "split_f16.hpp"

namespace ga3c {

struct Conv12F16 {
    static constexpr int PIT = 32, ROW = 41 * 16, ODD = 10 * PIT, TERM = 20 * ROW;      // 41: rows i and i + 2, nine pixels on, meet no bank twice
    static constexpr int MAP = 2 * F16_FRAME, LDS = MAP + 2 * TERM;
    __host__ __device__ static constexpr int pixel(int row, int col) { return row * ROW + (col & 1) * ODD + (col >> 1) * PIT; }
    // Filters of a parameter copy: layer 1 [k-block][term][lane], layer 2 [filter tile][k-block][term][lane], vectors of eight float16;
    // then floats by filter: reciprocals of the scales (48; negative: F16_WIDE), sums of layer 1's positive weights (16).
    static constexpr int F1 = 0, F2 = F1 + 8 * 128, INV = F2 + 2 * 8 * 128, SUM = INV + 12, VECS = SUM + 4;
};

// Filter q of both layers (0 .. 15, then 16 .. 47), whose 256 weights a wavefront has, four per lane.
__device__ __forceinline__ void conv12_f16_store_filter(u32x4 *__restrict__ frag, const int q, const int lane, const float4 v) {
    typedef Conv12F16 G;
    const float most = f16_wave_most(fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    float s, si;
    f16_scale(most, s, si);
    const int small = __popcll(__ballot(f16_is_small(v.x, most))) + __popcll(__ballot(f16_is_small(v.y, most))) +
                      __popcll(__ballot(f16_is_small(v.z, most))) + __popcll(__ballot(f16_is_small(v.w, most)));
    const int there = __popcll(__ballot(v.x != 0.f)) + __popcll(__ballot(v.y != 0.f)) + __popcll(__ballot(v.z != 0.f)) + __popcll(__ballot(v.w != 0.f));
    const float stored = f16_wide(small, there) || !(most < __builtin_inff()) ? -si : si;
    uint32_t h[2], l[2];
    split2_pair(v.x, v.y, s, h[0], l[0]);
    split2_pair(v.z, v.w, s, h[1], l[1]);
    if (lane == 0) ((float *)(frag + G::INV))[q] = stored;
    if (q < 16) {                                          // plane lane / 16, row lane / 2 % 8, columns 4 (lane % 2) ..
        uint2 *dst = (uint2 *)(frag + G::F1 + (lane >> 3) * 128 + (lane >> 1 & 3) * 16 + q) + (lane & 1);
        dst[0] = uint2{h[0], h[1]};
        dst[128] = uint2{l[0], l[1]};
        float sum = (fmaxf(v.x, 0.f) + fmaxf(v.y, 0.f)) + (fmaxf(v.z, 0.f) + fmaxf(v.w, 0.f));
        sum += dpp_row_f32<0xB1>(sum); sum += dpp_row_f32<0x4E>(sum); sum += dpp_row_f32<0x141>(sum); sum += dpp_row_f32<0x140>(sum);
        const int u = __float_as_int(sum);
        if (lane == 0)
            ((float *)(frag + G::SUM))[q] = (__int_as_float(__builtin_amdgcn_readlane(u, 0)) + __int_as_float(__builtin_amdgcn_readlane(u, 16))) +
                                            (__int_as_float(__builtin_amdgcn_readlane(u, 32)) + __int_as_float(__builtin_amdgcn_readlane(u, 48)));
    } else {                                               // channel lane / 4, row lane % 4, columns 0 .. 3
        const int c = lane >> 2, u = lane & 3;
        uint16_t *dst = (uint16_t *)(frag + G::F2 + ((q >> 4) - 1) * 1024 + u * 256 + (c >> 3) * 16 + (q & 15)) + (c & 7);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint16_t *d = dst + ((e >> 1) * 128 + (e & 1) * 32) * 8;
            d[0] = (uint16_t)(h[e >> 1] >> (16 * (e & 1)));
            d[64 * 8] = (uint16_t)(l[e >> 1] >> (16 * (e & 1)));
        }
    }
}
__global__ __launch_bounds__(256) void conv12_f16_filters_kernel(const float *__restrict__ w1, const float *__restrict__ w2, u32x4 *__restrict__ frag) {
    const int q = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;      // 12 blocks
    conv12_f16_store_filter(frag, __builtin_amdgcn_readfirstlane(q), lane, *(const float4 *)((q < 16 ? w1 + q * 256 : w2 + (q - 16) * 256) + 4 * lane));
}

inline hipError_t launch_conv12_f16_filters(const float *w1, const float *w2, u32x4 *frag, hipStream_t s) {
    ga3c::launch(conv12_f16_filters_kernel, dim3(12), dim3(256), 0, s, w1, w2, frag);
    return hipGetLastError();
}

// x: [n][4][84][84] bytes, or table: where each frame lies; frag: the filters; y2: [n][32][81]; w1, w2: the filter tensors, for plain sums.  Frames blockIdx.x, + gridDim.x, ..
// Wavefront w has pixel tiles w, w + 8, w + 16 of layer 1, the 25th goes to another one with every frame; of layer 2 filter tile w % 2 and
// pixel tile w / 2, the first four also w / 2 + 4: three for every SIMD.
template <bool TABLE>
__global__ __launch_bounds__(512, 2) void conv12_f16_kernel(const uint8_t *__restrict__ x, const uint8_t *const *__restrict__ table,
                                                            const u32x4 *__restrict__ frag, const float *__restrict__ b1,
                                                            const float *__restrict__ b2, float *y2, int nframes, float scale,
                                                            const float *__restrict__ w1, const float *__restrict__ w2) {
    typedef Conv12F16 G;
    constexpr int CHW = 4 * 84 * 84, NPIX2 = 81, NW = 8, T1 = 3, PG = 4, T2 = 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char c12h_smem[];        // two frames, a map
    __shared__ int wide;                                                             // filters need plain sums
    __shared__ __attribute__((aligned(16))) float consts[2][48];                     // by filter: reciprocal of its scale, bias

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grid = (int)gridDim.x;
    const uint32_t lds = lds_address(c12h_smem);

    int f = blockIdx.x;
    FramePointer<TABLE> next;
    next.ask(x, table, min(f, nframes - 1), CHW);
    f16_frame_to_lds<NW>(next.get(), lds, wave, lane);
    if (TABLE) next.ask(x, table, min(f + grid, nframes - 1), CHW);

    const int ot = wave & 1, pg = wave >> 1;
    F16x8Bits q1[8][2], q2[8][2];
#pragma unroll
    for (int kb = 0; kb < 8; ++kb)
#pragma unroll
        for (int t = 0; t < 2; ++t) q1[kb][t].u = (frag + G::F1 + (kb * 2 + t) * 64)[lane];
    const float *inv = (const float *)(frag + G::INV);
    float bound = ((const float *)(frag + G::SUM))[l16];
    const float bb = b1[l16];
    const bool marked = __any(inv[min(lane, 47)] < 0.f);
    if (tid < 48) {
        consts[0][tid] = fabsf(inv[tid]) * (tid < 16 ? scale : 1.f);
        consts[1][tid] = tid < 16 ? b1[tid] : b2[tid - 16];
    }
#pragma unroll
    for (int kb = 0; kb < 8; ++kb)
#pragma unroll
        for (int t = 0; t < 2; ++t) q2[kb][t].u = (frag + G::F2 + ((ot * 8 + kb) * 2 + t) * 64)[lane];
    // layer 1's values are 255 scale = 1 times this at most
    bound = 1.0001f * (255.f * scale * bound + fmaxf(bb, 0.f));
    if (wave == 0) wide = f16_apart(bound) || marked;
    float s, si;
    f16_scale(f16_wave_most(bound), s, si);
    s = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(s)));
    si = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(si)));

    // sums of four filters for a pixel -> rectified values
    auto rectify = [&](const floatx4 a, const float4 iv, const float4 bv, const float si) {
        return floatx4{fmaxf(a[0] * iv.x * si + bv.x, 0.f), fmaxf(a[1] * iv.y * si + bv.y, 0.f), fmaxf(a[2] * iv.z * si + bv.z, 0.f),
                       fmaxf(a[3] * iv.w * si + bv.w, 0.f)};
    };
    auto base_of = [&](int t) {
        const int p = t * 16 + l16;
        return (p / 20 * 4 + g) * 84 + p % 20 * 4;
    };
    floatx4 out[T2];
    // layer 2's results leave when the next frame has arrived: a wait for that would be one for the stores
    auto store = [&](int fr) {
        float *yb = y2 + (size_t)fr * 32 * NPIX2;
#pragma unroll
        for (int i = 0; i < T2; ++i) {
            const int p = (pg + PG * i) * 16 + l16;
            if (p < NPIX2) {
#pragma unroll
                for (int r = 0; r < 4; ++r) yb[(ot * 16 + 4 * g + r) * NPIX2 + p] = out[i][r];
            }
        }
    };
    int place = 0, turn = 0;
    for (bool first = true; f < nframes; f += grid, place ^= F16_FRAME, turn = (turn + 1) & (NW - 1), first = false) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // my pieces of the frame are there
        __syncthreads();                                   // everybody's are; the last map has been read
        if (!first) store(f - grid);
        if (f + grid < nframes) {
            if (!TABLE) next.ask(x, table, f + grid, CHW);
            f16_frame_to_lds<NW>(next.get(), lds + (place ^ F16_FRAME), wave, lane);
            if (TABLE) next.ask(x, table, min(f + 2 * grid, nframes - 1), CHW);
        }
        const unsigned char *xs = c12h_smem + place;
        unsigned char *map = c12h_smem + G::MAP;
        // ---- layer 1
        auto operand = [&](int base, int kb) {
            const uint32_t *src = (const uint32_t *)(xs + base + (kb >> 1) * (84 * 84) + (kb & 1) * (4 * 84));
            return make_uint2(src[0], src[1]);
        };
        const bool odd = wave == turn;
        floatx4 hi[T1 + 1], lo[T1 + 1];
        auto tiles1 = [&](auto count) {
            constexpr int NT = decltype(count)::value;
            int base[NT];
            uint2 v[2][NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                base[i] = base_of(i < T1 ? wave + NW * i : 24);
                hi[i] = lo[i] = floatx4{0.f, 0.f, 0.f, 0.f};
                v[0][i] = operand(base[i], 0);
            }
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) {
                if (kb + 1 < 8) {
#pragma unroll
                    for (int i = 0; i < NT; ++i) v[(kb + 1) & 1][i] = operand(base[i], kb + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    const f16x8 a = f16_of_bytes(v[kb & 1][i].x, v[kb & 1][i].y);
                    lo[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(q1[kb][1].v, a, lo[i], 0, 0, 0);
                    hi[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(q1[kb][0].v, a, hi[i], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (odd) tiles1(std::integral_constant<int, T1 + 1>{});
        else tiles1(std::integral_constant<int, T1>{});
        const float4 iv1 = ((const float4 *)consts[0])[g], bv1 = ((const float4 *)consts[1])[g];
        auto put = [&](const floatx4 sum, int t) {
            const floatx4 a = rectify(sum, iv1, bv1, 1.f);
            const int p = t * 16 + l16;
            unsigned char *dst = map + G::pixel(p / 20, p % 20) + 8 * g;
            uint2 h, l;
            split2_pair(a[0], a[1], s, h.x, l.x);
            split2_pair(a[2], a[3], s, h.y, l.y);
            *(uint2 *)dst = h;
            *(uint2 *)(dst + G::TERM) = l;
        };
#pragma unroll
        for (int i = 0; i < T1; ++i) put(hi[i] + lo[i], wave + NW * i);
        if (odd) put(hi[T1] + lo[T1], 24);
        __syncthreads();
        // ---- layer 2
        auto tiles = [&](auto count) {
            constexpr int NT = decltype(count)::value;
            floatx4 h2[NT], l2[NT];
            int pb[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int p = min((pg + PG * i) * 16 + l16, NPIX2 - 1);
                pb[i] = G::pixel(p / 9 * 2, p % 9 * 2) + (g >> 1) * G::ODD + 16 * (g & 1);
                h2[i] = l2[i] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            F16x8Bits v[2][NT][2];
            auto read = [&](int kb) {
#pragma unroll
                for (int i = 0; i < NT; ++i)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        v[kb & 1][i][t].u = *(const u32x4 *)(map + pb[i] + t * G::TERM + (kb >> 1) * G::ROW + (kb & 1) * G::PIT);
            };
            read(0);
            const float4 iv2 = ((const float4 *)consts[0])[4 * (1 + ot) + g], bv2 = ((const float4 *)consts[1])[4 * (1 + ot) + g];
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) {
                if (kb + 1 < 8) read(kb + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < NT; ++i) l2[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(q2[kb][1].v, v[kb & 1][i][0].v, l2[i], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < NT; ++i) h2[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(q2[kb][0].v, v[kb & 1][i][0].v, h2[i], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < NT; ++i) l2[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(q2[kb][0].v, v[kb & 1][i][1].v, l2[i], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < NT; ++i) out[i] = rectify(h2[i] + l2[i], iv2, bv2, si);
        };
        if (wave < 4) tiles(std::integral_constant<int, 2>{});
        else tiles(std::integral_constant<int, 1>{});
    }
    store(f - grid);
    if (wide) {                                            // my frames once more
        float *y1 = (float *)c12h_smem;
        constexpr int AT = 16 * 400 * 4;                   // the frame, behind the first map
        static_assert(AT + F16_FRAME <= G::LDS, "LDS");
        for (f = blockIdx.x; f < nframes; f += grid) {
            __syncthreads();
            f16_frame_to_lds<NW>(TABLE ? table[f] : x + (size_t)f * CHW, lds + AT, wave, lane);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            plain_conv_layer<uint8_t, 4, 84, 16, 8, 4, NW>(c12h_smem + AT, scale, w1, b1, y1, wave, lane);
            __syncthreads();
            plain_conv_layer<float, 16, 20, 32, 4, 2, NW>(y1, 1.f, w2, b2, y2 + (size_t)f * 32 * NPIX2, wave, lane);
        }
    }
}

inline hipError_t launch_conv12_f16(const uint8_t *x, const uint8_t *const *table, const u32x4 *frag, const float *b1, const float *b2, float *y2,
                                    int nframes, float scale, const float *w1, const float *w2, hipStream_t s) {
    if (nframes <= 0) return hipSuccess;
    static bool attr_set = false;
    if (!attr_set) {
        for (const void *k : {(const void *)conv12_f16_kernel<false>, (const void *)conv12_f16_kernel<true>}) {
            const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, Conv12F16::LDS);
            if (e != hipSuccess) return e;
        }
        attr_set = true;
    }
    ga3c::launch(table ? conv12_f16_kernel<true> : conv12_f16_kernel<false>, dim3(nframes < 256 ? nframes : 256), dim3(512), Conv12F16::LDS, s, x,
                 table, frag, b1, b2, y2, nframes, scale, w1, w2);
    return hipGetLastError();
}

}  // namespace ga3c
