// The three convolution layers of a network in one kernel, for predictions: a block of eight wavefronts takes a frame from
// its bytes to the fc layer's input, and nothing in between leaves the compute unit.  Networks are the larger one (32 8x8
// stride 4 on the 4x84x84 byte frame, 64 4x4 stride 2, 64 3x3 stride 1) and those of the larger-network family whose first map
// fits (32 8x8 stride 4 or 3, 32 4x4 stride 2, 64 4x4 stride 2), each layer with its rectifier.
//
// Operands are two float16 terms each (split_f16.hpp), bytes one.  Filters come scaled and split, in the order in which the
// lanes take them, from a buffer per parameter copy.  Layer 1's map is scaled by the largest value that it can have with these filters
// (sum of a filter's positive weights and its bias; a byte is 1 at most), layer 2's by its own largest value, which the eight wavefronts
// find between the layer's products and its way to LDS.
//
//   layer 1  both filter tiles from one read of a pixel tile's bytes: wavefront w has tiles w, w + 8, ..; of the tiles that are left
//            over wavefronts 2 i and 2 i + 1 have the i-th, a filter tile each
//   layers 2, 3  wavefront w has filter tile w % (filters / 16) and every so many pixel tiles
//
// Frames come to LDS as the bytes they are, the next one while this one is worked on; a lane's eight columns of a filter row are two
// dwords, or cut from three where the stride is odd.  Layer 2's map takes the place of layer 1's.  Every wavefront keeps a layer's
// filters in registers, 128 or 144 of them; those of the next layer take the place of the ones that have been multiplied, k-block by
// k-block, so that no layer waits for its filters.
//
// Bound by one frame's chain through a compute unit: bytes in, three layers and six barriers.  us a call (with the fc layer and the heads
// behind it) against a kernel per layer on three bfloat16 terms or the fp32 instruction: larger net 1 frame 27.6 -> 21.9, 64: 29.8 ->
// 23.5, 128: 37.3 -> 25.7, 256: 47.1 -> 29.0, 512: 69.9 -> 44.8, 1024: 113 -> 78; stride-4 member 1: 24.4 -> 18.7, 128: 35.0 -> 20.4, 256:
// 41.1 -> 21.2; stride-3 member 1: 23.5 -> 22.0, 64: 31.9 -> 23.9, 128: 38.3 -> 25.2, 256: 47.3 -> 26.0, 512: 69.1 -> 41.6.  Error of the
// logits against 64 bits (2-norm, 130 frames) 5.3e-7 -> 4.4e-7, 4.4e-7 -> 3.9e-7, 4.9e-7 -> 4.4e-7.
//
// Updates keep the layers' own kernels: another rounding of a sum puts a pre-activation next to zero on the other side of the
// rectifier now and then, and a map's gradients with it.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include <type_traits>

#include "conv_fwd_bf16x6.hpp"
#include "conv_plain.hpp"
#include "split_f16.hpp"

namespace ga3c {

// A map in LDS, as the input of layer SP: [term], eight channels of a pixel in 16 bytes.  Sixteen neighbouring output pixels read
// without bank conflicts: with stride 2 the even and the odd columns of a row lie apart, and rows are as long as makes pixel OW of
// a row fall where pixel 0 of the next one does.  PLANAR: the groups of eight channels apart from each other, which takes no
// padding behind a pixel but needs an even OW.
template <class SP, bool PLANAR>
struct F16Map {
    static constexpr int UNITS = SP::C / 8, PIT = PLANAR ? 1 : lds_row_units(UNITS), EVEN = (SP::W + 1) / 2;
    static constexpr int row_units() {
        int r = SP::W * PIT;
        while ((SP::S * r - PIT * SP::OW) % 16 != 0) ++r;
        return r;
    }
    static constexpr int ROW = 16 * row_units(), GROUP = PLANAR ? (SP::H * ROW + 255) / 256 * 256 : 16;
    static constexpr int TERM = PLANAR ? UNITS * GROUP : SP::H * ROW;
    // where a pixel's first eight channels lie; output pixel p's first one
    __host__ __device__ static constexpr int pixel(int row, int col) {
        return row * ROW + (SP::S == 2 ? (col & 1) * EVEN + (col >> 1) : col) * (16 * PIT);
    }
    __host__ __device__ static constexpr int origin(int p) { return p / SP::OW * SP::S * ROW + p % SP::OW * (16 * PIT); }
};

// A network: stride of layer 1 (32 filters), layers 2 and 3, whether layer 1's map is planar.
template <int S1_, class SP2_, class SP3_, bool PLANAR_>
struct Conv123Net {
    typedef SP2_ SP2;
    typedef SP3_ SP3;
    typedef F16Map<SP2, PLANAR_> M2;
    typedef F16Map<SP3, false> M3;
    static constexpr int S1 = S1_, OW1 = (84 - 8) / S1 + 1, NPIX1 = OW1 * OW1, NT1 = (NPIX1 + 15) / 16;
    static constexpr int NT2 = (SP2::NPIX + 15) / 16, NT3 = (SP3::NPIX + 15) / 16, OT2 = SP2::OC / 16;
    static_assert(SP2::H == OW1 && SP2::W == OW1 && SP2::C == 32 && SP2::K == 512 && SP2::S == 2 && (SP2::OC == 32 || SP2::OC == 64), "layer 2: 4x4, stride 2");
    static_assert(SP3::H == SP2::OH && SP3::C == SP2::OC && SP3::K % 32 == 0 && SP3::OC == 64, "layer 3");
    // Filters: [filter tile][k-block][term][lane] vectors of eight float16 each; then the reciprocals of the filters' scales (negative:
    // F16_WIDE), and sums of the positive weights of layer 1's.
    static constexpr int KB1 = 8, KB2 = 16, KB3 = SP3::K / 32, CG3 = SP3::C / 32;
    static constexpr int F1 = 0, F2 = F1 + 2 * KB1 * 128, F3 = F2 + OT2 * KB2 * 128, INV = F3 + 4 * KB3 * 128;
    static constexpr int FILTERS = 32 + SP2::OC + 64, SUM = INV + FILTERS / 4, VECS = SUM + 32 / 4;
    // the kernel that writes them: four k-blocks of a filter tile each block
    static constexpr int B1 = 2 * KB1 / 4, B2 = B1 + OT2 * KB2 / 4, PER3 = (KB3 + 3) / 4, BLOCKS = B2 + 4 * PER3;
    static constexpr int Y = 2 * F16_FRAME, LDS = Y + 2 * (M2::TERM > M3::TERM ? M2::TERM : M3::TERM);
    static_assert(LDS + 2048 <= 160 * 1024, "LDS");
    static_assert(32 * NPIX1 * 4 + F16_FRAME <= LDS && (32 * NPIX1 + SP2::OC * SP2::NPIX) * 4 <= LDS, "plain sums: the first map, then a frame or the second");
};

// Block b of N::BLOCKS, 256 threads.  w1, w2, w3: the filter tensors, 16-byte aligned.
template <class N>
__device__ __forceinline__ void conv123_fragments_block(const float *__restrict__ w1, const float *__restrict__ w2, const float *__restrict__ w3,
                                                        u32x4 *__restrict__ frag, int b) {
    __shared__ float scales[16];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    constexpr int K3 = N::SP3::K, TAPS3 = K3 / N::SP3::C, KMOST = K3 > 512 ? K3 : 512;
    int layer, ot, kb0, K, KB, at, first;
    const float *w;
    if (b < N::B1) { layer = 1; ot = b / 2; kb0 = b % 2 * 4; K = 256; KB = N::KB1; w = w1; at = N::F1; first = 0; }
    else if (b < N::B2) { layer = 2; ot = (b - N::B1) / 4; kb0 = (b - N::B1) % 4 * 4; K = 512; KB = N::KB2; w = w2; at = N::F2; first = 32; }
    else { layer = 3; ot = (b - N::B2) / N::PER3; kb0 = (b - N::B2) % N::PER3 * 4; K = K3; KB = N::KB3; w = w3; at = N::F3; first = 32 + N::SP2::OC; }
    w += (size_t)ot * 16 * K;
    // everything is asked for at once: my eight values, and sixteen threads, which are a row of lanes, find a filter's largest one
    const int kb = kb0 + (tid >> 6);
    float v[8], m = 0.f, sum = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        int k;                                             // of the filter as it lies in memory: (channel, row, column)
        if (layer == 1) k = 32 * kb + 8 * g + j;
        else if (layer == 2) k = (8 * g + j) * 16 + kb;
        else k = (kb % N::CG3 * 32 + 8 * g + j) * TAPS3 + kb / N::CG3;
        v[j] = w[(size_t)l16 * K + min(k, K - 1)];
    }
    float4 all[KMOST / 64];
#pragma unroll
    for (int i = 0; i < KMOST / 64; ++i) all[i] = *(const float4 *)(w + (size_t)(tid >> 4) * K + min(4 * (tid & 15) + 64 * i, K - 4));
#pragma unroll
    for (int i = 0; i < KMOST / 64; ++i) m = fmaxf(fmaxf(fmaxf(m, fabsf(all[i].x)), fmaxf(fabsf(all[i].y), fabsf(all[i].z))), fabsf(all[i].w));
    m = fmaxf(m, dpp_row_f32<0xB1>(m)); m = fmaxf(m, dpp_row_f32<0x4E>(m));
    m = fmaxf(m, dpp_row_f32<0x141>(m)); m = fmaxf(m, dpp_row_f32<0x140>(m));
    if (layer == 1) {                                      // K = 256: four vectors a thread
#pragma unroll
        for (int i = 0; i < 4; ++i) sum += (fmaxf(all[i].x, 0.f) + fmaxf(all[i].y, 0.f)) + (fmaxf(all[i].z, 0.f) + fmaxf(all[i].w, 0.f));
        sum += dpp_row_f32<0xB1>(sum); sum += dpp_row_f32<0x4E>(sum); sum += dpp_row_f32<0x141>(sum); sum += dpp_row_f32<0x140>(sum);
        if (kb0 == 0 && (tid & 15) == 0) ((float *)(frag + N::SUM))[ot * 16 + (tid >> 4)] = sum;
    }
    // small weights and those that are not zero, counted in one number: 1024 for each of the former
    float count = 0.f;
#pragma unroll
    for (int i = 0; i < KMOST / 64; ++i)
        if (4 * (tid & 15) + 64 * i < K) {
            auto weigh = [&](const float w) { return (float)(1024 * f16_is_small(w, m) + (w != 0.f)); };
            count += (weigh(all[i].x) + weigh(all[i].y)) + (weigh(all[i].z) + weigh(all[i].w));
        }
    count += dpp_row_f32<0xB1>(count); count += dpp_row_f32<0x4E>(count); count += dpp_row_f32<0x141>(count); count += dpp_row_f32<0x140>(count);
    static_assert(KMOST < 1024, "the count of weights");
    if ((tid & 15) == 0) {
        float s, inv;
        f16_scale(m, s, inv);
        scales[tid >> 4] = s;
        if (kb0 == 0) ((float *)(frag + N::INV))[first + ot * 16 + (tid >> 4)] = f16_wide((int)count >> 10, (int)count & 1023) || !(m < __builtin_inff()) ? -inv : inv;
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

// x: [n][4][84][84] bytes, or table: where each frame lies; frag: N's filters; b1 [32], b2, b3: biases; y: [n][64][layer 3's pixels]; f1, f2,
// f3: the filter tensors, for plain sums.
template <class N, bool TABLE>
__global__ __launch_bounds__(512, 1) void conv123_f16_kernel(const uint8_t *__restrict__ x, const uint8_t *const *__restrict__ table,
                                                             const u32x4 *__restrict__ frag, const float *__restrict__ b1,
                                                             const float *__restrict__ b2, const float *__restrict__ b3, float *y, int nframes,
                                                             float scale, const float *__restrict__ f1, const float *__restrict__ f2,
                                                             const float *__restrict__ f3) {
    typedef typename N::SP2 SP2;
    typedef typename N::SP3 SP3;
    typedef typename N::M2 M2;
    typedef typename N::M3 M3;
    constexpr int CHW = 4 * 84 * 84, KB1 = N::KB1, KB2 = N::KB2, KB3 = N::KB3;
    constexpr int FULL1 = N::NT1 / 8, REST1 = N::NT1 % 8, PG2 = 8 / N::OT2;      // tiles per wavefront, tiles left over; groups of wavefronts
    constexpr int T2 = (N::NT2 + PG2 - 1) / PG2, T3 = (N::NT3 + 1) / 2;          // the last of some wavefronts is not there
    static_assert(2 * REST1 <= 8, "half a tile each");
    extern __shared__ __attribute__((aligned(16))) unsigned char c123_smem[];
    __shared__ int wide[3];                                // layers that need plain sums
    __shared__ float most[8];                              // largest values of layer 2, by wavefront
    __shared__ __attribute__((aligned(16))) float consts[2][N::FILTERS];       // by filter: reciprocal of its scale, bias

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grid = (int)gridDim.x;
    const uint32_t lds = lds_address(c123_smem);

    int f = blockIdx.x;
    FramePointer<TABLE> next;
    next.ask(x, table, min(f, nframes - 1), CHW);
    f16_frame_to_lds<8>(next.get(), lds, wave, lane);
    if (TABLE) next.ask(x, table, min(f + grid, nframes - 1), CHW);

    // layer 1: w1[0] is filter tile `own`, w1[1] the other one
    const int own = wave & 1, ot2 = wave % N::OT2, pg2 = wave / N::OT2, ot3 = wave & 3, pg3 = wave >> 2;
    F16x8Bits w1[2][KB1][2], w2[KB2][2], w3[KB3][2];
    // A wavefront's place is added to the scalar address, a lane's is the same for all vectors.
    uint32_t again;
    const uint32_t mine = 16 * lane;
    auto vec = [&](int at) { return *(const u32x4 *)((const char *)(frag + again + at) + mine); };
    auto load1 = [&](int kb) {
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int t = 0; t < 2; ++t) w1[o][kb][t].u = vec(N::F1 + (((own ^ o) * KB1 + kb) * 2 + t) * 64);
    };
    auto load2 = [&](int kb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) w2[kb][t].u = vec(N::F2 + ((ot2 * KB2 + kb) * 2 + t) * 64);
    };
    auto load3 = [&](int kb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) w3[kb][t].u = vec(N::F3 + ((ot3 * KB3 + kb) * 2 + t) * 64);
    };
    float bound = ((const float *)(frag + N::SUM))[lane & 31];
    const float bb = b1[lane & 31];
    const float v = ((const float *)(frag + N::INV))[wave == 0 ? lane & 31 : wave == 1 ? 32 + lane % SP2::OC : 32 + SP2::OC + lane];
    const float b2v = b2[lane % SP2::OC];
    if (tid < N::FILTERS) {
        consts[0][tid] = fabsf(((const float *)(frag + N::INV))[tid]) * (tid < 32 ? scale : 1.f);
        consts[1][tid] = tid < 32 ? b1[tid] : tid < 32 + SP2::OC ? b2[tid - 32] : b3[tid - 32 - SP2::OC];
    }
    bound = 1.0001f * (255.f * scale * bound + fmaxf(bb, 0.f));
    const float top = f16_wave_most(bound);
    float s1, si1;
    f16_scale(top, s1, si1);
    if (wave < 3) {
        // of layer 2's channels: the filter's largest weight (2^15 times the reciprocal of its scale; 0: 2^-126) times the largest value it can meet
        const float size = wave == 0 ? bound : (fabsf(v) <= 1.1754943508222875e-38f ? 0.f : fabsf(v) * 32768.f * top) + fmaxf(b2v, 0.f);
        wide[wave] = __any(v < 0.f) || (wave < 2 && f16_apart(size));
    }
    s1 = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(s1)));
    si1 = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(si1)));

    constexpr int WT[3] = {1, 0, 0}, XT[3] = {0, 1, 0};    // smallest products first
    floatx4 out[T3];
    // layer 3's results leave when the next frame has arrived: a wait for that would be one for the stores
    auto store = [&](int fr) {
        if (N::NT3 == 1 && pg3 != 0) return;
        float *yb = y + (size_t)fr * SP3::OC * SP3::NPIX;
#pragma unroll
        for (int i = 0; i < T3; ++i) {
            const int p = (pg3 + 2 * i) * 16 + (lane & 15);
            if (p < SP3::NPIX) {
#pragma unroll
                for (int r = 0; r < 4; ++r) yb[(ot3 * 16 + 4 * (lane >> 4) + r) * SP3::NPIX + p] = out[i][r];
            }
        }
    };
    int place = 0;
    for (bool first = true; f < nframes; f += grid, place ^= F16_FRAME, first = false) {
        // what a frame does not change is read and worked out anew for each: there are no registers to keep it in
        int own_lane = lane;
        asm volatile("s_mov_b32 %0, 0" : "=s"(again), "+v"(own_lane));
        const int l16 = own_lane & 15, g = own_lane >> 4;
        const float4 *inv = (const float4 *)consts[0] + g, *bias = (const float4 *)consts[1] + g;      // my four filters of tile t: [4 t]
        // sums of those for a pixel -> rectified values
        auto rectify = [&](const floatx4 a, const float4 iv, const float4 bv, const float si) {
            return floatx4{fmaxf(a[0] * iv.x * si + bv.x, 0.f), fmaxf(a[1] * iv.y * si + bv.y, 0.f), fmaxf(a[2] * iv.z * si + bv.z, 0.f),
                           fmaxf(a[3] * iv.w * si + bv.w, 0.f)};
        };
        // values of filters 16 t + 4 g .. as terms, to the pixel that lies at `at`
        auto store4 = [&](int term, int group, int at, int t, const floatx4 v, float s) {
            uint2 hi, lo;
            split2_pair(v[0], v[1], s, hi.x, lo.x);
            split2_pair(v[2], v[3], s, hi.y, lo.y);
            unsigned char *dst = c123_smem + N::Y + at + (2 * t + (g >> 1)) * group + 8 * (g & 1);
            *(uint2 *)dst = hi;
            *(uint2 *)(dst + term) = lo;
        };
#pragma unroll
        for (int kb = 0; kb < KB1; ++kb) load1(kb);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // my pieces of the frame are there
        __syncthreads();                                   // everybody's are; the last layer-2 map has been read
        if (!first) store(f - grid);
        if (f + grid < nframes) {
            if (!TABLE) next.ask(x, table, f + grid, CHW);
            f16_frame_to_lds<8>(next.get(), lds + (place ^ F16_FRAME), wave, lane);
            if (TABLE) next.ask(x, table, min(f + 2 * grid, nframes - 1), CHW);
        }
        // ---- layer 1: a k-block is four filter rows of a plane
        {
            constexpr bool ODD = N::S1 % 2 != 0;
            constexpr int DW = ODD ? 3 : 2;
            struct Raw { uint32_t d[DW]; };
            auto base_of = [&](int t) {
                const int p = min(t * 16 + l16, N::NPIX1 - 1);
                return (p / N::OW1 * N::S1 + g) * 84 + p % N::OW1 * N::S1;
            };
            auto raw = [&](int base, int kb) {
                const uint32_t *src = (const uint32_t *)(c123_smem + place + (ODD ? base & ~3 : base) + (kb >> 1) * (84 * 84) + (kb & 1) * (4 * 84));
                Raw r;
#pragma unroll
                for (int d = 0; d < DW; ++d) r.d[d] = src[d];
                return r;
            };
            auto operand = [&](const Raw &r, int base) {
                if constexpr (ODD) return f16_of_bytes(__builtin_amdgcn_alignbyte(r.d[1], r.d[0], base & 3), __builtin_amdgcn_alignbyte(r.d[2], r.d[1], base & 3));
                else return f16_of_bytes(r.d[0], r.d[1]);
            };
            const int left = 8 * FULL1 + (wave >> 1);
            int base[FULL1];
            floatx4 acc[FULL1][2], accx[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
            if (wave < 2 * REST1) {                        // before the filters go
                const int b = base_of(left);
                Raw r[KB1];
#pragma unroll
                for (int kb = 0; kb < KB1; ++kb) r[kb] = raw(b, kb);
#pragma unroll
                for (int kb = 0; kb < KB1; ++kb) {
                    const f16x8 v = operand(r[kb], b);
#pragma unroll
                    for (int t = 1; t >= 0; --t) accx[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[0][kb][t].v, v, accx[t], 0, 0, 0);
                }
                accx[0] += accx[1];
            }
            Raw r[2][FULL1];
#pragma unroll
            for (int i = 0; i < FULL1; ++i) {
                base[i] = base_of(wave + 8 * i);
                acc[i][0] = acc[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
                r[0][i] = raw(base[i], 0);
            }
#pragma unroll
            for (int kb = 0; kb < KB1; ++kb) {
                if (kb + 1 < KB1) {
#pragma unroll
                    for (int i = 0; i < FULL1; ++i) r[(kb + 1) & 1][i] = raw(base[i], kb + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < FULL1; ++i) {
                    const f16x8 v = operand(r[kb & 1][i], base[i]);
#pragma unroll
                    for (int t = 1; t >= 0; --t)
#pragma unroll
                        for (int o = 0; o < 2; ++o) acc[i][o] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[o][kb][t].v, v, acc[i][o], 0, 0, 0);
                }
                load2(2 * kb);
                load2(2 * kb + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            const float4 iv[2] = {inv[4 * own], inv[4 * (own ^ 1)]}, bv[2] = {bias[4 * own], bias[4 * (own ^ 1)]};
            auto put = [&](const floatx4 a, int t, int o) {
                const int p = t * 16 + l16;
                if (N::NPIX1 % 16 == 0 || p < N::NPIX1)
                    store4(M2::TERM, M2::GROUP, M2::pixel(p / N::OW1, p % N::OW1), own ^ o, rectify(a, iv[o], bv[o], 1.f), s1);
            };
#pragma unroll
            for (int i = 0; i < FULL1; ++i) { put(acc[i][0], wave + 8 * i, 0); put(acc[i][1], wave + 8 * i, 1); }
            if (wave < 2 * REST1) put(accx[0], left, 0);
        }
        __syncthreads();
        // ---- layer 2: a k-block is a tap, 32 channels
        {
            floatx4 acc[T2];
            int pb[T2], px[T2];
#pragma unroll
            for (int i = 0; i < T2; ++i) {
                const int p = (pg2 + PG2 * i) * 16 + l16;
                px[i] = p < SP2::NPIX ? p : -1;
                pb[i] = N::Y + M2::origin(p < SP2::NPIX ? p : 0) + g * M2::GROUP;
                acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            F16x8Bits xv[2][T2][2];
            auto read = [&](int kb) {
#pragma unroll
                for (int i = 0; i < T2; ++i)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        xv[kb & 1][i][t].u = *(const u32x4 *)(c123_smem + t * M2::TERM + pb[i] + M2::pixel(kb / 4, kb % 4));
            };
            read(0);
#pragma unroll
            for (int kb = 0; kb < KB2; ++kb) {
                if (kb + 1 < KB2) read(kb + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int i = 0; i < T2; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w2[kb][WT[q]].v, xv[kb & 1][i][XT[q]].v, acc[i], 0, 0, 0);
                load3(kb);
                if (kb + KB3 - KB2 >= KB2) load3(kb + KB3 - KB2);
                __builtin_amdgcn_sched_barrier(0);
            }
            const float4 iv = inv[4 * (2 + ot2)], bv = bias[4 * (2 + ot2)];
            float m = 0.f;
#pragma unroll
            for (int i = 0; i < T2; ++i) {
                acc[i] = rectify(acc[i], iv, bv, si1);
                const float mi = fmaxf(fmaxf(acc[i][0], acc[i][1]), fmaxf(acc[i][2], acc[i][3]));
                m = px[i] >= 0 ? fmaxf(m, mi) : m;
            }
            m = f16_wave_most(m);
            if (lane == 0) most[wave] = m;
            __syncthreads();                               // everybody's largest value; layer 1's map has been read
            float s, si;
            f16_scale_of(most, s, si);
#pragma unroll
            for (int i = 0; i < T2; ++i)
                if (px[i] >= 0) store4(M3::TERM, M3::GROUP, M3::pixel(px[i] / SP3::W, px[i] % SP3::W), ot2, acc[i], s);
        }
        __syncthreads();
        // ---- layer 3: a k-block is 32 channels of a tap
        if (N::NT3 > 1 || pg3 == 0) {
            float s, si;
            f16_scale_of(most, s, si);
            floatx4 acc[T3];
            int pb[T3];
#pragma unroll
            for (int i = 0; i < T3; ++i) {
                pb[i] = N::Y + M3::origin(min((pg3 + 2 * i) * 16 + l16, SP3::NPIX - 1)) + g * M3::GROUP;
                acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            F16x8Bits xv[2][T3][2];
            auto read = [&](int kb) {
                const int tap = kb / N::CG3;
#pragma unroll
                for (int i = 0; i < T3; ++i)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        xv[kb & 1][i][t].u = *(const u32x4 *)(c123_smem + t * M3::TERM + pb[i] + M3::pixel(tap / SP3::KS, tap % SP3::KS) +
                                                              kb % N::CG3 * 4 * M3::GROUP);
            };
            read(0);
#pragma unroll
            for (int kb = 0; kb < KB3; ++kb) {
                if (kb + 1 < KB3) read(kb + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int i = 0; i < T3; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w3[kb][WT[q]].v, xv[kb & 1][i][XT[q]].v, acc[i], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            const float4 iv = inv[4 * (2 + N::OT2 + ot3)], bv = bias[4 * (2 + N::OT2 + ot3)];
#pragma unroll
            for (int i = 0; i < T3; ++i) out[i] = rectify(acc[i], iv, bv, si);
        }
    }
    store(f - grid);
    if (wide[0] | wide[1] | wide[2]) {                     // my frames once more
        float *y1 = (float *)c123_smem, *y2 = y1 + 32 * N::NPIX1;      // the frame lies in the second map's place first
        const unsigned char *frame = (const unsigned char *)y2;
        for (f = blockIdx.x; f < nframes; f += grid) {
            __syncthreads();
            f16_frame_to_lds<8>(TABLE ? table[f] : x + (size_t)f * CHW, lds + 32 * N::NPIX1 * 4, wave, lane);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            plain_conv_layer<uint8_t, 4, 84, 32, 8, N::S1, 8>(frame, scale, f1, b1, y1, wave, lane);
            __syncthreads();
            plain_conv_layer<float, 32, SP2::H, SP2::OC, 4, 2, 8>(y1, 1.f, f2, b2, y2, wave, lane);
            __syncthreads();
            plain_conv_layer<float, SP3::C, SP3::H, SP3::OC, SP3::KS, SP3::S, 8>(y2, 1.f, f3, b3, y + (size_t)f * SP3::OC * SP3::NPIX, wave, lane);
        }
    }
}

template <class N, bool TABLE>
inline hipError_t launch_conv123_f16(const uint8_t *x, const uint8_t *const *table, const u32x4 *frag, const float *b1, const float *b2,
                                     const float *b3, float *y, int nframes, float scale, const float *f1, const float *f2, const float *f3, hipStream_t s) {
    if (nframes <= 0) return hipSuccess;
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute((const void *)conv123_f16_kernel<N, TABLE>, hipFuncAttributeMaxDynamicSharedMemorySize, N::LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    ga3c::launch((conv123_f16_kernel<N, TABLE>), dim3(nframes < 256 ? nframes : 256), dim3(512), N::LDS, s, x, table, frag, b1, b2, b3, y, nframes, scale,
                 f1, f2, f3);
    return hipGetLastError();
}

}  // namespace ga3c
