// First convolution layer (8x8 filters, stride 4, on 4x84x84 byte frames;
// paper Sec. 3.2) on the bf16 matrix cores without losing fp32 accuracy.
//
// A byte 0..255 has at most 8 significant bits, which is exactly what a bf16
// holds, so the frame converts to bf16 without rounding.  An fp32 number is the
// exact sum of three bf16 numbers (hi + mid + lo, 8 bits each).  The product of
// a byte and a bf16 term has 16 bits and is exact in the fp32 accumulator.  So
//   sum_k W[k] x[k] = sum_k (hi[k] + mid[k] + lo[k]) x[k]
// evaluated with three v_mfma_f32_16x16x32_bf16 per 32 taps rounds only where
// the fp32 MFMA path rounds too (in the accumulation), at 5x its rate.  The
// layer then runs at the speed of fetching frames and storing activations.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include <type_traits>

#include "conv_frame.hpp"

namespace ga3c {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

union Bf16x8Bits {
    bf16x8 v;
    u32x4 u;
};

// Pitch, in units of 16 bytes, of the LDS rows (pixels, filters, channels) from which a lane (l16, g) of the matrix instructions
// reads unit g of row l16.  A 16-byte read takes its lanes in groups of 16: eight of one g and the other eight l16 of its
// neighbour.  With an odd pitch a row's unit g + 1 falls on the banks of another row's unit g and the read takes twice as long (8
// against 4.2 cycles); with twice an odd number the two halves of a group fall on the even and the odd units of the 256 bytes that
// the banks hold.  (Twice an odd number also keeps 8- and 16-byte writes of consecutive rows at 16 cycles a kilobyte, provided
// that a lane writes whole units; with 8 bytes each they take twice as long as from an odd pitch.)
constexpr int lds_row_units(int least) {
    while (least % 4 != 2) ++least;
    return least;
}

// Sum step inside a row of 16 lanes (DPP control CTRL).
template <int CTRL>
__device__ __forceinline__ float dpp_row_f32(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// hi/mid/lo with f == hi + mid + lo exactly (round-to-nearest-even casts).
__device__ __forceinline__ void split3(float f, __bf16 &hi, __bf16 &mid, __bf16 &lo) {
    hi = (__bf16)f;
    const float r1 = f - (float)hi;
    mid = (__bf16)r1;
    lo = (__bf16)(r1 - (float)mid);
}
// The same with a switch: rb != 0 keeps only hi, i.e. the operand rounded to
// bfloat16 (the reduced-precision variant of the network); the kernels then
// multiply zeros in the other two terms.
__device__ __forceinline__ void split3(float f, __bf16 &hi, __bf16 &mid, __bf16 &lo, int rb) {
    split3(f, hi, mid, lo);
    if (rb) { mid = (__bf16)0.f; lo = (__bf16)0.f; }
}

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// two floats -> two bfloat16 (round to nearest even) in one register, x in the low half
__device__ __forceinline__ uint32_t pack_bf16_rne(float x, float y) {
    union { bf16x2_t v; uint32_t u; } c;
    c.v = __builtin_convertvector(f32x2_t{x, y}, bf16x2_t);
    return c.u;
}

// split3 for two values at a time (the same roundings, one conversion instruction per pair and term):
// x in the low halves of hi, mid, lo and y in the high halves
__device__ __forceinline__ void split3_pair(float x, float y, uint32_t &hi, uint32_t &mid, uint32_t &lo) {
    hi = pack_bf16_rne(x, y);
    const float rx = x - __uint_as_float(hi << 16), ry = y - __uint_as_float(hi & 0xffff0000u);
    mid = pack_bf16_rne(rx, ry);
    lo = pack_bf16_rne(rx - __uint_as_float(mid << 16), ry - __uint_as_float(mid & 0xffff0000u));
}

// One dword per lane from base + off (bytes) to lds + 4 * lane; base and lds are the same for the whole wavefront.  The caller
// waits for vmcnt itself: the compiler, which would wait for every such load in front of the next LDS read, does not see it.
__device__ __forceinline__ void load_dword_to_lds(const void *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
// The same with 16 bytes per lane, to lds + 16 * lane.
__device__ __forceinline__ void load_vec_to_lds(const void *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}

// Where frame f lies.  TABLE: wherever the table's entry points (x is not used).  The table is host memory that no cache keeps,
// and an entry takes about two microseconds to arrive: one lane asks for it, and kernels that walk over frames ask early.
template <bool TABLE>
struct FramePointer {
    const uint8_t *at;
    __device__ __forceinline__ void ask(const uint8_t *x, const uint8_t *const *table, int f, int bytes) {
        if (!TABLE) at = x + (size_t)f * bytes;
        else if ((threadIdx.x & 63) == 0) at = __builtin_nontemporal_load(table + f);
    }
    __device__ __forceinline__ const uint8_t *get() const {
        if (!TABLE) return at;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)at), hi = __builtin_amdgcn_readfirstlane((uint32_t)((uintptr_t)at >> 32));
        return (const uint8_t *)(((uintptr_t)hi << 32) | lo);
    }
};

// 16 bytes -> 16 bf16 (two 16-byte vectors)
__device__ __forceinline__ void bytes_to_bf16(const u32x4 b, u32x4 &lo8, u32x4 &hi8) {
    Bf16x8Bits o[2];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t v = b[d];
        o[d / 2].v[(d % 2) * 4 + 0] = (__bf16)(float)(v & 0xff);
        o[d / 2].v[(d % 2) * 4 + 1] = (__bf16)(float)((v >> 8) & 0xff);
        o[d / 2].v[(d % 2) * 4 + 2] = (__bf16)(float)((v >> 16) & 0xff);
        o[d / 2].v[(d % 2) * 4 + 3] = (__bf16)(float)(v >> 24);
    }
    lo8 = o[0].u;
    hi8 = o[1].u;
}

// y[b][oc][pix] = max(0, scale * sum_k W[oc][k] x[b][tap k at pix] + bias[oc]),  OC = 16 or 32.
// Block = 4 wavefronts, frames blockIdx.x, blockIdx.x + gridDim.x, ...  The
// frame sits in LDS as bf16 [4][84][84]; a lane (pixel p, group g) reads the 8
// taps of filter row u = 4*(kb%2) + g of channel kb/2 in one go, which is the
// k = 8g..8g+7 share of a 16x16x32 MFMA.  The split filters stay in registers.
// ONE: operands rounded to bfloat16 (the reduced-precision variant): one term, one product (1280 frames of 32 filters 27.9 -> 24.2 us
// against two more terms that were zero).
// PARTS: blocks per frame (blockIdx.y), each with every PARTS-th group of four (pixel tile, filter tile) pairs, so that a few
// frames keep the chip busy.
template <int OC, bool TABLE, bool ONE, int PARTS>
__global__ __launch_bounds__(256, 2) void conv1_bf16x3_fwd_kernel(const uint8_t *__restrict__ x,
                                                                  const uint8_t *const *__restrict__ table,
                                                                  const float *__restrict__ w,
                                                                  const float *__restrict__ bias, float *__restrict__ y,
                                                                  int nframes, float scale) {
    constexpr int NTERM = ONE ? 1 : 3;
    constexpr int C = 4, H = 84, W = 84, S = 4, OW = 20, NPIX = 400, K = 256, CHW = C * H * W;
    constexpr int NV = CHW / 16, VPT = (NV + 255) / 256;           // 16-byte vectors of the byte frame
    constexpr int OT = OC / 16, JOBS = 25 * OT, SLOTS = 4 * PARTS, TPW = (JOBS + SLOTS - 1) / SLOTS;
    constexpr int FULL = JOBS % SLOTS == 0 ? TPW : TPW - 1, NLAST = JOBS - SLOTS * FULL;
    static_assert(OC == 16 || OC == 32, "16 or 32 filters");
    __shared__ __attribute__((aligned(16))) __bf16 xs[VPT * 256 * 16];

    const int tid = threadIdx.x, lane = tid & 63;
    // the wave that gets the odd tile rotates with the block, so that two
    // blocks sharing a compute unit do not load the same SIMD
    const int wave = __builtin_amdgcn_readfirstlane(((tid >> 6) + (OT == 1 ? blockIdx.x : 2 * (blockIdx.x & 1))) & 3);
    const int l16 = lane & 15, g = lane >> 4;
    const int ot = wave % OT, slot = wave + (PARTS == 1 ? 0 : 4 * blockIdx.y);

    // my filter (row l16 of tile ot), split into three bf16 terms, 8 taps per 32-tap block
    bf16x8 wq[NTERM][8];
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
        const float *src = w + (size_t)(ot * 16 + l16) * K + (kb / 2) * 64 + (4 * (kb % 2) + g) * 8;
        const float4 a = *(const float4 *)src, b = *(const float4 *)(src + 4);
        const float f[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            __bf16 t[3];
            split3(f[e], t[0], t[1], t[2]);
#pragma unroll
            for (int q = 0; q < NTERM; ++q) wq[q][kb][e] = t[q];
        }
    }
    // The MFMAs take the pixels as rows and the filters as columns: a lane ends up with four consecutive pixels
    // (16 tile + 4 g + r) of filter ot * 16 + l16, which it stores as one 16-byte vector.
    const float bv = bias[ot * 16 + l16];

    int pixbase[TPW], pixidx[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int job = slot + SLOTS * i;
        int p = (job / OT) * 16 + l16;
        pixidx[i] = (job < JOBS && p < NPIX) ? (job / OT) * 16 + 4 * g : -1;       // first of my four output pixels
        if (p >= NPIX) p = 0;
        pixbase[i] = (p / OW) * S * W + (p % OW) * S + g * W;     // + row g of the 4 rows of a tap block
    }
    int vidx[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) vidx[i] = min(tid + 256 * i, NV - 1);

    u32x4 pre[VPT];
    int f = blockIdx.x;
    {
        FramePointer<TABLE> first;
        first.ask(x, table, min(f, nframes - 1), CHW);
        const u32x4 *src = (const u32x4 *)first.get();
#pragma unroll
        for (int i = 0; i < VPT; ++i) pre[i] = src[vidx[i]];
    }
    FramePointer<TABLE> next;
    if (TABLE) next.ask(x, table, min(f + (int)gridDim.x, nframes - 1), CHW);
    for (; f < nframes; f += gridDim.x) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            u32x4 a, b;
            bytes_to_bf16(pre[i], a, b);
            u32x4 *dst = (u32x4 *)(xs + (size_t)(tid + 256 * i) * 16);
            dst[0] = a; dst[1] = b;
        }
        __syncthreads();
        {
            if (!TABLE) next.ask(x, table, min(f + (int)gridDim.x, nframes - 1), CHW);
            const u32x4 *src = (const u32x4 *)next.get();
#pragma unroll
            for (int i = 0; i < VPT; ++i) pre[i] = src[vidx[i]];
            if (TABLE) next.ask(x, table, min(f + 2 * (int)gridDim.x, nframes - 1), CHW);
        }
        floatx4 acc[TPW];
#pragma unroll
        for (int i = 0; i < TPW; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto tile_step = [&](int i, int kb) {
            const __bf16 *src = xs + pixbase[i] + (kb / 2) * (H * W) + 4 * (kb % 2) * W;   // 8-byte aligned
            const uint2 lo = *(const uint2 *)src, hi = *(const uint2 *)(src + 4);
            Bf16x8Bits xv;
            xv.u = u32x4{lo.x, lo.y, hi.x, hi.y};
#pragma unroll
            for (int q = NTERM - 1; q >= 0; --q) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv.v, wq[q][kb], acc[i], 0, 0, 0);
        };
#pragma unroll
        for (int kb = 0; kb < 8; ++kb)
#pragma unroll
            for (int i = 0; i < FULL; ++i) tile_step(i, kb);
        if (NLAST > 0 && slot < NLAST) {
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) tile_step(TPW - 1, kb);
        }
        float *yb = y + (size_t)f * OC * NPIX;
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            if (pixidx[i] >= 0) {
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = acc[i][r] * scale + bv;
                    v[r] = v[r] > 0.f ? v[r] : 0.f;
                }
                *(float4 *)(yb + (ot * 16 + l16) * NPIX + pixidx[i]) = float4{v[0], v[1], v[2], v[3]};      // NPIX % 4 == 0
            }
        }
    }
}

template <int OC>
inline hipError_t launch_conv1_bf16x3_fwd(const uint8_t *x, const uint8_t *const *table, const float *w, const float *bias, float *y, int nframes,
                                          float scale, hipStream_t s, int rb = 0) {
    if (nframes <= 0) return hipSuccess;
    const int grid = nframes < 512 ? nframes : 512;
    auto go = [&](auto kernel, int parts) { ga3c::launch(kernel, dim3(grid, parts), dim3(256), 0, s, x, table, w, bias, y, nframes, scale); };
    auto pick = [&](auto parts) {
        constexpr int P = decltype(parts)::value;
        if (table) rb ? go(conv1_bf16x3_fwd_kernel<OC, true, true, P>, P) : go(conv1_bf16x3_fwd_kernel<OC, true, false, P>, P);
        else rb ? go(conv1_bf16x3_fwd_kernel<OC, false, true, P>, P) : go(conv1_bf16x3_fwd_kernel<OC, false, false, P>, P);
    };
    // four blocks per frame while one per compute unit has room (32 filters: 1 frame 8.0 -> 5.4 us, 64 frames 9.7 -> 6.8)
    if (OC == 32 && 4 * nframes <= 256) pick(std::integral_constant<int, OC == 32 ? 4 : 1>{});
    else pick(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

}  // namespace ga3c
