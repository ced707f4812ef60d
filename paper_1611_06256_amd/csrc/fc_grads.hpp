// The fully connected layer's two gradients in one launch, on the bf16 matrix cores at fp32 accuracy
// (dense_gemm_bf16x6.hpp has the error argument):
//
//   dX[b][i] = [x[b][i] > 0] * sum_o dh[b][o] W[o][i]        (one block per 64x64 tile)
//   dW[o][i] = sum_b dh[b][o] x[b][i]                         (in chunks of frames)
//
// from operands that are split into three bf16 terms already: dh by its producer, W per parameter copy (fc_forward.hpp).
// Only x is still split here, by the one wavefront that uses those columns.  The sums are those of
// dense_fc_grads_kernel, in its order (the same bits).
//
// That kernel, which reads dh, W and x as fp32 and splits them in every block, spent 51 % of the SIMDs' cycles on vector
// instructions next to 28 % of products.  Here everything goes straight from memory to LDS, one k-step of 32 ahead, and
// three blocks share a compute unit (48 KB each): MFMA 29 - 43 %, vector instructions 19 - 27 %, no bank conflicts; the rest is
// waiting at the one barrier of a k-step (two blocks with two steps ahead: 64 instead of 57 us).  Rows of 128 units or frames
// in blocks of eight wavefronts were level; tiles of 128x128, one block of eight wavefronts with three steps in LDS per compute
// unit, which ask for half the bytes, were too (2560 frames of the small net 57.5 / 59.4 us, 1280 of the larger 57.5 / 60.2,
// 640 x 1024 x 18496 288 / 277), four wavefronts slower.  us of the launch before and after, and of the reduction behind it where dW needs no
// partial sums any more: small net 40 frames 14.6 -> 8.0, 640: 20.0 -> 16.0 (10.1 -> 8.3), 2560: 55.2 -> 47.7; larger net 1280:
// 67.0 -> 49.8 (34.8 -> 23.5), its operands rounded to bfloat16 38.8 -> 23.4 (36.7 -> 24.7); 640 x 1024 x 18496: 430 -> 250 (125
// -> 35).
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include "fc_forward.hpp"

namespace ga3c {

// dh as operands of dW (rows = fc units, k = frames) in the order in which the lanes take them:
// [unit / 16][frame / 32][terms][frame % 32 / 8][unit % 16][8 frames] bf16, zero behind the last frame.  A heads block has eight
// frames, 16 bytes of a unit.  dX wants the units as k and takes the same pieces through the transposing LDS read.
struct FcDhPlanes {
    u32x4 *w;                                 // nullptr: none
    int terms;                                // 3, or 1 (rounded to bfloat16)
};
inline size_t fc_dh_planes_bytes(int cap, int F, int terms) { return ((size_t)cap + 31) / 32 * 32 * F * 2 * terms; }

// Frames 8 b8 .. of unit o; kbw: frames / 32, rounded up.
__device__ __forceinline__ void fc_dh_store8(const FcDhPlanes &p, int o, int b8, int kbw, const float (&f)[8]) {
    u32x4 *dst = p.w + ((size_t)(o >> 4) * kbw + (b8 >> 2)) * (64 * p.terms) + (b8 & 3) * 16 + (o & 15), t[3];
    split3x8(f, t[0], t[1], t[2]);
#pragma unroll
    for (int q = 0; q < 3; ++q)
        if (q < p.terms) dst[64 * q] = t[q];
}

// From dh [B][F], behind heads kernels that do not write them.
__global__ __launch_bounds__(256) void fc_dh_planes_kernel(const float *__restrict__ dh, const FcDhPlanes p, int B, int F, const FastDiv dF) {
    const unsigned kbw = (unsigned)(B + 31) / 32, i = blockIdx.x * 256 + threadIdx.x;
    if (i >= kbw * 4 * (unsigned)F) return;
    uint32_t b8, o;
    dF.divmod(i, b8, o);
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float v = dh[(size_t)min(8 * (int)b8 + e, B - 1) * F + o];
        f[e] = 8 * (int)b8 + e < B ? v : 0.f;
    }
    fc_dh_store8(p, (int)o, (int)b8, (int)kbw, f);
}
inline hipError_t launch_fc_dh_planes(const float *dh, const FcDhPlanes &p, int B, int F, hipStream_t s) {
    ga3c::launch(fc_dh_planes_kernel, dim3(((unsigned)(B + 31) / 32 * 4 * F + 255) / 256), dim3(256), 0, s, dh, p, B, F, FastDiv(F));
    return hipGetLastError();
}

struct FcGradArgs {
    int B, F, flat;                           // F a multiple of 64, flat of 32
    int kchunk, nz;                           // dW: frames in nz chunks of kchunk (a multiple of 32)
    int ntx, ntw, ntn;                        // row tiles of dX and of dW, column tiles of both
    int per_x, per_w;                         // blocks per XCD
    int w_first;                              // dW's blocks come first
    int x_cols;                               // dX: an XCD's column tiles next to each other, not a column's row tiles
    int z_to_xcd;                             // dW: an XCD takes every eighth chunk instead of every eighth column tile
    FastDiv dntx, dntw, dtw;                  // by ntx, ntw, and dW's tiles of a chunk or of a column
    FcDhPlanes dh;
    const u32x4 *w;                           // FcPlanes
    const float *x;                           // [B][flat], 16-byte aligned
    float *dx;                                // [B][flat]
    float *dw;                                // [nz][F][flat], or with FOLD the gradient itself
};

constexpr int FCG_STEPS = 2;                  // k-steps of 32 in LDS: one is multiplied, one is on its way
template <bool ONE>
constexpr int fcg_step_bytes() { return ONE ? 4096 + 8192 : 12288 + 12288; }      // dh, then x (fp32, 8 KB) or W
template <bool ONE>
constexpr int fc_grads_lds() { return FCG_STEPS * fcg_step_bytes<ONE>(); }

// Four bf16 k of one column from four LDS rows, twice: in a group of 16 lanes the lanes name the 8-byte pieces of four rows, and
// every lane receives one column of them.
__device__ __forceinline__ u32x4 lds_transpose8(const unsigned char *p0, const unsigned char *p1) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    union { s16x4 s[2]; u32x4 u; } o;
    o.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p0);
    o.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p1);
    return o.u;
}

// One block's tile.  dW: a wavefront takes 16 of the 64 columns, which it splits, and all 64 rows, whose operands (dh) the four share
// through LDS.  dX: 32 rows and 32 columns (24 instead of 30 reads of LDS per step).  With that, the mask asked for with the last
// step, W's terms in pieces of 1 KB without gaps and the order of blocks below, larger net, 1280 frames: 58.4 -> 53.7 us, small net,
// 2560: 52.4 -> 50.5.
// FOLD (dW): all chunks of the tile, one after the other, their sums added up in the order of reduce_all_kernel.
template <bool WGRAD, bool ONE, bool FOLD>
__device__ __forceinline__ void fc_grad_block(const FcGradArgs &p, const int bid, unsigned char *smem) {
    constexpr int NT = ONE ? 1 : 3, STEP = fcg_step_bytes<ONE>(), AB = 4 * NT * 1024;
    const int xcd = bid % DG_XCDS, local = bid / DG_XCDS;
    uint32_t tm, tn, z = 0;
    if (WGRAD && !FOLD) {
        uint32_t q, t;
        p.dtw.divmod((uint32_t)local, q, t);
        if (p.z_to_xcd) { z = q * DG_XCDS + xcd; p.dntw.divmod(t, tn, tm); }
        else { tn = q * DG_XCDS + xcd; p.dntw.divmod(t, z, tm); }
        if ((int)z >= p.nz || (int)tn >= p.ntn) return;
    } else {
        uint32_t ci;
        if (WGRAD || !p.x_cols) (WGRAD ? p.dntw : p.dntx).divmod((uint32_t)local, ci, tm);
        else p.dntx.divmod((uint32_t)local, tm, ci);
        tn = ci * DG_XCDS + xcd;
        if ((int)tn >= p.ntn) return;
    }
    const int m0 = (int)tm * 64, n0 = (int)tn * 64;
    const int nf = (p.B + 31) / 32, nk = WGRAD ? nf : p.F / 32;
    const int kc = p.kchunk / 32, kb0 = WGRAD && !FOLD ? (int)z * kc : 0, kb1 = WGRAD && !FOLD ? min(nk, kb0 + kc) : nk;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;

    // dW: my 16 units; dX: 16 units of the k-step x 32 frames of the tile, unit u of the eight frames b at place u ^ 4 (b % 2), so
    // that the two groups of frames a wavefront reads at once are in different banks
    const u32x4 *ak = p.dh.w + (WGRAD ? (size_t)(m0 / 16 + wave) * nf : (size_t)(wave >> 1) * nf + min(m0 / 32 + (wave & 1), nf - 1)) * (NT * 64);
    const size_t astep = (WGRAD ? 1 : 2 * (size_t)nf) * (NT * 64);
    const uint32_t aoff = (WGRAD ? lane : lane ^ (4 * (g & 1))) * 16;
    // x: rows of 64 columns, four per load; piece c (16 bytes) of row r lies at place c ^ 4 (r / 8), so that the four rows eight apart that a
    // wavefront reads at once are in different banks
    // W: 16 units x 32 columns per wavefront, rows of 64 bytes; piece c of row r lies at place c ^ 2 (r / 8), likewise
    uint32_t boff[2] = {0, 0};
    int brow[2] = {0, 0};
    const unsigned char *bk;
    if (WGRAD) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = (2 * wave + i) * 64 + lane;         // piece of the step
            brow[i] = e / 16;
            boff[i] = 4u * (uint32_t)min(n0 + 4 * ((e % 16) ^ (4 * (brow[i] >> 3))), p.flat - 4);
        }
        bk = (const unsigned char *)p.x;
    } else {
        boff[0] = (lane >> 2) * 64 + ((lane & 3) ^ (2 * (lane >> 5))) * 16;
        bk = (const unsigned char *)(p.w + ((size_t)(wave >> 1) * (p.flat / 32) + min(n0 / 32 + (wave & 1), p.flat / 32 - 1)) * (NT * 64));
    }
    const size_t bstep = WGRAD ? (size_t)32 * p.flat * 4 : (size_t)2 * (p.flat / 32) * (NT * 1024);
    const uint32_t lds = lds_address(smem);
    auto issue = [&](int kb, int slot) {
        const uint32_t at = lds + slot * STEP;
#pragma unroll
        for (int q = 0; q < NT; ++q) load_vec_to_lds(ak + kb * astep + q * 64, aoff, at + (wave * NT + q) * 1024);
        const unsigned char *b = bk + kb * bstep;
        if (WGRAD) {
            const int last = p.B - 1 - 32 * kb;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                load_vec_to_lds(b, (uint32_t)min(brow[i], last) * (uint32_t)p.flat * 4u + boff[i], at + AB + (2 * wave + i) * 1024);
        } else {
#pragma unroll
            for (int q = 0; q < NT; ++q) load_vec_to_lds(b + q * 1024, boff[0], at + AB + (wave * NT + q) * 1024);
        }
    };
    if (kb0 < kb1) issue(kb0, 0);

    // dX: the mask of my four tiles, asked for behind the first step's operands
    float4 keep[WGRAD ? 1 : 4];
    auto out_at = [&](int i, int j, bool &in) {
        const int n = n0 + 32 * (wave & 1) + 16 * i + 4 * g, m = m0 + 32 * (wave >> 1) + 16 * j + l16;
        in = n < p.flat && m < p.B;
        return in ? (size_t)m * p.flat + n : (size_t)0;
    };
    floatx4 acc[4], tot[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) { acc[j] = floatx4{0.f, 0.f, 0.f, 0.f}; tot[j] = floatx4{0.f, 0.f, 0.f, 0.f}; }
    int slot = 0, fold_at = kc - 1;
    for (int kb = kb0; kb < kb1; ++kb) {
        // this step's loads have arrived (mine here, everybody's behind the barrier) and the last step has been read
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (kb + 1 < kb1) issue(kb + 1, slot ^ 1);
        if (!WGRAD && kb == kb1 - 1)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                bool in;
                keep[WGRAD ? 0 : i] = *(const float4 *)(p.x + out_at(i >> 1, i & 1, in));
            }
        const unsigned char *at = smem + slot * STEP;
        slot ^= 1;
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};      // smallest products first
        if constexpr (WGRAD) {
            Bf16x8Bits a[4][NT], b[3];
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[e] = ((const float *)(at + AB))[(8 * g + e) * 64 + (((4 * wave + (l16 >> 2)) ^ (4 * g)) * 4 + (l16 & 3))];
            if (32 * kb + 32 > p.B) {             // no frames behind the last
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = 32 * kb + 8 * g + e < p.B ? v[e] : 0.f;
            }
            split3x8(v, b[0].u, b[1].u, b[2].u, ONE);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < NT; ++t) a[j][t].u = ((const u32x4 *)at)[(j * NT + t) * 64 + lane];
#pragma unroll
            for (int q = ONE ? 5 : 0; q < 6; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j)        // rows of the result: four consecutive columns per lane
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[PB[q]].v, a[j][PA[q] % NT].v, acc[j], 0, 0, 0);
        } else {
            Bf16x8Bits a[2][NT], b[2][NT];
            const int odd = (l16 >> 1) & 1;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                // unit 8 g + 4 h + r of the step, r = l16 / 4; columns 16 i + 4 (l16 % 4) .. of my 32
                const unsigned char *blk = at + AB + (2 * (g >> 1) + (wave & 1)) * (NT * 1024);
                const int r0 = 8 * (g & 1) + (l16 >> 2), c = 2 * i + odd;
                const int o0 = r0 * 64 + ((c ^ (2 * (g & 1))) * 16) + (l16 & 1) * 8;
#pragma unroll
                for (int t = 0; t < NT; ++t) b[i][t].u = lds_transpose8(blk + t * 1024 + o0, blk + t * 1024 + o0 + 256);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int t = 0; t < NT; ++t) {     // unit 8 g + 4 h + l16 / 4 of the step, frames 16 j + 4 (l16 % 4) .. of my 32
                    const unsigned char *q = at + ((2 * (g >> 1) + (wave >> 1)) * NT + t) * 1024 + (2 * j + odd) * 256 + (8 * (g & 1) + (l16 >> 2)) * 16 +
                                             (l16 & 1) * 8;
                    a[j][t].u = lds_transpose8(q + 64 * odd, q + 64 * (1 - odd));
                }
#pragma unroll
            for (int q = ONE ? 5 : 0; q < 6; ++q)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[2 * i + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[i][PB[q] % NT].v, a[j][PA[q] % NT].v, acc[2 * i + j], 0, 0, 0);
        }
        if (WGRAD && FOLD && (kb == fold_at || kb + 1 == kb1)) {
            fold_at += kc;
#pragma unroll
            for (int j = 0; j < 4; ++j) { tot[j] += acc[j]; acc[j] = floatx4{0.f, 0.f, 0.f, 0.f}; }
        }
    }
    if constexpr (WGRAD) {
        const int n = n0 + 16 * wave + 4 * g;
        if (n >= p.flat) return;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            *(floatx4 *)(p.dw + (FOLD ? 0 : (size_t)z * p.F * p.flat) + (size_t)(m0 + 16 * j + l16) * p.flat + n) = FOLD ? tot[j] : acc[j];
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                bool in;
                const size_t at = out_at(i, j, in);
                if (!in) continue;
                const float4 k4 = keep[2 * i + j];
                floatx4 v = acc[2 * i + j];
                v[0] = k4.x > 0.f ? v[0] : 0.f; v[1] = k4.y > 0.f ? v[1] : 0.f; v[2] = k4.z > 0.f ? v[2] : 0.f; v[3] = k4.w > 0.f ? v[3] : 0.f;
                *(floatx4 *)(p.dx + at) = v;
            }
    }
}

template <bool ONE, bool FOLD>
__global__ __launch_bounds__(256, 2) void fc_grads_kernel(const FcGradArgs p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char fc_smem[];
    const int first = DG_XCDS * (p.w_first ? p.per_w : p.per_x), bid = (int)blockIdx.x < first ? (int)blockIdx.x : (int)blockIdx.x - first;
    if (((int)blockIdx.x < first) == (p.w_first != 0)) fc_grad_block<true, ONE, FOLD>(p, bid, fc_smem);
    else fc_grad_block<false, ONE, FOLD>(p, bid, fc_smem);
}

// Whether a block of dW takes all chunks of its 64x64 tile and writes the gradient itself.  That saves the partial sums, and
// makes the chain of k-steps up to eight times as long; with a tile for every compute unit the chain is no longer than the
// launch would be anyway, with one for half of them it is until about 1000 frames (640 where a k-step is one term).  us of an
// update, one block against one per chunk: larger net (392 tiles) 320 frames 233 / 239, 1280: 503 / 520, rounded to bfloat16 308 /
// 324; stride-1 member (4624) 640: 3804 / 4022, stride-2 member (256) 945 / 951, stride-3 member (100) 496.5 / 494.5, stride-4
// member (36) 239 / 234; small net (164) 640: 113.5 / 116.3, 960: 133.6 / 136.2, 1280: 154.9 / 155.9, 2560: 256.8 / 254.0, rounded
// 640: 90.0 / 92.2, 1280: 124.4 / 121.9.  Other layers between the two lines, 960 to 1020 frames (640 rounded): small net with 320 units
// (205 tiles) 151 / 158 (100 / 104), larger net with 256 and 192 units (196 and 147) 350 / 358 and 344 / 347 (185 / 192, 183 / 186),
// stride-3 member with 384 units (150) 686 / 689 (566 / 570), stride-4 member with 1024 (144) 352 / 355 (292 / 296); at 2000 frames level.
inline bool fc_grads_fold(int F, int flat, int B, int terms) {
    const int tiles = (F + 63) / 64 * ((flat + 63) / 64);
    return tiles >= 256 || (tiles >= 128 && B <= (terms == 1 ? 640 : 1024));
}

inline hipError_t launch_fc_grads(FcGradArgs p, bool fold, int rb, hipStream_t s) {
    p.ntx = (p.B + 63) / 64; p.ntw = p.F / 64; p.ntn = (p.flat + 63) / 64;
    const int cols = (p.ntn + DG_XCDS - 1) / DG_XCDS;
    p.per_x = cols * p.ntx;
    // Every eighth column tile of W or x goes to the same XCD, whose L2 holds those columns; dW's chunks do where each XCD gets one.
    p.z_to_xcd = !fold && p.nz >= DG_XCDS;
    p.per_w = fold ? cols * p.ntw : p.z_to_xcd ? (p.nz + DG_XCDS - 1) / DG_XCDS * p.ntw * p.ntn : cols * p.ntw * p.nz;
    // dh, which every column of W meets, passes through an XCD's L2 (4 MB) once where all its columns of W fit in half of it (small
    // net 2560 frames: dX alone 33.2 -> 31.8 us, 1280 of the larger 33.5 -> 32.2; where they don't, W would pass through more often:
    // 640 x 1024 x 18496 143 -> 178).
    p.x_cols = (size_t)cols * 64 * p.F * (rb ? 2 : 6) <= (size_t)2 << 20;
    p.dntx = FastDiv(p.x_cols ? cols : p.ntx); p.dntw = FastDiv(p.ntw); p.dtw = FastDiv(p.ntw * (p.z_to_xcd ? p.ntn : p.nz));
    p.w_first = fold && p.per_w <= 3 * 256 / DG_XCDS;
    const dim3 grid(DG_XCDS * (p.per_x + p.per_w));
    if (rb && fold) ga3c::launch((fc_grads_kernel<true, true>), grid, dim3(256), fc_grads_lds<true>(), s, p);
    else if (rb) ga3c::launch((fc_grads_kernel<true, false>), grid, dim3(256), fc_grads_lds<true>(), s, p);
    else if (fold) ga3c::launch((fc_grads_kernel<false, true>), grid, dim3(256), fc_grads_lds<false>(), s, p);
    else ga3c::launch((fc_grads_kernel<false, false>), grid, dim3(256), fc_grads_lds<false>(), s, p);
    return hipGetLastError();
}

}  // namespace ga3c
