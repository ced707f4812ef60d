// Forward product of the fully connected layer on the bf16 matrix cores at
// fp32 accuracy (dense_gemm_bf16x6.hpp has the error argument):
//
//   part[z][b][o] = sum_{k in chunk z} x[b][k] W[o][k]
//
// with the weights as ready-made operands: split into three bf16 terms once per
// parameter copy, in the order in which the matrix instruction takes them.  The
// sums are those of dense_gemm_bf16x6_kernel, in its order.
//
// Reading x and W as fp32 and splitting both in every block, that kernel was
// bound by the latency of one load per k-step and by the splitting: 16 us for
// 1024 x 256 x 2592 with 3.2 us of products.  Here nothing passes through
// registers on its way to LDS, so a k-step is under way while the last one is
// multiplied: a wavefront asks for the weights of a quarter of the columns and for
// its own 16 MT rows of x, still fp32; it is the only one that uses those rows and
// splits them as it reads them (three steps in LDS against the kernel above: 1024
// frames 16.0 -> 11.3 us, 512 10.4 -> 8.6, 2560 30.1 -> 25.7, 256 of the larger net
// 11.7 -> 9.3).  How many steps are in LDS is chosen per launch: fc_forward_steps.
// What is left is LDS reads (14 per wavefront and k-step of 384 cycles of products)
// and, at small batches, start and end of the launch.  32 rows per wavefront read
// less but left one block per compute unit (12.5 us at 1024 frames).
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include "dense_gemm_bf16x6.hpp"

namespace ga3c {

constexpr int FC_BN = 64;                     // columns of a block: four tiles

struct FcForwardArgs {
    int M, N, K;
    int kchunk, nz;                           // k is cut into nz chunks of kchunk; K and kchunk are multiples of 32
    FastDiv tiles, cols;                      // row x column tiles of a chunk; column tiles
    const float *x;                           // [M][K]
    const u32x4 *w;                           // [N / 16][K / 32][terms][16 rows][32 k] bf16
    float *part;                              // [nz][M][N]
};

// The weights as operands of both copies' forward product, and where they come from: vectors of four in the flat parameters.
struct FcPlanes {
    u32x4 *w;                                 // nullptr: none
    unsigned first, n;                        // first vector of the tensor; vectors in it
    int kblocks, terms;                       // K / 32; 3, or 1 (rounded to bfloat16)
    FastDiv row;                              // by K / 4
};
// Vector i of the tensor.  A row's 32 k of a block lie together (64 bytes a term), so the threads that update them, eight in a
// row, write whole memory sectors; the order in which a lane takes them would scatter them by 16 bytes.  The sixteen rows of a
// term follow each other, so that a load of a wavefront is 1 KB without gaps (640 x 1024 x 18496: 159 -> 149 us; with a row's
// three terms together it was sixteen pieces of 64 bytes).
__device__ __forceinline__ void fc_planes_store4(const FcPlanes &p, unsigned i, const float4 v) {
    const unsigned o = p.row.div(i), q = i - o * p.row.d;
    unsigned char *dst = (unsigned char *)p.w + (size_t)(((o >> 4) * p.kblocks + (q >> 3)) * p.terms) * 1024 + ((o & 15) * 64 + (q & 7) * 8);
    uint2 t[3];
    split3_pair(v.x, v.y, t[0].x, t[1].x, t[2].x);
    split3_pair(v.z, v.w, t[0].y, t[1].y, t[2].y);
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (k < p.terms) *(uint2 *)(dst + 1024 * k) = t[k];
}
__global__ __launch_bounds__(256) void fc_planes_kernel(const float4 *__restrict__ theta, const FcPlanes p) {
    const unsigned i = blockIdx.x * 256 + threadIdx.x;
    if (i < p.n) fc_planes_store4(p, i, theta[p.first + i]);
}

// NS: k-steps of 32 in LDS (20 KB each, with one term 12 KB).
template <bool ONE, int NS>
constexpr int fc_forward_lds() { return NS * (4 * 2048 + 4 * (ONE ? 1 : 3) * 1024); }

// ONE: operands rounded to bfloat16 (one term).
template <bool ONE, int NS>
__global__ __launch_bounds__(256, 2) void fc_forward_kernel(const FcForwardArgs p) {
    constexpr int NTERM = ONE ? 1 : 3, XB = 4 * 2048, WB = 4 * NTERM * 1024, LOADS = 2 + NTERM;
    extern __shared__ __attribute__((aligned(16))) unsigned char fc_smem[];    // [step][x: wavefront, row, k | w: column tile, term, lane]
    // chunk z belongs to XCD z % 8, whose L2 then holds one slice of the weights
    const int local = blockIdx.x / DG_XCDS, zi = p.tiles.div(local), t = local - zi * (int)p.tiles.d;
    const int z = zi * DG_XCDS + blockIdx.x % DG_XCDS;
    if (z >= p.nz) return;
    const int tm = p.cols.div(t), m0 = tm * 64, n0 = (t - tm * (int)p.cols.d) * FC_BN;
    const int kbeg = z * p.kchunk, nkb = (min(p.K, kbeg + p.kchunk) - kbeg) / 32;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;

    // an eighth of the lanes takes the 128 bytes of a row; 16-byte piece c of row r lies at place c ^ (r % 8) of the row, so
    // that the lanes of a tile, which all want the same piece, find it in different banks
    uint32_t xoff[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = min(m0 + wave * 16 + 8 * i + lane / 8, p.M - 1);
        xoff[i] = (uint32_t)row * (uint32_t)p.K * 4u + (uint32_t)(((lane & 7) ^ (lane >> 3)) * 16);
    }
    const unsigned char *xk = (const unsigned char *)(p.x + kbeg);
    const unsigned char *wk = (const unsigned char *)(p.w + ((size_t)(n0 / 16 + wave) * (p.K / 32) + kbeg / 32) * (NTERM * 64));
    const uint32_t woff = l16 * 64 + g * 16;
    const uint32_t lds = lds_address(fc_smem);
    auto issue = [&](int kb, int slot) {
        const uint32_t at = lds + slot * (XB + WB);
#pragma unroll
        for (int i = 0; i < 2; ++i) load_vec_to_lds(xk + (size_t)kb * 128, xoff[i], at + wave * 2048 + i * 1024);
#pragma unroll
        for (int q = 0; q < NTERM; ++q)
            load_vec_to_lds(wk + (size_t)kb * (NTERM * 1024) + q * 1024, woff, at + XB + (wave * NTERM + q) * 1024);
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < nkb) issue(s, s);

    floatx4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    int slot = 0;
    for (int kb = 0; kb < nkb; ++kb) {
        // this step's loads have arrived (mine here, everybody's behind the barrier) and the last step has been read
        if (kb + NS - 2 < nkb) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LOADS * (NS - 2)) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (kb + NS - 1 < nkb) issue(kb + NS - 1, slot == 0 ? NS - 1 : slot - 1);
        const unsigned char *at = fc_smem + slot * (XB + WB);
        slot = slot == NS - 1 ? 0 : slot + 1;
        Bf16x8Bits a[3], b[4][NTERM];
        float4 f[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) f[h] = ((const float4 *)(at + wave * 2048))[l16 * 8 + ((2 * g + h) ^ (l16 & 7))];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < NTERM; ++q) b[j][q].u = ((const u32x4 *)(at + XB))[(j * NTERM + q) * 64 + lane];
        const float v[8] = {f[0].x, f[0].y, f[0].z, f[0].w, f[1].x, f[1].y, f[1].z, f[1].w};
        split3x8(v, a[0].u, a[1].u, a[2].u);
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};      // smallest products first
#pragma unroll
        for (int q = ONE ? 5 : 0; q < 6; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j)        // rows of the result: four consecutive columns per lane
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][PB[q] % NTERM].v, a[PA[q]].v, acc[j], 0, 0, 0);
    }
    const int m = m0 + wave * 16 + l16;
    if (m >= p.M) return;
    float *dst = p.part + ((size_t)z * p.M + m) * p.N + n0 + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) *(floatx4 *)(dst + 16 * j) = acc[j];
}

// What the 16-byte loads and whole tiles need; offsets into x are 32 bits.
inline bool fc_forward_ok(int K, int N) { return K % 32 == 0 && N % FC_BN == 0; }
inline bool fc_forward_batch_ok(const float *x, int M, int K) { return (uintptr_t)x % 16 == 0 && (size_t)M * K * 4 < (size_t)1 << 32; }

// k-steps in LDS: with three, two are on their way while one is multiplied; with two, more blocks fit a compute unit and hide each
// other's waits (three terms: four blocks instead of two; one term: six instead of four).  Two steps against three, us of the
// launch, medians of 30 to 40 calls:
// Three terms.  Up to 256 blocks a block has a compute unit to itself and waits for memory alone: stride-1 member 32 frames 25.9 /
// 24.4, stride-2 member 256: 8.1 / 7.8, larger net 128: 7.7 / 7.4.  From two blocks a unit on two steps are ahead: small net 512
// frames (512 blocks) 9.2 / 10.2, 700: 11.1 / 12.9, larger net 256: 9.7 / 10.6, 10368 columns x 1024 units 256: 32.4 / 34.1, stride-1
// member 192 (768 blocks): 56.0 / 60.3, update of the small net 640: 10.6 / 12.9, 2560: 24.7 / 27.9, larger net 1280: 29.0 / 31.6 -
// unless there are two blocks a unit at most and the weights come from HBM because the activations in front of them no longer leave
// them in the 256 MB of the Infinity Cache: stride-1 member 128 frames (114 + 129 MB) 36.9 / 35.4
// (medians of eleven runs, 33 - 40 / 30 - 39), 256 (114 + 258): 68.8 / 67.1, with 512 units 200 (57 + 202): 35.5 / 31.1; not yet with
// 112 frames (114 + 113): 28.8 / 29.8, nor with 20736 columns x 1024 units at 256 (127 + 71): 59.9 / 63.2.
// One term.  Four blocks fit with three steps already, and three are ahead up to three blocks a unit: small net 256 frames 6.3 / 5.1,
// 512: 8.0 / 6.7, 1024: 8.8 / 6.7, larger net 128: 6.8 / 5.4, 512: 9.9 / 7.7, stride-1 member 128: 21.0 / 14.9, 256: 49.2 / 30.8,
// update of the small net 1280 (640 blocks) 9.4 / 8.9.  Above that two are ahead or level: larger net 400 frames (896) 9.6 / 10.1,
// its update of 1280 (1280) 14.5 / 15.1, small net 2250 (1152) 13.1 / 13.8, 2560: 14.0 / 13.7.
inline int fc_forward_steps(bool one, unsigned blocks, size_t weight_bytes, size_t pass_bytes) {
    constexpr unsigned CUS = 256;
    if (one) return blocks <= 3 * CUS ? 3 : 2;
    const bool from_hbm = weight_bytes + pass_bytes > (size_t)230 << 20;
    return blocks <= (from_hbm ? 2 * CUS : CUS) ? 3 : 2;
}

// pass_bytes: the activations that the forward pass has written in front of this product.
inline hipError_t launch_fc_forward(FcForwardArgs p, size_t pass_bytes, int rb, hipStream_t s) {
    const int ntm = (p.M + 63) / 64, ntn = p.N / FC_BN;
    p.tiles = FastDiv(ntm * ntn); p.cols = FastDiv(ntn);
    const unsigned blocks = DG_XCDS * ((p.nz + DG_XCDS - 1) / DG_XCDS) * ntm * ntn;
    auto go = [&](auto kernel, int lds) { ga3c::launch(kernel, dim3(blocks), dim3(256), lds, s, p); };
    if (fc_forward_steps(rb != 0, blocks, (size_t)p.N * p.K * 2 * (rb ? 1 : 3), pass_bytes) == 3)
        rb ? go(fc_forward_kernel<true, 3>, fc_forward_lds<true, 3>()) : go(fc_forward_kernel<false, 3>, fc_forward_lds<false, 3>());
    else rb ? go(fc_forward_kernel<true, 2>, fc_forward_lds<true, 2>()) : go(fc_forward_kernel<false, 2>, fc_forward_lds<false, 2>());
    return hipGetLastError();
}

}  // namespace ga3c
