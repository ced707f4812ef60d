// The layers of conv_band.hpp and conv_bytes.hpp on the fp32 matrix instruction,
// for maps of any size (the 4x4 stride-2 layer on 32 channels, and the 8x8 byte
// layer of any stride): forward pass, and the byte layer's weight gradient for
// the strides and filter counts that conv_band_grads.hpp does not take.
//
// Every sum is formed by the same instructions in the same order as in
// gemm_mfma.hpp (v_mfma_f32_16x16x4_f32, product t of a group of 16 k sums
// k = 16 kb + 4 g + t over g, groups and t ascending), so activations and
// gradients are the same bits as those of the any-shape kernels.  In the forward
// pass of an update that matters (predictions run the 4x4 layers here too, the byte
// layer on the bf16 instruction, conv_bytes.hpp): where a pre-activation lies within rounding of
// zero, another order of the sum can put it on the other side of the rectifier,
// and a map of millions of pixels has enough of those to move the gradient of a
// filter by 1e-4 of itself.  The gradients decide nothing: an input gradient's
// mask is the stored activation, and a weight gradient feeds nothing within the
// update (conv_band_grads.hpp has them on the bf16 instruction).
//
// What bounds them is the instruction: 146 - 150 TFLOP/s on this chip.  With k
// in the filter's own order (c, u, v), the four k of a lane are four columns of
// one filter row: a 16-byte piece of a filter, and four neighbouring values (or
// bytes) of an input row.  So the input is used as it lies in memory, without
// any re-laying, and one read per lane feeds four instructions per filter tile.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include <stdint.h>

#include "conv_band.hpp"
#include "conv_bytes.hpp"

namespace ga3c {

// Forward: 4x4, stride 2, 32 channels of floats, or 8x8, any stride, four planes of bytes.  A step is 16 taps: a channel's
// filter, or two rows of a plane's.  The weights lie in LDS as fragments; the pixels of all frames are numbered on, sixteen to
// a tile, and a block takes a run of tiles, wavefront by wavefront: a lane's four columns of a step come straight from memory
// (the caches see every row several times), DEPTH steps ahead, also across tiles.  No barrier after the weights have come, no
// tile with fewer pixels but the last, and only input values in the queue of loads.
// Bound by the instruction: 640 frames, 77x77 map 281 us (379 in bands of rows that were staged in LDS, whose weights were
// read while the tiles were multiplied and so arrived behind the next band's values), 223 without the loads, 195 the products
// alone; 84x84 bytes with stride 1 555 (605), 484 without loads and conversions; 100 frames with stride 3 16 (24).
struct F32FwdGeom {
    int nframes, H, W, S, OH, OW;
    float scale;             // of the sums
    int tiles;               // of 16 pixels
    FastDiv dNPIX, dOW;
};
template <class TIn> constexpr int f32_fwd_steps() { return sizeof(TIn) == 1 ? 16 : 32; }

template <class TIn, int OC, int MT, bool LDSW, bool BITS>
__global__ __launch_bounds__(LDSW ? 512 : 4 * OC / MT, LDSW && sizeof(TIn) == 1 ? 4 : 1) void conv_f32_fwd_kernel(const TIn *__restrict__ x, const float4 *__restrict__ w,
                                                              const float *__restrict__ bias, float *__restrict__ y, const F32FwdGeom b,
                                                              const PositiveBits bits) {
    constexpr bool BYTE = sizeof(TIn) == 1;
    constexpr int C = f32_fwd_steps<TIn>(), OT = OC / 16, DEPTH = BYTE ? 8 : 16;
    typedef typename std::conditional<BYTE, uint2, float4>::type Vec;
    constexpr int NW = LDSW ? 8 * MT / OT : 1, N = LDSW ? 2 : 1;      // tiles of a round, and how many of them a wavefront has in turn
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    float4 *ws = (float4 *)band_smem;                 // [filter tile][c][lane], as in memory
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int ot = wave % (OT / MT) * MT, slot = wave / (OT / MT);      // my first filter tile
    const int HW = b.H * b.W, CHW = (BYTE ? 4 : C) * HW, NPIX = b.OH * b.OW, npix = b.nframes * NPIX;
    const int first = (int)((long)blockIdx.x * b.tiles / gridDim.x), end = (int)((long)(blockIdx.x + 1) * b.tiles / gridDim.x);

    // Where a tile's values of step 0 lie: bytes from `base`, its first frame's, lane by lane.  Bytes come with the dword that
    // they begin in and the next one, or the frame's last two; `sel` picks mine.
    auto locate = [&](int t, const TIn *&base, uint32_t &off, uint32_t &sel) {
        const int p0 = min(t * 16, npix - 1);
        const uint32_t f0 = __builtin_amdgcn_readfirstlane(b.dNPIX.div((uint32_t)p0));
        uint32_t f, rem, i, j;
        b.dNPIX.divmod((uint32_t)min(t * 16 + l16, npix - 1), f, rem);
        b.dOW.divmod(rem, i, j);
        base = x + (size_t)f0 * CHW;
        if (BYTE) {
            const uint32_t at = (i * b.S + (g >> 1)) * b.W + j * b.S + 4 * (g & 1);
            off = min(at & ~3u, (uint32_t)((b.H - 6) * b.W - 8));      // the last step's rows are six further down
            sel = 0x03020100u + 0x01010101u * (at - off);
            off += (f - f0) * (uint32_t)CHW;
        } else off = 4u * ((f - f0) * (uint32_t)CHW + (2 * i + g) * b.W + 2 * j);
    };
    Vec xv[DEPTH][N];
    auto load = [&](const TIn *base, uint32_t off, int c, Vec &d) {
        if constexpr (BYTE) {
            const uint32_t *p = (const uint32_t *)(base + ((c >> 2) * HW + 2 * (c & 3) * b.W) + off);
            d = make_uint2(p[0], p[1]);
        } else {
            const f32x4_dw v = *(const f32x4_dw *)((const char *)(base + (size_t)c * HW) + off);
            d = make_float4(v.x, v.y, v.z, v.w);
        }
    };
    auto values = [&](const Vec &d, uint32_t sel, float (&v)[4]) {
        if constexpr (BYTE) {
            const uint32_t q = __builtin_amdgcn_perm(d.y, d.x, sel);
            v[0] = (float)(q & 0xff); v[1] = (float)((q >> 8) & 0xff); v[2] = (float)((q >> 16) & 0xff); v[3] = (float)(q >> 24);
        } else {
            v[0] = d.x; v[1] = d.y; v[2] = d.z; v[3] = d.w;
        }
    };
    const TIn *base[N], *next[N];
    uint32_t off[N], noff[N], sel[N], nsel[N];
    float4 wq[LDSW ? 1 : DEPTH][MT];                  // weights that do not lie in LDS come as the values do
    auto load_w = [&](int c, float4 (&d)[MT]) {
#pragma unroll
        for (int m = 0; m < MT; ++m) d[m] = w[((ot + m) * C + c % C) * 64 + lane];
    };
    int t = first + slot;
#pragma unroll
    for (int n = 0; n < N; ++n) {
        locate(t + NW * n, base[n], off[n], sel[n]);
#pragma unroll
        for (int c = 0; c < DEPTH - 1; ++c) load(base[n], off[n], c, xv[c][n]);
    }
    if constexpr (!LDSW) {
#pragma unroll
        for (int c = 0; c < DEPTH - 1; ++c) load_w(c, wq[c]);
    } else {
#pragma unroll
        for (int e = 0; e < C * OT / 8; ++e) {
            ws[512 * e + tid] = w[512 * e + tid];
        }
    }
    const uint32_t bit_off = BITS ? (uint32_t)(l16 >> 2) * (uint32_t)bits.plane + 4 * g + (l16 & 3) : 0u;
    float bv[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) bv[m] = bias[(ot + m) * 16 + l16];
    if (LDSW) __syncthreads();

    // tiles t, t + NW, ..: NT of them; behind the last channels of these come the first ones of the next
    auto pass = [&](auto ntc) {
        constexpr int NT = decltype(ntc)::value;
        const bool more = t + NW * N < end;
#pragma unroll
        for (int n = 0; n < N; ++n) locate(min(t + NW * (N + n), end - 1), next[n], noff[n], nsel[n]);
        floatx4 acc[NT][MT];
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[n][m] = floatx4{0.f, 0.f, 0.f, 0.f};
        float4 wv[2][MT];
        auto read_w = [&](int c, float4 (&d)[MT]) {
#pragma unroll
            for (int m = 0; m < MT; ++m) d[m] = ws[((ot + m) * C + c) * 64 + lane];
        };
        if (LDSW) read_w(0, wv[0]);
        auto chunk = [&](int c0, auto lastc) {
            constexpr bool LAST = decltype(lastc)::value;
#pragma unroll
            for (int k = 0; k < DEPTH; ++k) {
                constexpr int A = DEPTH - 1;
                if (!LAST || k == 0) {
#pragma unroll
                    for (int n = 0; n < NT; ++n) load(base[n], off[n], c0 + k + A, xv[(k + A) % DEPTH][n]);
                } else if (more) {
#pragma unroll
                    for (int n = 0; n < N; ++n) load(next[n], noff[n], k - 1, xv[(k + A) % DEPTH][n]);
                }
                if constexpr (!LDSW) {
#pragma unroll
                    for (int m = 0; m < MT; ++m) wv[k & 1][m] = wq[k][m];
                    load_w(c0 + k + A, wq[(k + A) % DEPTH]);
                } else if (!LAST || k + 1 < DEPTH) read_w(c0 + k + 1, wv[(k + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                float v[NT][4];
#pragma unroll
                for (int n = 0; n < NT; ++n) values(xv[k][n], sel[n], v[n]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        const float4 q = wv[k & 1][m];
                        const float we = e == 0 ? q.x : e == 1 ? q.y : e == 2 ? q.z : q.w;
#pragma unroll
                        for (int n = 0; n < NT; ++n) acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[n][e], we, acc[n][m], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        for (int c0 = 0; c0 < C - DEPTH; c0 += DEPTH) chunk(c0, std::false_type{});
        chunk(C - DEPTH, std::true_type{});
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const int p0 = (t + NW * n) * 16 + 4 * g;
            if (t + NW * n >= end) continue;
            uint32_t f, rem;
            b.dNPIX.divmod((uint32_t)min(p0, npix - 1), f, rem);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = BYTE ? acc[n][m][r] * b.scale + bv[m] : acc[n][m][r] + bv[m];
                    v[r] = v[r] > 0.f ? v[r] : 0.f;
                }
                if constexpr (BITS) {                 // behind the rectifier a value is positive if its bits are not all zero
                    uint32_t q = 0;
#pragma unroll
                    for (int r = 3; r >= 0; --r) q = 2 * q + min(__float_as_uint(v[r]), 1u);
                    (bits.at + (size_t)(ot + m) * 4 * bits.plane + (size_t)(t + NW * n) * 16)[bit_off] = (uint8_t)q;
                }
                if ((int)rem + 3 < NPIX && p0 + 3 < npix) {
                    *(f32x4_dw *)(y + ((size_t)f * OC + (ot + m) * 16 + l16) * NPIX + rem) = f32x4_dw{v[0], v[1], v[2], v[3]};
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        uint32_t fe, re;
                        b.dNPIX.divmod((uint32_t)(p0 + r), fe, re);
                        if (p0 + r < npix) y[((size_t)fe * OC + (ot + m) * 16 + l16) * NPIX + re] = v[r];
                    }
                }
            }
        }
#pragma unroll
        for (int n = 0; n < N; ++n) { base[n] = next[n]; off[n] = noff[n]; sel[n] = nsel[n]; }
    };
    // a last round that has one tile at most for every wavefront takes half the time
    for (; end - (t - slot) > NW * (N - 1); t += NW * N) pass(std::integral_constant<int, N>{});
    if (N > 1 && t < end) pass(std::integral_constant<int, 1>{});
}

// ---------------------------------------------------------- weight gradient --
// dW[oc][k] = scale * sum over the pixels P of all frames of dY[P][oc] x[P][tap k], db[oc] = sum of dY[P][oc], in the chunks of
// pixels and the order of problems.hpp's ConvWgradP: part[chunk][OC][K + 1].  8x8 filters over four planes of bytes, any
// stride.
//
// A chunk is one long chain of sums, so the parallelism left is chunks x columns: a wavefront keeps one tile of 16 taps (two
// rows of a plane's 8x8) of all filters.  The instruction adds its four products one after
// the other, so the column of the bias gradient, whose products are dY itself, is formed with plain additions in that order,
// by one wavefront of a chunk on the side (a wavefront of its own would end last: one chain of dependent instructions).
// The chunk goes by in steps of KT pixels, whose dY lies in LDS as [filter][pixel] and whose input rows as they are in memory:
// the rows that a frame's windows touch, numbered on from frame to frame (S (OH - 1) + KS to a frame), are contiguous for any
// run of pixels, also across frames, and a table gives each pixel's place in them.  The next step's values go from memory
// straight to the other half of the LDS buffers (no registers hold them).
// Bound by the instruction next to the address and byte-conversion instructions (8 per 8 products of 32 cycles), and by whole
// wavefronts per SIMD.
constexpr int F32_WGRAD_KT = 128, F32_WGRAD_WAVES = 4;
constexpr int F32_WGRAD_MAXX = 13;                // dwords of input per thread and step
struct F32WgradGeom {
    int nframes, C, H, W, S, OH, OW;
    int K, kchunk, nz;       // pixels in all, pixels per chunk, chunks
    int ny;                  // blocks per chunk
    int rows;                // input rows of a step in LDS, at most
    int RF, d;               // rows per frame in the numbering above; frame boundaries in a step, at most
    int stage;               // bytes of one half of the LDS buffers
    FastDiv dNPIX, dOW;
    float scale;
};

template <int OC, bool RB>
__global__ __launch_bounds__(64 * F32_WGRAD_WAVES, 5) void conv_f32_wgrad_kernel(const uint8_t *__restrict__ x, const float *__restrict__ dy,
                                                                                 float *__restrict__ part, const F32WgradGeom b) {
    constexpr int OT = OC / 16, KS = 8, KT = F32_WGRAD_KT, AP = KT + 4, NW = F32_WGRAD_WAVES, NT = 64 * NW, MAXX = F32_WGRAD_MAXX;
    constexpr int NG = KT / 16;
    // each half: dY [OC][AP] floats, [KT] byte offsets of the pixels' windows, the input [row][channel][W]
    extern __shared__ __attribute__((aligned(16))) unsigned char band_smem[];
    constexpr int OTAB = OC * AP * 4, XS = OTAB + KT * 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int NPIX = b.OH * b.OW, HW = b.H * b.W;
    // an XCD takes every eighth chunk, the blocks of a chunk next to each other: its dY then comes from the L2
    const int local = (int)blockIdx.x / 8, by = local % b.ny, z = local / b.ny * 8 + (int)blockIdx.x % 8;
    if (z >= b.nz) return;
    const int q = by * NW + wave;
    const int UW = b.W / 4, UR = 4 * UW, NU = b.rows * UR, ROW = 4 * b.W;      // dwords of a row of a plane and of all; bytes
    const int kbeg = z * b.kchunk, kend = min(b.K, kbeg + b.kchunk);

    uint32_t xoff[MAXX];
    int xrow[MAXX];
#pragma unroll
    for (int i = 0; i < MAXX; ++i) {
        const int u = min(tid + NT * i, NU - 1), rem = u % UR;
        xrow[i] = u / UR;
        xoff[i] = (uint32_t)(rem / UW * HW + xrow[i] * b.W + 4 * (rem % UW));
    }
    const uint32_t jump = (uint32_t)((b.C * b.H - b.RF) * b.W);         // over the rows between two frames' channels
    const size_t xbytes = (size_t)b.nframes * b.C * HW;
    auto fetch = [&](int k0, unsigned char *half) {
        const uint32_t lds = lds_address(half);
        uint32_t f0, p0, f1, p1;
        b.dNPIX.divmod((uint32_t)k0, f0, p0);
        b.dNPIX.divmod((uint32_t)min(k0 + KT, kend) - 1, f1, p1);
        const int r0 = (int)b.dOW.div(p0) * b.S;
        const int rows = (int)(f1 - f0) * b.RF + (int)b.dOW.div(p1) * b.S + KS - r0;      // that this step's windows touch
        const int nu = rows * UR;
        const size_t xb = (size_t)f0 * b.C * HW + (size_t)r0 * b.W;
        const uint32_t lim = xbytes - xb > 0x7fffffff ? 0x7fffffffu : (uint32_t)(xbytes - xb) - 4u;
#pragma unroll
        for (int i = 0; i < MAXX; ++i)
            if (64 * wave + NT * i < nu) {
                uint32_t off = xoff[i] + (xrow[i] >= b.RF - r0 ? jump : 0u);
                if (b.d > 1)
                    for (int q = 2; q <= b.d; ++q) off += xrow[i] >= q * b.RF - r0 ? jump : 0u;
                load_dword_to_lds((const char *)x + xb, min(off, lim), lds + XS + (64 * wave + NT * i) * 4);
            }
        const float *src = dy + (size_t)f0 * OC * NPIX;
#pragma unroll
        for (int h = 0; h < KT; h += 64) {
            const int k = k0 + h + lane;
            uint32_t f, p, i, j;
            b.dNPIX.divmod((uint32_t)min(k, b.K - 1), f, p);
            const uint32_t off = 4u * ((f - f0) * (uint32_t)(OC * NPIX) + p);
#pragma unroll
            for (int m = 0; m < OC; m += NW)
                if (OC % NW == 0 || m + wave < OC) load_dword_to_lds(src + (size_t)(m + wave) * NPIX, off, lds + ((m + wave) * AP + h) * 4);
            if (wave == 0) {
                b.dOW.divmod(p, i, j);
                ((int *)(half + OTAB))[h + lane] = k < kend ? ((int)(f - f0) * b.RF + (int)i * b.S - r0) * ROW + (int)j * b.S : 0;
            }
        }
    };
    fetch(kbeg, band_smem);

    floatx4 acc[OT];
    float bsum = 0.f;
#pragma unroll
    for (int m = 0; m < OT; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    // my tap's place behind a window's first value
    const int xl = (2 * (q % 4) + (l16 >> 3)) * ROW + (q / 4) * b.W + (l16 & 7);
    int at = 0;
    for (int k0 = kbeg; k0 < kend; k0 += KT, at ^= 1) {
        unsigned char *half = band_smem + at * b.stage;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // my loads for this step have arrived in LDS
        __syncthreads();                                      // everybody's have, and the other half has been read
        if (k0 + KT < kend) fetch(k0 + KT, band_smem + (at ^ 1) * b.stage);
        else if (k0 + KT > kend) {                            // no pixels behind the chunk's last
            for (int oc = wave; oc < OC; oc += NW)
                for (int kk = lane; kk < KT; kk += 64)
                    if (k0 + kk >= kend) ((float *)half)[oc * AP + kk] = 0.f;
            __syncthreads();
        }
        const float *al = (const float *)half + l16 * AP + 4 * g;
        auto read_a = [&](int grp, float4 (&d)[OT]) {
#pragma unroll
            for (int m = 0; m < OT; ++m) {
                d[m] = *(const float4 *)(al + m * 16 * AP + 16 * grp);
                if (RB) d[m] = bf16_rne(d[m]);
            }
        };
        const int4 *ol = (const int4 *)(half + OTAB) + g;
        const unsigned char *xb = half + XS + xl;
        uint32_t xr[2][4];
        auto read_x = [&](const int4 o, uint32_t (&d)[4]) { d[0] = xb[o.x]; d[1] = xb[o.y]; d[2] = xb[o.z]; d[3] = xb[o.w]; };
        int4 o = ol[0];
        float4 av[2][OT];
        read_x(o, xr[0]);
        read_a(0, av[0]);
        o = ol[4];
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) {
            if (grp + 1 < NG) {
                read_x(o, xr[(grp + 1) & 1]);
                read_a(grp + 1, av[(grp + 1) & 1]);
                if (grp + 2 < NG) o = ol[4 * (grp + 2)];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float xv = (float)xr[grp & 1][t];
#pragma unroll
                for (int m = 0; m < OT; ++m) {
                    const float4 a = av[grp & 1][m];
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(t == 0 ? a.x : t == 1 ? a.y : t == 2 ? a.z : a.w, xv, acc[m], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (by == 0 && wave == (z & (NW - 1))) {      // the bias gradient, a filter per lane: the sums the instruction would form
            const float *bl = (const float *)half + min(lane, OC - 1) * AP;
#pragma unroll
            for (int grp = 0; grp < NG; ++grp) {
                float v[16];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float4 d = *(const float4 *)(bl + 16 * grp + 4 * e);
                    v[4 * e] = d.x; v[4 * e + 1] = d.y; v[4 * e + 2] = d.z; v[4 * e + 3] = d.w;
                }
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) bsum += RB ? bf16_rne(v[4 * e + t]) : v[4 * e + t];
            }
        }
    }
    constexpr int K1 = 257;
    float *pb = part + (size_t)z * OC * K1;
#pragma unroll
    for (int m = 0; m < OT; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) pb[(size_t)(m * 16 + 4 * g + r) * K1 + 16 * q + l16] = acc[m][r] * b.scale;
    if (by == 0 && wave == (z & (NW - 1)) && lane < OC) pb[(size_t)lane * K1 + K1 - 1] = bsum;
}

template <class TIn, int OC, int MT, bool LDSW, bool BITS>
inline hipError_t launch_conv_f32_fwd2(const TIn *x, const float4 *w, const float *bias, float *y, const PositiveBits &bits, const F32FwdGeom &b, hipStream_t s) {
    static bool attr = false;
    const hipError_t e = LDSW ? band_allow_lds(conv_f32_fwd_kernel<TIn, OC, MT, LDSW, BITS>, attr) : hipSuccess;
    if (e != hipSuccess) return e;
    constexpr int NW = 128 * MT / OC;
    // Bytes: two blocks fit a compute unit, and hide each other's conversions (640 frames of 84x84 with stride 1 551 -> 526 us), if
    // their rounds of 2 NW tiles, of which the last may be one of NW, are no more than one block's by 3 %: 320 frames with stride 3
    // 42.2 us with one, 44.7 with two, 150 with stride 2 42.7 and 45.1.
    auto turns = [&](int blocks) {
        const int per = (b.tiles + blocks - 1) / blocks, rest = per % (2 * NW);
        return per / (2 * NW) * 2 + (rest > NW ? 2 : rest > 0 ? 1 : 0);
    };
    const int blocks = sizeof(TIn) == 1 && LDSW && 64 * turns(2 * BAND_CUS) <= 33 * turns(BAND_CUS) ? 2 * BAND_CUS : BAND_CUS;
    ga3c::launch((conv_f32_fwd_kernel<TIn, OC, MT, LDSW, BITS>), dim3(LDSW ? std::min((b.tiles + NW - 1) / NW, blocks) : b.tiles),
                 dim3(LDSW ? 512 : 4 * OC / MT), LDSW ? f32_fwd_steps<TIn>() * OC * 64 : 0, s, x, w, bias, y, b, bits);
    return hipGetLastError();
}
template <class TIn, int OC, int MT, bool LDSW>
inline hipError_t launch_conv_f32_fwd1(const TIn *x, const float4 *w, const float *bias, float *y, const PositiveBits &bits, const F32FwdGeom &b, hipStream_t s) {
    if constexpr (OC == 32)
        if (bits.at) return launch_conv_f32_fwd2<TIn, OC, MT, LDSW, true>(x, w, bias, y, bits, b, s);
    return launch_conv_f32_fwd2<TIn, OC, MT, LDSW, false>(x, w, bias, y, bits, b, s);
}
// x [n][32][H][W] floats -> y [n][OC][OH][OW] of the 4x4, stride-2 layer, or [n][4][H][W] bytes of the 8x8 layer of stride S;
// w: FRAG_F32 of the filters; bits (OC == 32): also written, if given.
template <class TIn, int OC>
inline hipError_t launch_conv_f32_fwd(const TIn *x, const float4 *w, const float *bias, float *y, int n, int H, int W, int S, float scale, hipStream_t s,
                                      const PositiveBits &bits = {}) {
    if (n <= 0) return hipSuccess;
    constexpr int KS = sizeof(TIn) == 1 ? 8 : 4;
    F32FwdGeom b{};
    b.nframes = n; b.H = H; b.W = W; b.S = S; b.OH = (H - KS) / S + 1; b.OW = (W - KS) / S + 1; b.scale = scale;
    const int npix = b.OH * b.OW;
    b.tiles = (int)(((long long)n * npix + 15) / 16);
    b.dNPIX = FastDiv((uint32_t)npix); b.dOW = FastDiv((uint32_t)b.OW);
    // Few tiles: a block each, a wavefront per filter tile.  Otherwise two filter tiles per wavefront, or one where the last
    // round of blocks would be half empty with two.  640 .. 20 frames of the family's maps, us, a block per tile / one filter
    // tile / two: 32 filters, 203 tiles 5.1 / 7.8 / 11.3, 451 7.5 / 7.6 / 11.0, 902 9.2 / 8.2 / 11.6, 1440 12.7 / 13.4 / 12.2,
    // 2278 20.3 / 16.3 / 22.7, 3240 26 / 23.3 / 23.2, 54760 418 / 305 / 281; 64 filters, 250 tiles 6.4 / 8.9 / 12.5, 500
    // 10.4 / 9.6 / 13.0, 640 12.6 / 13.6 / 12.5, 1280 20 / 16.8 / 22.6, 2560 37 / 29.5 / 28.7.  (In bands of rows staged in
    // LDS: 9.4, 9.5, 15.8, 17.5, 24.9, 34.9, 384; 13.3, 21.5, 21.6, 35.9, 52.8.)
    const int half = BAND_CUS * (128 / OC), rounds = (b.tiles + half - 1) / half;
    if (b.tiles <= BAND_CUS) return launch_conv_f32_fwd1<TIn, OC, 1, false>(x, w, bias, y, bits, b, s);
    if (rounds == 1 || rounds == 3) return launch_conv_f32_fwd1<TIn, OC, 1, true>(x, w, bias, y, bits, b, s);
    return launch_conv_f32_fwd1<TIn, OC, OC == 16 ? 1 : 2, true>(x, w, bias, y, bits, b, s);
}

// b.rows: rows of input that a step can touch; it covers up to R output rows and d frame boundaries.
inline F32WgradGeom f32_wgrad_geom(int C, int H, int W, int S, int n, int kchunk, float scale) {
    constexpr int KS = 8;
    F32WgradGeom b{};
    b.nframes = n; b.C = C; b.H = H; b.W = W; b.S = S; b.OH = (H - KS) / S + 1; b.OW = (W - KS) / S + 1;
    b.K = n * b.OH * b.OW; b.kchunk = kchunk; b.scale = scale;
    b.RF = S * (b.OH - 1) + KS;
    const int R = (F32_WGRAD_KT - 2) / b.OW + 2;
    b.d = (R - 2) / b.OH + 1;
    b.rows = S * (R - 1) + KS + b.d * std::max(0, KS - S);
    b.dNPIX = FastDiv((uint32_t)(b.OH * b.OW)); b.dOW = FastDiv((uint32_t)b.OW);
    return b;
}
inline int f32_wgrad_stage(const F32WgradGeom &b, int OC) {      // the input's part rounded up to whole wavefronts
    return (OC * (F32_WGRAD_KT + 4) + F32_WGRAD_KT) * 4 + (4 * b.rows * b.W + 255) / 256 * 256;
}
// Whether a step fits the threads and half of a compute unit's LDS.
inline bool f32_wgrad_ok(int C, int H, int W, int S, int OC) {
    const F32WgradGeom b = f32_wgrad_geom(C, H, W, S, 1, F32_WGRAD_KT, 1.f);
    return b.rows * W <= 64 * F32_WGRAD_WAVES * F32_WGRAD_MAXX && 2 * f32_wgrad_stage(b, OC) <= BAND_HALF_LDS;
}
// part [nz][OC][K + 1], nz chunks of kchunk pixels (a multiple of 16).
template <int OC>
inline hipError_t launch_conv_f32_wgrad(const uint8_t *x, const float *dy, float *part, int n, int C, int H, int W, int S, int nz, int kchunk, float scale,
                                        hipStream_t s, int rb) {
    if (n <= 0) return hipSuccess;
    F32WgradGeom b = f32_wgrad_geom(C, H, W, S, n, kchunk, scale);
    b.stage = f32_wgrad_stage(b, OC);
    b.nz = nz; b.ny = 16 / F32_WGRAD_WAVES;
    const dim3 grid((nz + 7) / 8 * 8 * b.ny), block(64 * F32_WGRAD_WAVES);
    const int lds = 2 * b.stage;
    static bool attr0 = false, attr1 = false;
    if (rb) {
        const hipError_t e = band_allow_lds(conv_f32_wgrad_kernel<OC, true>, attr1);
        if (e != hipSuccess) return e;
        ga3c::launch((conv_f32_wgrad_kernel<OC, true>), grid, block, lds, s, x, dy, part, b);
    } else {
        const hipError_t e = band_allow_lds(conv_f32_wgrad_kernel<OC, false>, attr0);
        if (e != hipSuccess) return e;
        ga3c::launch((conv_f32_wgrad_kernel<OC, false>), grid, block, lds, s, x, dy, part, b);
    }
    return hipGetLastError();
}

}  // namespace ga3c
