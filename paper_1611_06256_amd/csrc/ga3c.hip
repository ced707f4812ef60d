// GA3C hot path on MI355X (gfx950): the C ABI declared in include/ga3c.h and
// the kernels behind it that are not matrix products (heads + softmax +
// sampling, returns + loss, reductions, RMSProp, parameter initialisation).
// The matrix products are instances of gemm_mfma.hpp / problems.hpp.
#include <hip/hip_runtime.h>

#include "launch.hpp"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/ga3c.h"
#include "frame_table.hpp"
#include "problems.hpp"
#include "conv_frame.hpp"
#include "dense_gemm.hpp"
#include "conv1_bf16x3.hpp"
#include "conv1_wgrad_f16.hpp"
#include "dense_gemm_bf16x6.hpp"
#include "fc_forward.hpp"
#include "fc_grads.hpp"
#include "conv2_bf16x6.hpp"
#include "conv12_fused.hpp"
#include "conv12_f16.hpp"
#include "conv_fwd_bf16x6.hpp"
#include "conv123_f16.hpp"
#include "conv_dgrad_bf16x6.hpp"
#include "conv_grads.hpp"
#include "conv_wgrad_f16.hpp"
#include "conv_wgrad_s1_f16.hpp"
#include "conv_band.hpp"
#include "conv_bytes.hpp"
#include "conv_band_f32.hpp"
#include "conv_band_grads.hpp"

using namespace ga3c;

// Fixed-geometry kernels exist for the layers of the paper's networks.
typedef ConvSpec<uint8_t, 4, 84, 84, 16, 8, 4> SpecS1;    // small net, conv1
typedef ConvSpec<float, 16, 20, 20, 32, 4, 2> SpecS2;     // small net, conv2
typedef ConvSpec<uint8_t, 4, 84, 84, 32, 8, 4> SpecL1;    // large net, conv1
typedef ConvSpec<float, 32, 20, 20, 64, 4, 2> SpecL2;     // large net, conv2
typedef ConvSpec<float, 64, 9, 9, 64, 3, 1> SpecL3;       // large net, conv3
typedef ConvSpec<float, 32, 20, 20, 32, 4, 2> SpecP2;     // the paper's larger-network family (Sec. 5), stride-4 member, conv2
// 16-byte vectors of a small-net fragment buffer: the filters of conv1 / conv2 for the fused forward kernel, then
// those of conv2 for its input-gradient kernel
constexpr int CFRAG_FWD_VECS = 3 * C12_FRAG_SET, CFRAG_VECS = CFRAG_FWD_VECS + ConvDgradBf16Geom<SpecS2>::FRAG_VECS;
// parts of a larger-net fragment buffer: conv2 forward, conv2 input gradient, conv3 forward, conv3 input gradient; then (at
// LFRAG_VECS) all three layers for predictions, in a context that predicts at fp32 accuracy
constexpr int LFRAG_FWD2 = 0, LFRAG_DGRAD2 = LFRAG_FWD2 + ConvFwdBf16Geom<SpecL2>::FRAG_VECS,
              LFRAG_FWD3 = LFRAG_DGRAD2 + ConvDgradBf16Geom<SpecL2>::FRAG_VECS, LFRAG_DGRAD3 = LFRAG_FWD3 + ConvFwdBf16Geom<SpecL3>::FRAG_VECS,
              LFRAG_VECS = LFRAG_DGRAD3 + conv_dgrad_s1_frag_vecs<SpecL3>();

// Networks whose predictions run their three convolutions in one kernel: the larger one, the family's members of stride 4 and 3
// (the other members' first maps do not fit a compute unit's LDS).
typedef ConvSpec<float, 32, 9, 9, 64, 4, 2> SpecP43;
typedef ConvSpec<float, 32, 26, 26, 32, 4, 2> SpecP32;
typedef ConvSpec<float, 32, 12, 12, 64, 4, 2> SpecP33;
typedef Conv123Net<4, SpecL2, SpecL3, false> Conv123Large;
typedef Conv123Net<4, SpecP2, SpecP43, false> Conv123Paper4;
typedef Conv123Net<3, SpecP32, SpecP33, true> Conv123Paper3;
enum { CONV123_NONE = 0, CONV123_LARGE, CONV123_PAPER4, CONV123_PAPER3 };

// All parts in one launch (w1, w2, w3: the filter tensors); the last in LFRAG_B3 .. LFRAG_B3 + Conv123Large::BLOCKS.
typedef ConvSpec<float, SpecL3::OC, SpecL3::OH + 2 * (SpecL3::KS - 1), SpecL3::OW + 2 * (SpecL3::KS - 1), SpecL3::C, SpecL3::KS, 1> SpecL3Dgrad;
constexpr int LFRAG_B0 = ConvFwdBf16Geom<SpecL2>::KB, LFRAG_B1 = LFRAG_B0 + (SpecL2::OC * SpecL2::C * 4 + 255) / 256,
              LFRAG_B2 = LFRAG_B1 + ConvFwdBf16Geom<SpecL3>::KB, LFRAG_B3 = LFRAG_B2 + ConvFwdBf16Geom<SpecL3Dgrad>::KB;
__global__ __launch_bounds__(256) void large_filter_fragments_kernel(const float *__restrict__ w1, const float *__restrict__ w2,
                                                                     const float *__restrict__ w3, u32x4 *__restrict__ lfrag) {
    const int b = blockIdx.x, t = threadIdx.x;
    if (b < LFRAG_B0) conv_fwd_filter_fragments_thread<SpecL2, false>(w2, lfrag + LFRAG_FWD2, b * 256 + t);
    else if (b < LFRAG_B1) {
        const int i = (b - LFRAG_B0) * 256 + t;
        if (i < SpecL2::OC * SpecL2::C * 4) conv_dgrad_store_fragment4<SpecL2>(lfrag + LFRAG_DGRAD2, 4 * i, ((const float4 *)w2)[i]);
    } else if (b < LFRAG_B2) conv_fwd_filter_fragments_thread<SpecL3, false>(w3, lfrag + LFRAG_FWD3, (b - LFRAG_B1) * 256 + t);
    else if (b < LFRAG_B3) conv_fwd_filter_fragments_thread<SpecL3Dgrad, true>(w3, lfrag + LFRAG_DGRAD3, (b - LFRAG_B2) * 256 + t);
    else conv123_fragments_block<Conv123Large>(w1, w2, w3, lfrag + LFRAG_VECS, b - LFRAG_B3);
}
// The family's fragments (jobs) and, in front of them, N's.
template <class N>
__global__ __launch_bounds__(256) void family_filter_fragments_kernel(const float *__restrict__ w1, const float *__restrict__ w2,
                                                                      const float *__restrict__ w3, u32x4 *__restrict__ frag, const FragJobs jobs) {
    if (blockIdx.x < N::BLOCKS) conv123_fragments_block<N>(w1, w2, w3, frag, blockIdx.x);
    else band_filter_fragments_block<3>(jobs, blockIdx.x - N::BLOCKS);
}

// ---------------------------------------------------------------- errors ----

static thread_local char g_err[512] = "";

static int fail(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

#define HIP_TRY(expr)                                                                   \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess)                                                           \
            return fail(e_ == hipErrorOutOfMemory ? GA3C_ENOMEM : GA3C_EHIP, "%s: %s", \
                        #expr, hipGetErrorString(e_));                                  \
    } while (0)

extern "C" const char *ga3c_last_error(void) { return g_err; }

// ---------------------------------------------------------------- context ---

namespace {

constexpr int LOSS_THREADS = 64;    // frames per block in the returns/loss kernel

struct Work {            // activations of one call; predict and train own one each
    int cap = 0;         // frames
    float *act[GA3C_MAX_CONV] = {nullptr, nullptr, nullptr, nullptr};   // conv outputs, NCHW, post-ReLU
    float *h = nullptr;  // fc output [cap][F], post-ReLU
    float *zv = nullptr; // logits and value [cap][A+1]
    float *ws = nullptr; // split-k partial products of this call
    size_t ws_floats = 0;
    const float *fc_ws = nullptr;   // where the last forward left the fc partial sums, and how many
    int fc_nz = 1;
    // which conv outputs are positive, where the next layer's input gradient wants bits, and whether this forward pass has left them
    PositiveBits bits[GA3C_MAX_CONV];
    bool bits_set[GA3C_MAX_CONV] = {false, false, false, false};
};

}  // namespace

namespace {
// Optional per-stage timing: the execution times of the kernels of each stage (an event pair per launch).
struct ProfStage { const char *name; long calls; double ms, flop, bytes; };
struct ProfRec { int stage, stage2; hipEvent_t a, b; };      // stage2 >= 0: the launch does the work of two stages
struct Profiler {
    bool on = false;
    std::vector<ProfStage> stages;
    std::vector<ProfRec> recs;          // recorded, not yet read
    std::vector<hipEvent_t> pool;       // idle events
};
}  // namespace

namespace {
// An event and where it was last recorded (the handle is only ever compared).
struct Mark {
    hipEvent_t ev;
    hipStream_t where;
    bool set;
};
// Predictions of a parameter copy since it was written: none, some that no event stands behind yet, all behind an event.
enum Reads { READS_NONE, READS_OPEN, READS_MARKED };
}  // namespace

struct ga3c_ctx {
    Profiler *prof;
    bool fast;                    // use the fixed-geometry kernels where they apply
    int small_frames;             // predictions of up to so many frames go out as one launch (small_launch_frames)
    int rb;                       // desc.math == 1: operands of every contraction are rounded to bfloat16
    ga3c_net_desc desc;
    int nconv, F, A, flat;
    ConvGeom geom[GA3C_MAX_CONV];
    int *koff[GA3C_MAX_CONV];
    int64_t off[2 * GA3C_MAX_CONV + 7];
    int noff;
    size_t P;
    int max_pred, max_train;
    // Two copies of the parameters.  theta2[cur] is the published one, which every call reads; a writer (an update,
    // params_init, params_set) writes the other one, or in place (copy_to_write), and publishes it.
    float *theta2[2];
    int cur;
    Reads reads[2];               // of copy i by predictions
    Mark ready[2];                // copy i has been written
    Mark turned;                  // all predictions of the copy that is not published are over (READS_MARKED)
    Mark copied[2];               // all params_get of copy i are over
    float *g, *grad;
    // small net: conv1/conv2 filters of each parameter copy as split MFMA fragments (nullptr for other nets), forward
    // kernel's first, then (at CFRAG_FWD_VECS) the input-gradient kernel's; refreshed by whoever writes the copy
    u32x4 *cfrag[2];
    u32x4 *hfrag[2];              // the same filters for predictions at fp32 accuracy of more frames than one launch takes (conv12_f16.hpp), kept
                                  // current likewise; nullptr in a context that makes none
    bool cfrag_dgrad;             // the buffers hold the second part too (a context that can train)
    // larger net: the filters of conv2 and conv3 of each parameter copy as ready-made fragments for the forward and the
    // input-gradient kernels (LFRAG_* give the parts); rebuilt by whoever writes the copy
    u32x4 *lfrag[2];
    // predictions run the network's three convolutions in one kernel (CONV123_..), whose filters lie in lfrag at LFRAG_VECS or in bfrag
    // at bfrag_123
    int conv123;
    size_t bfrag_123;
    // layers on the any-size kernels of conv_band.hpp and conv_bytes.hpp: which ones, where their fragments sit in the
    // buffer of each parameter copy (in vectors), and the buffers (nullptr where no layer needs one)
    bool band[GA3C_MAX_CONV];
    size_t bfrag_fwd[GA3C_MAX_CONV], bfrag_f32[GA3C_MAX_CONV], bfrag_dgrad[GA3C_MAX_CONV], bfrag_vecs;
    u32x4 *bfrag[2];
    ga3c::FcPlanes fcw[2];        // fc weights of each parameter copy as operands of the forward product (w == nullptr: none); kept
                                  // current by whoever writes the copy
    bool fold_ok;                 // the fc weight gradient can be written without partial sums (fc_grads.hpp)
    int *ticket;                  // predict_small_kernel's per-frame counters, zero between launches
    Work pred, train;
    // training only
    float *dact[GA3C_MAX_CONV];   // dL/d(pre-activation) of each conv output
    float *dh;                    // dL/d(pre-activation) of the fc output
    ga3c::FcDhPlanes dhp;         // dh as operands of the fc gradients (w == nullptr: none)
    float *dzv;                   // dL/d(logits, value) [cap][A+1]
    float *R;                     // returns [cap]
    float *partials;              // one squared-norm partial per reduce block, then 3 per loss block
    int max_norm_parts;
    float *colpart;               // per-block column sums of dh [cap/HD_FRAMES + 1][F]
    float *scale;                 // clip scale of the last step (1 float)
    ga3c_train_stats *stats;      // stats of the last step
    int last_frames;
};

namespace {

// ------------------------------------------------------------ small kernels -

// Wavefront-wide sum and max in registers: butterflies inside each row of 16
// lanes with DPP (quad permutes, then the two mirror patterns), then the four
// row results are combined through scalar registers.  Every lane gets the
// result; no LDS traffic, unlike __shfl_xor.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_f32(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_f32<0xB1>(v);      // quad_perm [1,0,3,2]
    v += dpp_f32<0x4E>(v);      // quad_perm [2,3,0,1]
    v += dpp_f32<0x141>(v);     // row_half_mirror
    v += dpp_f32<0x140>(v);     // row_mirror
    return (lane_f32(v, 0) + lane_f32(v, 16)) + (lane_f32(v, 32) + lane_f32(v, 48));
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_f32<0xB1>(v));
    v = fmaxf(v, dpp_f32<0x4E>(v));
    v = fmaxf(v, dpp_f32<0x141>(v));
    v = fmaxf(v, dpp_f32<0x140>(v));
    return fmaxf(fmaxf(lane_f32(v, 0), lane_f32(v, 16)), fmaxf(lane_f32(v, 32), lane_f32(v, 48)));
}

// Sums over a row's 16 lanes of two or four values at once: lane l of every row ends up with its row's sum of value l % N.
// (Pairs of values trade halves first, so N values cost little more than one.)
__device__ __forceinline__ float row_sums(const float (&v)[2], const int lane) {
    const bool odd = lane & 1;
    float t = (odd ? v[1] : v[0]) + dpp_f32<0xB1>(odd ? v[0] : v[1]);      // quad_perm [1,0,3,2]
    t += dpp_f32<0x4E>(t);      // quad_perm [2,3,0,1]
    t += dpp_f32<0x124>(t);     // row_ror:4
    return t + dpp_f32<0x128>(t);
}
__device__ __forceinline__ float row_sums(const float (&v)[4], const int lane) {
    const bool odd = lane & 1, up = lane & 2;
    const float a = (odd ? v[1] : v[0]) + dpp_f32<0xB1>(odd ? v[0] : v[1]), b = (odd ? v[3] : v[2]) + dpp_f32<0xB1>(odd ? v[2] : v[3]);
    float t = (up ? b : a) + dpp_f32<0x4E>(up ? a : b);
    t += dpp_f32<0x124>(t);
    return t + dpp_f32<0x128>(t);
}
// The sum over the four rows of what lanes 16 r + l hold, in each of them.
__device__ __forceinline__ float across_rows(float v) {
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

// Global memory answers in roughly half a microsecond, so short kernels are
// bound by the number of dependent load rounds, not by bytes.  These helpers
// issue a batch of independent loads (indices past the end are clamped, the
// values then ignored) before any of them is used.
template <int BATCH>
__device__ __forceinline__ void copy_to_lds(float *dst, const float *__restrict__ src, int n, int tid, int nthreads) {
    for (int e0 = 0; e0 < n; e0 += BATCH * nthreads) {
        float v[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) v[j] = src[min(e0 + j * nthreads + tid, n - 1)];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int idx = e0 + j * nthreads + tid;
            if (idx < n) dst[idx] = v[j];
        }
    }
}

// A division by a constant as a FastDiv, for code that takes either.
template <uint32_t D>
struct FastDivConst {
    static __device__ __forceinline__ FastDiv get() {
        static_assert((D & (D - 1)) == 0, "a power of two");
        FastDiv f = {};
        f.d = D; f.mul = 1; f.shift = 31 - __builtin_clz(D);
        return f;
    }
};

// Policy and value heads (Sec. 3.2: softmax policy output, linear value
// output), then softmax and inverse-CDF sampling; optionally preceded by the
// last step of a split-k fully connected layer.  A block takes 4 frames.
//   ws != null: h[b][o] = max(0, bias[o] + sum_z ws[z][b][o]) is formed first
//               (and written to h); otherwise h is read.
//   h [B][F]; Wp [A][F], bp [A], Wv [F], bv [1].  zv [B][A+1] is written when
//   not null (training keeps it); logits / values / probs / actions are the
//   caller's optional outputs.
// Dynamic LDS: heads_lds_floats(F, A) floats: the 4 rows of h, both weight
// matrices (rows padded to a multiple of 4 plus 4, so that rows start 16-byte
// aligned in different banks), the partial dot products.  Global memory answers
// in about a microsecond, so every load a thread needs (weights, partial sums,
// biases, its uniform number) is issued before the first one is used.
__host__ __device__ inline int heads_f4(int F) { return (F + 3) / 4 * 4; }
__host__ __device__ inline int heads_lds_floats(int F, int A) { return 4 * heads_f4(F) + (A + 1) * (heads_f4(F) + 4 + 12); }

// The columns F .. WP - 1 (at most seven) of `rows` rows of the heads' weights in LDS.
template <int NT>
__device__ __forceinline__ void heads_zero_padding(float *wsh, const int t, int F, int WP, int rows) {
    for (int r = t >> 3; r < rows; r += NT / 8)
        if ((t & 7) < WP - F) wsh[r * WP + F + (t & 7)] = 0.f;
}

// The loads of a heads block as 16-byte vectors (a quarter of the load instructions: a wavefront spends about a
// hundred cycles issuing each one, whatever its width): the split-k partial sums of the fc layer for NF frames are
// added up in chunk order, bias and ReLU follow, the result goes to h and (rounded if rb) to hs [NF][F4]; the heads'
// weights go to wsh [A+1][WP] (the value head's row with 4-byte loads: it follows the policy biases in the parameter
// vector and is not aligned).  Needs F % 4 == 0 and 16-byte aligned pointers (heads_loads).
// What it takes is rounds of latency, so the weights, the biases and the partial sums of IP outputs per thread, CH chunks
// each, are all requested before the first of them is used: one round where the chunks fit CH and the outputs IP (training
// on 40 frames, 40 chunks: the block's loads 7.5 us when every output and every eight chunks were a round of their own).
// A block runs these kernels' code once and fetches it from memory as it goes, so each way to load is a kernel of its own
// (LOADS) instead of a branch.
// any shape; 16-byte vectors, of at most 8 chunks and of more (16 at a time; heads_train_kernel takes 28 or 20)
enum { LOADS_SCALAR = 0, LOADS_VEC8 = 1, LOADS_VEC16 = 2 };
inline int heads_loads(int F, int nz, const void *ws, const void *fcb, const void *h, const void *Wp) {
    if (F % 4 != 0 || !ws || (((uintptr_t)ws | (uintptr_t)fcb | (uintptr_t)h | (uintptr_t)Wp) & 15) != 0) return LOADS_SCALAR;
    return nz <= 8 ? LOADS_VEC8 : LOADS_VEC16;
}
// meanwhile(): called once by every thread, also where it has no output, between the first requests and their use.
template <int NT, int NF, int CH, int IP, class Meanwhile>
__device__ __forceinline__ void heads_load_vec4(float *hs, float *wsh, const int tid, const int b0, const int nf,
                                                const float *__restrict__ ws, int nz, const float *__restrict__ fcb,
                                                float *__restrict__ h, int B, int F, int F4, int WP, int A,
                                                const float *__restrict__ Wp, const float *__restrict__ Wv, int rb, const FastDiv dFQ,
                                                Meanwhile meanwhile) {
    constexpr int WQ = 8, WVQ = 2;
    const int FQ = F >> 2, nwq = A * FQ, nit = NF * FQ;
    const size_t stride4 = (size_t)B * FQ;
    float4 wv4[WQ];
    float wv[WVQ];
#pragma unroll
    for (int j = 0; j < WQ; ++j) wv4[j] = ((const float4 *)Wp)[min(j * NT + tid, nwq - 1)];
#pragma unroll
    for (int j = 0; j < WVQ; ++j) wv[j] = Wv[min(j * NT + tid, F - 1)];
    for (int it0 = tid; it0 == tid || it0 < nit; it0 += IP * NT) {
        // output it of the block is vector b0 * FQ + it of a chunk's sums
        const float4 *src = (const float4 *)ws + (size_t)b0 * FQ;
        float4 bias[IP], acc[IP];
        uint32_t off[IP];
#pragma unroll
        for (int p = 0; p < IP; ++p) {
            off[p] = (uint32_t)min(it0 + p * NT, nf * FQ - 1);
            uint32_t fb, oq;
            dFQ.divmod(off[p], fb, oq);
            bias[p] = ((const float4 *)fcb)[oq];
            acc[p] = float4{0.f, 0.f, 0.f, 0.f};
        }
        for (int z = 0; z < nz; z += CH) {
            float4 v[IP][CH];
#pragma unroll
            for (int i = 0; i < CH; i += 4)
                if (z + i < nz) {
#pragma unroll
                    for (int p = 0; p < IP; ++p)
#pragma unroll
                        for (int j = i; j < i + 4; ++j) v[p][j] = (src + (size_t)min(z + j, nz - 1) * stride4)[off[p]];
                }
            __builtin_amdgcn_sched_barrier(0);
            if (z == 0 && it0 == tid) meanwhile();
#pragma unroll
            for (int i = 0; i < CH; i += 4)
                if (z + i < nz) {
#pragma unroll
                    for (int j = i; j < i + 4; ++j) {
                        const bool in = z + j < nz;
#pragma unroll
                        for (int p = 0; p < IP; ++p) {
                            acc[p].x += in ? v[p][j].x : 0.f; acc[p].y += in ? v[p][j].y : 0.f;
                            acc[p].z += in ? v[p][j].z : 0.f; acc[p].w += in ? v[p][j].w : 0.f;
                        }
                    }
                }
        }
#pragma unroll
        for (int p = 0; p < IP; ++p) {
            const int it = it0 + p * NT;
            if (it >= nit) break;
            float4 r = float4{acc[p].x + bias[p].x, acc[p].y + bias[p].y, acc[p].z + bias[p].z, acc[p].w + bias[p].w};
            r.x = r.x > 0.f ? r.x : 0.f; r.y = r.y > 0.f ? r.y : 0.f; r.z = r.z > 0.f ? r.z : 0.f; r.w = r.w > 0.f ? r.w : 0.f;
            if (it < nf * FQ) ((float4 *)h + (size_t)b0 * FQ)[it] = r;
            ((float4 *)hs)[it] = rb ? bf16_rne(r) : r;            // F4 == F here
        }
    }
    for (int q0 = 0;; q0 += WQ * NT) {
#pragma unroll
        for (int j = 0; j < WQ; ++j) {
            const int q = q0 + j * NT + tid;
            if (q < nwq) *(float4 *)(wsh + 4 * q + (WP - F) * (int)dFQ.div((uint32_t)q)) = rb ? bf16_rne(wv4[j]) : wv4[j];
        }
        if (q0 + WQ * NT >= nwq) break;
#pragma unroll
        for (int j = 0; j < WQ; ++j) wv4[j] = ((const float4 *)Wp)[min(q0 + (WQ + j) * NT + tid, nwq - 1)];
    }
#pragma unroll
    for (int j = 0; j < WVQ; ++j)
        if (j * NT + tid < F) wsh[A * WP + j * NT + tid] = rb ? bf16_rne(wv[j]) : wv[j];
    for (int k = WVQ * NT + tid; k < F; k += NT) wsh[A * WP + k] = rb ? bf16_rne(Wv[k]) : Wv[k];
}

template <int LOADS>
__global__ __launch_bounds__(256) void heads_fwd_kernel(const float *__restrict__ ws, int nz, const float *__restrict__ fcb,
                                                        float *__restrict__ h, int B, int F, int A,
                                                        const float *__restrict__ Wp, const float *__restrict__ bp,
                                                        const float *__restrict__ Wv, const float *__restrict__ bv, float *zv,
                                                        float *logits, float *values, float *probs, const float *uniforms,
                                                        int32_t *actions, int rb, const FastDiv dFQ, const FastDiv dA1) {
    extern __shared__ __attribute__((aligned(16))) float hs[];
    constexpr int NT = 256;
    const int tid = threadIdx.x, b0 = blockIdx.x * 4;
    // dFQ, dA1: divisions by F / 4 and A + 1 (a division by a run-time number costs tens of instructions, and these kernels are
    // short).  rb: the products of the heads take h and the weights rounded to bfloat16 (h itself is stored as computed)
    const int F4 = heads_f4(F), WP = F4 + 4;                        // hs: [4][F4], weights [A+1][F4+4], partial dots
    float *wsh = hs + 4 * F4;
    const int nf = min(4, B - b0);
    const int nout = nf * (A + 1);
    // thread tid < nout finishes output a of frame fb
    uint32_t tq, tr;
    dA1.divmod((uint32_t)tid, tq, tr);
    const int ofb = min((int)tq, nf - 1), oa = (int)tr;
    const float obias = oa < A ? bp[oa] : bv[0];
    // padding columns of the LDS rows stay zero
    for (int e = tid; e < 4 * (F4 - F); e += NT) hs[(e / (F4 - F)) * F4 + F + e % (F4 - F)] = 0.f;
    heads_zero_padding<NT>(wsh, tid, F, WP, A + 1);
    const int nw = (A + 1) * F;                 // Wp [A][F] and Wv [F] are adjacent in LDS, not in global memory
    constexpr bool vec4 = LOADS != LOADS_SCALAR;
    if (vec4) heads_load_vec4<NT, 4, LOADS == LOADS_VEC8 ? 8 : 16, LOADS == LOADS_VEC8 ? 2 : 1>(hs, wsh, tid, b0, nf, ws, nz, fcb, h, B, F, F4, WP, A, Wp, Wv, rb, dFQ, [] {});
    for (int e0 = 0; !vec4 && (e0 < nw || e0 == 0); e0 += 24 * NT) {
        float wv[24];
#pragma unroll
        for (int j = 0; j < 24; ++j) {
            const int e = min(e0 + j * NT + tid, nw - 1);
            wv[j] = e < A * F ? Wp[e] : Wv[e - A * F];
        }
        if (e0 == 0) {
            for (int o = tid; o < F; o += NT) {
                if (ws) {
                    const float bias = fcb[o];
                    const size_t stride = (size_t)B * F;
                    const float *src = ws + (size_t)b0 * F + o;
                    float acc4[4] = {0.f, 0.f, 0.f, 0.f};
                    for (int z = 0; z < nz; z += 16) {
                        float v[4][16];
#pragma unroll
                        for (int fb = 0; fb < 4; ++fb)
#pragma unroll
                            for (int i = 0; i < 16; ++i)
                                v[fb][i] = src[min(z + i, nz - 1) * stride + (size_t)min(fb, nf - 1) * F];
#pragma unroll
                        for (int fb = 0; fb < 4; ++fb)
#pragma unroll
                            for (int i = 0; i < 16; ++i) acc4[fb] += (z + i < nz) ? v[fb][i] : 0.f;
                    }
#pragma unroll
                    for (int fb = 0; fb < 4; ++fb) {
                        float v = acc4[fb] + bias;
                        v = v > 0.f ? v : 0.f;
                        if (fb < nf) h[(size_t)(b0 + fb) * F + o] = v;
                        hs[fb * F4 + o] = rb ? bf16_rne(v) : v;
                    }
                } else {
                    float v[4];
#pragma unroll
                    for (int fb = 0; fb < 4; ++fb) {
                        const float *src = h + (size_t)(b0 + min(fb, nf - 1)) * F + o;
                        v[fb] = *src;
                    }
#pragma unroll
                    for (int fb = 0; fb < 4; ++fb) hs[fb * F4 + o] = rb ? bf16_rne(v[fb]) : v[fb];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 24; ++j) {
            const int e = e0 + j * NT + tid;
            if (e < nw) wsh[(e / F) * WP + e % F] = rb ? bf16_rne(wv[j]) : wv[j];
        }
    }
    __syncthreads();
    // asked for after everything that the products need, and needed last: it may be in host memory
    const float ou = (actions && tid < nout) ? uniforms[b0 + ofb] : 0.f;
    // Dot products from LDS, 16 bytes per read, without cross-lane traffic:
    // thread (frame, output, part of k) adds its share; KP shares make one output (three where the block has
    // threads for them, fewer when there are many actions).
    float *zs = wsh + (A + 1) * WP;                  // [4][A+1][3] partial dots, then [4][A+1] values
    const int KP = max(1, min(3, (int)dA1.div(64)));      // the first 256 threads finish the outputs
    if (tid < KP * nout) {
        // thread tid: output a of frame fb, part kp, in this order of significance: tid = (kp nf + fb) (A + 1) + a
        const int a = oa, kp = nf == 4 ? (int)(tq >> 2) : (int)tq / nf, fb = (int)tq - kp * nf;
        const int nk = F4 / 4;
        const int klo = KP == 3 ? (nk * kp) / 3 : (nk * kp) / KP, khi = KP == 3 ? (nk * (kp + 1)) / 3 : (nk * (kp + 1)) / KP;
        const float4 *hb = (const float4 *)(hs + fb * F4), *wr = (const float4 *)(wsh + a * WP);
        float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll 4
        for (int k = klo; k < khi; ++k) {
            const float4 x = hb[k], w = wr[k];
            s0 += x.x * w.x; s1 += x.y * w.y; s2 += x.z * w.z; s3 += x.w * w.w;
        }
        zs[(fb * (A + 1) + a) * 3 + kp] = (s0 + s1) + (s2 + s3);
    }
    __syncthreads();
    float z = 0.f;
    const bool mine = tid < nout;
    const int b = b0 + ofb;
    if (mine) {
        z = zs[tid * 3];
        for (int kp = 1; kp < KP; ++kp) z += zs[tid * 3 + kp];
        z += obias;
        if (zv) zv[(size_t)b * (A + 1) + oa] = z;
        if (oa < A && logits) logits[(size_t)b * A + oa] = z;
        if (oa == A && values) values[b] = z;
    }
    if (!probs && !actions) return;
    // Softmax and the draw, one thread per (frame, action).  The sums run left to
    // right in fp32 exactly as a single thread would form them, so the sampled
    // action is a pure function of the probabilities written out.
    const bool pol = mine && oa < A;
    float *zr = zs + ofb * (A + 1);
    __syncthreads();                                  // all partials are consumed
    if (mine) zs[tid] = z;
    __syncthreads();
    float e = 0.f;
    if (pol) {
        float zmax = zr[0];
        for (int j = 1; j < A; ++j) zmax = fmaxf(zmax, zr[j]);
        e = expf(z - zmax);
    }
    __syncthreads();
    if (pol) zr[oa] = e;
    __syncthreads();
    float pr = 0.f;
    if (pol) {
        float S = 0.f;
        for (int j = 0; j < A; ++j) S += zr[j];
        pr = e / S;
        if (probs) probs[(size_t)b * A + oa] = pr;
    }
    if (!actions) return;
    __syncthreads();
    if (pol) zr[oa] = pr;
    __syncthreads();
    if (pol) {
        float c = 0.f, cprev = 0.f;
        for (int j = 0; j <= oa; ++j) { cprev = c; c += zr[j]; }
        // the first action whose running sum exceeds u; the last one if none does
        if (c > ou && !(oa > 0 && cprev > ou)) actions[b] = oa;
        else if (oa == A - 1 && !(c > ou)) actions[b] = A - 1;
    }
}

// The end of a prediction, by one wavefront: lane a < A holds logit a of frame b, lane A the value.  Softmax and the draw stay
// in registers; the running sums of the draw go left to right in fp32 exactly as a single thread would form them, so the
// sampled action is a pure function of the probabilities written out.  A frame's value and action are stored once each, behind
// the reads of its pixels, its pointer and its uniform number (here and in heads_fwd_kernel): whoever has seen them all may use
// that memory for something else while the kernel still runs.
__device__ __forceinline__ void heads_finish_frame(const int lane, const float z, const int A, const int b, const float u, float *logits,
                                                   float *values, float *probs, int32_t *actions) {
    const bool pol = lane < A;
    if (pol && logits) logits[(size_t)b * A + lane] = z;
    if (lane == A && values) values[b] = z;
    if (!probs && !actions) return;
    const float zmax = wave_max(pol ? z : -3.4e38f);
    const float e = pol ? expf(z - zmax) : 0.f;
    const float pr = e / wave_sum(e);
    if (pol && probs) probs[(size_t)b * A + lane] = pr;
    if (!actions) return;
    // the first action whose running sum exceeds u, the last one if none does: the running sums never fall
    float c = 0.f;
    int act = 0;
    for (int j0 = 0; j0 < A; j0 += 8) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            c += lane_f32(pr, min(j0 + j, 63));            // zero from action A on
            act += c > u ? 0 : 1;
        }
    }
    act = min(act, A - 1);
    if (lane == 0) actions[b] = act;
}

// The heads' weights [A + 1][WP] in LDS, columns F .. WP - 1 not used; by NT threads, at most WQ vectors per thread in flight.
// Needs F % 4 == 0 and a 16-byte aligned policy matrix.  fetch and store are apart so that other loads can go out in between.
template <int NT, int WQ>
struct HeadWeights {
    float4 w[WQ];
    float v[2];
    __device__ __forceinline__ void fetch(int t, int q0, int F, int A, const float *__restrict__ Wp, const float *__restrict__ Wv) {
        const int nwq = A * (F >> 2);
#pragma unroll
        for (int j = 0; j < WQ; ++j) w[j] = ((const float4 *)Wp)[min(q0 + j * NT + t, nwq - 1)];
        if (q0 == 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j) v[j] = Wv[min(j * NT + t, F - 1)];
        }
    }
    __device__ __forceinline__ void store(float *wsh, int t, int F, int WP, int A, const float *__restrict__ Wp, const float *__restrict__ Wv, int rb,
                                          const FastDiv dFQ) {
        const int nwq = A * (F >> 2);
        for (int q0 = 0;; q0 += WQ * NT) {
#pragma unroll
            for (int j = 0; j < WQ; ++j) {
                const int q = q0 + j * NT + t;
                if (q < nwq) *(float4 *)(wsh + 4 * q + (WP - F) * (int)dFQ.div((uint32_t)q)) = rb ? bf16_rne(w[j]) : w[j];
            }
            if (q0 == 0) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (j * NT + t < F) wsh[A * WP + j * NT + t] = rb ? bf16_rne(v[j]) : v[j];
                for (int k = 2 * NT + t; k < F; k += NT) wsh[A * WP + k] = rb ? bf16_rne(Wv[k]) : Wv[k];
            }
            if (q0 + WQ * NT >= nwq) break;
            fetch(t, q0 + WQ * NT, F, A, Wp, Wv);
        }
    }
};

// Four products of a head's sum, rounded in one way in every kernel (left to itself the compiler picks which of a pair is fused).
__device__ __forceinline__ float head_product(const float4 h, const float4 w) {
    return fmaf(h.x, w.x, h.y * w.y) + fmaf(h.z, w.z, h.w * w.w);
}


// Heads of a prediction after the split-k fc layer of F = 256 NJ units: wavefront w of a block takes frame 4 blockIdx.x + w and
// keeps everything of it in registers (its fc outputs, then its logits); only the weights, which the block's four frames share,
// go through LDS, behind the one barrier.  CH chunks of partial sums in flight per lane.
// Latency: 1024 frames 5.2 us with 8 chunks of partial sums; 6.8 us with 16, where barriers between the steps
// (heads_fwd_kernel) took 7.9.
template <int NJ, int CH>
__global__ __launch_bounds__(256) void heads_predict_kernel(const float *__restrict__ ws, int nz, const float *__restrict__ fcb, int B, int A,
                                                            const float *__restrict__ Wp, const float *__restrict__ bp,
                                                            const float *__restrict__ Wv, const float *__restrict__ bv, float *logits,
                                                            float *values, float *probs, const float *uniforms, int32_t *actions, int rb) {
    constexpr int F = 256 * NJ, FQ = F / 4, WP = F + 4;
    extern __shared__ __attribute__((aligned(16))) float heads_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x * 4 + wave;
    HeadWeights<256, 5> hw;
    hw.fetch(tid, 0, F, A, Wp, Wv);
    const float obias = lane < A ? bp[lane] : bv[0];
    float4 bias[NJ], acc[NJ];
    const float4 *src = (const float4 *)ws + (size_t)min(b, B - 1) * FQ;
    const size_t stride4 = (size_t)B * FQ;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        bias[j] = ((const float4 *)fcb)[64 * j + lane];
        acc[j] = float4{0.f, 0.f, 0.f, 0.f};
    }
    for (int z = 0; z < nz; z += CH) {
        float4 v[CH][NJ];
#pragma unroll
        for (int i = 0; i < CH; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) v[i][j] = (src + (size_t)min(z + i, nz - 1) * stride4)[64 * j + lane];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const bool in = z + i < nz;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                acc[j].x += in ? v[i][j].x : 0.f; acc[j].y += in ? v[i][j].y : 0.f;
                acc[j].z += in ? v[i][j].z : 0.f; acc[j].w += in ? v[i][j].w : 0.f;
            }
        }
    }
    hw.store(heads_smem, tid, F, WP, A, Wp, Wv, rb, FastDivConst<FQ>::get());
    // asked for last and needed last: it may be in host memory
    const float u = actions && uniforms ? uniforms[min(b, B - 1)] : 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        acc[j] = float4{acc[j].x + bias[j].x, acc[j].y + bias[j].y, acc[j].z + bias[j].z, acc[j].w + bias[j].w};
        acc[j].x = acc[j].x > 0.f ? acc[j].x : 0.f; acc[j].y = acc[j].y > 0.f ? acc[j].y : 0.f;
        acc[j].z = acc[j].z > 0.f ? acc[j].z : 0.f; acc[j].w = acc[j].w > 0.f ? acc[j].w : 0.f;
        if (rb) acc[j] = bf16_rne(acc[j]);
    }
    __syncthreads();
    if (b >= B) return;
    // sixteen outputs at a time: output a of them lands in lane a % 16 of every row, and row a / 16 keeps it
    float z = 0.f;
    for (int a0 = 0; a0 <= A; a0 += 16) {
        float s16 = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float d[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                d[i] = 0.f;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const float4 w = *(const float4 *)(heads_smem + min(a0 + 4 * q + i, A) * WP + 256 * j + 4 * lane);
                    d[i] += head_product(acc[j], w);
                }
            }
            const float t = row_sums(d, lane);
            s16 = (lane >> 2 & 3) == q ? t : s16;
        }
        s16 = across_rows(s16);
        z = lane >> 4 == a0 >> 4 ? s16 : z;
    }
    heads_finish_frame(lane, z + obias, A, b, u, logits, values, probs, actions);
}

// The same for few frames: a block each, whose threads have NJ neighbouring fc units, and every fourth group of four outputs
// per wavefront, straight from memory.  The same sums.  (16 frames, 512 units 9.1 -> 5.4 us, 1024 12.5 -> 6.1; 256 frames,
// 512 units 7.7 -> 5.4, 256 units 5.9 -> 4.9.)
template <int NJ>
__global__ __launch_bounds__(256) void heads_predict_few_kernel(const float *__restrict__ ws, int nz, const float *__restrict__ fcb, int B, int A,
                                                                const float *__restrict__ Wp, const float *__restrict__ bp,
                                                                const float *__restrict__ Wv, const float *__restrict__ bv, float *logits,
                                                                float *values, float *probs, const float *uniforms, int32_t *actions, int rb) {
    constexpr int F = 256 * NJ, CH = 32;
    typedef float Units __attribute__((ext_vector_type(NJ)));
    __shared__ __attribute__((aligned(16))) float hs[F], zs[64];
    const int tid = threadIdx.x, lane = tid & 63, b = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Units bias = ((const Units *)fcb)[tid];
    float4 w[4][NJ];
    auto weights = [&](int a0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float *row = a0 + i < A ? Wp + (size_t)(a0 + i) * F : Wv;      // the value's row need not be aligned
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const f32x4_dw v = *(const f32x4_dw *)(row + 256 * j + 4 * lane);
                w[i][j] = make_float4(v.x, v.y, v.z, v.w);
            }
        }
    };
    weights(4 * wave);
    const Units *src = (const Units *)(ws + (size_t)b * F) + tid;
    const size_t stride = (size_t)B * 256;
    Units acc = {};
    for (int z = 0; z < nz; z += CH) {
        Units v[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) v[i] = src[(size_t)min(z + i, nz - 1) * stride];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < CH; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[j] += z + i < nz ? v[i][j] : 0.f;
    }
    const float obias = lane < A ? bp[lane] : bv[0];
    const float u = actions && uniforms ? uniforms[b] : 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        float h = acc[j] + bias[j];
        h = h > 0.f ? h : 0.f;
        hs[NJ * tid + j] = rb ? bf16_rne(h) : h;
    }
    __syncthreads();
    float4 h[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) h[j] = ((const float4 *)hs)[64 * j + lane];
    for (int a0 = 4 * wave; a0 <= A; a0 += 16) {
        float d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            d[i] = 0.f;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const float4 q = rb ? bf16_rne(w[i][j]) : w[i][j];
                d[i] += head_product(h[j], q);
            }
        }
        weights(a0 + 16);
        const float t = across_rows(row_sums(d, lane));
        if (lane >> 2 == wave) zs[a0 + (lane & 3)] = t;      // the lanes that keep it in the kernel above: a row's lanes add in orders of their own
    }
    __syncthreads();
    if (wave == 0) heads_finish_frame(lane, zs[lane] + obias, A, b, u, logits, values, probs, actions);
}

// The whole forward pass of the small network (Sec. 3.2) for up to SP_MAX_FRAMES frames in ONE launch, for the latency of a
// small prediction batch (the paper's Sec. 5.2 finds the per-call overhead, not the arithmetic, dominant there).
//
// A block takes FB frames, three of the nine output rows of layer 2 (`rg`; they need 36 of the frame's 84 rows and 8 of
// layer 1's 20) and 256 / NS outputs of the fully connected layer, for which it forms the sums over its rows.  Wavefronts 0..3
// run layer 1 from LDS (as in conv12_fused.hpp), then all eight layer 2, a quarter of its taps and half of the pixel tiles each,
// and the fc sums, two outputs per wavefront and pass, whose weights are on their way while layer 2 runs.  The block that finishes a frame group last
// (a ticket per group; nobody waits for anybody) adds the three row groups up and runs the heads, the softmax and the draw.
// Blocks in order of (row group, slice): an XCD reads few parts of the fc weights.
// Latency: nothing is large.  One frame 15.9 -> 12.8 us a call, 37 frames 23.9 -> 18.6 us against a kernel whose blocks each ran
// both layers of a whole frame, with an event recorded behind every call (9.6 and 14.9 us without one).
constexpr int SP_FC = 256, SP_FLAT = 2592, SP_MAX_FRAMES = 42, SP_ONE_FRAME = 21;      // up to so many: a frame a block
constexpr int SP_TICKET_PITCH = 32;                        // ints between two groups' counters: a cache line each
constexpr int SP_ROWS1 = 8, SP_PIX1 = SP_ROWS1 * 20, SP_PIX2 = 27, SP_XROWS = 36;      // of a row group: layer 1, layer 2, input
constexpr int SP_XVEC = 4 * SP_XROWS * 84 / 16;            // 16-byte vectors of a frame's part
constexpr int SP_Y1 = 16 * SP_PIX1;                        // elements of one plane of its layer-1 output
constexpr int SP_Y2 = 32 * 28;                             // floats of its layer-2 output: 27 pixels and a zero per filter
constexpr int SP_WP = SP_FC + 4;
template <int FB>
struct SpLds {
    static constexpr int XS = 0, FR = XS + FB * SP_XVEC * 32, EX = FR,      // layer 1's filters, later layer 2's partial sums
                         Y1 = FR + (FB == 1 ? 3 * 8 * 64 * 16 : FB * 16384), Y2 = Y1 + FB * 3 * SP_Y1 * 2, ZS = Y2 + FB * SP_Y2 * 4, WS = ZS + FB * 256;
    static size_t bytes(int A) { return WS + sizeof(float) * (A + 1) * SP_WP; }
};

template <bool ONE, int FB, bool TABLE>
__global__ __launch_bounds__(512, 1) void predict_small_kernel(
    const uint8_t *__restrict__ x, const uint8_t *const *__restrict__ table, const u32x4 *__restrict__ frag, const float *__restrict__ b1,
    const float *__restrict__ b2, const float *__restrict__ Wfc, const float *__restrict__ fcb, float *__restrict__ part,
    int *__restrict__ ticket, int B, int NS, int A, const float *__restrict__ Wp, const float *__restrict__ bp,
    const float *__restrict__ Wv, const float *__restrict__ bv, float *logits, float *values, float *probs, const float *uniforms,
    int32_t *actions, float scale, int rb) {
    typedef SpLds<FB> L;
    constexpr int NTERM = ONE ? 1 : 3, CHW1 = 4 * 84 * 84, FPT = NTERM * 2;
    constexpr int XPT = (FB * SP_XVEC + 255) / 256, T1 = (FB * 10 + 3) / 4;      // vectors of input, layer-1 tiles per wavefront
    extern __shared__ __attribute__((aligned(16))) unsigned char sp_smem[];
    __shared__ int last;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rt = tid & 255, rw = wave & 3, l16 = lane & 15, g = lane >> 4;
    const int groups = (B + FB - 1) / FB, per = (int)gridDim.x / 8, at = (int)blockIdx.x % 8 * per + (int)blockIdx.x / 8;
    if (at >= 3 * NS * groups) return;
    const int combo = at / groups, fg = at % groups, rg = combo / NS, o0 = combo % NS * (SP_FC / NS), f0 = fg * FB;
    const int passes = SP_FC / NS / 16;
    __bf16 *xs = (__bf16 *)(sp_smem + L::XS), *y1 = (__bf16 *)(sp_smem + L::Y1);
    float *ex = (float *)(sp_smem + L::EX), *y2 = (float *)(sp_smem + L::Y2), *zs = (float *)(sp_smem + L::ZS), *wsh = (float *)(sp_smem + L::WS);

    // ---- everything that can be asked for now
    u32x4 xpre[XPT], fpre[FPT];
    HeadWeights<256, 5> hw;
    if (wave < 4) {
#pragma unroll
        for (int f = 0; f < FB; ++f) {
            FramePointer<TABLE> fp;
            fp.ask(x, table, min(f0 + f, B - 1), CHW1);
            const u32x4 *src = (const u32x4 *)fp.get() + rg * (24 * 84 / 16);
#pragma unroll
            for (int i = 0; i < XPT / FB; ++i) {
                const int v = min(rt + 256 * i, SP_XVEC - 1);
                xpre[f * (XPT / FB) + i] = src[v / 189 * 441 + v % 189];            // plane by plane: 36 rows are 189 vectors of 441
            }
        }
#pragma unroll
        for (int i = 0; i < FPT; ++i) fpre[i] = frag[rt + 256 * i];
    } else {
        hw.fetch(rt, 0, SP_FC, A, Wp, Wv);
        for (int e = rt; e < FB * 32; e += 256) y2[e * 28 + 27] = 0.f;
    }
    // my lane's vectors of an fc row: vector v is four pixels of filter v / 7, at an address that is a multiple of 4 bytes only; the
    // seventh of a filter has one value too many
    typedef float f32x4_dw4 __attribute__((ext_vector_type(4), aligned(4)));
    int voff[4];
    bool odd[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int v = min(lane + 64 * j, 223);
        voff[j] = v / 7 * 81 + 27 * rg + 4 * (v % 7);
        odd[j] = v % 7 == 6;
    }
    float4 wreg[2][2][4];
    auto load_rows = [&](int set, int p) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4_dw4 t = *(const f32x4_dw4 *)(Wfc + (size_t)(o0 + (p * 8 + wave) * 2 + r) * SP_FLAT + voff[j]);
                wreg[set][r][j] = float4{t[0], t[1], t[2], t[3]};
            }
        asm volatile("" ::: "memory");      // the loads go out here, and not where the compiler finds their first use
    };
    if (wave < 4) {
#pragma unroll
        for (int f = 0; f < FB; ++f)
#pragma unroll
            for (int i = 0; i < XPT / FB; ++i) {
                u32x4 a, b;
                bytes_to_bf16(xpre[f * (XPT / FB) + i], a, b);
                const int v = rt + 256 * i;
                if (v < SP_XVEC) {
                    u32x4 *dst = (u32x4 *)(xs + (size_t)(f * SP_XVEC + v) * 16);
                    dst[0] = a; dst[1] = b;
                }
            }
#pragma unroll
        for (int i = 0; i < FPT; ++i) ((u32x4 *)(sp_smem + L::FR))[rt + 256 * i] = fpre[i];
    }
    __syncthreads();
    const int pg = wave >> 2;                                      // layer 2: pixel tiles pg, pg + 2, ..; taps 64 rw ..
    bf16x8 wq[NTERM][8], w2[NTERM][4];                             // w2: slot 2 kb + filter tile
    {
        const u32x4 *src = frag + (size_t)(1 + (rw >> 1)) * C12_FRAG_SET + (rw & 1) * 4 * 64 + lane;
#pragma unroll
        for (int t = 0; t < NTERM; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                Bf16x8Bits v;
                v.u = src[(t * 8 + j) * 64];
                w2[t][j] = v.v;
            }
    }
    if (wave < 4) {
        const u32x4 *src = (const u32x4 *)(sp_smem + L::FR) + lane;
#pragma unroll
        for (int t = 0; t < NTERM; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                Bf16x8Bits v;
                v.u = src[(t * 8 + j) * 64];
                wq[t][j] = v.v;
            }
    }
    // ---- layer 1: pixels are the rows of the products, filters the columns
    if (wave < 4) {
        const float bias = b1[l16];
        int base[T1];
        floatx4 acc[T1];
#pragma unroll
        for (int j = 0; j < T1; ++j) {
            const int t = min(rw + 4 * j, FB * 10 - 1), f = t / 10, p = t % 10 * 16 + l16;
            base[j] = f * SP_XVEC * 16 + (p / 20 * 4 + g) * 84 + p % 20 * 4;
            acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) {
            bf16x8 xv[T1];
#pragma unroll
            for (int j = 0; j < T1; ++j) {
                const __bf16 *src = xs + base[j] + (kb / 2) * (SP_XROWS * 84) + 4 * (kb % 2) * 84;      // 8-byte aligned
                const uint2 lo = *(const uint2 *)src, hi = *(const uint2 *)(src + 4);
                Bf16x8Bits v;
                v.u = u32x4{lo.x, lo.y, hi.x, hi.y};
                xv[j] = v.v;
            }
#pragma unroll
            for (int t = NTERM - 1; t >= 0; --t)
#pragma unroll
                for (int j = 0; j < T1; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[j], wq[t][kb], acc[j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < T1; ++j) {
            const int t = rw + 4 * j;
            if (t >= FB * 10) continue;
            const int f = t / 10, p = t % 10 * 16 + 4 * g, row = p / 20, col = p % 20;            // four pixels of one row
            __bf16 *yp = y1 + (size_t)f * 3 * SP_Y1 + l16 * SP_PIX1 + (row >> 1) * 40 + (col >> 1) * 4 + (row & 1) * 2;
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = acc[j][r] * scale + bias;
                v[r] = v[r] > 0.f ? v[r] : 0.f;
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                uint32_t hi, mid, lo;
                split3_pair(v[2 * q], v[2 * q + 1], hi, mid, lo);
                *(uint32_t *)(yp + 4 * q) = hi;
                if (!ONE) {
                    *(uint32_t *)(yp + SP_Y1 + 4 * q) = mid;
                    *(uint32_t *)(yp + 2 * SP_Y1 + 4 * q) = lo;
                }
            }
        }
    } else hw.store(wsh, rt, SP_FC, SP_WP, A, Wp, Wv, rb, FastDivConst<SP_FC / 4>::get());
    __syncthreads();
    // ---- layer 2: filters are the rows
    load_rows(0, 0);
    {
        floatx4 acc[FB][2];
        Bf16x8Bits xv[2][FB][NTERM];
#pragma unroll
        for (int i = 0; i < FB; ++i) {
            const int p = min((pg + 2 * i) * 16 + l16, FB * SP_PIX2 - 1), f = p / SP_PIX2, q = p % SP_PIX2;
            const __bf16 *src = y1 + f * 3 * SP_Y1 + (g / 2 + 4 * rw) * SP_PIX1 + (q / 9 + g % 2) * 40 + q % 9 * 4;
            acc[i][0] = acc[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int t = 0; t < NTERM; ++t) {
                    const uint2 *q2 = (const uint2 *)(src + t * SP_Y1 + 2 * kb * SP_PIX1);      // 8-byte aligned
                    const uint2 lo = q2[0], hi = q2[1];
                    xv[kb][i][t].u = u32x4{lo.x, lo.y, hi.x, hi.y};
                }
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            // the six largest term products, smallest first
            constexpr int WT[6] = {2, 1, 0, 1, 0, 0}, XT[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
            for (int q = ONE ? 5 : 0; q < 6; ++q)
#pragma unroll
                for (int i = 0; i < FB; ++i)
#pragma unroll
                    for (int o = 0; o < 2; ++o)
                        acc[i][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2[WT[q]][2 * kb + o], xv[kb][i][XT[q]].v, acc[i][o], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
            for (int o = 0; o < 2; ++o) *(floatx4 *)(ex + ((rw * 4 * FB + (pg + 2 * i) * 2 + o) * 64 + lane) * 4) = acc[i][o];
    }
    __syncthreads();
    for (int e = tid; e < 4 * FB * 64; e += 512) {                 // (pixel tile, filter tile, lane)
        const int el = e & 63, o = e >> 6 & 1, p = (e >> 7) * 16 + (el & 15), f = p / SP_PIX2, q = p % SP_PIX2, oc = o * 16 + (el >> 4) * 4;
        floatx4 s[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] = *(const floatx4 *)(ex + (k * 4 * FB * 64 + e) * 4);
        if (p < FB * SP_PIX2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = ((s[0][r] + s[1][r]) + (s[2][r] + s[3][r])) + b2[oc + r];
                y2[f * SP_Y2 + (oc + r) * 28 + q] = v > 0.f ? v : 0.f;
            }
        }
    }
    __syncthreads();
    // ---- my outputs of the fully connected layer, over my rows
    float4 yv[FB][4];
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            yv[f][j] = ((const float4 *)(y2 + f * SP_Y2))[min(lane + 64 * j, 223)];
            if (rb) yv[f][j] = bf16_rne(yv[f][j]);
            if (lane + 64 * j > 223) yv[f][j] = float4{0.f, 0.f, 0.f, 0.f};
        }
    // lane 2 FB (p % PG) + 2 f + r of every row, register p / PG: the row's share of output r of pass p, frame f
    constexpr int PG = 8 / FB;
    float res[2] = {0.f, 0.f};
    auto fc_pass = [&](int set, int p) {
        float d[2 * FB];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
#pragma unroll
            for (int f = 0; f < FB; ++f) d[2 * f + r] = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float4 w = wreg[set][r][j];
                if (rb) w = bf16_rne(w);
                if (odd[j]) w.w = 0.f;
#pragma unroll
                for (int f = 0; f < FB; ++f) d[2 * f + r] += (yv[f][j].x * w.x + yv[f][j].y * w.y) + (yv[f][j].z * w.z + yv[f][j].w * w.w);
            }
        }
        const float t = row_sums(d, lane);
        const bool mine = (lane & 15) / (2 * FB) == p % PG;
        res[0] = mine && p < PG ? t : res[0];
        res[1] = mine && p >= PG ? t : res[1];
    };
    for (int p = 0; p < passes; p += 2) {                          // the next pass's rows travel while this pass adds up
        if (p + 1 < passes) load_rows(1, p + 1);
        fc_pass(0, p);
        if (p + 2 < passes) load_rows(0, p + 2);
        if (p + 1 < passes) fc_pass(1, p + 1);
    }
    {
        const float v0 = across_rows(res[0]), v1 = across_rows(res[1]);
        const int p = (lane & 15) / (2 * FB) + (lane >> 4) * PG, f = (lane & 15) % (2 * FB) / 2, r = lane & 1;
        // written through to where every compute unit sees it (a device-wide fence instead would write back and invalidate
        // the whole L2 of this block's XCD, once per block)
        if (lane < 32 && p < passes && f0 + f < B)
            __hip_atomic_store(part + ((size_t)(f0 + f) * 3 + rg) * SP_FC + o0 + (p * 8 + wave) * 2 + r, lane < 16 ? v0 : v1, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    // Hand-off to whichever block finishes the group last.  Order of events that makes its reads of `part` safe:
    //  1. every wavefront waits until the memory system has acknowledged its own stores (they are device-scope atomic
    //     stores, which the hardware writes through to the level all compute units share, and a store leaves the
    //     wavefront's count of outstanding memory operations only when that write is acknowledged);
    //  2. the barrier: all of the block's stores are therefore acknowledged before thread 0 goes on;
    //  3. thread 0 draws the ticket with a device-scope read-modify-write and waits for its result;
    //  4. the block that draws the last ticket knows that steps 1-3 of every other block are complete, and reads the
    //     sums with device-scope atomic loads issued after its ticket returned: they are served from the shared level.
    // No fence is used: a device-scope release or acquire fence writes back / invalidates the whole L2 of the XCD,
    // which costs more than the three kernels this one replaces when a training step shares the chip.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        int *mine = ticket + fg * SP_TICKET_PITCH;
        const int t = __hip_atomic_fetch_add(mine, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = t == 3 * NS - 1;
        // for the next launch (stream order puts it after this kernel's end, which completes the store)
        if (last) __hip_atomic_store(mine, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!last) return;
    // ---- heads: 8 / FB wavefronts share a frame's outputs, then one finishes it
    const int hf = wave % FB, b = f0 + hf;
    float4 h;
    {
        float q[3][4];
        const float *src = part + (size_t)min(b, B - 1) * 3 * SP_FC + 4 * lane;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) q[r][e] = __hip_atomic_load(src + r * SP_FC + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float4 bias = ((const float4 *)fcb)[lane];
        h = float4{((q[0][0] + q[1][0]) + q[2][0]) + bias.x, ((q[0][1] + q[1][1]) + q[2][1]) + bias.y,
                   ((q[0][2] + q[1][2]) + q[2][2]) + bias.z, ((q[0][3] + q[1][3]) + q[2][3]) + bias.w};
        h.x = h.x > 0.f ? h.x : 0.f; h.y = h.y > 0.f ? h.y : 0.f; h.z = h.z > 0.f ? h.z : 0.f; h.w = h.w > 0.f ? h.w : 0.f;
        if (rb) h = bf16_rne(h);
    }
    const float obias = lane < A ? bp[lane] : bv[0];
    const float u = actions && uniforms ? uniforms[min(b, B - 1)] : 0.f;
    for (int a0 = wave / FB * 4; a0 <= A; a0 += 32 / FB) {         // four outputs at a time
        float d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 w = *(const float4 *)(wsh + min(a0 + i, A) * SP_WP + 4 * lane);
            d[i] = (h.x * w.x + h.y * w.y) + (h.z * w.z + h.w * w.w);
        }
        const float t = across_rows(row_sums(d, lane));
        if (lane < 4 && a0 + lane <= A) zs[hf * 64 + a0 + lane] = t;
    }
    __syncthreads();
    if (wave < FB && b < B) heads_finish_frame(lane, zs[hf * 64 + lane] + obias, A, b, u, logits, values, probs, actions);
}

// n-step return (text after Eq. 1) of frame i when the segments have unequal
// lengths (Sec. 4.1: an agent hands in fewer than t_max experiences when its
// episode ends): segment n is the frames seg_start[n] .. seg_start[n+1]-1 and
// the return after its last frame is bootstrap[n].  The segment of frame i is
// the last n with seg_start[n] <= i, so empty segments are passed over.  The
// walk is bounded by the frame count whatever the table holds.
__device__ __forceinline__ float ragged_return(const float *__restrict__ rewards, const uint8_t *__restrict__ dones,
                                               const int32_t *__restrict__ seg_start, const float *__restrict__ bootstrap,
                                               int N, int B, int i, float gamma) {
    int lo = 0, hi = N - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (seg_start[mid] <= i) lo = mid; else hi = mid - 1;
    }
    const int end = min(seg_start[lo + 1], B);
    float next = bootstrap ? bootstrap[lo] : 0.f;
    for (int j = end - 1; j >= i; --j) next = rewards[j] + gamma * (dones[j] ? 0.f : 1.f) * next;
    return next;
}

// n-step returns (text after Eq. 1) and the loss with its gradient w.r.t. the
// head outputs (Eq. 1, 2, 5), one thread per frame (n, t).  The thread walks
// its agent's steps T-1 .. t to get R_t, in the order of the recursion.  The
// block first copies the head outputs of its frames to LDS in one sweep.
// Per-block sums of the three loss pieces go to part[3*block..].
// Dynamic LDS: LOSS_THREADS * (A + 1) floats.
__global__ __launch_bounds__(LOSS_THREADS) void returns_loss_kernel(
    const float *__restrict__ zv, const int32_t *__restrict__ actions, const float *__restrict__ rewards,
    const uint8_t *__restrict__ dones, const float *__restrict__ bootstrap, const int32_t *__restrict__ seg_start, int N,
    int T, int B, int A, float gamma, float beta, float cv, float eps, float *__restrict__ R, float *__restrict__ dzv,
    float *__restrict__ part) {
    extern __shared__ float zsh[];     // [LOSS_THREADS][A+1]
    const int i0 = blockIdx.x * LOSS_THREADS;
    const int i = i0 + threadIdx.x;
    const int nrows = min(LOSS_THREADS, B - i0);
    copy_to_lds<8>(zsh, zv + (size_t)i0 * (A + 1), nrows * (A + 1), threadIdx.x, LOSS_THREADS);
    float s_pl = 0.f, s_vl = 0.f, s_en = 0.f;
    float next = 0.f;
    int a = 0;
    if (i < B) {
        a = actions[i];
        if (seg_start) {
            next = ragged_return(rewards, dones, seg_start, bootstrap, N, B, i, gamma);
        } else {
            const int n = i / T, t = i % T;
            next = bootstrap ? bootstrap[n] : 0.f;
            for (int tt = T - 1; tt >= t; --tt) {
                const size_t j = (size_t)n * T + tt;
                next = rewards[j] + gamma * (dones[j] ? 0.f : 1.f) * next;
            }
        }
        R[i] = next;
    }
    __syncthreads();
    if (i < B) {
        const float *z = zsh + threadIdx.x * (A + 1);
        float *dz = dzv + (size_t)i * (A + 1);
        const float V = z[A];
        const float adv = next - V;
        float zmax = z[0];
        for (int j = 1; j < A; ++j) zmax = fmaxf(zmax, z[j]);
        float S = 0.f;
        for (int j = 0; j < A; ++j) S += expf(z[j] - zmax);
        const float logS = logf(S), invS = 1.f / S;
        // dL/dp_k = beta (lg_k + r_k) - [k=a] adv/(p_a+eps);  lg = log(p+eps), r = p/(p+eps)
        float H = 0.f, dot = 0.f, lga = 0.f, ra = 1.f;
        for (int j = 0; j < A; ++j) {
            const float p = expf(z[j] - zmax) * invS;
            float lg, r;
            if (eps == 0.f) { lg = z[j] - zmax - logS; r = 1.f; }
            else { lg = logf(p + eps); r = p / (p + eps); }
            H -= p * lg;
            dot += p * beta * (lg + r);
            if (j == a) { lga = lg; ra = r; }
        }
        dot -= adv * ra;
        for (int j = 0; j < A; ++j) {
            const float p = expf(z[j] - zmax) * invS;
            float lg, r;
            if (eps == 0.f) { lg = z[j] - zmax - logS; r = 1.f; }
            else { lg = logf(p + eps); r = p / (p + eps); }
            dz[j] = p * (beta * (lg + r) - dot) - (j == a ? adv * ra : 0.f);
        }
        dz[A] = -2.f * cv * adv;
        s_pl = -lga * adv;
        s_vl = adv * adv;
        s_en = H;
    }
    __shared__ float sh[3][LOSS_THREADS / 64];
    s_pl = wave_sum(s_pl); s_vl = wave_sum(s_vl); s_en = wave_sum(s_en);
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = s_pl; sh[1][threadIdx.x >> 6] = s_vl; sh[2][threadIdx.x >> 6] = s_en;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        float s = 0.f;
        for (int w = 0; w < LOSS_THREADS / 64; ++w) s += sh[threadIdx.x][w];
        part[3 * blockIdx.x + threadIdx.x] = s;
    }
}

// dL/d(pre-activation of fc)[b][k] = [h > 0] * (sum_a dz[b][a] Wp[a][k] + dv[b] Wv[k]).
// A block takes HD_FRAMES frames and 256 columns, a thread one of them, whose weights it alone reads: straight from memory, eight
// outputs ahead.  A block that took all columns copied the weights to LDS first and ran as many passes as there are 256 columns.
// 640 frames, 1024 units, 18 actions: 28.2 -> 9.2 us, and an update of 5 frames of the stride-1 member 429 -> 410.
// colpart[block][k] receives the block's sum over its frames, which a reduction turns into the fc bias gradient.
// Dynamic LDS: (A + 1) * HD_FRAMES floats.
constexpr int HD_FRAMES = 8, HD_COLS = 256, HD_AHEAD = 8;
__global__ __launch_bounds__(HD_COLS) void heads_dgrad_kernel(const float *__restrict__ dzv, const float *__restrict__ h,
                                                              const float *__restrict__ Wp, const float *__restrict__ Wv,
                                                              int B, int F, int A, float *__restrict__ dh,
                                                              float *__restrict__ colpart, float *__restrict__ wpart, int rb) {
    // rb: every product takes its operands rounded to bfloat16, and the sums that are products with ones
    // (the bias gradients) take rounded terms; dh is stored as computed
    extern __shared__ float4 hd_dz[];       // [A+1][HD_FRAMES]
    float *dzs = (float *)hd_dz;
    const int tid = threadIdx.x;
    const int b0 = blockIdx.x * HD_FRAMES;
    const int nf = min(HD_FRAMES, B - b0);
    const int k = blockIdx.y * HD_COLS + tid, kc = min(k, F - 1);
    float wv[HD_AHEAD], hv[HD_FRAMES];
    auto weights = [&](int a0) {
#pragma unroll
        for (int i = 0; i < HD_AHEAD; ++i) wv[i] = (a0 + i < A ? Wp + (size_t)(a0 + i) * F : Wv)[kc];
    };
    weights(0);
#pragma unroll
    for (int fb = 0; fb < HD_FRAMES; ++fb) hv[fb] = h[(size_t)(b0 + min(fb, nf - 1)) * F + kc];
    for (int e = tid; e < (A + 1) * HD_FRAMES; e += HD_COLS) {
        const int fb = e % HD_FRAMES;
        const float d = fb < nf ? dzv[(size_t)(b0 + fb) * (A + 1) + e / HD_FRAMES] : 0.f;
        dzs[e] = rb ? bf16_rne(d) : d;
    }
    __syncthreads();
    if (k < F) {
        float s[HD_FRAMES];
#pragma unroll
        for (int fb = 0; fb < HD_FRAMES; ++fb) s[fb] = 0.f;
        // wpart (optional): this block's share of the heads' weight gradient,
        // [block][A+1][F+1] with the bias gradient in the last column
        float *wp = wpart ? wpart + (size_t)blockIdx.x * (A + 1) * (F + 1) + k : nullptr;
        for (int a0 = 0; a0 <= A; a0 += HD_AHEAD) {
            float w[HD_AHEAD];
#pragma unroll
            for (int i = 0; i < HD_AHEAD; ++i) w[i] = rb ? bf16_rne(wv[i]) : wv[i];
            if (a0 + HD_AHEAD <= A) weights(a0 + HD_AHEAD);
#pragma unroll
            for (int i = 0; i < HD_AHEAD; ++i)
                if (a0 + i <= A) {
                    const float4 lo = hd_dz[2 * (a0 + i)], hi = hd_dz[2 * (a0 + i) + 1];
                    const float d[HD_FRAMES] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                    float gw = 0.f;
#pragma unroll
                    for (int fb = 0; fb < HD_FRAMES; ++fb) {
                        s[fb] += d[fb] * w[i];
                        gw += fb < nf ? d[fb] * (rb ? bf16_rne(hv[fb]) : hv[fb]) : 0.f;
                    }
                    if (wp) wp[(size_t)(a0 + i) * (F + 1)] = gw;
                }
        }
        float col = 0.f;
#pragma unroll
        for (int fb = 0; fb < HD_FRAMES; ++fb)
            if (fb < nf) {
                const float v = hv[fb] > 0.f ? s[fb] : 0.f;
                dh[(size_t)(b0 + fb) * F + k] = v;
                col += rb ? bf16_rne(v) : v;
            }
        colpart[(size_t)blockIdx.x * F + k] = col;      // this block's share of the fc bias gradient
    }
    if (wpart && blockIdx.y == 0 && tid <= A) {
        float gb = 0.f;
        for (int fb = 0; fb < nf; ++fb) gb += dzs[tid * HD_FRAMES + fb];
        wpart[((size_t)blockIdx.x * (A + 1) + tid) * (F + 1) + F] = gb;
    }
}

// Training only: everything between the fc products and the fc backward in one
// kernel, for HD_FRAMES frames per block.  (1) last step of the split-k fc layer:
// h = max(0, bias + sum_z ws[z]); (2) heads: z = W h + b; (3) n-step returns
// (text after Eq. 1), loss and its gradient w.r.t. the head outputs (Eq. 1, 2,
// 5), a wavefront per frame with an output per lane, sums taken in action order;
// (4) heads backward: dh = [h > 0] dz W,
// and the block's shares of the heads' weight and bias gradients (wpart
// [block][A+1][F+1]) and of the fc bias gradient (colpart [block][F]): a
// thread takes VK consecutive k and every fourth output, so that weights,
// activations and gradients move as vectors; the four partial sums of dh meet in
// LDS.
// What it takes is one block's chain of steps (us since its start, 40 frames of 256
// units, 27 chunks of partial sums: operands in LDS 5.0, dots 5.9, returns and loss
// 8.3, end 11.0; with four barriers and a thread per (frame, action) the loss ended at
// 9.4), and in the long ones of them the block's instructions and its requests to
// memory, each of which occupies a wavefront for a hundred cycles; hence eight
// wavefronts.  Launches, with loss by threads of four or eight wavefronts / now: 40 frames
// 13.9 / 13.4, 640 in segments of unequal length 13.9 / 12.1, 1050 13.6 / 12.0, 2560
// 17.9 / 18.1, in unequal segments 19.1 / 17.8, 1280 frames of 512 units 18.7 / 17.2.
// Writes h, zv, R, dzv (kept for inspection), dh, colpart, wpart and three loss
// sums per block.  rb: operands of every product rounded to bfloat16.
// Dynamic LDS: heads_train_lds_floats(F, A) floats.
__host__ __device__ inline int heads_train_kparts(int F, int A) {
    const int kp = 256 / (A + 1), nk = heads_f4(F) / 4;
    return kp < nk ? kp : nk;
}
constexpr int HEADS_TRAIN_THREADS = 64 * HD_FRAMES;
inline int heads_train_vk(int F) { return F > 256 ? 4 : 2; }      // k per thread in the backward part: a pass over 256 or 512 units
__host__ __device__ inline int heads_train_lds_floats(int F, int A) {
    return HD_FRAMES * heads_f4(F) + (A + 1) * (heads_f4(F) + 4) + HD_FRAMES * (F > 256 ? 2048 : 1024) + (A + 1) * HD_FRAMES +
           4 * HD_FRAMES + HD_FRAMES * (A + 1) * heads_train_kparts(F, A) + 512;
}

template <int LOADS, int VK>
__global__ __launch_bounds__(HEADS_TRAIN_THREADS) void heads_train_kernel(
    const float *__restrict__ ws, int nz, const float *__restrict__ fcb, int B, int F, int A,
    const float *__restrict__ Wp, const float *__restrict__ bp, const float *__restrict__ Wv, const float *__restrict__ bv,
    const int32_t *__restrict__ actions, const float *__restrict__ rewards, const uint8_t *__restrict__ dones,
    const float *__restrict__ bootstrap, const int32_t *__restrict__ seg_start, int N, int T, float gamma, float beta,
    float cv, float eps, float *__restrict__ h, float *__restrict__ zv, float *__restrict__ R, float *__restrict__ dzv,
    float *__restrict__ dh, float *__restrict__ colpart, float *__restrict__ wpart, float *__restrict__ losspart, int rb,
    const FastDiv dFQ, const FastDiv dA1, const FastDiv dKP, const FastDiv dT, const ga3c::FcDhPlanes dhp) {
    extern __shared__ __attribute__((aligned(16))) float sm[];
    constexpr int NT = HEADS_TRAIN_THREADS, NF = HD_FRAMES, KPASS = NT / 4 * VK;      // k of a pass of the backward part
    const int F4 = heads_f4(F), WP = F4 + 4, A1 = A + 1, KP = (int)dKP.d;
    float *hs = sm;                          // [NF][F4]   fc output of my frames (rounded if rb)
    float *wsh = hs + NF * F4;               // [A1][WP]   head weights (rounded if rb)
    float *red = wsh + A1 * WP;              // [4][NF][KPASS] partial sums of dh, one set per quarter of the outputs
    float *zt = red + 4 * NF * KPASS;          // [A1][NF]   gradients of the head outputs, transposed
    float *ls = zt + A1 * NF;                // [3][NF]    loss terms of my frames
    float *zp = ls + 4 * NF;                 // [NF][A1][KP] partial dots
    float *rw = zp + NF * A1 * KP;           // [256]      rewards of the agents my frames belong to
    float *dn = rw + 256;                    // [256]      1 - done
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * NF;
    const int nf = min(NF, B - b0);

    // ---- everything from global memory is requested first
    const int n0 = (int)dT.div((uint32_t)b0), n1 = (int)dT.div((uint32_t)(b0 + nf - 1));      // agents of my frames
    const int nrw = (n1 - n0 + 1) * T;
    const bool rw_lds = !seg_start && nrw <= 256;      // segments of unequal length read their rewards from global memory
    const size_t at_rw = rw_lds ? (size_t)n0 * T + min(tid, nrw - 1) : 0;
    const float my_rw = rewards[at_rw];
    const uint32_t my_done = dones[at_rw];
    // the loss of a frame is one wavefront's, lane a has output a
    const int ob = b0 + min(wave, nf - 1);
    const float obias = lane < A ? bp[lane] : bv[0];
    const int oact = actions[ob];
    float oboot = bootstrap && !seg_start ? bootstrap[dT.div((uint32_t)ob)] : 0.f;
    // Segments of unequal length: a frame's own (ragged_return says how), and its rewards from there on, a step per lane.  The
    // search goes through the scalar cache while the partial sums are on their way.
    int send = 0;
    float srw = 0.f, sdn = 0.f;
    auto segments = [&]() __attribute__((always_inline)) {
        if (!seg_start) return;
        int lo = 0, hi = N - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (seg_start[mid] <= ob) lo = mid; else hi = mid - 1;
        }
        send = min(seg_start[lo + 1], B);
        oboot = bootstrap ? bootstrap[lo] : 0.f;
        const int at = min(ob + lane, B - 1);
        srw = rewards[at];
        sdn = dones[at] ? 0.f : 1.f;
    };
    for (int e = tid; e < NF * (F4 - F); e += NT) hs[(e / (F4 - F)) * F4 + F + e % (F4 - F)] = 0.f;
    heads_zero_padding<NT>(wsh, tid, F, WP, A1);
    const int nw = A1 * F;
    constexpr bool vec4 = LOADS != LOADS_SCALAR;
    // Outputs per thread and round: a block of 512 threads has one each of up to 256 units, two of 512.  Chunks per round: with one
    // output as many as the 27 that the small net's updates of at most 320 frames leave, in whole fours; with two outputs 28 would be
    // 224 registers of the 256 that eight wavefronts leave each, 20 are 160.
    constexpr int IP = VK == 2 ? 1 : 2, CH = LOADS == LOADS_VEC8 ? 8 : VK == 2 ? 28 : 20;
    if constexpr (vec4) heads_load_vec4<NT, NF, CH, IP>(hs, wsh, tid, b0, nf, ws, nz, fcb, h, B, F, F4, WP, A, Wp, Wv, rb, dFQ, segments);
    for (int e0 = 0; !vec4 && (e0 < nw || e0 == 0); e0 += 24 * NT) {
        float wv[24];
#pragma unroll
        for (int j = 0; j < 24; ++j) {
            const int e = min(e0 + j * NT + tid, nw - 1);
            wv[j] = e < A * F ? Wp[e] : Wv[e - A * F];
        }
        if (e0 == 0) {
            for (int o = tid; o < F; o += NT) {
                const float bias = fcb[o];
                const size_t stride = (size_t)B * F;
                const float *src = ws + (size_t)b0 * F + o;
                float acc[NF];
#pragma unroll
                for (int fb = 0; fb < NF; ++fb) acc[fb] = 0.f;
                for (int z = 0; z < nz; z += 8) {
                    float v[NF][8];
#pragma unroll
                    for (int fb = 0; fb < NF; ++fb)
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            v[fb][i] = src[min(z + i, nz - 1) * stride + (size_t)min(fb, nf - 1) * F];
#pragma unroll
                    for (int fb = 0; fb < NF; ++fb)
#pragma unroll
                        for (int i = 0; i < 8; ++i) acc[fb] += (z + i < nz) ? v[fb][i] : 0.f;
                }
#pragma unroll
                for (int fb = 0; fb < NF; ++fb) {
                    float v = acc[fb] + bias;
                    v = v > 0.f ? v : 0.f;
                    if (fb < nf) h[(size_t)(b0 + fb) * F + o] = v;
                    hs[fb * F4 + o] = rb ? bf16_rne(v) : v;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 24; ++j) {
            const int e = e0 + j * NT + tid;
            if (e < nw) wsh[(e / F) * WP + e % F] = rb ? bf16_rne(wv[j]) : wv[j];
        }
    }
    if constexpr (!vec4) segments();
    if (rw_lds && tid < nrw) { rw[tid] = my_rw; dn[tid] = my_done ? 0.f : 1.f; }
    __syncthreads();

    // ---- heads: thread (action a, part kp of k) for the frames of its 256 threads, then the parts are added in order
    {
        constexpr int NH = NF * 256 / NT;
        uint32_t kp_, a_;
        dA1.divmod((uint32_t)(tid & 255), kp_, a_);
        const int a = (int)a_, kp = (int)kp_, f0 = NH * (tid >> 8);
        if (kp < KP) {
            const int nk = F4 / 4;
            const int klo = (int)dKP.div((uint32_t)(nk * kp)), khi = (int)dKP.div((uint32_t)(nk * (kp + 1)));
            const float4 *wr = (const float4 *)(wsh + a * WP);
            float s[NH];
#pragma unroll
            for (int fb = 0; fb < NH; ++fb) s[fb] = 0.f;
            for (int k = klo; k < khi; ++k) {
                const float4 w = wr[k];
#pragma unroll
                for (int fb = 0; fb < NH; ++fb) {
                    const float4 x = ((const float4 *)(hs + (f0 + fb) * F4))[k];
                    s[fb] += (x.x * w.x + x.y * w.y) + (x.z * w.z + x.w * w.w);
                }
            }
#pragma unroll
            for (int fb = 0; fb < NH; ++fb) zp[((f0 + fb) * A1 + a) * KP + kp] = s[fb];
        }
    }
    __syncthreads();
    // ---- loss and dL/dz.  Sums over the parts and over the actions run in index order; no barrier until they are done (five, with
    // a thread per (frame, output) of the block: 3.5 us of an update of 40 frames, 2.4 now).
    float dzo = 0.f;
    if (wave < nf) {
        float z = 0.f;
        const float *part = zp + (wave * A1 + min(lane, A)) * KP;
        for (int kp = 0; kp < KP; ++kp) z += part[kp];
        z += obias;
        // n-step return
        float Rt = oboot;
        if (seg_start) {
            for (int j = send - 1; j >= ob + 64; --j) Rt = rewards[j] + gamma * (dones[j] ? 0.f : 1.f) * Rt;
            for (int j = min(send - ob, 64) - 1; j >= 0; --j) Rt = lane_f32(srw, j) + gamma * lane_f32(sdn, j) * Rt;
        } else {
            const int n = (int)dT.div((uint32_t)ob), t = ob - n * T;
            if (rw_lds)
                for (int tt = T - 1; tt >= t; --tt) { const int j = (n - n0) * T + tt; Rt = rw[j] + gamma * dn[j] * Rt; }
            else
                for (int tt = T - 1; tt >= t; --tt) {
                    const size_t j = (size_t)n * T + tt;
                    Rt = rewards[j] + gamma * (dones[j] ? 0.f : 1.f) * Rt;
                }
        }
        const bool pol = lane < A;
        const float adv = Rt - lane_f32(z, A), zmax = wave_max(pol ? z : lane_f32(z, 0));
        const float e = expf(z - zmax);
        float S = 0.f;
        for (int j = 0; j < A; ++j) S += lane_f32(e, j);
        const float logS = logf(S), invS = 1.f / S;
        const float p = e * invS;
        float lg, r;
        if (eps == 0.f) { lg = z - zmax - logS; r = 1.f; }
        else { lg = logf(p + eps); r = p / (p + eps); }
        const float ent = p * lg, trm = p * beta * (lg + r);
        float H = 0.f, dot = 0.f;
        for (int j = 0; j < A; ++j) { H -= lane_f32(ent, j); dot += lane_f32(trm, j); }
        const bool known = (unsigned)oact < (unsigned)A;
        const int taken = __builtin_amdgcn_readfirstlane(known ? oact : 0);
        const float lga = known ? lane_f32(lg, taken) : 0.f, ra = known ? lane_f32(r, taken) : 1.f;
        dot -= adv * ra;
        if (pol) dzo = p * (beta * (lg + r) - dot) - (lane == oact ? adv * ra : 0.f);
        else dzo = -2.f * cv * adv;
        if (lane < A1) {
            zv[(size_t)ob * A1 + lane] = z;
            dzv[(size_t)ob * A1 + lane] = dzo;
        }
        if (lane == 0) {
            R[ob] = Rt;
            ls[wave] = -lga * adv; ls[NF + wave] = adv * adv; ls[2 * NF + wave] = H;
        }
    }
    // zt[output][frame] for the backward pass, zero for frames the block does not have
    if (lane < A1) zt[lane * NF + wave] = rb ? bf16_rne(dzo) : dzo;
    __syncthreads();
    if (tid < 3) {
        const float *src = ls + tid * NF;
        float sum = 0.f;
        for (int fb = 0; fb < nf; ++fb) sum += src[fb];
        losspart[3 * blockIdx.x + tid] = sum;
    }
    // ---- heads backward (zt holds dz of my frames).  A quarter of the block takes the outputs ag, ag + 4, ..; thread kl of it the
    // VK k starting at kbase + VK kl.
    typedef float fk __attribute__((ext_vector_type(VK)));
    typedef float fk_dword_aligned __attribute__((ext_vector_type(VK), aligned(4)));
    const int ag = tid / (NT / 4), kl = tid % (NT / 4);
    for (int kbase = 0; kbase < F; kbase += KPASS) {
        const int kv = kbase + VK * kl;
        const bool kin = kv < F4;
        fk hv[NF], sd[NF];
#pragma unroll
        for (int fb = 0; fb < NF; ++fb) {
            hv[fb] = kin ? *(const fk *)(hs + fb * F4 + kv) : (fk)(0.f);
            sd[fb] = (fk)(0.f);
        }
        float *wp = wpart + (size_t)blockIdx.x * A1 * (F + 1) + kv;
        for (int a = ag; a < A1; a += 4) {
            const fk wv = kin ? *(const fk *)(wsh + a * WP + kv) : (fk)(0.f);
            const float4 d0 = *(const float4 *)(zt + a * NF), d1 = *(const float4 *)(zt + a * NF + 4);
            const float d[NF] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
            fk gw = (fk)(0.f);
#pragma unroll
            for (int fb = 0; fb < NF; ++fb)
#pragma unroll
                for (int e = 0; e < VK; ++e) { sd[fb][e] += d[fb] * wv[e]; gw[e] += d[fb] * hv[fb][e]; }
            float *dst = wp + (size_t)a * (F + 1);
            if (kv + VK - 1 < F) {
                *(fk_dword_aligned *)dst = gw;
            } else {
#pragma unroll
                for (int e = 0; e < VK - 1; ++e)
                    if (kv + e < F) dst[e] = gw[e];
            }
        }
#pragma unroll
        for (int fb = 0; fb < NF; ++fb) *(fk *)(red + (ag * NF + fb) * KPASS + VK * kl) = sd[fb];
        __syncthreads();
        const int kk = tid % KPASS, k = kbase + kk;
        // where a pass has half as many k as the block threads, one half writes dh and the other what is made of it
        const bool writes_dh = KPASS >= NT || tid < KPASS, writes_sums = KPASS >= NT || tid >= KPASS;
        if (k < F) {
            float v[NF], col = 0.f;
#pragma unroll
            for (int fb = 0; fb < NF; ++fb) {
                v[fb] = 0.f;
                if (fb < nf) {
                    const float sum = (red[fb * KPASS + kk] + red[(NF + fb) * KPASS + kk]) +
                                      (red[(2 * NF + fb) * KPASS + kk] + red[(3 * NF + fb) * KPASS + kk]);
                    v[fb] = hs[fb * F4 + k] > 0.f ? sum : 0.f;
                    if (writes_dh) dh[(size_t)(b0 + fb) * F + k] = v[fb];
                    col += rb ? bf16_rne(v[fb]) : v[fb];
                }
            }
            if (writes_sums) {
                colpart[(size_t)blockIdx.x * F + k] = col;
                if (dhp.w) {                              // dh as operands of the fc gradients
                    static_assert(NF == 8, "a block's frames are one group of eight k");
                    const int kbw = (B + 31) / 32;
                    fc_dh_store8(dhp, k, blockIdx.x, kbw, v);
                    if (blockIdx.x + 1 == gridDim.x) {    // nothing behind the last frame
                        const float none[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                        for (int b8 = blockIdx.x + 1; b8 < 4 * kbw; ++b8) fc_dh_store8(dhp, k, b8, kbw, none);
                    }
                }
            }
        }
        __syncthreads();                              // red is written again in the next pass
    }
    if (tid <= A) {
        float gb = 0.f;
        for (int fb = 0; fb < nf; ++fb) gb += zt[tid * NF + fb];
        wpart[((size_t)blockIdx.x * A1 + tid) * (F + 1) + F] = gb;
    }
}

// One launch adds up the partial weight gradients of every layer and, on the
// way, the squares of the results (for the global norm).
// A segment is a stack of nz partial matrices [rows][N], `stride` floats apart (nz = 1 and in place: the gradient itself).
// It goes to gW[m*(N-1) + n] for n < N-1 and gb[m] for n = N-1 (bias column), or all N columns to gW[m*N + n].
// A block handles 256/zg outputs with zg threads each: thread j adds z = j, j+zg, ... (sixteen loads in
// flight at a time), then the zg sums are added in order of j.  Nothing depends
// on timing, so the gradient is reproducible bit for bit.
// Block ids go round-robin over the 8 XCDs; the ids of one XCD take consecutive
// groups of outputs, so that blocks which share 128-byte lines of the partial
// sums also share an L2.  Where the first row of the segment and the planes of the stack start on 16-byte
// boundaries a thread takes four consecutive outputs and reads its partial sums as 16-byte vectors (a quarter of the
// load instructions); the sums of an output are formed in the same order either way.
constexpr int MAX_REDUCE_SEGS = 12;
struct alignas(64) ReduceSeg {
    const float *ws;     // first row of the segment in the first matrix
    float *gW, *gb;
    size_t stride, cnt;  // cnt = rows * N
    int nz, N;
    uint32_t mul;        // FastDiv(N) is {N, mul, shift}
    int per_xcd;         // the segment owns 8 * per_xcd block ids, the first of them is a multiple of 8
    uint8_t shift, lzg;  // zg = 1 << lzg
    bool bias_col, vec, in_place;        // vec: a thread takes four consecutive outputs and reads 16-byte vectors (the stack allows it)
};
static_assert(sizeof(ReduceSeg) == 64, "a segment is one line of the arguments");
struct ReduceArgs {
    int first[MAX_REDUCE_SEGS];          // first block of a segment; INT32_MAX for those there are not
    float *normpart;     // one partial sum of squares per block
    ReduceSeg seg[MAX_REDUCE_SEGS];
};

// What bounds it on small updates is the chain of one block: arguments, loads, LDS, stores.  The arguments come from host
// memory a line at a time, about a microsecond each, so a block finds its segment in one line (`first`) and reads one more,
// and the four outputs of a thread are divided by N once: training of the small net on 40 frames 67.0 -> 65.4 us, of the larger
// net on 1280 466.0 -> 462.2 (against a search from segment to segment, 64-bit divisions per output and eight loads a round).
__global__ __launch_bounds__(256) void reduce_all_kernel(const ReduceArgs a) {
    __shared__ float4 sh[256];
    __shared__ float wsum[4];
    int si = 0, first = a.first[0];
#pragma unroll
    for (int k = 1; k < MAX_REDUCE_SEGS; ++k)
        if ((int)blockIdx.x >= a.first[k]) { si = k; first = a.first[k]; }
    const ReduceSeg &g = a.seg[si];
    const int lopb = 8 - g.lzg, zg = 1 << g.lzg, opb = 1 << lopb, N = g.N, nz = g.nz;
    const int o = threadIdx.x & (opb - 1), zi = threadIdx.x >> lopb;
    const int lb = blockIdx.x - first;
    const int per = g.vec ? 4 : 1;                      // outputs per thread
    const size_t cnt = g.cnt, stride = g.stride;
    const size_t i = ((size_t)((lb & 7) * g.per_xcd + (lb >> 3)) * opb + o) * per;
    float4 s = float4{0.f, 0.f, 0.f, 0.f};
    const float *src = g.ws + i;
    if (g.vec && nz == 1 && i + 3 < cnt) {
        if (zi == 0) s = *(const float4 *)src;
    } else if (g.vec && i + 3 < cnt) {
        for (int z0 = 0; z0 < nz; z0 += 16 * zg) {
            float4 v[16];
#pragma unroll
            for (int q = 0; q < 16; q += 4)
                if (z0 + q * zg < nz) {
#pragma unroll
                    for (int j = q; j < q + 4; ++j) v[j] = *(const float4 *)(src + (size_t)min(z0 + zi + j * zg, nz - 1) * stride);
                }
#pragma unroll
            for (int q = 0; q < 16; q += 4)
                if (z0 + q * zg < nz) {
#pragma unroll
                    for (int j = q; j < q + 4; ++j) {
                        const bool in = z0 + zi + j * zg < nz;
                        s.x += in ? v[j].x : 0.f; s.y += in ? v[j].y : 0.f; s.z += in ? v[j].z : 0.f; s.w += in ? v[j].w : 0.f;
                    }
                }
        }
    } else if (i < cnt) {                               // one output, or the last, partial group of four
        const int ne = (int)min((size_t)per, cnt - i);
        for (int e = 0; e < ne; ++e) {
            float t = 0.f;
            for (int z = zi; z < nz; z += 8 * zg) {
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = src[(size_t)min(z + j * zg, nz - 1) * stride + e];
#pragma unroll
                for (int j = 0; j < 8; ++j) t += (z + j * zg < nz) ? v[j] : 0.f;
            }
            if (e == 0) s.x = t; else if (e == 1) s.y = t; else if (e == 2) s.z = t; else s.w = t;
        }
    }
    float sq = 0.f;
    if (zg > 1) {
        sh[threadIdx.x] = s;
        __syncthreads();
    }
    if (zi == 0 && i < cnt) {
        for (int j = 1; j < zg; ++j) {
            const float4 u = sh[j * opb + o];
            s.x += u.x; s.y += u.y; s.z += u.z; s.w += u.w;
        }
        const float te[4] = {s.x, s.y, s.z, s.w};       // those behind the last output are zero
#pragma unroll
        for (int e = 0; e < 4; ++e) sq += te[e] * te[e];
        if (!g.in_place) {                              // else the gradient is there already: only its squares are wanted
            typedef float f4_dword_aligned __attribute__((ext_vector_type(4), aligned(4)));
            size_t m = 0, n = i;
            if (g.bias_col) {                           // FastDiv takes 31 bits
                if (cnt >> 31) m = i / (size_t)N;
                else m = (__umulhi((uint32_t)i, g.mul) + (uint32_t)i) >> g.shift;
                n = i - m * N;
            }
            const int NW = g.bias_col ? N - 1 : N;      // columns of gW
            float *dst = g.gW + (m * (size_t)(g.bias_col ? NW : 0) + n);
            if (g.vec && i + 3 < cnt && (!g.bias_col || n + 3 < (size_t)NW)) {
                *(f4_dword_aligned *)dst = f4_dword_aligned{te[0], te[1], te[2], te[3]};
            } else {
                const int ne = (int)min((size_t)per, cnt - i);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < ne) {
                        if (!g.bias_col || n < (size_t)NW) *dst++ = te[e];
                        else g.gb[m] = te[e];
                        if (g.bias_col && ++n == (size_t)N) { n = 0; ++m; }
                    }
            }
        }
    }
    sq = wave_sum(sq);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) a.normpart[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// Eq. 3 on a flat buffer: d = s*grad; g = alpha g + (1-alpha) d^2;
// theta_out = theta_in - lr d / sqrt(g + eps) (the two may be the same buffer).  20 bytes of traffic per parameter.
// s comes from one of three places: scale_host (normpart == nullptr and scale_dev == nullptr), scale_dev[0], or,
// inside a training step, the per-block squared norms of the gradient (normpart, nnorm of them): every block adds
// them up in the same fixed order and forms s = min(1, clip / norm) itself, and block 0 also writes the loss sums
// and the statistics, which saves the launch of a kernel of one block between the reduction and this one.
// A thread keeps four 16-byte vectors of each array in flight, which is what a streaming kernel needs to approach
// the memory's bandwidth on a buffer far larger than the caches.  VARIANT bit 0: loads, bit 1: stores bypass the caches.
struct RmsClip {
    const float *normpart; int nnorm;          // squared-norm partials of the gradient
    const float *losspart; int nloss;          // three loss sums per loss block
    float clip;                                // threshold of the global-norm rescale, <= 0: off
    float *scale_out;                          // receives s (1 float)
    ga3c_train_stats *own, *user;              // statistics (user may be null)
};

// streaming accesses: the line is not kept in the caches after use
typedef float f32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 nt_load(const float4 *p) {
    const f32x4_t v = __builtin_nontemporal_load((const f32x4_t *)p);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void nt_store(const float4 v, float4 *p) {
    __builtin_nontemporal_store(f32x4_t{v.x, v.y, v.z, v.w}, (f32x4_t *)p);
}

__device__ __forceinline__ void rmsprop4(float4 &t, float4 &gg, float4 d, float s, float lr, float alpha, float oma, float eps) {
    d.x *= s; d.y *= s; d.z *= s; d.w *= s;
    gg.x = alpha * gg.x + oma * d.x * d.x; gg.y = alpha * gg.y + oma * d.y * d.y;
    gg.z = alpha * gg.z + oma * d.z * d.z; gg.w = alpha * gg.w + oma * d.w * d.w;
    t.x -= lr * d.x / sqrtf(gg.x + eps); t.y -= lr * d.y / sqrtf(gg.y + eps);
    t.z -= lr * d.z / sqrtf(gg.z + eps); t.w -= lr * d.w / sqrtf(gg.w + eps);
}

template <int VARIANT, int VPT>
__global__ __launch_bounds__(256) void rmsprop_kernel(const float *theta_in, float *theta_out, float *__restrict__ g,
                                                      const float *__restrict__ grad, size_t n,
                                                      const float *__restrict__ scale_dev, float scale_host, float lr,
                                                      float alpha, float eps, u32x4 *__restrict__ frag, u32x4 *__restrict__ hfrag,
                                                      int frag_rb, const ga3c::FcPlanes fcw, const RmsClip clipargs) {
    // frag (optional): split MFMA fragments of the small net's conv filters, kept current with theta_out; hfrag (optional, VPT == 1): the
    // same for predictions (conv12_f16.hpp).  fcw (optional): the fc weights as operands of the forward product, likewise
    constexpr unsigned W1 = 0, W2 = 16u * 256u + 16u;      // where the filter tensors start in the flat buffer then
    float s = scale_dev ? scale_dev[0] : scale_host;
    if (clipargs.normpart) {
        __shared__ float sh[4][4];
        const int tid = threadIdx.x;
        float acc[4] = {0.f, 0.f, 0.f, 0.f};     // norm^2, policy loss, value loss, entropy
        for (int i = tid; i < clipargs.nnorm; i += 8 * 256) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = clipargs.normpart[min(i + 256 * j, clipargs.nnorm - 1)];
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[0] += (i + 256 * j < clipargs.nnorm) ? v[j] : 0.f;
        }
        if (blockIdx.x == 0)
            for (int i = tid; i < clipargs.nloss; i += 256)
                for (int c = 0; c < 3; ++c) acc[1 + c] += clipargs.losspart[3 * i + c];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            acc[c] = wave_sum(acc[c]);
            if ((tid & 63) == 0) sh[c][tid >> 6] = acc[c];
        }
        __syncthreads();
        float t[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) t[c] = (sh[c][0] + sh[c][1]) + (sh[c][2] + sh[c][3]);
        const float norm = sqrtf(t[0]);
        s = 1.f;
        if (clipargs.clip > 0.f && norm > clipargs.clip) s = clipargs.clip / norm;
        if (blockIdx.x == 0 && tid == 0) {
            clipargs.scale_out[0] = s;
            ga3c_train_stats st;
            st.policy_loss = t[1]; st.value_loss = t[2]; st.entropy = t[3];
            st.grad_norm = norm; st.clip_scale = s; st.nonfinite = !(norm <= 3.0e38f) ? 1 : 0;
            *clipargs.own = st;
            if (clipargs.user) *clipargs.user = st;
        }
    }
    const float oma = 1.f - alpha;
    const size_t n4 = n / 4;
    const size_t stride = (size_t)gridDim.x * 256;
    const float4 *t4 = (const float4 *)theta_in;
    float4 *o4 = (float4 *)theta_out;
    float4 *g4 = (float4 *)g;
    const float4 *d4 = (const float4 *)grad;
    // hfrag takes filters whole, from the 64 lanes of a wavefront: the second tensor begins four vectors (the first one's biases) behind a
    // multiple of 64, and these four come behind it
    auto vector_of = [&](const size_t i) {
        if (VPT != 1 || !hfrag) return i;
        constexpr size_t A = W1 + 16 * 64, B = A + 32 * 64;
        return i < A || i >= B + 4 ? i : i < B ? i + 4 : i - (B - A);
    };
    auto store_filter = [&](const size_t i, const float4 t) {
        if (VPT == 1 && hfrag && i < 48 * 64) conv12_f16_store_filter(hfrag, __builtin_amdgcn_readfirstlane((int)i >> 6), threadIdx.x & 63, t);
    };
    // a block works on tiles of 256 * VPT consecutive vectors (16 KB of each array for VPT = 4): thread t takes vectors
    // t, t + 256, ... of the tile, all requested before the first is used
    const size_t ntile = n4 / (256 * VPT);
    for (size_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        const size_t first = tile * (256 * VPT) + threadIdx.x, i = vector_of(first);
        float4 t[VPT], gg[VPT], d[VPT];
#pragma unroll
        for (int j = 0; j < VPT; ++j) {
            t[j] = VARIANT & 1 ? nt_load(t4 + i + 256 * j) : t4[i + 256 * j];
            gg[j] = VARIANT & 1 ? nt_load(g4 + i + 256 * j) : g4[i + 256 * j];
            d[j] = VARIANT & 1 ? nt_load(d4 + i + 256 * j) : d4[i + 256 * j];
        }
#pragma unroll
        for (int j = 0; j < VPT; ++j) {
            rmsprop4(t[j], gg[j], d[j], s, lr, alpha, oma, eps);
            if (VARIANT & 2) { nt_store(gg[j], g4 + i + 256 * j); nt_store(t[j], o4 + i + 256 * j); }
            else { g4[i + 256 * j] = gg[j]; o4[i + 256 * j] = t[j]; }
            if (frag) {
                const unsigned r1 = (unsigned)(4 * (i + 256 * j)) - W1, r2 = (unsigned)(4 * (i + 256 * j)) - W2;
                if (r1 < 16u * 256u) conv12_store_fragment4(frag, 0, (int)r1, t[j], frag_rb);
                else if (r2 < 32u * 256u) {
                    conv12_store_fragment4(frag, 1, (int)r2, t[j], frag_rb);
                    conv_dgrad_store_fragment4<SpecS2>(frag + CFRAG_FWD_VECS, (int)r2, t[j]);
                }
                store_filter(first + 256 * j, t[j]);
            }
            if (fcw.w) {
                const unsigned r = (unsigned)(i + 256 * j) - fcw.first;
                if (r < fcw.n) ga3c::fc_planes_store4(fcw, r, t[j]);
            }
        }
    }
    for (size_t at = ntile * (256 * VPT) + (size_t)blockIdx.x * 256 + threadIdx.x; at < n4; at += stride) {
        const size_t i = vector_of(at);
        float4 t = t4[i], gg = g4[i];
        rmsprop4(t, gg, d4[i], s, lr, alpha, oma, eps);
        g4[i] = gg; o4[i] = t;
        if (frag) {
            const unsigned r1 = (unsigned)(4 * i) - W1, r2 = (unsigned)(4 * i) - W2;
            if (r1 < 16u * 256u) conv12_store_fragment4(frag, 0, (int)r1, t, frag_rb);
            else if (r2 < 32u * 256u) {
                conv12_store_fragment4(frag, 1, (int)r2, t, frag_rb);
                conv_dgrad_store_fragment4<SpecS2>(frag + CFRAG_FWD_VECS, (int)r2, t);
            }
            store_filter(at, t);
        }
        if (fcw.w) {
            const unsigned r = (unsigned)i - fcw.first;
            if (r < fcw.n) ga3c::fc_planes_store4(fcw, r, t);
        }
    }
    for (size_t k = n4 * 4 + (size_t)blockIdx.x * 256 + threadIdx.x; k < n; k += stride) {
        const float d = s * grad[k];
        const float gg = alpha * g[k] + oma * d * d;
        g[k] = gg;
        theta_out[k] = theta_in[k] - lr * d / sqrtf(gg + eps);
    }
}

// Counter-based normal deviates: splitmix64 of (seed, index) gives two
// 24-bit uniforms, Box-Muller turns them into one N(0,1) value.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}
__global__ __launch_bounds__(256) void init_normal_kernel(float *__restrict__ dst, size_t base, size_t n, float std,
                                                          uint64_t seed) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint64_t r = splitmix64(seed * 0xD1342543DE82EF95ull + (base + i));
    const float u1 = ((float)((r >> 40) & 0xFFFFFF) + 1.f) * (1.f / 16777216.f);   // (0, 1]
    const float u2 = (float)((r >> 8) & 0xFFFFFF) * (1.f / 16777216.f);             // [0, 1)
    dst[i] = std * sqrtf(-2.f * logf(u1)) * cosf(6.28318530717958647692f * u2);
}
__global__ __launch_bounds__(256) void fill_kernel(float *__restrict__ dst, size_t n, float v) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = v;
}

// dst = src, n floats; n4 of the 16-byte vectors first (0 where the two are not aligned alike).
__global__ __launch_bounds__(256) void copy_kernel(float *__restrict__ dst, const float *__restrict__ src, size_t n, size_t n4) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
    for (size_t k = i; k < n4; k += stride) ((float4 *)dst)[k] = ((const float4 *)src)[k];
    for (size_t k = 4 * n4 + i; k < n; k += stride) dst[k] = src[k];
}

// ------------------------------------------------------------ host helpers --

// Order between calls of one context on different streams.
//   - A writer of the parameters leaves an event when it is done (ready); every call that reads them waits for it.
//   - Predictions leave no event of their own (behind a prediction it costs 1.5 to 3 us of the stream's time, a fifth of a
//     prediction of one frame).  The first one that reads a newly published copy records one event before its work, if the other
//     copy has been read: calls of this kind are in order among themselves, so all predictions of the other copy are over then
//     (turned).
//   - A writer takes the other copy, behind that event.  If the other copy has been read and no prediction has come since, there
//     is no event, but nothing reads the published copy either, and that is written in place.
// Events are recorded only on the stream that the running call was given: a handle kept from an earlier call may by then be a
// stream that is gone, or another one.  A wait is skipped when the event was last recorded on the same stream (stream order
// already holds) or never.
int wait_mark(const Mark &m, hipStream_t s) {
    if (!m.set || m.where == s) return GA3C_OK;
    HIP_TRY(hipStreamWaitEvent(s, m.ev, 0));
    return GA3C_OK;
}
int set_mark(Mark &m, hipStream_t s, const ga3c::StopEvent *stop = nullptr) {
    if (!stop || !stop->attached) HIP_TRY(hipEventRecord(m.ev, s));
    m.set = true; m.where = s;
    return GA3C_OK;
}
// The mark's event for a call's last launch to complete; a stream that is being captured gets it as a node of its own instead.
ga3c::StopEvent stop_for(const Mark &m, hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    const hipError_t e = hipStreamIsCapturing(s, &st);
    if (e != hipSuccess) (void)hipGetLastError();
    ga3c::StopEvent stop;
    if (e == hipSuccess && st == hipStreamCaptureStatusNone) stop.ev = m.ev;
    return stop;
}
int wait_ready(ga3c_ctx *c, hipStream_t s) { return wait_mark(c->ready[c->cur], s); }
// A prediction on s is about to read the published copy.
int begin_prediction(ga3c_ctx *c, hipStream_t s) {
    if (c->reads[c->cur ^ 1] == READS_OPEN) {
        const int rc = set_mark(c->turned, s);
        if (rc != GA3C_OK) return rc;
        c->reads[c->cur ^ 1] = READS_MARKED;
    }
    c->reads[c->cur] = READS_OPEN;
    return GA3C_OK;
}
// The copy that the next writer writes; what has to be over before it does; its publication.
int copy_to_write(const ga3c_ctx *c) { return c->reads[c->cur ^ 1] == READS_OPEN ? c->cur : c->cur ^ 1; }
int wait_writable(ga3c_ctx *c, hipStream_t s) {
    const int to = copy_to_write(c);
    const int rc = c->reads[to] == READS_MARKED ? wait_mark(c->turned, s) : GA3C_OK;
    return rc == GA3C_OK ? wait_mark(c->copied[to], s) : rc;
}
int publish(ga3c_ctx *c, hipStream_t s, const ga3c::StopEvent *stop = nullptr) {
    const int to = copy_to_write(c), rc = set_mark(c->ready[to], s, stop);
    if (rc != GA3C_OK) return rc;
    c->reads[to] = READS_NONE; c->copied[to].set = false;
    c->cur = to;                 // calls enqueued from now on see the new parameters
    return GA3C_OK;
}
#define TRY(expr) do { int rc_ = (expr); if (rc_ != GA3C_OK) return rc_; } while (0)

// While one of these is alive and profiling is on, every kernel launched by this host thread carries an event pair
// of its own (launch.hpp), booked to the stage: the stage's time is the sum of its kernels' execution times.  A launch
// that does the work of two stages counts for both, its time in the proportion of their operations.  Costs one branch
// when profiling is off.
struct ProfScope final : ga3c::LaunchTimer {
    Profiler *p; int sid, sid2;
    ProfScope(ga3c_ctx *c, hipStream_t, const char *name, double flop, double bytes, const char *name2 = nullptr, double flop2 = 0, double bytes2 = 0)
        : p(c->prof), sid(-1), sid2(-1) {
        if (!p || !p->on) { p = nullptr; return; }
        try {
            p->stages.reserve(p->stages.size() + 2);
        } catch (const std::bad_alloc &) { p = nullptr; return; }      // untimed
        sid = book(name, flop, bytes);
        if (name2) sid2 = book(name2, flop2, bytes2);
        ga3c::launch_timer = this;
    }
    int book(const char *name, double flop, double bytes) {
        size_t i = 0;
        while (i < p->stages.size() && strcmp(p->stages[i].name, name)) ++i;
        if (i == p->stages.size()) p->stages.push_back({name, 0, 0.0, 0.0, 0.0});
        p->stages[i].calls += 1; p->stages[i].flop += flop; p->stages[i].bytes += bytes;
        return (int)i;
    }
    bool next_events(hipEvent_t *start, hipEvent_t *stop) override {
        ProfRec r; r.stage = sid; r.stage2 = sid2; r.a = r.b = nullptr;
        try {       // the record, and its events' way back to the pool
            if (p->recs.size() == p->recs.capacity()) p->recs.reserve(2 * p->recs.size() + 16);
            p->pool.reserve(2 * p->recs.capacity() + p->pool.size());
        } catch (const std::bad_alloc &) { return false; }
        for (hipEvent_t *e : {&r.a, &r.b}) {
            if (!p->pool.empty()) { *e = p->pool.back(); p->pool.pop_back(); }
            else if (hipEventCreate(e) != hipSuccess) { *e = nullptr; }
        }
        if (!r.a || !r.b) {
            for (hipEvent_t e : {r.a, r.b}) if (e) p->pool.push_back(e);
            return false;
        }
        p->recs.push_back(r);
        *start = r.a; *stop = r.b;
        return true;
    }
    ~ProfScope() { if (p) ga3c::launch_timer = nullptr; }
    ProfScope(const ProfScope &) = delete;
    ProfScope &operator=(const ProfScope &) = delete;
};
#define STAGE(name, flop, bytes) ProfScope prof_scope_(c, s, name, (double)(flop), (double)(bytes))
#define STAGE2(name, flop, bytes, name2, flop2, bytes2) ProfScope prof_scope_(c, s, name, (double)(flop), (double)(bytes), name2, (double)(flop2), (double)(bytes2))

const char *const CONV_FWD[GA3C_MAX_CONV] = {"conv1_fwd", "conv2_fwd", "conv3_fwd", "conv4_fwd"};
const char *const CONV_WGRAD[GA3C_MAX_CONV] = {"conv1_wgrad", "conv2_wgrad", "conv3_wgrad", "conv4_wgrad"};
const char *const CONV_DGRAD[GA3C_MAX_CONV] = {"conv1_dgrad", "conv2_dgrad", "conv3_dgrad", "conv4_dgrad"};

inline unsigned blocks_for(size_t n, int per = 256) { return (unsigned)((n + per - 1) / per); }

// Number of k-chunks for a split-k product with `tiles` output tiles and a
// reduction of length K: enough blocks to fill 256 compute units a few times
// over, chunks a multiple of the k-tile and at least two k-tiles long.
// split_want: what is asked for, never fewer with a larger K (a workspace is sized by it); rounding the chunks up may leave fewer.
inline int split_want(int tiles, int K) {
    const int maxz = std::max(1, K / (2 * GEMM_BK));
    return std::max(1, std::min((512 + tiles - 1) / tiles, maxz));
}
inline void split_into(int want, int K, int &nz, int &kchunk) {
    kchunk = (K + want - 1) / want;
    kchunk = (kchunk + GEMM_BK - 1) / GEMM_BK * GEMM_BK;
    nz = (K + kchunk - 1) / kchunk;
}
inline void pick_split(int tiles, int K, int &nz, int &kchunk) { split_into(split_want(tiles, K), K, nz, kchunk); }

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// k-chunks for the XCD-partitioned dense product: a multiple of 8 chunks (one
// or more per XCD) when the reduction is long enough, about `target` blocks in
// all (fewer chunks mean fewer partial sums to write and add up again).
inline int split_want_xcd(int tiles, int K, int target) {
    const int want = 8 * std::max(1, (target + 8 * tiles - 1) / (8 * tiles)), maxz = std::max(1, K / (2 * GEMM_BK));
    return want <= maxz ? want : maxz >= 8 ? maxz / 8 * 8 : maxz;
}
inline void pick_split_xcd(int tiles, int K, int &nz, int &kchunk, int target = 512) { split_into(split_want_xcd(tiles, K, target), K, nz, kchunk); }

int alloc_work(Work &w, const ga3c_ctx *c, int cap, bool training) {
    w.cap = cap;
    if (cap <= 0) return GA3C_OK;
    for (int l = 0; l < c->nconv; ++l)
        HIP_TRY(hipMalloc(&w.act[l], sizeof(float) * ((size_t)cap * c->geom[l].OC * c->geom[l].OHW + BAND_SLACK)));
    // layers of 32 filters whose forward pass in updates is conv_f32_fwd_kernel and whose gradient comes from conv_band_dgrad_kernel
    for (int l = 0; training && !c->rb && l + 1 < c->nconv; ++l)
        if (c->band[l] && c->band[l + 1]) {
            w.bits[l].plane = PositiveBits::plane_of((size_t)cap * c->geom[l].OHW);
            HIP_TRY(hipMalloc(&w.bits[l].at, PositiveBits::PLANES * w.bits[l].plane));
        }
    HIP_TRY(hipMalloc(&w.h, sizeof(float) * (size_t)cap * c->F));
    HIP_TRY(hipMalloc(&w.zv, sizeof(float) * (size_t)cap * (c->A + 1)));
    return GA3C_OK;
}

void free_work(Work &w) {
    (void)hipFree(w.ws);
    for (int l = 0; l < GA3C_MAX_CONV; ++l) { (void)hipFree(w.act[l]); (void)hipFree(w.bits[l].at); }
    (void)hipFree(w.h);
    (void)hipFree(w.zv);
}

// Tile shapes: output channels are few (16..64), pixels are many.
template <class P>
hipError_t launch_conv_like(const P &p, int nz, hipStream_t s, bool a_rows_unused = false) {
    (void)a_rows_unused;
    if (p.M <= 16) return launch_gemm<1, 4, 1, 4, false, true>(p, nz, s);   // 16 x 256
    if (p.M <= 32) return launch_gemm<2, 2, 1, 4, false, true>(p, nz, s);   // 32 x 128
    return launch_gemm<2, 2, 2, 2, false, true>(p, nz, s);                  // 64 x 64
}
inline int conv_like_tiles(int M, int N) {
    if (M <= 16) return cdiv(N, 256);
    if (M <= 32) return cdiv(N, 128);
    return cdiv(M, 64) * cdiv(N, 64);
}

// LDS the fused training heads kernel may ask for; larger heads fall back to the separate kernels.
constexpr size_t HEADS_TRAIN_MAX_LDS = 160 * 1024;
constexpr size_t HEADS_FWD_MAX_LDS = 160 * 1024;      // all of a compute unit's LDS

// A kernel may take more than 64 KB of dynamic LDS only after its limit has
// been raised; `set` remembers the largest size asked for so far.
static hipError_t allow_dynamic_lds(const void *kernel, size_t bytes, size_t &set) {
    if (bytes <= 64 * 1024 || bytes <= set) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) set = bytes;
    return e;
}

template <class SP>
inline bool spec_matches(const ConvGeom &g, bool byte_input) {
    return g.C == SP::C && g.H == SP::H && g.W == SP::W && g.OC == SP::OC && g.KS == SP::KS && g.S == SP::S &&
           byte_input == (sizeof(typename SP::TIn) == 1);
}
inline bool is_aligned16(const void *p) { return (((uintptr_t)p) & 15) == 0; }

// Whether the forward kernels of an any-size layer take its filters as terms: with rounded operands, and the byte layer of predictions
// that run a kernel per layer.
bool takes_terms(const ga3c_ctx *c, int l) { return c->rb || (l == 0 && !c->conv123); }

// Things derived from parameter copy i, rebuilt on s after that copy was written there.  fc: the fc weights' too (an update
// writes those itself).  stop: the event for the last launch, if the larger nets' fragments are among them.
int refresh_derived(ga3c_ctx *c, int i, hipStream_t s, bool fc = true, ga3c::StopEvent *stop = nullptr) {
    if (fc && c->fcw[i].w) {
        ga3c::launch(fc_planes_kernel, dim3(blocks_for(c->fcw[i].n)), dim3(256), 0, s, (const float4 *)c->theta2[i], c->fcw[i]);
        HIP_TRY(hipGetLastError());
    }
    if (c->cfrag[i]) {
        HIP_TRY(launch_conv12_filter_fragments(c->theta2[i] + c->off[0], c->theta2[i] + c->off[2], c->cfrag[i], s, c->rb));
        if (c->cfrag_dgrad)
            HIP_TRY(launch_conv_dgrad_filter_fragments<SpecS2>(c->theta2[i] + c->off[2], c->cfrag[i] + CFRAG_FWD_VECS, s));
        if (c->hfrag[i]) HIP_TRY(launch_conv12_f16_filters(c->theta2[i] + c->off[0], c->theta2[i] + c->off[2], c->hfrag[i], s));
    }
    if (c->lfrag[i]) {
        const float *th = c->theta2[i];
        ga3c::launch_stop(c->bfrag[i] ? nullptr : stop, large_filter_fragments_kernel, dim3(LFRAG_B3 + (c->conv123 ? Conv123Large::BLOCKS : 0)),
                          dim3(256), 0, s, th + c->off[0], th + c->off[2], th + c->off[4], c->lfrag[i]);
        HIP_TRY(hipGetLastError());
    }
    if (c->bfrag[i]) {
        FragJobs jobs;
        jobs.n = 0;
        int blocks = 0;
        auto add = [&](int l, int kind, u32x4 *dst, int n) {
            jobs.job[jobs.n++] = FragJob{c->theta2[i] + c->off[2 * l], dst, kind, c->geom[l].C, c->geom[l].OC, c->geom[l].KS, n, blocks};
            blocks += cdiv(n, 256);
        };
        for (int l = 0; l < c->nconv; ++l) {
            if (!c->band[l]) continue;
            const ConvGeom &g = c->geom[l];
            if (takes_terms(c, l)) add(l, l == 0 ? FRAG_BYTES8 : FRAG_CONV, c->bfrag[i] + c->bfrag_fwd[l], g.OC * g.K / 8);
            if (!c->rb && (l > 0 || c->max_train > 0)) add(l, FRAG_F32, c->bfrag[i] + c->bfrag_f32[l], g.OC * g.K / 4);
            if (l > 0 && c->max_train > 0) add(l, FRAG_DGRAD, c->bfrag[i] + c->bfrag_dgrad[l], g.OC * g.K / 8);
        }
        const float *th = c->theta2[i];
        auto both = [&](auto kernel, int more) {
            ga3c::launch_stop(stop, kernel, dim3(blocks + more), dim3(256), 0, s, th + c->off[0], th + c->off[2], th + c->off[4], c->bfrag[i] + c->bfrag_123, jobs);
        };
        if (c->conv123 == CONV123_PAPER4) both(family_filter_fragments_kernel<Conv123Paper4>, Conv123Paper4::BLOCKS);
        else if (c->conv123 == CONV123_PAPER3) both(family_filter_fragments_kernel<Conv123Paper3>, Conv123Paper3::BLOCKS);
        else ga3c::launch_stop(stop, c->rb ? band_filter_fragments_kernel<1> : band_filter_fragments_kernel<3>, dim3(blocks), dim3(256), 0, s, jobs);
        HIP_TRY(hipGetLastError());
    }
    return GA3C_OK;
}

// Layers that the any-size kernels take: the byte layer with 8x8 filters over four planes of width 84, and 4x4 stride-2
// layers on 32 channels; layers with kernels of their own shape keep those.
bool on_band_kernels(const ConvGeom &g, int l) {
    if (g.OC != 32 && !(l == 0 && g.OC == 16) && !(l > 0 && g.OC == 64)) return false;
    if (l == 0) return g.C == 4 && g.KS == 8 && bytes_ok(g.H, g.W, g.S) && !spec_matches<SpecS1>(g, true) && !spec_matches<SpecL1>(g, true);
    if (g.C != 32 || g.KS != 4 || g.S != 2 || spec_matches<SpecL2>(g, false)) return false;
    return band_ok<32>(g.H, g.W) && band_grads_ok(g.H, g.W);
}

// Predictions of up to how many frames go out as one launch (predict_small_kernel); 0: not this network's.  42: the most that 256 blocks hold, two
// frames and four slices of the fc layer each; beyond, slices are halves and the kernel takes as long as the three launches do and more
// (us a call, one launch / three: 42 frames 15.2 / 15.5, 43: 16.9 / 15.4, 64: 17.8 / 15.9; rounded 14.1 / 15.7, 16.8 / 15.8, 17.1 / 15.8;
// ga3c_predict_static 19.8 / 19.1 to 20.6, 21.6 / 19.0 to 20.4, 22.5 / 19.4 to 20.8).  Where the heads of many actions leave no room for
// two frames in LDS, 21 (63 actions, 21 frames 15.0 / 16.5, 22: 16.6 / 16.5, 42: 19.0 / 16.9; rounded 15.0 / 14.4, 17.0 / 14.4, 18.9 / 14.8).
int small_launch_frames(const ga3c_ctx *c) {
    const int nb = 2 * c->nconv;
    if (c->nconv != 2 || c->F != SP_FC || c->flat != SP_FLAT || c->off[nb + 1] % 4 != 0 || c->off[nb + 2] % 4 != 0) return 0;
    return SpLds<2>::bytes(c->A) <= HEADS_FWD_MAX_LDS ? SP_MAX_FRAMES : SP_ONE_FRAME;
}

// Forward pass of `B` frames into `w`; heads outputs to the optional pointers.  table (frames is nullptr then): the frames lie
// where its entries point; only where takes_frame_table says so.
int forward(ga3c_ctx *c, int which, Work &w, const uint8_t *frames, const uint8_t *const *table, int B, bool keep_zv, float *logits, float *values,
            float *probs, const float *uniforms, int32_t *actions, hipStream_t s, bool with_heads = true) {
    const float *th = c->theta2[which];
    const int nb = 2 * c->nconv;
    int first = 0;
    std::fill(w.bits_set, w.bits_set + GA3C_MAX_CONV, false);
    if (c->fast && c->ticket && c->cfrag[which] && is_aligned16(frames) && !keep_zv && with_heads && B <= c->small_frames) {
        // a handful of frames: one launch for the whole network, in about as many blocks as there are compute units
        const bool two = B > SP_ONE_FRAME;
        const int NS = B <= 5 ? 16 : B <= 10 ? 8 : 4;
        const int groups = two ? (B + 1) / 2 : B;
        if ((size_t)B * 3 * SP_FC > w.ws_floats) return fail(GA3C_EINVAL, "internal: workspace too small (small predictions)");
        const ConvGeom &g0 = c->geom[0], &g1 = c->geom[1];
        STAGE("predict_small", 2.0 * B * (g0.OHW * g0.OC * g0.K + g1.OHW * g1.OC * g1.K + (double)c->flat * c->F + c->F * (c->A + 1)),
              (double)B * g0.CHW + 4.0 * c->flat * c->F);
        typedef decltype(&predict_small_kernel<false, 1, false>) PredictSmall;
        static const PredictSmall kernels[8] = {predict_small_kernel<false, 1, false>, predict_small_kernel<false, 1, true>,
                                                predict_small_kernel<false, 2, false>, predict_small_kernel<false, 2, true>,
                                                predict_small_kernel<true, 1, false>,  predict_small_kernel<true, 1, true>,
                                                predict_small_kernel<true, 2, false>,  predict_small_kernel<true, 2, true>};
        static size_t lds_set[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const int k = (c->rb ? 4 : 0) + (two ? 2 : 0) + (table ? 1 : 0);
        const size_t lds = two ? SpLds<2>::bytes(c->A) : SpLds<1>::bytes(c->A);
        HIP_TRY(allow_dynamic_lds((const void *)kernels[k], lds, lds_set[k]));
        ga3c::launch(kernels[k], dim3((3 * NS * groups + 7) / 8 * 8), dim3(512), lds, s, frames, table, c->cfrag[which], th + c->off[1],
                     th + c->off[3], th + c->off[nb], th + c->off[nb + 1], w.ws, c->ticket, B, NS, c->A, th + c->off[nb + 2], th + c->off[nb + 3],
                     th + c->off[nb + 4], th + c->off[nb + 5], logits, values, probs, uniforms, actions, 1.f / 255.f, c->rb);
        HIP_TRY(hipGetLastError());
        return GA3C_OK;
    }
    if (c->fast && (keep_zv || c->rb ? c->cfrag[which] : c->hfrag[which]) && is_aligned16(frames)) {
        // small net: both convolution layers in one kernel; layer-1 activations go to HBM only when training
        const ConvGeom &g0 = c->geom[0], &g1 = c->geom[1];
        STAGE("conv12_fwd", 2.0 * B * (g0.OHW * g0.OC * g0.K + g1.OHW * g1.OC * g1.K),
              (double)B * (g0.CHW + (keep_zv ? 4.0 * g0.OC * g0.OHW : 0.0) + 4.0 * g1.OC * g1.OHW));
        // predictions at fp32 accuracy: two float16 terms; updates keep the rounding of their sums (conv123_f16.hpp says why)
        if (!keep_zv && !c->rb)
            HIP_TRY(launch_conv12_f16(frames, table, c->hfrag[which], th + c->off[1], th + c->off[3], w.act[1], B, 1.f / 255.f, th + c->off[0],
                                      th + c->off[2], s));
        else
            HIP_TRY(launch_conv12_fused_fwd(frames, table, c->cfrag[which], th + c->off[1], th + c->off[3],
                                            keep_zv ? w.act[0] : nullptr, w.act[1], B, 1.f / 255.f, s, c->rb));
        first = 2;
    }
    if (c->fast && c->conv123 && !keep_zv && is_aligned16(frames)) {
        // predictions: all three layers in one kernel
        const ConvGeom &g0 = c->geom[0], &g1 = c->geom[1], &g2 = c->geom[2];
        STAGE("conv123_fwd", 2.0 * B * (g0.OHW * g0.OC * g0.K + g1.OHW * g1.OC * g1.K + g2.OHW * g2.OC * g2.K),
              (double)B * (g0.CHW + 4.0 * g2.OC * g2.OHW));
        auto go = [&](auto launch, const u32x4 *frag) {
            return launch(frames, table, frag, th + c->off[1], th + c->off[3], th + c->off[5], w.act[2], B, 1.f / 255.f, th + c->off[0],
                          th + c->off[2], th + c->off[4], s);
        };
        if (c->conv123 == CONV123_LARGE)
            HIP_TRY(go(table ? launch_conv123_f16<Conv123Large, true> : launch_conv123_f16<Conv123Large, false>, c->lfrag[which] + LFRAG_VECS));
        else if (c->conv123 == CONV123_PAPER4)
            HIP_TRY(go(table ? launch_conv123_f16<Conv123Paper4, true> : launch_conv123_f16<Conv123Paper4, false>, c->bfrag[which] + c->bfrag_123));
        else HIP_TRY(go(launch_conv123_f16<Conv123Paper3, false>, c->bfrag[which] + c->bfrag_123));      // its frames never come in a table
        first = 3;
    }
    for (int l = first; l < c->nconv; ++l) {
        const ConvGeom &g = c->geom[l];
        STAGE(CONV_FWD[l], 2.0 * B * g.OHW * g.OC * g.K, (double)B * ((l == 0 ? 1.0 : 4.0) * g.CHW + 4.0 * g.OC * g.OHW));
        const float *wl = th + c->off[2 * l], *bl = th + c->off[2 * l + 1];
        const void *xin = l == 0 ? (const void *)frames : (const void *)w.act[l - 1];
        if (c->fast && is_aligned16(wl) && is_aligned16(xin)) {
            if (spec_matches<SpecS1>(g, l == 0)) {
                HIP_TRY(launch_conv1_bf16x3_fwd<16>((const uint8_t *)xin, table, wl, bl, w.act[l], B, 1.f / 255.f, s, c->rb));
                continue;
            }
            if (spec_matches<SpecL1>(g, l == 0)) {
                HIP_TRY(launch_conv1_bf16x3_fwd<32>((const uint8_t *)xin, table, wl, bl, w.act[l], B, 1.f / 255.f, s, c->rb));
                continue;
            }
            if (spec_matches<SpecS2>(g, l == 0)) {
                HIP_TRY(launch_conv2_bf16x6_fwd((const float *)xin, wl, bl, w.act[l], B, s, c->rb));
                continue;
            }
            if (spec_matches<SpecL2>(g, l == 0)) {      // the frame as split bf16 planes in LDS: one block per CU
                HIP_TRY((launch_conv_fwd_bf16x6<SpecL2, 4>((const float *)xin, wl, bl, w.act[l], B, s, 256, c->rb,
                                                           c->lfrag[which] && l == 1 ? c->lfrag[which] + LFRAG_FWD2 : nullptr)));
                continue;
            }
            if (spec_matches<SpecL3>(g, l == 0)) {
                HIP_TRY((launch_conv_fwd_bf16x6<SpecL3, 4>((const float *)xin, wl, bl, w.act[l], B, s, 256, c->rb,
                                                           c->lfrag[which] && l == 2 ? c->lfrag[which] + LFRAG_FWD3 : nullptr)));
                continue;
            }
        }
        // (Predictions whose maps fit a compute unit's LDS are done already, in one kernel.)
        // At fp32 accuracy the 4x4 layers run on the fp32 instruction, straight from memory, in both calls: faster than bands
        // staged as three bf16 terms up to 256 frames (128 frames: 77x77 map 65 / 73 us, 26x26 11.8 / 12.7, 12x12 with 64 filters 6.1 /
        // 10.2, the only loss 37x37 with 64 filters 27.9 / 24.8; one frame 4.6 / 9.8) and nearer to the exact sums (2.9e-7 /
        // 3.3e-7); with 512 frames a call is still ahead (stride-1 member 545 -> 504 us, stride 3 76.1 -> 70.5, stride 4 56.8 -> 50.9).
        // The byte layer does so in updates only, whose activations keep the any-shape kernels' order of sums
        // (conv_band_f32.hpp); predictions take three bf16 terms of its weights (128 frames, stride 3: 9.5 us, on the fp32
        // instruction 19.4).  With operands rounded to bfloat16 everything takes one term (640 frames of the stride-3 member, on
        // the fp32 instruction / with one term: conv1 70 / 22, conv2 35 / 19, conv3 16 / 10 us).
        if (c->fast && c->band[l] && is_aligned16(xin) && is_aligned16(wl)) {
            const u32x4 *wf = c->bfrag[which] + c->bfrag_fwd[l];
            const float4 *w32 = (const float4 *)(c->bfrag[which] + c->bfrag_f32[l]);
            w.bits_set[l] = w.bits[l].at != nullptr;
            if (l == 0) {
                const bool f32 = !c->rb && keep_zv;
                if (f32 && g.OC == 16) HIP_TRY((launch_conv_f32_fwd<uint8_t, 16>(frames, w32, bl, w.act[l], B, g.H, g.W, g.S, 1.f / 255.f, s)));
                else if (f32) HIP_TRY((launch_conv_f32_fwd<uint8_t, 32>(frames, w32, bl, w.act[l], B, g.H, g.W, g.S, 1.f / 255.f, s, w.bits[l])));
                else if (g.OC == 16) HIP_TRY(launch_conv_bytes_fwd<16>(frames, wf, bl, w.act[l], B, g.H, g.S, 1.f / 255.f, s, c->rb));
                else HIP_TRY(launch_conv_bytes_fwd<32>(frames, wf, bl, w.act[l], B, g.H, g.S, 1.f / 255.f, s, c->rb));
            } else if (c->rb && g.OC == 32) HIP_TRY((launch_conv_band_fwd<32, 32>(w.act[l - 1], wf, bl, w.act[l], B, g.H, g.W, s)));
            else if (c->rb) HIP_TRY((launch_conv_band_fwd<32, 64>(w.act[l - 1], wf, bl, w.act[l], B, g.H, g.W, s)));
            else if (g.OC == 32) HIP_TRY((launch_conv_f32_fwd<float, 32>(w.act[l - 1], w32, bl, w.act[l], B, g.H, g.W, g.S, 1.f, s, w.bits[l])));
            else HIP_TRY((launch_conv_f32_fwd<float, 64>(w.act[l - 1], w32, bl, w.act[l], B, g.H, g.W, g.S, 1.f, s)));
            continue;
        }
        if (l == 0) {
            ConvFwdP<uint8_t> p; p.rb = c->rb;
            p.M = g.OC; p.N = B * g.OHW; p.K = g.K; p.g = g;
            p.x = frames; p.w = th + c->off[0]; p.bias = th + c->off[1];
            p.y = w.act[0]; p.scale = 1.f / 255.f;
            HIP_TRY(launch_conv_like(p, 1, s));
        } else {
            ConvFwdP<float> p; p.rb = c->rb;
            p.M = g.OC; p.N = B * g.OHW; p.K = g.K; p.g = g;
            p.x = w.act[l - 1]; p.w = th + c->off[2 * l]; p.bias = th + c->off[2 * l + 1];
            p.y = w.act[l]; p.scale = 1.f;
            HIP_TRY(launch_conv_like(p, 1, s));
        }
    }
    const float *fc_ws = nullptr;
    int fc_nz = 1;
    {   // fully connected: h[b][o] = max(0, b[o] + sum_i x[b][i] Wfc[o][i])
        const float *x = w.act[c->nconv - 1];
        const float *wfc = th + c->off[nb];
        STAGE("fc_fwd", 2.0 * B * c->F * c->flat, 0);
        int nz, kchunk;
        if (c->fast && dense_operand_ok(x, c->flat, c->flat) && dense_operand_ok(wfc, c->flat, c->flat)) {
            // Up to 16 tiles a prediction's fc product takes one block per compute unit: a second one would double the partial
            // sums that the heads add up one after the other.  One block against two, us a call (the convolutions took longer then): larger
            // net 16 frames 42.2 / 44.2, 128: 45.8 / 48.1; small net 192: 21.3 / 21.7, 256: 21.0 / 22.8.  With more tiles it depends (small
            // net 300 frames 22.4 / 23.1, 400: 23.0 / 24.2, 512: 23.9 / 23.6, 768: 28.1 / 28.9; larger net 140: 25.8 / 25.6, 192: 26.5 / 26.7, 256:
            // 30.2 / 27.6, 300: 41.1 / 42.8); the line stays because of the larger net's 256, and because a prediction's value enters its
            // segment's update as the bootstrap, and another rounding of it can move a pre-activation across zero a few updates later.
            // Updates keep one order of sums.
            const int tiles = cdiv(B, 64) * cdiv(c->F, 64);
            pick_split_xcd(tiles, c->flat, nz, kchunk, !keep_zv && tiles <= 16 ? 256 : 512);
            if ((size_t)nz * B * c->F > w.ws_floats) return fail(GA3C_EINVAL, "internal: split-k workspace too small (fc)");
            if (c->fcw[which].w && fc_forward_batch_ok(x, B, c->flat)) {
                FcForwardArgs p;
                p.M = B; p.N = c->F; p.K = c->flat; p.kchunk = kchunk; p.nz = nz;
                p.x = x; p.w = c->fcw[which].w; p.part = w.ws;
                size_t pass_bytes = 0;           // (of layers in one kernel a prediction writes the last one's only)
                for (int l = first > 0 && !keep_zv ? first - 1 : 0; l < c->nconv; ++l) pass_bytes += sizeof(float) * (size_t)B * c->geom[l].OC * c->geom[l].OHW;
                HIP_TRY(launch_fc_forward(p, pass_bytes, c->rb, s));
            } else {
                DenseGemmArgs p{}; p.rb = c->rb;
                p.M = B; p.N = c->F; p.K = c->flat; p.kchunk = kchunk; p.nz = nz;
                p.A = x; p.lda = c->flat; p.B = wfc; p.ldb = c->flat;
                p.C = w.ws; p.ldc = c->F; p.aux = nullptr;
                HIP_TRY((launch_dense_gemm_bf16x6<2, 2, 2, 2, false, false, DG_PARTIAL>(p, DG_SPLIT_Z, s)));
            }
            fc_ws = w.ws; fc_nz = nz;
        } else {
            pick_split(cdiv(B, 64) * cdiv(c->F, 64), c->flat, nz, kchunk);
            GemmP<EPI_PARTIAL, false> p; p.rb = c->rb;
            p.M = B; p.N = c->F; p.K = c->flat; p.kchunk = kchunk;
            p.A = x; p.sAm = c->flat; p.sAk = 1;
            p.B = wfc; p.sBn = c->flat; p.sBk = 1;
            p.C = w.ws; p.ldc = c->F; p.aux = nullptr;
            if ((size_t)nz * B * c->F > w.ws_floats) return fail(GA3C_EINVAL, "internal: split-k workspace too small (fc)");
            HIP_TRY((launch_gemm<2, 2, 2, 2, false, false>(p, nz, s)));
            fc_ws = w.ws; fc_nz = nz;
        }
    }
    w.fc_ws = fc_ws; w.fc_nz = fc_nz;
    if (!with_heads) return GA3C_OK;          // the caller finishes the fc layer and the heads itself
    const int hf = heads_loads(c->F, fc_nz, fc_ws, th + c->off[nb + 1], w.h, th + c->off[nb + 2]);
    const int nj = c->F % 256 == 0 ? c->F / 256 : 0;
    if (c->fast && !keep_zv && hf != LOADS_SCALAR && (nj == 1 || nj == 2 || nj == 4)) {
        typedef decltype(&heads_predict_kernel<1, 8>) HeadsPredict;
        static const HeadsPredict hp_kernels[6] = {heads_predict_kernel<1, 8>, heads_predict_kernel<1, 20>, heads_predict_kernel<2, 8>,
                                                   heads_predict_kernel<2, 16>, heads_predict_kernel<4, 8>, heads_predict_kernel<4, 8>};
        static size_t hp_lds_set[6] = {0, 0, 0, 0, 0, 0};
        const int k = (nj == 1 ? 0 : nj == 2 ? 2 : 4) + (hf == LOADS_VEC16 ? 1 : 0);
        const size_t lds = sizeof(float) * (c->A + 1) * (c->F + 4);
        HIP_TRY(allow_dynamic_lds((const void *)hp_kernels[k], lds, hp_lds_set[k]));
        STAGE("heads_fwd", 2.0 * B * c->F * (c->A + 1), 4.0 * fc_nz * B * c->F);
        // A block per compute unit at most.  With eight chunks or fewer (1024 units from 193 frames on) there is little to share out:
        // calls of 193 / 224 / 256 frames of the stride-1 member 237 / 253 / 271 us with four frames a block, 233 / 250 / 269 with one.
        if (B <= 256 && hf == LOADS_VEC16) {
            static const HeadsPredict few[3] = {heads_predict_few_kernel<1>, heads_predict_few_kernel<2>, heads_predict_few_kernel<4>};
            ga3c::launch(few[nj / 2], dim3(B), dim3(256), 0, s, fc_ws, fc_nz, th + c->off[nb + 1], B, c->A, th + c->off[nb + 2],
                         th + c->off[nb + 3], th + c->off[nb + 4], th + c->off[nb + 5], logits, values, probs, uniforms, actions, c->rb);
            HIP_TRY(hipGetLastError());
            return GA3C_OK;
        }
        ga3c::launch(hp_kernels[k], dim3(cdiv(B, 4)), dim3(256), lds, s, fc_ws, fc_nz, th + c->off[nb + 1], B, c->A, th + c->off[nb + 2],
                     th + c->off[nb + 3], th + c->off[nb + 4], th + c->off[nb + 5], logits, values, probs, uniforms, actions, c->rb);
        HIP_TRY(hipGetLastError());
        return GA3C_OK;
    }
    const size_t hf_lds = sizeof(float) * heads_lds_floats(c->F, c->A);
    typedef decltype(&heads_fwd_kernel<LOADS_SCALAR>) HeadsFwd;
    static const HeadsFwd hf_kernels[3] = {heads_fwd_kernel<LOADS_SCALAR>, heads_fwd_kernel<LOADS_VEC8>, heads_fwd_kernel<LOADS_VEC16>};
    static size_t hf_lds_set[3] = {0, 0, 0};
    HIP_TRY(allow_dynamic_lds((const void *)hf_kernels[hf], hf_lds, hf_lds_set[hf]));
    STAGE("heads_fwd", 2.0 * B * c->F * (c->A + 1), 4.0 * (fc_nz + 1) * B * c->F);
    ga3c::launch(hf_kernels[hf], dim3(cdiv(B, 4)), dim3(256), hf_lds, s, fc_ws, fc_nz,
                       th + c->off[nb + 1], w.h, B, c->F, c->A, th + c->off[nb + 2],
                       th + c->off[nb + 3], th + c->off[nb + 4], th + c->off[nb + 5],
                       keep_zv ? w.zv : nullptr, logits, values, probs, uniforms, actions, c->rb, FastDiv(std::max(1, c->F / 4)), FastDiv(c->A + 1));
    HIP_TRY(hipGetLastError());
    return GA3C_OK;
}

// Partial weight gradients that an update of B frames leaves for a layer on conv_band_grads.hpp's kernels; 0 for every other layer.
int band_grad_parts(const ga3c_ctx *c, int l, int B) {
    const ConvGeom &g = c->geom[l];
    if (!c->band[l]) return 0;
    if (l == 0) return bytes_wgrad_ok(g.S, g.OC) ? bytes_wgrad_parts(B, g.H, g.S, c->rb) : 0;
    return g.OC == 32 ? band_wgrad_parts<32>(B, g.H, g.W, c->rb) : band_wgrad_parts<64>(B, g.H, g.W, c->rb);
}

// Floats of split-k workspace a call on up to `cap` frames can need.
size_t workspace_floats(const ga3c_ctx *c, int cap, bool training) {
    size_t need = 0;
    for (int B = 1; B <= cap; ++B) {        // fc forward: depends on the batch
        int nz, kc;
        pick_split(cdiv(B, 64) * cdiv(c->F, 64), c->flat, nz, kc);
        need = std::max(need, (size_t)nz * B * c->F);
        pick_split_xcd(cdiv(B, 64) * cdiv(c->F, 64), c->flat, nz, kc);
        need = std::max(need, (size_t)nz * B * c->F);
    }
    const int B = cap;
    if (training && B > 0) {       // every weight gradient has a region of its own (rounded up to 64 floats)
        size_t sum = 0;
        auto add = [&](size_t floats) { sum += (floats + 63) / 64 * 64; };
        for (int l = 0; l < c->nconv; ++l) {
            const ConvGeom &g = c->geom[l];
            int nz = split_want(conv_like_tiles(g.OC, g.K + 1), B * g.OHW);
            // any-shape kernel; one partial per block; or bands: as many as fit from BAND_WGRAD_ITEMS frames on, before that also more
            // of fewer rows (five frames of the stride-3 member 12 MB, with the 512 of the largest updates 120)
            if (!c->band[l]) nz = std::max(nz, std::min(B, 512));
            for (int b = 1; c->band[l] && b <= std::min(B, BAND_WGRAD_ITEMS); ++b) nz = std::max(nz, band_grad_parts(c, l, b));
            nz = std::max(nz, band_grad_parts(c, l, B));
            add((size_t)nz * g.OC * (g.K + 1));
        }
        const bool fold = c->fold_ok && fc_grads_fold(c->F, c->flat, 1 << 30, c->dhp.terms);
        const int dense = fold ? 0 : split_want_xcd(cdiv(c->F, 64) * cdiv(c->flat, 64), B, 256);
        add((size_t)std::max(split_want(cdiv(c->F, 64) * cdiv(c->flat + 1, 64), B), dense) * c->F * (c->flat + 1));
        add((size_t)std::max(split_want(conv_like_tiles(c->A + 1, c->F + 1), B), cdiv(B, HD_FRAMES)) * (c->A + 1) * (c->F + 1));
        need = (need + 63) / 64 * 64 + sum;      // the regions follow the fc partial sums
    }
    return need;
}

}  // namespace

// Host-only part of setting up a context: layer geometry, parameter offsets, counts.  Touches no device memory.
// On a layer that does not fit its input, returns GA3C_EINVAL with c->nconv set to that layer's index.
static int init_shape(ga3c_ctx *c, const ga3c_net_desc *d) {
    c->rb = d->math;
    c->desc = *d;
    c->nconv = d->n_conv; c->F = d->fc_units; c->A = d->n_actions;
    int C = d->in_c, H = d->in_h, W = d->in_w;
    int64_t pos = 0; int no = 0;
    for (int l = 0; l < c->nconv; ++l) {
        const int oc = d->conv[l].oc, ks = d->conv[l].k, st = d->conv[l].stride;
        if (oc < 1 || ks < 1 || st < 1 || ks > H || ks > W) { c->nconv = l; return GA3C_EINVAL; }
        ConvGeom &g = c->geom[l];
        g.C = C; g.H = H; g.W = W; g.OC = oc; g.KS = ks; g.S = st;
        g.OH = (H - ks) / st + 1; g.OW = (W - ks) / st + 1;
        g.K = C * ks * ks; g.OHW = g.OH * g.OW; g.CHW = C * H * W;
        g.dOHW = FastDiv(g.OHW); g.dOW = FastDiv(g.OW);
        g.koff = nullptr;
        c->off[no++] = pos; pos += (int64_t)oc * g.K;
        c->off[no++] = pos; pos += oc;
        C = oc; H = g.OH; W = g.OW;
    }
    c->flat = C * H * W;
    c->off[no++] = pos; pos += (int64_t)c->flat * c->F;
    c->off[no++] = pos; pos += c->F;
    c->off[no++] = pos; pos += (int64_t)c->A * c->F;
    c->off[no++] = pos; pos += c->A;
    c->off[no++] = pos; pos += c->F;
    c->off[no++] = pos; pos += 1;
    c->off[no++] = pos;
    c->noff = no; c->P = (size_t)pos;
    return GA3C_OK;
}

// ------------------------------------------------------------------ C ABI ---

extern "C" int ga3c_create(const ga3c_net_desc *d, int max_predict_batch, int max_train_frames, ga3c_ctx **out) {
    if (out) *out = nullptr;
    if (!d || !out) return fail(GA3C_EINVAL, "ga3c_create: null argument");
    if (d->n_conv < 1 || d->n_conv > GA3C_MAX_CONV) return fail(GA3C_EINVAL, "ga3c_create: n_conv must be 1..4");
    if (d->n_actions < 1 || d->n_actions > GA3C_MAX_ACTIONS)
        return fail(GA3C_EINVAL, "ga3c_create: n_actions must be 1..%d", GA3C_MAX_ACTIONS);
    if (d->in_c < 1 || d->in_h < 1 || d->in_w < 1 || d->fc_units < 1) return fail(GA3C_EINVAL, "ga3c_create: bad sizes");
    if (d->math != 0 && d->math != 1) return fail(GA3C_EINVAL, "ga3c_create: math must be 0 (fp32) or 1 (bfloat16 operands)");
    if (max_predict_batch < 0 || max_train_frames < 0) return fail(GA3C_EINVAL, "ga3c_create: negative capacity");
    if ((size_t)heads_lds_floats(d->fc_units, d->n_actions) * sizeof(float) > HEADS_FWD_MAX_LDS)
        return fail(GA3C_EINVAL, "ga3c_create: (n_actions + 5) * (fc_units + 16) must not exceed 40960");

    ga3c_ctx *c = new (std::nothrow) ga3c_ctx();
    if (!c) return fail(GA3C_ENOMEM, "ga3c_create: host allocation failed");
    memset((void *)c, 0, sizeof(*c));
    c->prof = new (std::nothrow) Profiler();
    c->fast = true;
    c->max_pred = max_predict_batch; c->max_train = max_train_frames;

    if (init_shape(c, d) != GA3C_OK) {
        const int l = c->nconv;      // init_shape leaves the index of the offending layer here
        delete c->prof;
        delete c;
        return fail(GA3C_EINVAL, "ga3c_create: conv layer %d does not fit its input", l);
    }
    // 32-bit index limits of the kernels
    const int maxB = std::max(max_predict_batch, max_train_frames);
    for (int l = 0; l < c->nconv; ++l)
        if ((double)maxB * std::max(c->geom[l].OHW, c->geom[l].H * c->geom[l].W) >= 2.0e9) {
            delete c->prof;
            delete c;
            return fail(GA3C_EINVAL, "ga3c_create: capacity too large for 32-bit pixel indices");
        }

    int rc = GA3C_OK;
    auto guard = [&](int r) { if (r != GA3C_OK && rc == GA3C_OK) rc = r; return r == GA3C_OK; };
    auto dmalloc = [&](void **p, size_t bytes) -> int {
        HIP_TRY(hipMalloc(p, bytes ? bytes : 16));
        return GA3C_OK;
    };
    // filter-tap offset tables
    for (int l = 0; l < c->nconv && rc == GA3C_OK; ++l) {
        ConvGeom &g = c->geom[l];
        const int n = (g.K + 3) / 4 * 4;
        std::unique_ptr<int[]> t(new (std::nothrow) int[n]());
        if (!t) { guard(fail(GA3C_ENOMEM, "ga3c_create: host allocation failed")); break; }
        for (int cc = 0; cc < g.C; ++cc)
            for (int u = 0; u < g.KS; ++u)
                for (int v = 0; v < g.KS; ++v) t[(cc * g.KS + u) * g.KS + v] = cc * g.H * g.W + u * g.W + v;
        if (!guard(dmalloc((void **)&c->koff[l], sizeof(int) * n))) break;
        hipError_t e = hipMemcpy(c->koff[l], t.get(), sizeof(int) * n, hipMemcpyHostToDevice);
        if (e != hipSuccess) { guard(fail(GA3C_EHIP, "hipMemcpy: %s", hipGetErrorString(e))); break; }
        g.koff = c->koff[l];
    }
    // these events order kernels of one device and nobody inspects them: no fence to the host's memory (1 us of each call)
    constexpr unsigned order_only = hipEventDisableTiming | hipEventDisableSystemFence;
    for (int i = 0; i < 2 && rc == GA3C_OK; ++i) {
        guard(dmalloc((void **)&c->theta2[i], sizeof(float) * c->P));
        for (Mark *m : {&c->ready[i], &c->copied[i], &c->turned})
            if (rc == GA3C_OK && !m->ev && hipEventCreateWithFlags(&m->ev, order_only) != hipSuccess)
                guard(fail(GA3C_EHIP, "hipEventCreate failed"));
    }
    if (rc == GA3C_OK) guard(dmalloc((void **)&c->g, sizeof(float) * c->P));
    if (rc == GA3C_OK) guard(dmalloc((void **)&c->grad, sizeof(float) * c->P));
    if (rc == GA3C_OK) {
        hipError_t e = hipMemset(c->theta2[0], 0, sizeof(float) * c->P);
        if (e == hipSuccess) e = hipMemset(c->theta2[1], 0, sizeof(float) * c->P);
        if (e == hipSuccess) e = hipMemset(c->g, 0, sizeof(float) * c->P);
        if (e == hipSuccess) e = hipMemset(c->grad, 0, sizeof(float) * c->P);
        if (e != hipSuccess) guard(fail(GA3C_EHIP, "hipMemset: %s", hipGetErrorString(e)));
    }
    if (rc == GA3C_OK && c->nconv >= 2 && spec_matches<SpecS1>(c->geom[0], true) && spec_matches<SpecS2>(c->geom[1], false) &&
        c->off[0] % 4 == 0 && c->off[2] % 4 == 0) {
        c->cfrag_dgrad = true;
        c->small_frames = small_launch_frames(c);
        for (int i = 0; i < 2 && rc == GA3C_OK; ++i) {
            guard(dmalloc((void **)&c->cfrag[i], sizeof(u32x4) * CFRAG_VECS));
            if (rc == GA3C_OK && !c->rb && max_predict_batch > c->small_frames) guard(dmalloc((void **)&c->hfrag[i], sizeof(u32x4) * Conv12F16::VECS));
            if (rc == GA3C_OK) guard(refresh_derived(c, i, nullptr));
        }
        if (rc == GA3C_OK) guard(dmalloc((void **)&c->ticket, sizeof(int) * SP_MAX_FRAMES * SP_TICKET_PITCH));
        if (rc == GA3C_OK) {
            const hipError_t e = hipMemset(c->ticket, 0, sizeof(int) * SP_MAX_FRAMES * SP_TICKET_PITCH);
            if (e != hipSuccess) guard(fail(GA3C_EHIP, "hipMemset: %s", hipGetErrorString(e)));
        }
    }
    if (rc == GA3C_OK && c->nconv == 3 && spec_matches<SpecL2>(c->geom[1], false) && spec_matches<SpecL3>(c->geom[2], false) &&
        c->off[2] % 4 == 0 && c->off[4] % 4 == 0) {
        if (spec_matches<SpecL1>(c->geom[0], true) && !c->rb && max_predict_batch > 0) c->conv123 = CONV123_LARGE;
        for (int i = 0; i < 2 && rc == GA3C_OK; ++i) {
            guard(dmalloc((void **)&c->lfrag[i], sizeof(u32x4) * (LFRAG_VECS + (c->conv123 ? Conv123Large::VECS : 0))));
            if (rc == GA3C_OK) guard(refresh_derived(c, i, nullptr));
        }
    }
    for (int l = 0; l < c->nconv; ++l) c->band[l] = on_band_kernels(c->geom[l], l);
    if (c->nconv == 3 && !c->rb && max_predict_batch > 0 && c->band[2] && c->off[2] % 4 == 0 && c->off[4] % 4 == 0) {
        const ConvGeom &g = c->geom[0];
        const bool frames = g.C == 4 && g.H == 84 && g.W == 84 && g.OC == 32 && g.KS == 8;
        if (frames && g.S == 4 && spec_matches<SpecP2>(c->geom[1], false) && spec_matches<SpecP43>(c->geom[2], false)) c->conv123 = CONV123_PAPER4;
        if (frames && g.S == 3 && spec_matches<SpecP32>(c->geom[1], false) && spec_matches<SpecP33>(c->geom[2], false)) c->conv123 = CONV123_PAPER3;
    }
    for (int l = 0; l < c->nconv; ++l) {
        const ConvGeom &g = c->geom[l];
        if (!c->band[l]) continue;
        const size_t vecs = (size_t)(c->rb ? 1 : 3) * g.OC * g.K / 8;
        if (takes_terms(c, l)) { c->bfrag_fwd[l] = c->bfrag_vecs; c->bfrag_vecs += vecs; }
        if (!c->rb && (l > 0 || max_train_frames > 0)) { c->bfrag_f32[l] = c->bfrag_vecs; c->bfrag_vecs += (size_t)g.OC * g.K / 4; }
        if (l > 0 && max_train_frames > 0) { c->bfrag_dgrad[l] = c->bfrag_vecs; c->bfrag_vecs += vecs; }
    }
    c->bfrag_123 = c->bfrag_vecs;
    c->bfrag_vecs += c->conv123 == CONV123_PAPER4 ? Conv123Paper4::VECS : c->conv123 == CONV123_PAPER3 ? Conv123Paper3::VECS : 0;
    if (c->bfrag_vecs)
        for (int i = 0; i < 2 && rc == GA3C_OK; ++i) {
            guard(dmalloc((void **)&c->bfrag[i], sizeof(u32x4) * c->bfrag_vecs));
            if (rc == GA3C_OK) guard(refresh_derived(c, i, nullptr));
        }
    // a small net whose calls all fit one launch has no use for them
    if (rc == GA3C_OK && fc_forward_ok(c->flat, c->F) && c->off[2 * c->nconv] % 4 == 0 && c->P < (size_t)1 << 31 &&
        !(c->ticket && max_train_frames == 0 && max_predict_batch <= c->small_frames)) {
        const int terms = c->rb ? 1 : 3;
        const size_t bytes = (size_t)c->flat * c->F * 2 * terms;
        unsigned char *w = nullptr;
        guard(dmalloc((void **)&w, 2 * bytes));
        if (rc == GA3C_OK) {
            for (int i = 0; i < 2; ++i) {
                FcPlanes &f = c->fcw[i];
                f.w = (u32x4 *)(w + i * bytes);
                f.first = (unsigned)(c->off[2 * c->nconv] / 4); f.n = (unsigned)((size_t)c->flat * c->F / 4);
                f.kblocks = c->flat / 32; f.terms = terms; f.row = FastDiv(c->flat / 4);
            }
            const hipError_t e = hipMemset(w, 0, 2 * bytes);         // of parameters that are zero
            if (e != hipSuccess) guard(fail(GA3C_EHIP, "hipMemset: %s", hipGetErrorString(e)));
        }
    }
    if (rc == GA3C_OK) guard(alloc_work(c->pred, c, max_predict_batch, false));
    if (rc == GA3C_OK) guard(alloc_work(c->train, c, max_train_frames, true));
    if (rc == GA3C_OK && max_train_frames > 0) {
        const size_t B = (size_t)max_train_frames;
        for (int l = 0; l < c->nconv && rc == GA3C_OK; ++l)
            guard(dmalloc((void **)&c->dact[l], sizeof(float) * (B * c->geom[l].OC * c->geom[l].OHW + BAND_SLACK)));
        if (rc == GA3C_OK) guard(dmalloc((void **)&c->dh, sizeof(float) * B * c->F));
        if (c->fcw[0].w) {
            c->dhp.terms = c->fcw[0].terms;
            c->fold_ok = is_aligned16(c->grad + c->off[2 * c->nconv]);
            if (rc == GA3C_OK) guard(dmalloc((void **)&c->dhp.w, fc_dh_planes_bytes(max_train_frames, c->F, c->dhp.terms)));
        }
        if (rc == GA3C_OK) guard(dmalloc((void **)&c->dzv, sizeof(float) * B * (c->A + 1)));
        if (rc == GA3C_OK) guard(dmalloc((void **)&c->R, sizeof(float) * B));
        c->max_norm_parts = (int)(c->P / 4 + 24 * MAX_REDUCE_SEGS);   // a reduce block covers at least 4 outputs
        if (rc == GA3C_OK) guard(dmalloc((void **)&c->partials, sizeof(float) * (c->max_norm_parts + 3 * (B / HD_FRAMES + 1))));
        if (rc == GA3C_OK) guard(dmalloc((void **)&c->colpart, sizeof(float) * (B / HD_FRAMES + 1) * c->F));
        if (rc == GA3C_OK) guard(dmalloc((void **)&c->scale, sizeof(float)));
        if (rc == GA3C_OK) guard(dmalloc((void **)&c->stats, sizeof(ga3c_train_stats)));
        if (rc == GA3C_OK) {
            hipError_t e = hipMemset(c->stats, 0, sizeof(ga3c_train_stats));
            if (e != hipSuccess) guard(fail(GA3C_EHIP, "hipMemset: %s", hipGetErrorString(e)));
        }
    }
    if (rc == GA3C_OK) {
        c->pred.ws_floats = workspace_floats(c, max_predict_batch, false);
        guard(dmalloc((void **)&c->pred.ws, sizeof(float) * c->pred.ws_floats));
    }
    if (rc == GA3C_OK) {
        c->train.ws_floats = workspace_floats(c, max_train_frames, true);
        guard(dmalloc((void **)&c->train.ws, sizeof(float) * c->train.ws_floats));
    }
    if (rc != GA3C_OK) {
        char keep[sizeof(g_err)];
        memcpy(keep, g_err, sizeof(keep));
        ga3c_destroy(c);
        memcpy(g_err, keep, sizeof(keep));
        return rc;
    }
    *out = c;
    return GA3C_OK;
}

extern "C" int ga3c_destroy(ga3c_ctx *c) {
    if (!c) return GA3C_OK;
    (void)hipDeviceSynchronize();
    for (int l = 0; l < GA3C_MAX_CONV; ++l) { (void)hipFree(c->koff[l]); (void)hipFree(c->dact[l]); }
    for (Mark *m : {&c->ready[0], &c->ready[1], &c->turned, &c->copied[0], &c->copied[1]})
        if (m->ev) (void)hipEventDestroy(m->ev);
    (void)hipFree(c->theta2[0]); (void)hipFree(c->theta2[1]);
    (void)hipFree(c->g); (void)hipFree(c->grad);
    (void)hipFree(c->cfrag[0]); (void)hipFree(c->cfrag[1]); (void)hipFree(c->hfrag[0]); (void)hipFree(c->hfrag[1]); (void)hipFree(c->ticket); (void)hipFree(c->lfrag[0]); (void)hipFree(c->lfrag[1]);
    (void)hipFree(c->bfrag[0]); (void)hipFree(c->bfrag[1]); (void)hipFree(c->fcw[0].w);      // both copies' in one piece
    free_work(c->pred); free_work(c->train);
    (void)hipFree(c->dhp.w); (void)hipFree(c->dh); (void)hipFree(c->dzv); (void)hipFree(c->R);
    (void)hipFree(c->partials); (void)hipFree(c->colpart); (void)hipFree(c->scale); (void)hipFree(c->stats);
    if (c->prof) {
        for (ProfRec &r : c->prof->recs) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
        for (hipEvent_t e : c->prof->pool) (void)hipEventDestroy(e);
        delete c->prof;
    }
    delete c;
    return GA3C_OK;
}

extern "C" size_t ga3c_params_count(const ga3c_ctx *c) { return c ? c->P : 0; }

extern "C" int ga3c_params_offsets(const ga3c_ctx *c, int64_t *off, int cap) {
    if (!c || !off || cap < c->noff) return fail(GA3C_EINVAL, "ga3c_params_offsets: null argument or cap too small");
    for (int i = 0; i < c->noff; ++i) off[i] = c->off[i];
    return c->noff;
}

extern "C" int ga3c_params_init(ga3c_ctx *c, uint64_t seed, void *stream) {
    if (!c) return fail(GA3C_EINVAL, "ga3c_params_init: null context");
    hipStream_t s = (hipStream_t)stream;
    const int to = copy_to_write(c);
    float *theta = c->theta2[to];
    TRY(wait_ready(c, s));
    TRY(wait_writable(c, s));
    ga3c::launch(fill_kernel, dim3(blocks_for(c->P)), dim3(256), 0, s, theta, c->P, 0.f);
    ga3c::launch(fill_kernel, dim3(blocks_for(c->P)), dim3(256), 0, s, c->g, c->P, 0.f);
    HIP_TRY(hipGetLastError());
    const int nb = 2 * c->nconv;
    // weight tensors and their fan-in; biases stay zero
    struct { int64_t off; size_t n; int fan_in; } t[GA3C_MAX_CONV + 3];
    int nt = 0;
    for (int l = 0; l < c->nconv; ++l) t[nt++] = {c->off[2 * l], (size_t)c->geom[l].OC * c->geom[l].K, c->geom[l].K};
    t[nt++] = {c->off[nb], (size_t)c->flat * c->F, c->flat};
    t[nt++] = {c->off[nb + 2], (size_t)c->A * c->F, c->F};
    t[nt++] = {c->off[nb + 4], (size_t)c->F, c->F};
    for (int i = 0; i < nt; ++i) {
        ga3c::launch(init_normal_kernel, dim3(blocks_for(t[i].n)), dim3(256), 0, s, theta + t[i].off,
                           (size_t)t[i].off, t[i].n, sqrtf(2.f / (float)t[i].fan_in), seed);
        HIP_TRY(hipGetLastError());
    }
    TRY(refresh_derived(c, to, s));
    return publish(c, s);
}

static float *select_buffer(ga3c_ctx *c, int which) {
    return which == 0 ? c->theta2[c->cur] : which == 1 ? c->g : which == 2 ? c->grad : nullptr;
}

extern "C" int ga3c_params_get(ga3c_ctx *c, int which, float *dst, size_t n, void *stream) {
    if (!c || !dst) return fail(GA3C_EINVAL, "ga3c_params_get: null argument");
    float *src = select_buffer(c, which);
    if (!src || n != c->P) return fail(GA3C_EINVAL, "ga3c_params_get: which must be 0..2 and n the parameter count");
    hipStream_t s = (hipStream_t)stream;
    TRY(wait_ready(c, s));
    // the writer that the copying has to come before: on the last writer's stream, unless that one writes in place (the event
    // costs the stream 2 us)
    Mark &done = c->copied[c->cur];
    const bool marked = which == 0 && (copy_to_write(c) == c->cur || c->ready[c->cur].where != s);
    ga3c::StopEvent stop;
    if (marked) {
        TRY(wait_mark(done, s));      // the event then stands for the earlier copies too
        stop = stop_for(done, s);
    }
    const size_t n4 = is_aligned16(dst) && is_aligned16(src) ? n / 4 : 0;
    ga3c::launch_stop(&stop, copy_kernel, dim3(std::min(blocks_for(n4 ? n4 : n), 4096u)), dim3(256), 0, s, dst, (const float *)src, n, n4);
    HIP_TRY(hipGetLastError());
    return marked ? set_mark(done, s, &stop) : GA3C_OK;
}

extern "C" int ga3c_params_set(ga3c_ctx *c, int which, const float *src, size_t n, void *stream) {
    if (!c || !src) return fail(GA3C_EINVAL, "ga3c_params_set: null argument");
    if ((which != 0 && which != 1) || n != c->P)
        return fail(GA3C_EINVAL, "ga3c_params_set: which must be 0 or 1 and n the parameter count");
    hipStream_t s = (hipStream_t)stream;
    TRY(wait_ready(c, s));
    if (which == 0) TRY(wait_writable(c, s));
    const int to = copy_to_write(c);
    HIP_TRY(hipMemcpyAsync(which == 0 ? c->theta2[to] : c->g, src, sizeof(float) * n, hipMemcpyDeviceToDevice, s));
    if (which != 0) return GA3C_OK;
    TRY(refresh_derived(c, to, s));
    return publish(c, s);
}

static int predict_impl(ga3c_ctx *c, const uint8_t *frames, const uint8_t *const *table, int B, const float *uniforms, float *logits,
                        float *values, float *probs, int32_t *actions, void *stream) {
    if (!c) return fail(GA3C_EINVAL, "ga3c_predict: null context");
    if (B < 0 || B > c->max_pred) return fail(GA3C_EINVAL, "ga3c_predict: B = %d outside [0, %d]", B, c->max_pred);
    if (B == 0) return GA3C_OK;
    if (!frames && !table) return fail(GA3C_EINVAL, "ga3c_predict: null frames");
    if (actions && !uniforms) return fail(GA3C_EINVAL, "ga3c_predict: actions requested without uniforms");
    hipStream_t s = (hipStream_t)stream;
    TRY(wait_ready(c, s));
    TRY(begin_prediction(c, s));
    return forward(c, c->cur, c->pred, frames, table, B, false, logits, values, probs, uniforms, actions, s);
}

extern "C" int ga3c_predict(ga3c_ctx *c, const uint8_t *frames, int B, const float *uniforms, float *logits,
                            float *values, float *probs, int32_t *actions, void *stream) {
    return predict_impl(c, frames, nullptr, B, uniforms, logits, values, probs, actions, stream);
}

// One update on B frames.  seg_start == nullptr: N segments of T frames each
// (B = N*T); otherwise N segments of unequal length, T = 1.
static int train_step_impl(ga3c_ctx *c, const uint8_t *frames, const uint8_t *const *table, const int32_t *actions, const float *rewards,
                           const uint8_t *dones, const float *bootstrap, const int32_t *seg_start, int N, int T, int B,
                           const ga3c_hparams *hp, ga3c_train_stats *stats, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    Work &w = c->train;
    const int nb = 2 * c->nconv, A = c->A, F = c->F;
    c->last_frames = B;

    const int cur = c->cur;
    const float *th = c->theta2[cur];
    TRY(wait_ready(c, s));
    // One kernel finishes the fc layer, runs the heads, the loss and the heads' backward pass, if its LDS fits, for at most the 31
    // actions that it is tested with.  Its layout would do for 63 (the loss has an output per lane), and it would be ahead there: us an
    // update, separate kernels / this one, small net with 32 actions 40 frames 85.7 / 68.0, 2560 frames 304.7 / 292.7, with 63 actions
    // 104.0 / 72.1 and 330.1 / 302.1; larger net with 32 actions 640 frames 357.6 / 336.3.
    const size_t ht_lds = sizeof(float) * (size_t)heads_train_lds_floats(F, A);
    const bool fused_heads = c->fast && ht_lds <= HEADS_TRAIN_MAX_LDS && A <= 31;
    int rc = forward(c, cur, w, frames, table, B, true, nullptr, nullptr, nullptr, nullptr, nullptr, s, !fused_heads);
    if (rc != GA3C_OK) return rc;

    const int nloss = fused_heads ? cdiv(B, HD_FRAMES) : cdiv(B, LOSS_THREADS);
    float *losspart = c->partials + c->max_norm_parts;
    if (!fused_heads) {
        STAGE("returns_loss", 0, 4.0 * B * (2 * (A + 1) + 4));
        ga3c::launch(returns_loss_kernel, dim3(nloss), dim3(LOSS_THREADS), sizeof(float) * LOSS_THREADS * (A + 1), s, w.zv, actions, rewards, dones,
                           bootstrap, seg_start, N, T, B, A, hp->gamma, hp->beta, hp->value_coef, hp->log_eps, c->R, c->dzv, losspart);
        HIP_TRY(hipGetLastError());
    }

    const float *Wp = th + c->off[nb + 2], *Wv = th + c->off[nb + 4];
    int nz, kchunk;
    // Every weight gradient leaves its partial sums in a region of its own; one kernel adds them all up at the end.
    ReduceArgs red;
    std::fill(red.first, red.first + MAX_REDUCE_SEGS, INT32_MAX);
    red.normpart = c->partials;
    int nseg = 0;
    // the fused heads kernel still reads the fc partial sums, which sit at the start of the workspace
    size_t ws_used = fused_heads ? ((size_t)w.fc_nz * B * F + 63) / 64 * 64 : 0;
    int red_blocks = 0;
    double red_bytes = 0;
    auto region = [&](size_t floats) -> float * {
        float *r = ws_used + floats <= w.ws_floats ? w.ws + ws_used : nullptr;
        ws_used += (floats + 63) / 64 * 64;
        return r;
    };
    bool seg_overflow = false;
    auto add_seg = [&](const float *ws, int nz_, int M, int Ncols, int r0, int rows, float *gW, float *gb, int bias_col) {
        if (nseg >= MAX_REDUCE_SEGS) { seg_overflow = true; return; }
        red.first[nseg] = red_blocks;
        ReduceSeg &g = red.seg[nseg++];
        g.ws = ws + (size_t)r0 * Ncols; g.gW = gW; g.gb = gb; g.nz = nz_; g.N = Ncols; g.bias_col = bias_col != 0; g.in_place = ws == gW;
        g.stride = (size_t)M * Ncols; g.cnt = (size_t)rows * Ncols;
        const FastDiv by_n((uint32_t)Ncols);
        g.mul = by_n.mul; g.shift = (uint8_t)by_n.shift; g.lzg = 0;
        while (g.lzg < 6 && (16 << g.lzg) < nz_) ++g.lzg;      // one round of sixteen loads per thread
        g.vec = ((size_t)r0 * Ncols) % 4 == 0 && g.stride % 4 == 0 && (uintptr_t)ws % 16 == 0;
        const size_t per_block = (size_t)(256 >> g.lzg) * (g.vec ? 4 : 1);
        const int nblk = (int)((g.cnt + per_block - 1) / per_block);
        g.per_xcd = (nblk + 7) / 8;
        red_blocks += 8 * g.per_xcd;
        red_bytes += 4.0 * (nz_ + 1) * rows * Ncols;
    };
    const size_t hd_lds = sizeof(float) * (A + 1) * HD_FRAMES;      // heads_dgrad_kernel's LDS, 2 KB at most
    if (fused_heads) {
        const int nblk = cdiv(B, HD_FRAMES);
        float *part = region((size_t)nblk * (A + 1) * (F + 1));
        if (!part) return fail(GA3C_EINVAL, "internal: split-k workspace too small (heads)");
        typedef decltype(&heads_train_kernel<LOADS_SCALAR, 2>) HeadsTrain;
        static const HeadsTrain ht_kernels[6] = {heads_train_kernel<LOADS_SCALAR, 2>, heads_train_kernel<LOADS_VEC8, 2>, heads_train_kernel<LOADS_VEC16, 2>,
                                                 heads_train_kernel<LOADS_SCALAR, 4>, heads_train_kernel<LOADS_VEC8, 4>, heads_train_kernel<LOADS_VEC16, 4>};
        static size_t ht_lds_set[6] = {0, 0, 0, 0, 0, 0};
        const int vk = heads_train_vk(F);
        const int ht = heads_loads(F, w.fc_nz, w.fc_ws, th + c->off[nb + 1], w.h, Wp) + (vk == 2 ? 0 : 3);
        HIP_TRY(allow_dynamic_lds((const void *)ht_kernels[ht], ht_lds, ht_lds_set[ht]));
        STAGE("heads_train", 6.0 * B * (A + 1) * F, 4.0 * (w.fc_nz + 1) * B * F);
        ga3c::launch(ht_kernels[ht], dim3(nblk), dim3(HEADS_TRAIN_THREADS), ht_lds, s, w.fc_ws, w.fc_nz, th + c->off[nb + 1], B, F, A, Wp,
                           th + c->off[nb + 3], Wv, th + c->off[nb + 5], actions, rewards, dones, bootstrap, seg_start, N, T, hp->gamma, hp->beta,
                           hp->value_coef, hp->log_eps, w.h, w.zv, c->R, c->dzv, c->dh, c->colpart, part, losspart, c->rb,
                           FastDiv(std::max(1, F / 4)), FastDiv(A + 1), FastDiv(heads_train_kparts(F, A)), FastDiv(T), c->dhp);
        HIP_TRY(hipGetLastError());
        add_seg(part, nblk, A + 1, F + 1, 0, A, c->grad + c->off[nb + 2], c->grad + c->off[nb + 3], 1);
        add_seg(part, nblk, A + 1, F + 1, A, 1, c->grad + c->off[nb + 4], c->grad + c->off[nb + 5], 1);
    } else if (c->fast) {   // heads: input gradient and, per block of frames, the block's share of the weight and bias gradients
        const int nblk = cdiv(B, HD_FRAMES);
        float *part = region((size_t)nblk * (A + 1) * (F + 1));
        if (!part) return fail(GA3C_EINVAL, "internal: split-k workspace too small (heads)");
        STAGE("heads_bwd", 4.0 * B * (A + 1) * F, 0);
        ga3c::launch(heads_dgrad_kernel, dim3(nblk, cdiv(F, HD_COLS)), dim3(HD_COLS), hd_lds, s, c->dzv, w.h, Wp, Wv, B,
                           F, A, c->dh, c->colpart, part, c->rb);
        HIP_TRY(hipGetLastError());
        add_seg(part, nblk, A + 1, F + 1, 0, A, c->grad + c->off[nb + 2], c->grad + c->off[nb + 3], 1);
        add_seg(part, nblk, A + 1, F + 1, A, 1, c->grad + c->off[nb + 4], c->grad + c->off[nb + 5], 1);
    } else {   // heads: weight and bias gradients as a product, then the input gradient
        GemmP<EPI_PARTIAL, true> p; p.rb = c->rb;
        p.M = A + 1; p.N = F + 1; p.K = B;
        pick_split(conv_like_tiles(p.M, p.N), B, nz, kchunk);
        p.kchunk = kchunk;
        p.A = c->dzv; p.sAm = 1; p.sAk = A + 1;
        p.B = w.h; p.sBn = 1; p.sBk = F;
        p.C = region((size_t)nz * p.M * p.N); p.ldc = 0; p.aux = nullptr;
        if (!p.C) return fail(GA3C_EINVAL, "internal: split-k workspace too small (heads)");
        {
            STAGE("heads_wgrad", 2.0 * B * (A + 1) * F, 0);
            HIP_TRY(launch_conv_like(p, nz, s));
        }
        add_seg(p.C, nz, A + 1, F + 1, 0, A, c->grad + c->off[nb + 2], c->grad + c->off[nb + 3], 1);
        add_seg(p.C, nz, A + 1, F + 1, A, 1, c->grad + c->off[nb + 4], c->grad + c->off[nb + 5], 1);
        STAGE("heads_dgrad", 2.0 * B * (A + 1) * F, 0);
        ga3c::launch(heads_dgrad_kernel, dim3(cdiv(B, HD_FRAMES), cdiv(F, HD_COLS)), dim3(HD_COLS), hd_lds, s, c->dzv, w.h, Wp, Wv, B,
                           F, A, c->dh, c->colpart, (float *)nullptr, c->rb);
        HIP_TRY(hipGetLastError());
    }
    const float *xfc = w.act[c->nconv - 1];
    const float *wfc = th + c->off[nb];
    const bool fc_dense = c->fast && dense_operand_ok(c->dh, F, F) && dense_operand_ok(xfc, c->flat, c->flat) &&
                          dense_operand_ok(wfc, c->flat, c->flat);
    if (fc_dense) {   // fc weight gradient: D[o][i] = sum_b dh[b][o] x[b][i]; bias from the column sums of dh
        pick_split_xcd(cdiv(F, 64) * cdiv(c->flat, 64), B, nz, kchunk, 256);
        const bool planes = c->dhp.w && c->fcw[cur].w;
        // chunks added up by the block itself go straight into the gradient
        const bool fold = planes && c->fold_ok && fc_grads_fold(F, c->flat, B, c->dhp.terms);
        float *dw = fold ? c->grad + c->off[nb] : region((size_t)nz * F * c->flat);
        if (!dw) return fail(GA3C_EINVAL, "internal: split-k workspace too small (fc wgrad)");
        STAGE2("fc_wgrad", 2.0 * B * F * c->flat, 0, "fc_dgrad", 2.0 * B * F * c->flat, 0);
        if (planes) {
            if (!fused_heads) HIP_TRY(launch_fc_dh_planes(c->dh, c->dhp, B, F, s));
            FcGradArgs p{};
            p.B = B; p.F = F; p.flat = c->flat; p.kchunk = kchunk; p.nz = nz;
            p.dh = c->dhp; p.w = c->fcw[cur].w; p.x = xfc; p.dx = c->dact[c->nconv - 1]; p.dw = dw;
            HIP_TRY(launch_fc_grads(p, fold, c->rb, s));
        } else {
            DenseGemmArgs p{}; p.rb = c->rb;
            p.M = F; p.N = c->flat; p.K = B; p.kchunk = kchunk; p.nz = nz;
            p.A = c->dh; p.lda = F; p.B = xfc; p.ldb = c->flat;
            p.C = dw; p.ldc = 0; p.aux = nullptr;
            // fc input gradient, masked by the ReLU of the last conv layer
            DenseGemmArgs q{}; q.rb = c->rb;
            q.M = B; q.N = c->flat; q.K = F; q.kchunk = (F + GEMM_BK - 1) / GEMM_BK * GEMM_BK; q.nz = 1;
            q.A = c->dh; q.lda = F; q.B = wfc; q.ldb = c->flat;
            q.C = c->dact[c->nconv - 1]; q.ldc = c->flat; q.aux = xfc;
            // What fc_grads.hpp does not take (units that are not a multiple of 64, columns that are not one of 32).  The input
            // gradient's tile is 64x64 as long as there is one tile per compute unit at most, 128x64 above that: fewer tiles leave
            // units idle, more read their operands twice.  64x64 against 128x64 on layers of both kernels, us of the launch (tiles of 64x64): small net
            // 160 frames 15.9 / 18.7 (123), 320: 15.0 / 17.9 (205), 480: 19.8 / 19.0 (328), 2560: 63.5 / 57.2; larger net 320: 28.3 /
            // 30.0 (245), 480: 37.9 / 35.8 (392), 1280: 74.1 / 66.9; stride-4 member 960: 13.1 / 16.9 (135); stride-2 member 320: 20.3
            // / 19.7 (320); stride-1 member 80: 294 / 286 (578).
            if (cdiv(B, 64) * cdiv(c->flat, 64) <= 256) HIP_TRY((launch_dense_fc_grads<2, 2>(q, p, s)));
            else HIP_TRY((launch_dense_fc_grads<4, 1>(q, p, s)));
        }
        add_seg(dw, fold ? 1 : nz, F, c->flat, 0, F, c->grad + c->off[nb], nullptr, 0);
        add_seg(c->colpart, cdiv(B, HD_FRAMES), 1, F, 0, 1, c->grad + c->off[nb + 1], nullptr, 0);
    } else {   // general shapes: one more column of ones yields the bias gradient
        GemmP<EPI_PARTIAL, true> p; p.rb = c->rb;
        p.M = F; p.N = c->flat + 1; p.K = B;
        pick_split(cdiv(p.M, 64) * cdiv(p.N, 64), B, nz, kchunk);
        p.kchunk = kchunk;
        p.A = c->dh; p.sAm = 1; p.sAk = F;
        p.B = xfc; p.sBn = 1; p.sBk = c->flat;
        p.C = region((size_t)nz * p.M * p.N); p.ldc = 0; p.aux = nullptr;
        if (!p.C) return fail(GA3C_EINVAL, "internal: split-k workspace too small (fc wgrad)");
        {
            STAGE("fc_wgrad", 2.0 * B * F * c->flat, 0);
            HIP_TRY((launch_gemm<2, 2, 2, 2, true, true>(p, nz, s)));
        }
        add_seg(p.C, nz, p.M, p.N, 0, p.M, c->grad + c->off[nb], c->grad + c->off[nb + 1], 1);
    }
    if (!fc_dense) {   // fc input gradient, masked by the ReLU of the last conv layer
        STAGE("fc_dgrad", 2.0 * B * F * c->flat, 0);
        GemmP<EPI_MASK, false> p; p.rb = c->rb;
        p.M = B; p.N = c->flat; p.K = F; p.kchunk = (F + GEMM_BK - 1) / GEMM_BK * GEMM_BK;
        p.A = c->dh; p.sAm = F; p.sAk = 1;
        p.B = wfc; p.sBn = 1; p.sBk = c->flat;
        p.C = c->dact[c->nconv - 1]; p.ldc = c->flat; p.aux = xfc;
        HIP_TRY((launch_gemm<2, 2, 2, 2, false, true>(p, 1, s)));
    }
    for (int l = c->nconv - 1; l >= 0; --l) {
        const ConvGeom &g = c->geom[l];
        // weight + bias gradient
        {
            const void *xin = l == 0 ? (const void *)frames : (const void *)w.act[l - 1];
            const bool ok = c->fast && is_aligned16(xin);
            const int band_nz = band_grad_parts(c, l, B);
            const int kind = !ok || !is_aligned16(c->dact[l]) ? 0
                                     : spec_matches<SpecS1>(g, l == 0) ? 1
                                     : spec_matches<SpecL1>(g, l == 0) ? 2
                                     : spec_matches<SpecS2>(g, l == 0) ? 3
                                     : spec_matches<SpecL2>(g, l == 0) ? 4
                                     : spec_matches<SpecL3>(g, l == 0) ? 5
                                     : spec_matches<SpecP2>(g, l == 0) ? 6
                                     : band_nz > 0 ? 8
                                     : c->band[l] && f32_wgrad_ok(g.C, g.H, g.W, g.S, g.OC) ? 7 : 0;
            if (kind == 1 || kind == 2) nz = conv1_wgrad_blocks(B);
            else if (kind == 3) nz = conv_wgrad_f16_blocks<SpecS2>(B);
            else if (kind == 4) nz = conv_wgrad_f16_blocks<SpecL2>(B);
            else if (kind == 5) nz = conv_wgrad_s1_f16_blocks<SpecL3>(B);
            else if (kind == 6) nz = conv_wgrad_f16_blocks<SpecP2>(B);
            else if (kind == 8) nz = band_nz;
            else pick_split(conv_like_tiles(g.OC, g.K + 1), B * g.OHW, nz, kchunk);
            float *part = region((size_t)nz * g.OC * (g.K + 1));
            if (!part) return fail(GA3C_EINVAL, "internal: split-k workspace too small (conv)");
            // the 4x4 stride-2 layers' two gradients share a launch (conv_grads.hpp)
            if ((kind == 3 || kind == 4 || kind == 6) && is_aligned16(th + c->off[2 * l])) {
                STAGE2(CONV_DGRAD[l], 2.0 * B * g.OHW * g.OC * g.K, 4.0 * B * (g.OC * g.OHW + 2.0 * g.C * g.H * g.W),
                       CONV_WGRAD[l], 2.0 * B * g.OHW * g.OC * g.K, (double)B * (4.0 * g.CHW + 4.0 * g.OC * g.OHW));
                const float *x = (const float *)xin, *dy = c->dact[l], *wl = th + c->off[2 * l];
                // the fragments of the copy being trained on, when the context keeps them
                if (kind == 3)
                    HIP_TRY(launch_conv_grads<SpecS2>(x, dy, wl, c->cfrag[cur] && c->cfrag_dgrad ? c->cfrag[cur] + CFRAG_FWD_VECS : nullptr,
                                                             c->dact[l - 1], part, B, s, c->rb));
                else if (kind == 4)
                    HIP_TRY((launch_conv_grads<SpecL2, 32>(x, dy, wl, c->lfrag[cur] && l == 1 ? c->lfrag[cur] + LFRAG_DGRAD2 : nullptr,
                                                                  c->dact[l - 1], part, B, s, c->rb)));
                else
                    HIP_TRY(launch_conv_grads<SpecP2>(x, dy, wl, nullptr, c->dact[l - 1], part, B, s, c->rb));
                add_seg(part, nz, g.OC, g.K + 1, 0, g.OC, c->grad + c->off[2 * l], c->grad + c->off[2 * l + 1], 1);
                continue;
            }
            STAGE(CONV_WGRAD[l], 2.0 * B * g.OHW * g.OC * g.K, (double)B * ((l == 0 ? 1.0 : 4.0) * g.CHW + 4.0 * g.OC * g.OHW));
            if (kind == 1) {
                HIP_TRY(launch_conv1_wgrad<16>((const uint8_t *)xin, table, c->dact[l], part, B, 1.f / 255.f, s, c->rb));
            } else if (kind == 2) {
                HIP_TRY(launch_conv1_wgrad<32>((const uint8_t *)xin, table, c->dact[l], part, B, 1.f / 255.f, s, c->rb));
            } else if (kind == 3) {
                HIP_TRY(launch_conv_wgrad_f16<SpecS2>((const float *)xin, c->dact[l], part, B, 1.f, s, c->rb));
            } else if (kind == 4) {
                HIP_TRY((launch_conv_wgrad_f16<SpecL2, 32>((const float *)xin, c->dact[l], part, B, 1.f, s, c->rb)));
            } else if (kind == 5) {
                HIP_TRY(launch_conv_wgrad_s1_f16<SpecL3>((const float *)xin, c->dact[l], part, B, 1.f, s, c->rb));
            } else if (kind == 6) {
                HIP_TRY(launch_conv_wgrad_f16<SpecP2>((const float *)xin, c->dact[l], part, B, 1.f, s, c->rb));
            } else if (kind == 7) {
                if (g.OC == 16) HIP_TRY((launch_conv_f32_wgrad<16>(frames, c->dact[l], part, B, g.C, g.H, g.W, g.S, nz, kchunk, 1.f / 255.f, s, c->rb)));
                else HIP_TRY((launch_conv_f32_wgrad<32>(frames, c->dact[l], part, B, g.C, g.H, g.W, g.S, nz, kchunk, 1.f / 255.f, s, c->rb)));
            } else if (kind == 8 && l == 0) {
                if (g.S == 1) HIP_TRY(launch_conv_bytes_wgrad<1>(frames, c->dact[l], part, B, g.H, 1.f / 255.f, s, c->rb));
                else if (g.S == 2) HIP_TRY(launch_conv_bytes_wgrad<2>(frames, c->dact[l], part, B, g.H, 1.f / 255.f, s, c->rb));
                else HIP_TRY(launch_conv_bytes_wgrad<3>(frames, c->dact[l], part, B, g.H, 1.f / 255.f, s, c->rb));
            } else if (kind == 8) {
                if (g.OC == 32) HIP_TRY(launch_conv_band_wgrad<32>((const float *)xin, c->dact[l], part, B, g.H, g.W, s, c->rb));
                else HIP_TRY(launch_conv_band_wgrad<64>((const float *)xin, c->dact[l], part, B, g.H, g.W, s, c->rb));
            } else if (l == 0) {
                ConvWgradP<uint8_t> p; p.rb = c->rb;
                p.M = g.OC; p.N = g.K + 1; p.K = B * g.OHW; p.kchunk = kchunk; p.g = g;
                p.x = frames; p.dy = c->dact[0]; p.ws = part; p.scale = 1.f / 255.f;
                HIP_TRY(launch_conv_like(p, nz, s));
            } else {
                ConvWgradP<float> p; p.rb = c->rb;
                p.M = g.OC; p.N = g.K + 1; p.K = B * g.OHW; p.kchunk = kchunk; p.g = g;
                p.x = w.act[l - 1]; p.dy = c->dact[l]; p.ws = part; p.scale = 1.f;
                HIP_TRY(launch_conv_like(p, nz, s));
            }
            add_seg(part, nz, g.OC, g.K + 1, 0, g.OC, c->grad + c->off[2 * l], c->grad + c->off[2 * l + 1], 1);
        }
        if (l == 0) break;   // the input is data: no gradient needed
        // input gradient
        // bytes: dY in, the layer's input (for the ReLU mask) in, dX out
        STAGE(CONV_DGRAD[l], 2.0 * B * g.OHW * g.OC * g.K, 4.0 * B * (g.OC * g.OHW + 2.0 * g.C * g.H * g.W));
        if (c->fast && c->band[l]) {
            const u32x4 *wf = c->bfrag[cur] + c->bfrag_dgrad[l];
            const PositiveBits bits = w.bits_set[l - 1] ? w.bits[l - 1] : PositiveBits{};
            if (g.OC == 32) HIP_TRY(launch_conv_band_dgrad<32>(c->dact[l], wf, w.act[l - 1], bits, c->dact[l - 1], B, g.H, g.W, s, c->rb));
            else HIP_TRY(launch_conv_band_dgrad<64>(c->dact[l], wf, w.act[l - 1], bits, c->dact[l - 1], B, g.H, g.W, s, c->rb));
            continue;
        }
        if (c->fast && spec_matches<SpecL3>(g, false)) {
            HIP_TRY((launch_conv_dgrad_s1_bf16x6<SpecL3, 4>(c->dact[l], th + c->off[2 * l], w.act[l - 1], c->dact[l - 1], B, s, 256, c->rb,
                                                            c->lfrag[cur] && l == 2 ? c->lfrag[cur] + LFRAG_DGRAD3 : nullptr)));
            continue;
        }
        // general shapes: one launch per stride phase
        for (int ry = 0; ry < g.S; ++ry)
            for (int rx = 0; rx < g.S; ++rx) {
                ConvDgradP p; p.rb = c->rb;
                p.g = g; p.ry = ry; p.rx = rx;
                p.nH = ry < g.H ? (g.H - ry + g.S - 1) / g.S : 0;
                p.nW = rx < g.W ? (g.W - rx + g.S - 1) / g.S : 0;
                if (p.nH == 0 || p.nW == 0) continue;
                p.TA = (g.KS + g.S - 1) / g.S; p.TB = p.TA;
                p.dNHW = FastDiv(p.nH * p.nW); p.dNW = FastDiv(p.nW);
                p.dTAB = FastDiv(p.TA * p.TB); p.dTB = FastDiv(p.TB);
                p.M = g.C; p.N = B * p.nH * p.nW; p.K = g.OC * p.TA * p.TB;
                p.w = th + c->off[2 * l]; p.dy = c->dact[l]; p.xmask = w.act[l - 1]; p.dx = c->dact[l - 1];
                HIP_TRY(launch_conv_like(p, 1, s));
            }
    }
    // all partial gradients -> gradient and its squared norm; then clip scale and stats; then RMSProp
    if (seg_overflow) return fail(GA3C_EINVAL, "internal: more partial-gradient segments than the reduction kernel takes");
    if (red_blocks > c->max_norm_parts) return fail(GA3C_EINVAL, "internal: too many reduce blocks");
    {
        STAGE("wgrad_reduce", 0, red_bytes);
        ga3c::launch(reduce_all_kernel, dim3(red_blocks), dim3(256), 0, s, red);
        HIP_TRY(hipGetLastError());
    }
    STAGE("rmsprop", 8.0 * c->P, 20.0 * c->P);
    // one float4 per thread at these sizes; the clip factor and the statistics are formed in the kernel's prologue
    const unsigned rb = std::min<unsigned>(blocks_for(c->P / 4 + 1), 2048u);
    const int to = copy_to_write(c);
    TRY(wait_writable(c, s));
    RmsClip ca;
    ca.normpart = c->partials; ca.nnorm = red_blocks; ca.losspart = losspart; ca.nloss = nloss; ca.clip = hp->clip_norm;
    ca.scale_out = c->scale; ca.own = c->stats; ca.user = stats;
    const bool fragments = c->lfrag[to] || c->bfrag[to];      // they follow the new parameters, in launches of their own
    ga3c::StopEvent stop = stop_for(c->ready[to], s);
    ga3c::launch_stop(fragments ? nullptr : &stop, (rmsprop_kernel<0, 1>), dim3(rb), dim3(256), 0, s, th, c->theta2[to], c->g, c->grad, c->P,
                      (const float *)nullptr, 1.f, hp->lr, hp->rms_decay, hp->rms_eps, c->cfrag[to], c->hfrag[to], c->rb,
                      c->fcw[to], ca);
    HIP_TRY(hipGetLastError());
    if (fragments) TRY(refresh_derived(c, to, s, false, &stop));
    return publish(c, s, &stop);
}

extern "C" int ga3c_train_step(ga3c_ctx *c, const uint8_t *frames, const int32_t *actions, const float *rewards,
                               const uint8_t *dones, const float *bootstrap, int N, int T, const ga3c_hparams *hp,
                               ga3c_train_stats *stats, void *stream) {
    if (!c) return fail(GA3C_EINVAL, "ga3c_train_step: null context");
    if (N < 0 || T < 0) return fail(GA3C_EINVAL, "ga3c_train_step: negative N or T");
    const long long BL = (long long)N * T;
    if (BL > c->max_train) return fail(GA3C_EINVAL, "ga3c_train_step: N*T = %lld above capacity %d", BL, c->max_train);
    if (BL == 0) return GA3C_OK;
    if (!frames || !actions || !rewards || !dones || !hp) return fail(GA3C_EINVAL, "ga3c_train_step: null argument");
    return train_step_impl(c, frames, nullptr, actions, rewards, dones, bootstrap, nullptr, N, T, (int)BL, hp, stats, stream);
}

extern "C" int ga3c_train_step_ragged(ga3c_ctx *c, const uint8_t *frames, const int32_t *actions, const float *rewards,
                                      const uint8_t *dones, const int32_t *seg_start, const float *bootstrap, int N,
                                      int n_frames, const ga3c_hparams *hp, ga3c_train_stats *stats, void *stream) {
    if (!c) return fail(GA3C_EINVAL, "ga3c_train_step_ragged: null context");
    if (N < 0 || n_frames < 0) return fail(GA3C_EINVAL, "ga3c_train_step_ragged: negative N or n_frames");
    if (n_frames > c->max_train)
        return fail(GA3C_EINVAL, "ga3c_train_step_ragged: %d frames above capacity %d", n_frames, c->max_train);
    if (n_frames == 0) return GA3C_OK;
    if (N == 0) return fail(GA3C_EINVAL, "ga3c_train_step_ragged: frames without a segment");
    if (!frames || !actions || !rewards || !dones || !seg_start || !hp)
        return fail(GA3C_EINVAL, "ga3c_train_step_ragged: null argument");
    return train_step_impl(c, frames, nullptr, actions, rewards, dones, bootstrap, seg_start, N, 1, n_frames, hp, stats, stream);
}

// What the scheduler calls (frame_table.hpp).
bool ga3c::takes_frame_table(const ga3c_ctx *c) {
    const ConvGeom &g = c->geom[0];
    return c->fast && is_aligned16(c->theta2[0] + c->off[0]) && (spec_matches<SpecS1>(g, true) || spec_matches<SpecL1>(g, true));
}
int ga3c::predict_from_table(ga3c_ctx *c, const uint8_t *const *table, int B, const float *uniforms, float *values, int32_t *actions, hipStream_t s) {
    return predict_impl(c, nullptr, table, B, uniforms, nullptr, values, nullptr, actions, s);
}
int ga3c::train_from_table(ga3c_ctx *c, const uint8_t *const *table, const int32_t *actions, const float *rewards, const uint8_t *dones,
                           const float *bootstrap, const int32_t *seg_start, int N, int T, int B, const ga3c_hparams *hp, hipStream_t s) {
    if (B < 1 || B > c->max_train) return fail(GA3C_EINVAL, "ga3c_train_step: %d frames outside 1..%d", B, c->max_train);
    return train_step_impl(c, nullptr, table, actions, rewards, dones, bootstrap, seg_start, N, T, B, hp, nullptr, s);
}

extern "C" int ga3c_train_debug_get(ga3c_ctx *c, int which, float *dst, size_t n, void *stream) {
    if (!c || !dst) return fail(GA3C_EINVAL, "ga3c_train_debug_get: null argument");
    const size_t B = (size_t)c->last_frames;
    const float *src = nullptr;
    size_t cap = 0;
    if (which == 0) { src = c->R; cap = B; }
    else if (which == 3) { src = c->dzv; cap = B * (c->A + 1); }
    else if (which == 1 || which == 2) { src = c->train.zv; cap = B * (c->A + 1); }
    else if (which >= 4 && which < 4 + c->nconv) { src = c->train.act[which - 4]; cap = B * c->geom[which - 4].OC * c->geom[which - 4].OHW; }
    else if (which == 8) { src = c->train.h; cap = B * c->F; }
    else if (which == 9) { src = c->dh; cap = B * c->F; }
    else if (which >= 10 && which < 10 + c->nconv) { src = c->dact[which - 10]; cap = B * c->geom[which - 10].OC * c->geom[which - 10].OHW; }
    if (!src || n > (which == 1 ? B * c->A : which == 2 ? B : cap))
        return fail(GA3C_EINVAL, "ga3c_train_debug_get: bad selector or size");
    hipStream_t s = (hipStream_t)stream;
    if (which == 1 || which == 2) {
        // strided copy out of the packed [B][A+1] buffer
        const size_t rows = which == 1 ? n / c->A : n;
        HIP_TRY(hipMemcpy2DAsync(dst, sizeof(float) * (which == 1 ? c->A : 1), src + (which == 2 ? c->A : 0),
                                 sizeof(float) * (c->A + 1), sizeof(float) * (which == 1 ? c->A : 1), rows,
                                 hipMemcpyDeviceToDevice, s));
        return GA3C_OK;
    }
    HIP_TRY(hipMemcpyAsync(dst, src, sizeof(float) * n, hipMemcpyDeviceToDevice, s));
    return GA3C_OK;
}

extern "C" int ga3c_rmsprop_flat(float *theta, float *g, const float *grad, size_t n, float scale, float lr,
                                 float rms_decay, float rms_eps, void *stream) {
    if (!theta || !g || !grad) return fail(GA3C_EINVAL, "ga3c_rmsprop_flat: null argument");
    if (n == 0) return GA3C_OK;
    if ((((uintptr_t)theta) | ((uintptr_t)g) | ((uintptr_t)grad)) & 15)
        return fail(GA3C_EINVAL, "ga3c_rmsprop_flat: buffers must be 16-byte aligned");
    // one tile of 1024 vectors per block (measured: 6.0 TB/s on 2^28 parameters, against 5.3 with 4096 blocks that
    // loop over tiles and 4.3 with one vector per thread and iteration).  Buffers far larger than the last-level
    // cache are streamed past the caches (non-temporal loads and stores: 5.5 -> 6.0 TB/s); smaller ones are not,
    // since whoever uses theta next finds it in the cache.
    const unsigned rb = (unsigned)std::min<size_t>(std::max<size_t>(n / 4096, 1), (size_t)1 << 20);
    const bool stream_past_caches = 20.0 * (double)n > 1.0e9;
    RmsClip none;
    memset(&none, 0, sizeof(none));
#define GA3C_RMS_LAUNCH(V)                                                                                               \
    ga3c::launch((rmsprop_kernel<V, 4>), dim3(rb), dim3(256), 0, (hipStream_t)stream, theta, theta, g, grad, n,         \
                       (const float *)nullptr, scale, lr, rms_decay, rms_eps, (u32x4 *)nullptr, (u32x4 *)nullptr, 0, FcPlanes(), none)
    if (stream_past_caches) GA3C_RMS_LAUNCH(3); else GA3C_RMS_LAUNCH(0);
#undef GA3C_RMS_LAUNCH
    HIP_TRY(hipGetLastError());
    return GA3C_OK;
}

extern "C" int ga3c_profile_enable(ga3c_ctx *c, int on) {
    if (!c || !c->prof) return fail(GA3C_EINVAL, "ga3c_profile_enable: null context");
    c->prof->on = on != 0;
    return GA3C_OK;
}

extern "C" int ga3c_profile_read(ga3c_ctx *c, char *buf, size_t cap) {
    if (!c || !c->prof || !buf || cap == 0) return fail(GA3C_EINVAL, "ga3c_profile_read: null argument");
    Profiler *p = c->prof;
    for (ProfRec &r : p->recs) {
        HIP_TRY(hipEventSynchronize(r.b));
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, r.a, r.b));
        const double f1 = p->stages[r.stage].flop / p->stages[r.stage].calls;
        const double f2 = r.stage2 >= 0 ? p->stages[r.stage2].flop / p->stages[r.stage2].calls : 0.0;
        const double share = r.stage2 >= 0 && f1 + f2 > 0 ? f1 / (f1 + f2) : 1.0;
        p->stages[r.stage].ms += share * ms;
        if (r.stage2 >= 0) p->stages[r.stage2].ms += (1.0 - share) * ms;
        p->pool.push_back(r.a); p->pool.push_back(r.b);
    }
    p->recs.clear();
    size_t pos = 0;
    buf[0] = 0;
    for (const ProfStage &st : p->stages) {
        int n = snprintf(buf + pos, cap - pos, "%s %ld %.6f %.6e %.6e\n", st.name, st.calls, st.ms, st.flop, st.bytes);
        if (n < 0 || (size_t)n >= cap - pos) return fail(GA3C_EINVAL, "ga3c_profile_read: buffer too small");
        pos += (size_t)n;
    }
    p->stages.clear();
    return GA3C_OK;
}

extern "C" int ga3c_use_generic_kernels(ga3c_ctx *c, int on) {
    if (!c) return fail(GA3C_EINVAL, "ga3c_use_generic_kernels: null context");
    c->fast = on == 0;
    return GA3C_OK;
}

extern "C" int ga3c_get_desc(const ga3c_ctx *c, ga3c_net_desc *desc, int *max_predict_batch, int *max_train_frames) {
    if (!c) return fail(GA3C_EINVAL, "ga3c_get_desc: null context");
    if (desc) *desc = c->desc;
    if (max_predict_batch) *max_predict_batch = c->max_pred;
    if (max_train_frames) *max_train_frames = c->max_train;
    return GA3C_OK;
}

// ---------------------------------------------- prediction without allocation ---
//
// ga3c_predict_static: the prediction of the Sec. 3.2 network for callers that cannot allocate device memory.
// Everything ga3c_predict keeps in buffers that ga3c_create allocates (filter fragments, layer-2 activations, split-k
// partial sums of the fc layer, fc outputs, the one-launch path's tickets) lives in one file-scope device array here.
// Each GPU holds its own copy of the array; its address on a device is looked up once, with that device current,
// and kernels and copies only ever get that looked-up address.
namespace {
constexpr int STATIC_MAX_FRAMES = GA3C_STATIC_MAX_FRAMES;
constexpr int STATIC_MAX_SPLITS = 40;                                    // k-chunks of the fc product: 2592 / 64
constexpr size_t up256(size_t n) { return (n + 255) / 256 * 256; }
constexpr size_t ST_FRAG_OFF = 0;
constexpr size_t ST_HFRAG_OFF = ST_FRAG_OFF + up256(sizeof(u32x4) * 3 * C12_FRAG_SET);
constexpr size_t ST_TICKET_OFF = ST_HFRAG_OFF + up256(sizeof(u32x4) * Conv12F16::VECS);
constexpr size_t ST_H_OFF = ST_TICKET_OFF + up256(sizeof(int) * SP_MAX_FRAMES * SP_TICKET_PITCH);
constexpr size_t ST_Y2_OFF = ST_H_OFF + up256(sizeof(float) * STATIC_MAX_FRAMES * SP_FC);
constexpr size_t ST_WS_OFF = ST_Y2_OFF + up256(sizeof(float) * STATIC_MAX_FRAMES * SP_FLAT);
constexpr size_t ST_WS_FLOATS = (size_t)STATIC_MAX_SPLITS * STATIC_MAX_FRAMES * SP_FC;
constexpr size_t ST_BYTES = ST_WS_OFF + up256(sizeof(float) * ST_WS_FLOATS);
static_assert(ST_BYTES <= (size_t)GA3C_STATIC_SCRATCH_BYTES, "the header promises a smaller array");

constexpr int ST_MAX_DEVICES = 64;
unsigned char *g_static_ptr[ST_MAX_DEVICES];      // device address of the array on each GPU, nullptr until looked up
std::mutex g_static_mutex;
}  // namespace

static __device__ __align__(256) unsigned char ga3c_static_scratch[ST_BYTES];

// Address of the array on the current device (looked up on the first call there).
static int static_scratch(unsigned char **out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= ST_MAX_DEVICES) return fail(GA3C_EINVAL, "ga3c_predict_static: device index %d not supported", dev);
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(ga3c_static_scratch)));
        if (!p) return fail(GA3C_EHIP, "ga3c_predict_static: the scratch array has no address on device %d", dev);
        g_static_ptr[dev] = (unsigned char *)p;
    }
    *out = g_static_ptr[dev];
    return GA3C_OK;
}

extern "C" int ga3c_predict_static(int n_actions, int math, const float *theta, const uint8_t *frames, int B,
                                   const float *uniforms, float *logits, float *values, float *probs, int32_t *actions,
                                   void *stream) {
    if (n_actions < 1 || n_actions > GA3C_MAX_ACTIONS)
        return fail(GA3C_EINVAL, "ga3c_predict_static: n_actions must be 1..%d", GA3C_MAX_ACTIONS);
    if (math != 0 && math != 1) return fail(GA3C_EINVAL, "ga3c_predict_static: math must be 0 or 1");
    if (B < 0 || B > STATIC_MAX_FRAMES)
        return fail(GA3C_EINVAL, "ga3c_predict_static: B = %d outside [0, %d] (the scratch array is sized for %d frames)", B,
                    STATIC_MAX_FRAMES, STATIC_MAX_FRAMES);
    if (B == 0) return GA3C_OK;
    if (!theta || !frames) return fail(GA3C_EINVAL, "ga3c_predict_static: null theta or frames");
    if (actions && !uniforms) return fail(GA3C_EINVAL, "ga3c_predict_static: actions requested without uniforms");
    if (!is_aligned16(theta) || !is_aligned16(frames))
        return fail(GA3C_EINVAL, "ga3c_predict_static: theta and frames must be 16-byte aligned");

    // a context on the stack that owns nothing: shape and offsets on the host, every buffer inside the array
    ga3c_ctx c;
    memset((void *)&c, 0, sizeof(c));
    ga3c_net_desc d;
    memset(&d, 0, sizeof(d));
    d.in_c = 4; d.in_h = 84; d.in_w = 84; d.n_conv = 2;
    d.conv[0].oc = 16; d.conv[0].k = 8; d.conv[0].stride = 4;
    d.conv[1].oc = 32; d.conv[1].k = 4; d.conv[1].stride = 2;
    d.fc_units = SP_FC; d.n_actions = n_actions; d.math = math;
    TRY(init_shape(&c, &d));
    if (c.flat != SP_FLAT || c.off[2] % 4 != 0 || c.off[4] % 4 != 0)
        return fail(GA3C_EINVAL, "ga3c_predict_static: internal: unexpected layout");
    unsigned char *base = nullptr;
    TRY(static_scratch(&base));
    c.fast = true; c.small_frames = small_launch_frames(&c); c.max_pred = STATIC_MAX_FRAMES;
    c.theta2[0] = const_cast<float *>(theta);
    c.cfrag[0] = (u32x4 *)(base + ST_FRAG_OFF);
    c.ticket = (int *)(base + ST_TICKET_OFF);
    c.pred.cap = STATIC_MAX_FRAMES;
    c.pred.h = (float *)(base + ST_H_OFF);
    c.pred.act[1] = (float *)(base + ST_Y2_OFF);
    c.pred.ws = (float *)(base + ST_WS_OFF);
    c.pred.ws_floats = ST_WS_FLOATS;
    hipStream_t s = (hipStream_t)stream;
    // the filters as split MFMA fragments, from the caller's parameters (a context does this when they change): those that this call reads
    if (B > c.small_frames && !math) {
        c.hfrag[0] = (u32x4 *)(base + ST_HFRAG_OFF);
        HIP_TRY(launch_conv12_f16_filters(theta + c.off[0], theta + c.off[2], c.hfrag[0], s));
    } else TRY(refresh_derived(&c, 0, s));
    return forward(&c, 0, c.pred, frames, nullptr, B, false, logits, values, probs, uniforms, actions, s);
}
