// Mixed-precision evaluation of acceleration, jerk and snap (order 2).
//
// The paper offers a cheaper arithmetic beside full double precision
// (Sec. 3 item 6: an extended type of about 48-bit significand, and single
// precision) for devices weak in double. The mixed form here keeps what
// cancellation makes precision-critical in FP64 and moves the bulk of the
// pair arithmetic to FP32:
//   * position and velocity differences are formed in FP64 from FP64
//     predicted states, then rounded to FP32 (relative error 2^-24 of the
//     small difference, not of the large coordinates);
//   * acceleration differences, the reciprocal square root (v_rsq_f32 and
//     one Newton step), alpha, beta and the pair terms are FP32;
//   * the a/j/s sums are FP64: FP32 products are gathered over 8 sources,
//     then added to plain FP64 accumulators (the FP64 rounding, about 1e-16
//     per addition, stays far below the FP32 terms' own).
// The launch structure (LDS tiles of sources, target per lane, source
// slices, separate compensated slice reduction) is the FP64 kernel's.
#include "eval_mixed_body.h"
#include "shared_step_body.h"

namespace h6 {
namespace {

using namespace mixedbody;

template <int BLOCK, int IPL, bool SKIPSELF>
__global__ __launch_bounds__(BLOCK)
__attribute__((amdgpu_waves_per_eu(4))) void k_eval_mixed(
    SrcPtrs src, const int32_t *__restrict__ active, int n, int n_act, double eps2, int slice_len,
    OutPtrs out, int64_t slice_stride) {
    mixed_tile_body<BLOCK, IPL, SKIPSELF>(src, active, n, n_act, eps2, slice_len, out, slice_stride,
                                          blockIdx.x, blockIdx.y);
}

template <int TPW, bool SKIPSELF>
__global__ __launch_bounds__(64) void k_eval_small_mixed(SrcPtrs src,
                                                         const int32_t *__restrict__ active, int n,
                                                         int n_act, double eps2, int slice_len,
                                                         OutPtrs out, int64_t slice_stride) {
    mixed_small_body<TPW, SKIPSELF>(src, active, n, n_act, eps2, slice_len, out, slice_stride,
                                    blockIdx.x, blockIdx.y);
}

template <int BLOCK, int IPL>
hipError_t launch_tile(bool skipself, dim3 grid, hipStream_t st, const SrcPtrs &src,
                       const int32_t *active, int n, int n_act, double eps2, int slice_len,
                       const OutPtrs &out, int64_t slice_stride) {
    if (skipself)
        hipLaunchKernelGGL((k_eval_mixed<BLOCK, IPL, true>), grid, dim3(BLOCK), 0, st, src, active,
                           n, n_act, eps2, slice_len, out, slice_stride);
    else
        hipLaunchKernelGGL((k_eval_mixed<BLOCK, IPL, false>), grid, dim3(BLOCK), 0, st, src,
                           active, n, n_act, eps2, slice_len, out, slice_stride);
    return hipGetLastError();
}

// Particles and pairs of the whole-workgroup kernels (eval_wg_body.h). The FP32
// sums cover RUN consecutive sources from a multiple of RUN on: 8 as in the
// tiled body, so the same FP32 values enter the FP64 sums, and 1 for systems of
// at most kDefaultSmallMax, whose strands have one source each, as the lanes of
// the source-parallel body have.
template <bool SKIPSELF, int RUN>
struct MixedOps {
    using Word = double;  // x0 x1 | x2 v0 | v1 v2 | (a0, a1) (a2, m) in FP32
    using Acc = float;
    static constexpr int NREC = 4, NI = 9, kRun = RUN, kMinTgt = kMixedWgMinTgt, kDirectMaxTgt = 0;
    static constexpr int kUnroll = 1;  // where RUN is 1
    struct Sum {
        double s;
    };
    struct Target {
        double x[3], v[3];
        float a[3];
    };
    SrcPtrs src;
    double eps2;
    static __device__ __forceinline__ double pair_word(float a, float b) {
        return __hiloint2double(__float_as_int(b), __float_as_int(a));
    }
    __device__ __forceinline__ void load_rec(int jj, evalbody::Word2<double> *rec) const {
        rec[0] = {src.x[0][jj], src.x[1][jj]};
        rec[1] = {src.x[2][jj], src.v[0][jj]};
        rec[2] = {src.v[1][jj], src.v[2][jj]};
        rec[3] = {pair_word((float)src.a[0][jj], (float)src.a[1][jj]),
                  pair_word((float)src.a[2][jj], (float)src.m[jj])};
    }
    static __device__ __forceinline__ void pad_rec(evalbody::Word2<double> *rec) {
        rec[0] = {kPadPosMixed, kPadPosMixed};
        rec[1] = {kPadPosMixed, 0.0};
        rec[2] = rec[3] = {0.0, 0.0};
    }
    __device__ __forceinline__ void load(int k, int, Target &t) const {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            t.x[c] = src.x[c][k];
            t.v[c] = src.v[c][k];
            t.a[c] = (float)src.a[c][k];
        }
    }
    __device__ __forceinline__ void one(const evalbody::Word2<double> *e, const Target &t, bool self,
                                        float *acc) const {
        const float dx = (float)(e[0].x - t.x[0]), dy = (float)(e[0].y - t.x[1]);
        const float dz = (float)(e[1].x - t.x[2]), dvx = (float)(e[1].y - t.v[0]);
        const float dvy = (float)(e[2].x - t.v[1]), dvz = (float)(e[2].y - t.v[2]);
        const float a0 = __int_as_float(__double2loint(e[3].x));
        const float a1 = __int_as_float(__double2hiint(e[3].x));
        const float a2 = __int_as_float(__double2loint(e[3].y));
        float m = __int_as_float(__double2hiint(e[3].y));
        float r2 = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, (float)eps2)));
        if (SKIPSELF) {
            r2 = self ? 1.0f : r2;
            m = self ? 0.0f : m;
        }
        pair_acc2_f32(dx, dy, dz, dvx, dvy, dvz, a0 - t.a[0], a1 - t.a[1], a2 - t.a[2], r2, m, acc);
    }
    static __device__ __forceinline__ void add(Sum &s, float x) { s.s += (double)x; }
    static __device__ __forceinline__ double value(const Sum &s) { return s.s; }
};

}  // namespace

hipError_t dispatch_mixed_wg(int tgt, bool skipself, dim3 grid, hipStream_t st, const SrcPtrs &src,
                             const int32_t *active, int n, int n_act, double eps2, int slice_len,
                             const OutPtrs &out, int64_t slice_stride) {
    return skipself ? evalbody::launch_wg(tgt, grid, st, MixedOps<true, kChunk>{src, eps2}, active, n, n_act,
                                          slice_len, 0, out, slice_stride)
                    : evalbody::launch_wg(tgt, grid, st, MixedOps<false, kChunk>{src, eps2}, active, n,
                                          n_act, slice_len, 0, out, slice_stride);
}

hipError_t launch_mixed_shared_step(h6_ctx ctx, h6_state *st, int n, const SrcPtrs &src, double dt,
                                    bool predict, const h6_pred *out, const h6_force *f) {
    auto launch = [&](auto ops) {
        return stepbody::launch_shared_step_ops(ctx, ops, st, n, dt, predict, out, f);
    };
    const double eps2 = ctx->eps2;
    const bool small = n <= kDefaultSmallMax;
    if (self_pair_masked(eps2, H6_MIXED))
        return small ? launch(MixedOps<true, 1>{src, eps2}) : launch(MixedOps<true, kChunk>{src, eps2});
    return small ? launch(MixedOps<false, 1>{src, eps2}) : launch(MixedOps<false, kChunk>{src, eps2});
}

hipError_t dispatch_mixed(const EvalConfig &cfg, bool skipself, dim3 grid, hipStream_t st,
                          const SrcPtrs &src, const int32_t *active, int n, int n_act, double eps2,
                          int slice_len, const OutPtrs &out, int64_t slice_stride) {
    if (cfg.kind == 1) {
#define H6_SMALLM(T)                                                                            \
    if (cfg.ipl == T) {                                                                         \
        if (skipself)                                                                           \
            hipLaunchKernelGGL((k_eval_small_mixed<T, true>), grid, dim3(64), 0, st, src,       \
                               active, n, n_act, eps2, slice_len, out, slice_stride);           \
        else                                                                                    \
            hipLaunchKernelGGL((k_eval_small_mixed<T, false>), grid, dim3(64), 0, st, src,      \
                               active, n, n_act, eps2, slice_len, out, slice_stride);           \
        return hipGetLastError();                                                               \
    }
        H6_SMALLM(1)
        H6_SMALLM(2)
        H6_SMALLM(4)
#undef H6_SMALLM
        return hipErrorInvalidValue;
    }
#define H6_TILEM(B, I)                                                                          \
    if (cfg.block == B && cfg.ipl == I)                                                         \
        return launch_tile<B, I>(skipself, grid, st, src, active, n, n_act, eps2, slice_len, out, \
                                 slice_stride);
    H6_TILEM(64, 1)
    H6_TILEM(128, 1)
    H6_TILEM(256, 1)
    H6_TILEM(64, 2)
    H6_TILEM(128, 2)
    H6_TILEM(256, 2)
#undef H6_TILEM
    return hipErrorInvalidValue;
}

}  // namespace h6
