// Evaluation of softened acceleration, jerk, snap (and, at start-up,
// crackle) on a set of target particles from all source particles.
//
// The stage and its kernel steps follow the paper (Sec. 3, item 4): sources
// are staged tile by tile through on-chip local memory (LDS here), each
// thread keeps its target's partial sums in registers across tiles, the
// self term is excluded, and the sums are written to global memory at the
// end. The pair terms are the time derivatives of the softened Newtonian
// acceleration of the 6th-order Hermite scheme the paper cites.
//
// gfx950 design:
//   * one target per lane (or two: IPL = 2), wave64; the source record of a
//     tile entry is read by all lanes at one LDS address (broadcast), five
//     128-bit reads per source;
//   * grid = (target blocks) x (source slices): the sum over sources is
//     split across workgroups so that even a few hundred targets fill 256
//     CUs; the slices are combined by a separate compensated reduction;
//   * FP64 throughout; reciprocal square root from the hardware estimate
//     (v_rsq_f64) refined by one Newton step;
//   * per tile the register sums are flushed into a compensated (hi, lo)
//     pair, so rounding grows with the number of tiles, not sources;
//   * no floating-point atomics: results are bitwise reproducible for a
//     given launch shape.
#include <algorithm>
#include <climits>

#include "eval_body.h"
#include "eval_wg_body.h"

namespace h6 {
namespace {

using namespace evalbody;

template <int ORDER, int BLOCK, int IPL, bool SKIPSELF>
__global__ __launch_bounds__(BLOCK)
__attribute__((amdgpu_waves_per_eu(IPL == 1 ? 4 : 2))) void k_eval_f64(
    SrcPtrs src, const int32_t *__restrict__ active, int n, int n_act, double eps2, int slice_len,
    OutPtrs out, int64_t slice_stride) {
    eval_tile_body<ORDER, BLOCK, IPL, SKIPSELF>(src, active, n, n_act, eps2, slice_len, out,
                                                slice_stride, blockIdx.x, blockIdx.y);
}

// Slice reduction, few slices: one thread per (component, target), a
// Neumaier sum over the slices with all loads issued up front.
__global__ __launch_bounds__(256) void k_reduce_slices(const double *__restrict__ partial,
                                                       int64_t ld, int n_split, int ncomp, int out0,
                                                       int n_act, OutPtrs out, unsigned acc_mask,
                                                       const int32_t *__restrict__ list) {
    const int64_t total = (int64_t)ncomp * n_act;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(idx / n_act);
        const int k = (int)(idx - (int64_t)c * n_act);
        double s = 0.0, comp = 0.0;
        for (int s0 = 0; s0 < n_split; s0 += 8) {
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                x[u] = s0 + u < n_split ? partial[((int64_t)(s0 + u) * ncomp + c) * ld + k] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const double t = s + x[u];
                comp += fabs(s) >= fabs(x[u]) ? (s - t) + x[u] : (x[u] - t) + s;
                s = t;
            }
        }
        double *dst = &out.p[out0 + c][list ? list[k] : k];
        *dst = ((acc_mask >> c) & 1u) ? *dst + (s + comp) : s + comp;
    }
}

// Slice reduction, many slices: 64 consecutive outputs per workgroup, one a
// lane (coalesced), each wave summing every kRedWaves-th slice (Neumaier);
// the waves' pairs are then merged in order.
constexpr int kRedWaves = 8;
__global__ __launch_bounds__(64 * kRedWaves) void k_reduce_slices_many(
    const double *__restrict__ partial, int n_split, int ncomp, int out0, int n_act, OutPtrs out,
    unsigned acc_mask, const int32_t *__restrict__ list) {
    __shared__ double2 part[64 * kRedWaves];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t total = (int64_t)ncomp * n_act;
    const int64_t idx = (int64_t)blockIdx.x * 64 + lane;
    const double *__restrict__ p = partial + (idx < total ? idx : total - 1);
    double s = 0.0, comp = 0.0;
    for (int s0 = w; s0 < n_split; s0 += 8 * kRedWaves) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int sl = s0 + u * kRedWaves;
            x[u] = sl < n_split ? p[(int64_t)sl * total] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double t = s + x[u];
            comp += fabs(s) >= fabs(x[u]) ? (s - t) + x[u] : (x[u] - t) + s;
            s = t;
        }
    }
    part[threadIdx.x] = make_double2(s, comp);
    __syncthreads();
    if (w != 0 || idx >= total) return;
#pragma unroll
    for (int q = 1; q < kRedWaves; ++q) comp_merge(s, comp, part[q * 64 + lane].x, part[q * 64 + lane].y);
    const int c = (int)(idx / n_act);
    const int k = (int)(idx - (int64_t)c * n_act);
    double *dst = &out.p[out0 + c][list ? list[k] : k];
    *dst = ((acc_mask >> c) & 1u) ? *dst + (s + comp) : s + comp;
}

template <int TPW, bool SKIPSELF>
__global__ __launch_bounds__(64) void k_eval_small(SrcPtrs src, const int32_t *__restrict__ active,
                                                    int n, int n_act, double eps2, int slice_len,
                                                    OutPtrs out, int64_t slice_stride) {
    eval_small_body<TPW, SKIPSELF>(src, active, n, n_act, eps2, slice_len, out, slice_stride,
                                   blockIdx.x, blockIdx.y);
}

// Slice reduction, many slices of few outputs: one wave per output, its lanes
// over the slices (eight loads each in flight), merged by the row butterfly.
constexpr int kRedOutWaves = 4;
__global__ __launch_bounds__(64 * kRedOutWaves) void k_reduce_slices_wave(
    const double *__restrict__ partial, int n_split, int ncomp, int out0, int n_act, OutPtrs out,
    unsigned acc_mask, const int32_t *__restrict__ list) {
    const int lane = threadIdx.x & 63;
    const int total = ncomp * n_act;
    const int idx = (int)blockIdx.x * kRedOutWaves + (int)(threadIdx.x >> 6);
    if (idx >= total) return;
    const double *__restrict__ p = partial + idx;
    double s = 0.0, comp = 0.0;
    for (int s0 = lane; s0 < n_split; s0 += 8 * 64) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int sl = s0 + u * 64;
            x[u] = sl < n_split ? p[(int64_t)sl * total] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) two_sum_into(s, comp, x[u]);
    }
    seg_comp_reduce_n<1>(&s, &comp, 64);  // valid in lane 63
    if (lane != 63) return;
    const int c = idx / n_act, k = idx - c * n_act;
    double *dst = &out.p[out0 + c][list ? list[k] : k];
    *dst = ((acc_mask >> c) & 1u) ? *dst + (s + comp) : s + comp;
}

template <int ORDER, int BLOCK, int IPL>
hipError_t dispatch_f64(bool skipself, dim3 grid, hipStream_t st, const SrcPtrs &src,
                        const int32_t *active, int n, int n_act, double eps2, int slice_len,
                        const OutPtrs &out, int64_t slice_stride) {
    if (skipself)
        hipLaunchKernelGGL((k_eval_f64<ORDER, BLOCK, IPL, true>), grid, dim3(BLOCK), 0, st, src,
                           active, n, n_act, eps2, slice_len, out, slice_stride);
    else
        hipLaunchKernelGGL((k_eval_f64<ORDER, BLOCK, IPL, false>), grid, dim3(BLOCK), 0, st, src,
                           active, n, n_act, eps2, slice_len, out, slice_stride);
    return hipGetLastError();
}

hipError_t dispatch_shape(const EvalConfig &cfg, bool skipself, dim3 grid, hipStream_t st,
                          const SrcPtrs &src, const int32_t *active, int n, int n_act,
                          double eps2, int slice_len, const OutPtrs &out, int64_t slice_stride) {
#define H6_SHAPE(B, I)                                                                          \
    if (cfg.block == B && cfg.ipl == I)                                                         \
        return dispatch_f64<2, B, I>(skipself, grid, st, src, active, n, n_act, eps2,           \
                                     slice_len, out, slice_stride);
    H6_SHAPE(64, 1)
    H6_SHAPE(128, 1)
    H6_SHAPE(256, 1)
    H6_SHAPE(64, 2)
    H6_SHAPE(128, 2)
    H6_SHAPE(256, 2)
#undef H6_SHAPE
    return hipErrorInvalidValue;
}

int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

hipError_t dispatch_small(int tpw, bool skipself, dim3 grid, hipStream_t st, const SrcPtrs &src,
                          const int32_t *active, int n, int n_act, double eps2, int slice_len,
                          const OutPtrs &out, int64_t slice_stride) {
#define H6_SMALL(T)                                                                            \
    if (tpw == T) {                                                                            \
        if (skipself)                                                                          \
            hipLaunchKernelGGL((k_eval_small<T, true>), grid, dim3(64), 0, st, src, active, n, \
                               n_act, eps2, slice_len, out, slice_stride);                     \
        else                                                                                   \
            hipLaunchKernelGGL((k_eval_small<T, false>), grid, dim3(64), 0, st, src, active, n,\
                               n_act, eps2, slice_len, out, slice_stride);                     \
        return hipGetLastError();                                                              \
    }
    H6_SMALL(1)
    H6_SMALL(2)
    H6_SMALL(4)
#undef H6_SMALL
    return hipErrorInvalidValue;
}

template <int ORDER>
hipError_t dispatch_wg(int tgt, bool skipself, dim3 grid, hipStream_t st, const SrcPtrs &src,
                       const int32_t *active, int n, int n_act, double eps2, int slice_len,
                       const OutPtrs &out, int64_t slice_stride) {
    constexpr int OUT0 = Traits<ORDER>::OUT0;
    return skipself ? launch_wg(tgt, grid, st, EvalOps<ORDER, true>{src, eps2}, active, n, n_act,
                                slice_len, OUT0, out, slice_stride)
                    : launch_wg(tgt, grid, st, EvalOps<ORDER, false>{src, eps2}, active, n, n_act,
                                slice_len, OUT0, out, slice_stride);
}

// Up to this many outputs, each has a wave: 64 coalesced outputs a workgroup
// would leave all but total / 64 CUs idle. Single precision over 65536 sources
// (1024 slices), evaluation and reduction, many / wave: 1 target 23.3 / 14.3
// us, 40 targets 26.1 / 18.2, 200 (1800 outputs) 43.4 / 43.5, 700 98.6 / 100.9,
// 1000 137 / 175 us.
constexpr int64_t kWaveReduceMaxOut = 2048;
// From this many slices the reduction splits them over waves.
constexpr int kManyReduceMinSplit = 16;
// Evaluations of up to this many pairs, over up to this many sources, take the
// whole-workgroup kernel. Beyond, the tile kernel fills the GPU too and is as fast
// or faster, with two targets a lane that share each record's LDS reads, unless
// its groups of 64 or 128 targets are padded by 6% more than groups of 32. Tile /
// whole workgroups, us: FP64 1000 of 20000 123 / 55, 1500 of 65536 255 / 235, 2000
// of 65536 299 / 305, 8192 of 65536 999 / 1044, 1000 of 131072 300 / 308; padded,
// 400 of 524288 508 / 468, 500 (512) 550 / 566; 40 of 1000000 171 / 122. Mixed: 33
// of 1024 41 / 9.2, 300 of 10007 42.6 / 15.2, 6000 of 20000 230 / 212, 1000 of 65536
// 168 / 130, 2000 of 65536 235 / 240, 8192 of 65536 772 / 835, 100 of 524288 127 / 131.
constexpr int64_t kWgMaxPairs = 125000000;
constexpr int kWgMaxSrc = 262144;
constexpr int kWgAlwaysMax = 64;
constexpr int kWgMaxAct = 1 << 27;  // targets of one launch
bool wg_wins(int n, int n_act) {
    if (n_act <= kWgAlwaysMax || (n <= kWgMaxSrc && (int64_t)n * n_act <= kWgMaxPairs)) return true;
    const int tile = n_act <= 512 ? 64 : 128;
    return 1.06 * 32.0 * ceil_div(n_act, 32) < (double)tile * ceil_div(n_act, tile);
}
// Waves a launch aims to put in flight (256 CUs x 4 SIMDs x 2).
constexpr int kTargetWaves = 2048;
// Shortest source slice of the source-parallel kernel (4 sources per lane).
constexpr int kSmallMinSlice = 256;

}  // namespace

// Number of source slices for a target-parallel kernel of `block` threads
// per workgroup whose register footprint allows `waves_per_simd` waves on a
// SIMD. A launch of W workgroups runs in rounds of the resident ones (CUs x
// waves per SIMD x 4 SIMDs / waves per workgroup), so it takes about
// ceil(W / resident) x (slice length + per-workgroup overhead); pick the
// slice count minimising that (fewest slices on ties, to keep the
// reduction small), with at least four tiles per slice.
int balanced_split(h6_ctx ctx, int waves_per_simd, int block, int n, int blocks_i) {
    const int wg_per_cu = std::max(1, waves_per_simd * 4 / (block / 64));
    const int64_t resident = (int64_t)ctx->n_cu * wg_per_cu;
    const int max_split = std::max(1, ceil_div(n, 4 * block));
    const int64_t overhead = 2 * block;  // target loads, partial stores, reduction share
    int best = 1;
    int64_t best_cost = INT64_MAX;
    int last_eff = -1;
    for (int sp = 1; sp <= max_split; ++sp) {
        const int slice = ceil_div(ceil_div(n, sp), block) * block;
        const int eff = ceil_div(n, slice);
        if (eff == last_eff) continue;
        last_eff = eff;
        const int64_t w = (int64_t)blocks_i * eff;
        const int64_t rounds = (w + resident - 1) / resident;
        const int64_t cost = rounds * (slice + overhead);
        if (cost < best_cost) {
            best_cost = cost;
            best = eff;
        }
    }
    return best;
}

// Shape of the whole-workgroup kernel: targets per workgroup and source
// slices, the cheapest by a price in microseconds fitted to a sweep of both
// (n 256 to 65536, n_act 1 to n; the priced shape within 10% of the best
// measured, mostly within 4%). A CU takes c = ceil(workgroups / CUs) of them;
// one issues for `issue` (two waves a SIMD, 216 cycles a pair step) and waits
// about 0.7 us a tile, which a second workgroup on the CU hides. With few
// targets a group, a wave reads more distinct LDS records a step (kWgShare).
// Slices cost a second launch and their traffic.
// EX pairs cost 13 times the operations.
EvalConfig choose_wg(h6_ctx ctx, int order, int precision, int n, int n_act) {
    static const float kWgShare[6] = {1.3f, 1.25f, 1.2f, 1.12f, 1.05f, 1.0f};
    static const int kSplits[14] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128};
    const int ncomp = order == 2 ? 9 : 6;
    EvalConfig cfg;
    cfg.kind = 0;
    cfg.block = kWgThreads;
    cfg.ipl = 1;
    cfg.n_split = 1;
    float best = 3.0e38f;
    const int run = precision == H6_MIXED ? 8 : 1;  // consecutive sources of a strand
    for (int l = 0; l < 6; ++l) {
        const int tgt = 1 << l, strands = kWgThreads / tgt;
        if (precision == H6_MIXED && tgt < kMixedWgMinTgt) continue;
        const int groups = ceil_div(n_act, tgt);
        for (int sp : kSplits) {
            if (sp > 1 && (n / sp < 64 || (int64_t)sp * ncomp * n_act > ctx->partial_cap)) break;
            const int slice = ceil_div(ceil_div(n, sp), 64) * 64;
            const int eff = ceil_div(n, slice);
            const float c = (float)ceil_div((int64_t)groups * eff, ctx->n_cu);
            const int tiles = ceil_div(slice, kWgThreads);
            const int steps = slice / kWgThreads * tgt + ceil_div(slice % kWgThreads, strands * run) * run;
            const float issue = (precision == H6_EX ? 2.6f : 0.196f) * (float)steps;
            // a tile's latency; without LDS (kDirectMaxTgt) that of a thread's pairs
            const float wait = precision == H6_FP64 && order == 2 && tgt <= 2 ? 0.2f * (float)tgt : 0.7f;
            float cost = std::max(c * issue * kWgShare[l], issue + wait * (float)tiles) + 1.2f * c;
            if (eff > 1) cost += 2.0f + (float)eff * (float)n_act * 3.6e-5f;
            if (cost < best) {
                best = cost;
                cfg.ipl = tgt;
                cfg.n_split = eff;
            }
        }
    }
    return cfg;
}

EvalConfig choose_eval_config(h6_ctx ctx, int order, int precision, int n, int n_act) {
    EvalConfig cfg;
    if (precision == H6_EX) return choose_wg(ctx, order, precision, n, n_act);
    if (precision == H6_SP) {
        cfg.kind = 0;
        cfg.block = kSpBlock;
        cfg.ipl = 1;
        const int blocks_i = ceil_div(n_act, kSpBlock);
        int split = std::max(1, ceil_div(4 * ctx->n_cu, blocks_i));
        split = std::min(split, ceil_div(n, kSpBlock));
        const int64_t cap_split = ctx->partial_cap / ((int64_t)9 * n_act);
        if (split > cap_split) split = (int)(cap_split < 1 ? 1 : cap_split);
        cfg.n_split = split < 1 ? 1 : split;
        return cfg;
    }
    // the start-up passes take the third law from kSymMinF64 particles on (whose
    // three slots of six sums every scratch holds) and this below
    if (order != 2) return choose_wg(ctx, order, precision, n, n_act);
    // a launch shape forced by h6_set_eval_config takes the kernels it names
    // (the mixed source-parallel kernel of the smallest sets sums other sources
    // together in FP32, and is as fast)
    const bool forced = eval_shape_forced(ctx);
    if (precision == H6_FP64 && !forced && wg_wins(n, n_act))
        return choose_wg(ctx, order, precision, n, n_act);
    if (precision == H6_MIXED && n_act > kDefaultSmallMax && !forced && wg_wins(n, n_act))
        return choose_wg(ctx, order, precision, n, n_act);
    const int small_max = ctx->cfg_small >= 0 ? ctx->cfg_small : kDefaultSmallMax;
    if (n_act <= small_max) {
        // source-parallel kernel: one wave per TPW targets
        cfg.kind = 1;
        cfg.block = 64;
        cfg.ipl = ctx->cfg_ipl ? ctx->cfg_ipl : (n_act <= 4 ? 1 : 2);
        const int waves_i = ceil_div(n_act, cfg.ipl);
        int split = ceil_div(kTargetWaves, waves_i);
        const int max_split = ceil_div(n, kSmallMinSlice);
        if (split > max_split) split = max_split;
        if (ctx->cfg_split) split = ctx->cfg_split < ceil_div(n, 64) ? ctx->cfg_split : ceil_div(n, 64);
        const int64_t cap_split = ctx->partial_cap / ((int64_t)9 * n_act);
        if (split > cap_split) split = (int)cap_split;
        cfg.n_split = split < 1 ? 1 : split;
        return cfg;
    }
    cfg.kind = 0;
    // measured on gfx950 at N = 65536: one target per lane in 64-thread
    // workgroups up to 512 targets, two per lane beyond
    cfg.block = ctx->cfg_block ? ctx->cfg_block : (n_act <= 16384 ? 64 : 256);
    cfg.ipl = ctx->cfg_ipl ? (ctx->cfg_ipl > 2 ? 2 : ctx->cfg_ipl) : (n_act <= 512 ? 1 : 2);
    const int per_block = cfg.block * cfg.ipl;
    const int blocks_i = ceil_div(n_act, per_block);
    int split;
    if (ctx->cfg_split) {
        split = ctx->cfg_split;
    } else {
        // measured footprints on gfx950: one target per lane <= 128 VGPRs (4
        // waves per SIMD), two per lane <= 256 (2 waves), except the mixed
        // form's (FP32 pair terms, <= 128: 4 waves, and slices enough to fill
        // them, 8% faster at N = 262144)
        const int waves_per_simd = (cfg.ipl == 2 && precision != H6_MIXED) ? 2 : 4;
        split = balanced_split(ctx, waves_per_simd, cfg.block, n, blocks_i);
    }
    const int max_by_tiles = ceil_div(n, cfg.block);
    if (split > max_by_tiles) split = max_by_tiles;
    if (split < 1) split = 1;
    // respect the partial-sum capacity
    const int64_t cap_split = ctx->partial_cap / ((int64_t)9 * (n_act > 0 ? n_act : 1));
    if (split > 1 && split > cap_split) split = (int)(cap_split < 1 ? 1 : cap_split);
    cfg.n_split = split;
    return cfg;
}

hipError_t launch_eval(h6_ctx ctx, int order, int precision, const SrcPtrs &src, int n,
                       const int32_t *active, int n_act, const OutPtrs &out, EvalConfig *used) {
    if (n_act <= 0) return hipSuccess;
    // whole workgroups of 512 threads for 32 targets pass a launch's 2^32 threads
    // from 2^28 targets on; only EX takes them at any size
    if (precision == H6_EX && active && n_act > kWgMaxAct) {
        hipError_t e = hipSuccess;
        for (int k0 = 0; k0 < n_act && e == hipSuccess; k0 += kWgMaxAct) {
            OutPtrs part = out;
            for (int c = 0; c < 9; ++c) part.p[c] += k0;
            e = launch_eval(ctx, order, precision, src, n, active + k0,
                            std::min(kWgMaxAct, n_act - k0), part, used);
        }
        return e;
    }
    // (EX and SP have no forced shapes)
    const bool sym = (precision == H6_EX ||
                      (precision == H6_FP64 && !(order == 2 && eval_shape_forced(ctx)))) &&
                     n >= sym_min(precision);
    if (!active && n_act == n && sym) {
        hipEvent_t ev0 = nullptr, ev1 = nullptr;
        hipError_t e = ctx->prof ? prof_begin(ctx, &ev0, &ev1) : hipSuccess;
        bool done = false;
        if (e == hipSuccess) e = launch_eval_sym(ctx, order, precision, src, n, out, &done);
        const EvalConfig shape = {3, 256, precision == H6_EX ? 1 : 2, 1};
        if (e == hipSuccess && ctx->prof && done)
            e = prof_end(ctx, ev0, ev1, order, shape, precision, n_act, (double)n * (double)n);
        if (e != hipSuccess || done) {
            if (used) *used = shape;
            return e;
        }
    }
    EvalConfig cfg = choose_eval_config(ctx, order, precision, n, n_act);
    // equal slices, each a whole number of tiles
    const bool wg = cfg.kind == 0 && cfg.block == kWgThreads;
    const int unit = wg ? 64 : cfg.block;  // whole tiles (64 for kind 1 and the workgroup kernel)
    int slice_len = ceil_div(n, cfg.n_split);
    slice_len = ceil_div(slice_len, unit) * unit;
    cfg.n_split = ceil_div(n, slice_len);
    if (used) *used = cfg;

    const int ncomp = order == 2 ? 9 : 6;
    const int out0 = order == 3 ? 6 : 0;
    const int per_block = cfg.block * cfg.ipl;
    dim3 grid(ceil_div(n_act, per_block), cfg.n_split);
    const bool skipself = self_pair_masked(ctx->eps2, precision);

    OutPtrs dst;
    int64_t slice_stride = 0;
    if (cfg.n_split == 1) {
        dst = out;
    } else {
        for (int c = 0; c < kMaxOut; ++c) dst.p[c] = nullptr;
        for (int c = 0; c < ncomp; ++c) dst.p[out0 + c] = ctx->partial + (int64_t)c * n_act;
        slice_stride = (int64_t)ncomp * n_act;
    }
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    if (ctx->prof) {
        hipError_t pe = prof_begin(ctx, &ev0, &ev1);
        if (pe != hipSuccess) return pe;
    }
    hipError_t e;
    if (precision == H6_EX) {
        e = dispatch_ex_wg(cfg.ipl, skipself, dim3(ceil_div(n_act, cfg.ipl), cfg.n_split),
                           ctx->stream, src, active, n, n_act, ctx->eps2, slice_len, dst,
                           slice_stride);
    } else if (precision == H6_SP) {
        e = dispatch_sp(ctx->n_cu, skipself, grid, ctx->stream, src, active, n, n_act, ctx->eps2,
                         slice_len, dst, slice_stride);
    } else if (precision == H6_MIXED && wg) {
        e = dispatch_mixed_wg(cfg.ipl, skipself, dim3(ceil_div(n_act, cfg.ipl), cfg.n_split),
                              ctx->stream, src, active, n, n_act, ctx->eps2, slice_len, dst,
                              slice_stride);
    } else if (precision == H6_MIXED) {
        dim3 g = cfg.kind == 1 ? dim3(ceil_div(n_act, cfg.ipl), cfg.n_split) : grid;
        e = dispatch_mixed(cfg, skipself, g, ctx->stream, src, active, n, n_act, ctx->eps2,
                           slice_len, dst, slice_stride);
    } else if (cfg.kind == 1) {
        dim3 g(ceil_div(n_act, cfg.ipl), cfg.n_split);
        e = dispatch_small(cfg.ipl, skipself, g, ctx->stream, src, active, n, n_act, ctx->eps2,
                           slice_len, dst, slice_stride);
    } else if (wg) {
        dim3 g(ceil_div(n_act, cfg.ipl), cfg.n_split);
        if (order == 1)
            e = dispatch_wg<1>(cfg.ipl, skipself, g, ctx->stream, src, active, n, n_act, ctx->eps2,
                               slice_len, dst, slice_stride);
        else if (order == 2)
            e = dispatch_wg<2>(cfg.ipl, skipself, g, ctx->stream, src, active, n, n_act, ctx->eps2,
                               slice_len, dst, slice_stride);
        else
            e = dispatch_wg<3>(cfg.ipl, skipself, g, ctx->stream, src, active, n, n_act, ctx->eps2,
                               slice_len, dst, slice_stride);
    } else {
        e = dispatch_shape(cfg, skipself, grid, ctx->stream, src, active, n, n_act, ctx->eps2,
                           slice_len, dst, slice_stride);
    }
    if (e == hipSuccess && ctx->prof)
        e = prof_end(ctx, ev0, ev1, order, cfg, precision, n_act, (double)n_act * (double)n);
    if (e != hipSuccess || cfg.n_split == 1) return e;
    return launch_reduce(ctx, ctx->partial, cfg.n_split, ncomp, out0, n_act, out, 0u, nullptr);
}

hipError_t launch_ex_chains(h6_ctx ctx, const SrcPtrs &src, int n, const OutPtrs &out) {
    // the single-precision chains' slices
    EvalConfig cfg = choose_eval_config(ctx, 2, H6_SP, n, n);
    const int slice_len = ceil_div(ceil_div(n, cfg.n_split), kSpBlock) * kSpBlock;
    cfg.n_split = ceil_div(n, slice_len);
    OutPtrs dst = out;
    if (cfg.n_split > 1)
        for (int c = 0; c < 9; ++c) dst.p[c] = ctx->partial + (int64_t)c * n;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    hipError_t e = ctx->prof ? prof_begin(ctx, &ev0, &ev1) : hipSuccess;
    if (e == hipSuccess)
        e = dispatch_ex_chain(self_pair_masked(ctx->eps2, H6_EX),
                              dim3(ceil_div(n, kSpBlock), cfg.n_split), ctx->stream, src, n,
                              ctx->eps2, slice_len, dst, (int64_t)9 * n);
    if (e == hipSuccess && ctx->prof)
        e = prof_end(ctx, ev0, ev1, 2, cfg, H6_EX, n, (double)n * (double)n);
    if (e != hipSuccess || cfg.n_split == 1) return e;
    return launch_reduce(ctx, ctx->partial, cfg.n_split, 9, 0, n, out, 0u, nullptr);
}

hipError_t launch_reduce(h6_ctx ctx, const double *partial, int n_split, int ncomp, int out0,
                         int n_act, const OutPtrs &out, unsigned acc_mask, const int32_t *list) {
    const int64_t total = (int64_t)ncomp * n_act;
    if (n_split >= kManyReduceMinSplit && total <= kWaveReduceMaxOut) {
        hipLaunchKernelGGL(k_reduce_slices_wave, dim3(ceil_div(total, kRedOutWaves)),
                           dim3(64 * kRedOutWaves), 0, ctx->stream, partial, n_split, ncomp, out0,
                           n_act, out, acc_mask, list);
    } else if (n_split >= kManyReduceMinSplit) {
        hipLaunchKernelGGL(k_reduce_slices_many, dim3(ceil_div(total, 64)), dim3(64 * kRedWaves), 0,
                           ctx->stream, partial, n_split, ncomp, out0, n_act, out, acc_mask, list);
    } else {
        int rb = ceil_div(total, 256);
        if (rb > 4096) rb = 4096;
        hipLaunchKernelGGL(k_reduce_slices, dim3(rb), dim3(256), 0, ctx->stream, partial,
                           (int64_t)n_act, n_split, ncomp, out0, n_act, out, acc_mask, list);
    }
    return hipGetLastError();
}

}  // namespace h6
