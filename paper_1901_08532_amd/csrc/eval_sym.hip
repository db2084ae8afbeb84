// Evaluation over all particles with each unordered pair taken once
// (sym_plan.h): the a, j, s terms of a pair serve both particles, by Newton's
// third law.
//
// The walk is sym_body.h's; a lane holds two targets, so that the 18 DPP moves
// that take a source's sums to the next lane serve two pairs. Per unordered
// pair that is 63 + 9 VALU operations at order 2
// against 2 x 54 in ordered form; the bound stays FP64 issue. Evaluation of
// all particles, ordered form and this: n = 8192 139 -> 116 us, 16384 493 ->
// 357 us, 32768 1902 -> 1335 us, 65536 7585 -> 5200 us (64 TFLOP/s at 78
// operations an ordered pair, 82% of the FP64 vector peak). Both start-up passes: n = 32768 3999 -> 2510 us.
#include <algorithm>

#include "eval_ops.h"

namespace h6 {
namespace {

using namespace evalbody;
using namespace symbody;

template <int ORDER, bool SKIPSELF>
__global__ __launch_bounds__(kSymThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_eval_sym(
    SrcPtrs src, SymPlan P, double eps2, double *__restrict__ partial) {
    sym_run(EvalOps<ORDER, SKIPSELF>{src, eps2}, P, partial);
}

// One sum of a batch's slots per thread, components from c0 on.
__global__ __launch_bounds__(256) void k_sym_reduce(const double *__restrict__ partial, SymPlan P,
                                                    int ncomp, int c0, int nc, int out0, OutPtrs out,
                                                    unsigned acc_mask) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)nc * P.n) return;
    const int cl = (int)(idx / P.n), c = c0 + cl, k = (int)(idx - (int64_t)cl * P.n);
    double s;
    sym_sums<1>(partial, P, ncomp, c, k, &s);
    double *dst = &out.p[out0 + c][k];
    *dst = ((acc_mask >> c) & 1u) ? *dst + s : s;
}

// Particles of a superblock and the price of a cell. FP64: n = 16384 in 9
// whole chunks a run takes 1.6% less than in 17 halves; EX, whose FP32 operations
// issue faster the more waves there are: a shared step of n = 4096 on two
// workgroups a CU 243 us, on three 220, 8192 769 and 708.
constexpr int kEvalBlock = kSymThreads * EvalOps<2, false>::K;
int block_of(int precision) { return precision == H6_EX ? kSymThreads : kEvalBlock; }
SymCost cost_of(int precision) {
    return precision == H6_EX ? SymCost{180.0f, 1.0f, 260.0f} : SymCost{36.0f, 3.0f};
}

}  // namespace

bool sym_plan(h6_ctx ctx, int n, int block, int ncomp, SymCost cost, int d0, SymPlan *plan) {
    int runs = 2 * ctx->n_cu;  // two workgroups of four waves a CU (two waves a SIMD)
    SymPlan P;
    P.n = n;
    P.block = block;
    P.nsb = (n + block - 1) / block;
    P.d0 = d0;
    P.ordered = 0;
    const int nd = P.nsb / 2 + 1, dj = d0 > 0 ? d0 : 1;
    const int64_t slots = ctx->partial_cap / ((int64_t)ncomp * n);
    if (d0 >= nd) return false;
    // the batch [d0, dj + m) in `sub` parts on r workgroups; false if its
    // sums need more slots than there are
    auto fits = [&](int m, int sub, int r) {
        P.d1 = dj + m;
        P.half = P.nsb % 2 == 0 && P.nsb > 1 && P.d1 == nd;
        P.sub = sub;
        P.runs = 1;
        P.cells = 1;  // not read by first_cell
        P.cells = P.first_cell(P.nsb);
        P.runs = (int)std::min<int64_t>(r, P.cells);
        P.slots_j = m * sub;
        // a superblock's cells touch at most this many runs of len or more
        const int64_t most = (int64_t)(P.d1 - d0) * P.per_d(), len = P.cells / P.runs;
        return P.slots_j + (most - 1 + len - 1) / len + 1 <= slots;
    };
    // as many offsets as fit; for large systems, whose scratch is short, on
    // fewer workgroups if one offset needs it (then three slots do)
    int m = (int)std::min<int64_t>(nd - dj, slots);
    while (m > 1 && !fits(m, 1, runs)) --m;
    while (runs > 1 && !fits(m, 1, runs)) runs = (runs + 1) / 2;
    if (!fits(m, 1, runs)) return false;
    // parts: the longest run, and the sum over slots (their loads go in
    // batches of 8, about 0.55 us each, and at about 3 TB/s)
    float best = 3.0e38f;
    for (int three = 0; three < (cost.chunk3 > 0.0f ? 2 : 1); ++three) {
        const int r = three ? 3 * ctx->n_cu : runs;
        const float chunk = three ? cost.chunk3 : cost.chunk;
        for (int sub = 1; sub <= kSymMaxSub && fits(m, sub, r); sub *= 2) {
            const float longest = (float)((P.cells + P.runs - 1) / P.runs);
            const float used = (float)(P.slots_j + P.run_count(0));
            const float t = longest * (chunk / (float)sub + cost.part) +
                            used * (0.07f + (float)ncomp * (float)n * 2.7e-6f);
            if (t < best) {
                best = t;
                *plan = P;
            }
        }
    }
    return true;
}

SymPlan sym_plan_ordered(int n, int block, int d0) {
    SymPlan P;
    P.n = n;
    P.block = block;
    P.nsb = (n + block - 1) / block;
    P.sub = 1;
    P.d0 = d0;
    P.d1 = std::min(P.nsb, d0 + kOrderedMax);
    P.ordered = 1;
    P.half = 0;
    P.slots_j = 0;
    P.runs = P.nsb;  // a run is a superblock's cells: one slot
    P.cells = P.first_cell(P.nsb);
    return P;
}

hipError_t launch_sym_reduce(h6_ctx ctx, const SymPlan &P, int ncomp, int out0, const OutPtrs &out,
                             unsigned acc_mask) {
    // a launch holds fewer than 2^32 threads: the largest systems a few components at a time
    const int most = (int)std::min<int64_t>(ncomp, ((int64_t)1 << 31) / P.n);
    for (int c0 = 0; c0 < ncomp; c0 += most) {
        const int nc = std::min(most, ncomp - c0);
        hipLaunchKernelGGL(k_sym_reduce, dim3((unsigned)(((int64_t)nc * P.n + 255) / 256)),
                           dim3(256), 0, ctx->stream, ctx->partial, P, ncomp, c0, nc, out0, out,
                           acc_mask);
    }
    return hipGetLastError();
}

bool eval_sym_single(h6_ctx ctx, int precision, int n, SymPlan *plan) {
    return sym_plan(ctx, n, block_of(precision), 9, cost_of(precision), 0, plan) &&
           plan->d1 == plan->nsb / 2 + 1;
}

hipError_t launch_eval_sym_pairs(h6_ctx ctx, int order, int precision, const SrcPtrs &src,
                                 const SymPlan &P) {
    const bool skip = self_pair_masked(ctx->eps2, precision);
#define H6_SYM(O, S)                                                                           \
    hipLaunchKernelGGL((k_eval_sym<O, S>), dim3(P.runs), dim3(kSymThreads), 0, ctx->stream, src, \
                       P, ctx->eps2, ctx->partial)
    if (precision == H6_EX) {
        launch_ex_sym_pairs(ctx, src, P);
    } else if (order == 1) {
        if (skip) H6_SYM(1, true); else H6_SYM(1, false);
    } else if (order == 2) {
        if (skip) H6_SYM(2, true); else H6_SYM(2, false);
    } else {
        if (skip) H6_SYM(3, true); else H6_SYM(3, false);
    }
#undef H6_SYM
    return hipGetLastError();
}

hipError_t launch_eval_sym(h6_ctx ctx, int order, int precision, const SrcPtrs &src, int n,
                           const OutPtrs &out, bool *done) {
    return sym_batches(ctx, n, block_of(precision), order == 2 ? 9 : 6, cost_of(precision),
                       order == 3 ? 6 : 0, out, 0u, done, [&](const SymPlan &P) {
                           return launch_eval_sym_pairs(ctx, order, precision, src, P);
                       });
}

}  // namespace h6
