// Evaluation over all particles with each unordered pair taken once
// (sym_plan.h): the a, j, s terms of a pair serve both particles, by Newton's
// third law.
//
// The walk is sym_body.h's; a lane holds two targets, so that the 18 DPP moves
// that take a source's sums to the next lane serve two pairs. Per unordered
// pair that is 63 + 9 VALU operations at order 2
// against 2 x 54 in ordered form; the bound stays FP64 issue. Evaluation of
// all particles, ordered form and this: n = 8192 139 -> 116 us, 16384 493 ->
// 364 us, 32768 1902 -> 1335 us, 65536 7585 -> 5200 us (64 TFLOP/s at 78
// operations an ordered pair, 82% of the FP64 vector peak). Both start-up passes: n = 32768 3999 -> 2510 us.
#include <algorithm>

#include "eval_body.h"
#include "sym_body.h"

namespace h6 {
namespace {

using namespace evalbody;
using namespace symbody;

// Terms of the pair (target i, source j) added to both particles' sums; d* is
// source minus target. Order 1: a, j; 2: a, j, s; 3: s, c.
template <int ORDER>
__device__ __forceinline__ void pair_both(const double *r, const double *v, const double *a,
                                          const double *jr, double r2, double mi, double mj,
                                          double *acci, double *accj) {
    const double rinv = rsqrt_f64(r2);
    const double rinv2 = rinv * rinv;
    const double r3 = rinv * rinv2;
    const double pj = mj * r3, pi = mi * r3;
    const double rv = fma(r[2], v[2], fma(r[1], v[1], r[0] * v[0]));
    const double alpha = rv * rinv2;
    const double a3 = 3.0 * alpha;
    double w[3], u[3], z[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) w[c] = fma(-a3, r[c], v[c]);
    if constexpr (ORDER >= 2) {
        const double vvra =
            fma(r[2], a[2], fma(r[1], a[1], fma(r[0], a[0],
                fma(v[2], v[2], fma(v[1], v[1], v[0] * v[0])))));
        const double beta = fma(alpha, alpha, vvra * rinv2);
        const double b3 = 3.0 * beta, a6 = a3 + a3;
#pragma unroll
        for (int c = 0; c < 3; ++c) u[c] = fma(-a6, w[c], fma(-b3, r[c], a[c]));
        if constexpr (ORDER == 3) {
            const double va = fma(v[2], a[2], fma(v[1], a[1], v[0] * a[0]));
            const double rj = fma(r[2], jr[2], fma(r[1], jr[1], r[0] * jr[0]));
            const double gamma =
                fma(alpha, fma(-4.0 * alpha, alpha, b3), fma(3.0, va, rj) * rinv2);
            const double a9 = 3.0 * a3, b9 = 3.0 * b3, g3 = 3.0 * gamma;
#pragma unroll
            for (int c = 0; c < 3; ++c)
                z[c] = fma(-a9, u[c], fma(-b9, w[c], fma(-g3, r[c], jr[c])));
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if constexpr (ORDER <= 2) {
            acci[c] = fma(pj, r[c], acci[c]);
            accj[c] = fma(-pi, r[c], accj[c]);
            acci[3 + c] = fma(pj, w[c], acci[3 + c]);
            accj[3 + c] = fma(-pi, w[c], accj[3 + c]);
            if constexpr (ORDER == 2) {
                acci[6 + c] = fma(pj, u[c], acci[6 + c]);
                accj[6 + c] = fma(-pi, u[c], accj[6 + c]);
            }
        } else {
            acci[c] = fma(pj, u[c], acci[c]);
            accj[c] = fma(-pi, u[c], accj[c]);
            acci[3 + c] = fma(pj, z[c], acci[3 + c]);
            accj[3 + c] = fma(-pi, z[c], accj[3 + c]);
        }
    }
}

template <int ORDER, bool SKIPSELF>
struct EvalOps {
    using Word = double;
    using Sum = CompSum;
    static constexpr int NF = ORDER == 1 ? 7 : ORDER == 2 ? 10 : 13;  // x, m, v, a, j
    static constexpr int NREC = Traits<ORDER>::NREC;
    static constexpr int NI = Traits<ORDER>::NACC, NJ = NI, K = 2, kUnroll = 2;
    struct Target {
        double x[3], v[3], a[3], j[3], m;
    };
    SrcPtrs src;
    double eps2;
    // record order x0 x1 | x2 m | v0 v1 | v2 a0 | a1 a2 | j0 j1 | j2
    __device__ __forceinline__ const double *field(int f) const {
        return f < 3   ? src.x[f]
               : f == 3 ? src.m
               : f < 7  ? src.v[f - 4]
               : f < 10 ? src.a[f - 7]
                        : src.j[f - 10];
    }
    static __device__ __forceinline__ double word(double x) { return x; }
    static __device__ __forceinline__ double pad(int f) { return f < 3 ? kPadPos : 0.0; }
    __device__ __forceinline__ void load(int k, int n, Target &t) const {
        const bool in = k < n;
        PredSrc{src, nullptr}.template get<ORDER>(in ? k : n - 1, t.x, t.v, t.a, t.j);
        t.m = in ? src.m[k] : 0.0;
        // padding: massless, and far from the sources' padding too
#pragma unroll
        for (int c = 0; c < 3; ++c) t.x[c] = in ? t.x[c] : -kPadPos;
    }
    __device__ __forceinline__ void both(const Word2<double> *e, const Target &t, double *acci,
                                         double *accj) const {
        const double r[3] = {e[0].x - t.x[0], e[0].y - t.x[1], e[1].x - t.x[2]};
        const double v[3] = {e[2].x - t.v[0], e[2].y - t.v[1], e[3].x - t.v[2]};
        double a[3] = {0, 0, 0}, jr[3] = {0, 0, 0};
        if constexpr (ORDER >= 2) {
            a[0] = e[3].y - t.a[0];
            a[1] = e[4].x - t.a[1];
            a[2] = e[4].y - t.a[2];
        }
        if constexpr (ORDER == 3) {
            jr[0] = e[5].x - t.j[0];
            jr[1] = e[5].y - t.j[1];
            jr[2] = e[6].x - t.j[2];
        }
        const double r2 = fma(r[2], r[2], fma(r[1], r[1], fma(r[0], r[0], eps2)));
        pair_both<ORDER>(r, v, a, jr, r2, t.m, e[1].y, acci, accj);
    }
    __device__ __forceinline__ void one(const Word2<double> *e, const Target &t, bool self,
                                        double *acci) const {
        double2 d[NREC];
#pragma unroll
        for (int q = 0; q < NREC; ++q) d[q] = make_double2(e[q].x, e[q].y);
        pair_terms<ORDER, SKIPSELF>(d, t.x, t.v, t.a, t.j, eps2, self, acci);
    }
    static __device__ __forceinline__ void add(Sum &s, double x) { two_sum_into(s.hi, s.lo, x); }
    static __device__ __forceinline__ double value(const Sum &s) { return s.hi + s.lo; }
    static __device__ __forceinline__ double value(double x) { return x; }
};

template <int ORDER, bool SKIPSELF>
__global__ __launch_bounds__(kSymThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_eval_sym(
    SrcPtrs src, SymPlan P, double eps2, double *__restrict__ partial) {
    sym_run(EvalOps<ORDER, SKIPSELF>{src, eps2}, P, partial);
}

// Sum of a batch's slots: the source-side slots that particle k's superblock
// has, then the target-side ones of the runs that touched it (compensated).
__global__ __launch_bounds__(256) void k_sym_reduce(const double *__restrict__ partial, SymPlan P,
                                                    int ncomp, int out0, OutPtrs out,
                                                    unsigned acc_mask) {
    const int n = P.n;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)ncomp * n) return;
    const int c = (int)(idx / n), k = (int)(idx - (int64_t)c * n);
    const int J = k / P.block;
    const double *__restrict__ p = partial + (int64_t)c * n + k;
    const int64_t ld = (int64_t)ncomp * n;
    int nj = P.slots_j;
    // the batch's last slots are d = nsb / 2, which only half the superblocks have
    if (P.half && nj > 0 && !P.has_source_sum(J, P.nsb / 2)) nj -= P.sub;
    const int ni = P.run_count(J);
    double s = 0.0, comp = 0.0;
    for (int part = 0; part < 2; ++part) {
        const int cnt = part ? ni : nj;
        const double *__restrict__ b = p + (part ? P.slots_j * ld : 0);
        for (int s0 = 0; s0 < cnt; s0 += 8) {
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = s0 + u < cnt ? b[(int64_t)(s0 + u) * ld] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) two_sum_into(s, comp, x[u]);
        }
    }
    double *dst = &out.p[out0 + c][k];
    *dst = ((acc_mask >> c) & 1u) ? *dst + (s + comp) : s + comp;
}

}  // namespace

bool sym_plan(h6_ctx ctx, int n, int block, int runs, int ncomp, int d0, SymPlan *plan) {
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
    // parts: the longest run in chunk times (a part costs about 1/12 more for
    // its staging and sums: n = 16384 in 9 whole chunks a run 352 us, in 17
    // halves 358; n = 8192 in 3 chunks 116 us, in 5 halves 105)
    float best = 3.0e38f;
    for (int sub = 1; sub <= kSymMaxSub && fits(m, sub, runs); sub *= 2) {
        const float longest = (float)((P.cells + P.runs - 1) / P.runs);
        const float cost = longest * (1.0f / (float)sub + 1.0f / 12.0f);
        if (cost < best) {
            best = cost;
            *plan = P;
        }
    }
    return true;
}

SymPlan sym_plan_ordered(int n, int block) {
    SymPlan P;
    P.n = n;
    P.block = block;
    P.nsb = (n + block - 1) / block;
    P.sub = 1;
    P.d0 = 0;
    P.d1 = P.nsb;
    P.ordered = 1;
    P.half = 0;
    P.slots_j = 0;
    P.runs = P.nsb;  // a run is a superblock's cells: one slot
    P.cells = P.first_cell(P.nsb);
    return P;
}

hipError_t launch_sym_reduce(h6_ctx ctx, const SymPlan &P, int ncomp, int out0, const OutPtrs &out,
                             unsigned acc_mask) {
    const int64_t total = (int64_t)ncomp * P.n;
    hipLaunchKernelGGL(k_sym_reduce, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                       ctx->stream, ctx->partial, P, ncomp, out0, out, acc_mask);
    return hipGetLastError();
}

hipError_t launch_eval_sym(h6_ctx ctx, int order, const SrcPtrs &src, int n, const OutPtrs &out,
                           bool *done) {
    const int ncomp = order == 2 ? 9 : 6, out0 = order == 3 ? 6 : 0;
    const int block = kSymThreads * EvalOps<2, false>::K;
    const int runs = 2 * ctx->n_cu;  // two workgroups of four waves a CU (two waves a SIMD)
    SymPlan P;
    *done = sym_plan(ctx, n, block, runs, ncomp, 0, &P);
    if (!*done) return hipSuccess;
    const bool skip = self_pair_masked(ctx->eps2, H6_FP64);
    for (bool more = true; more; more = sym_plan(ctx, n, block, runs, ncomp, P.d1, &P)) {
#define H6_SYM(O, S)                                                                           \
    hipLaunchKernelGGL((k_eval_sym<O, S>), dim3(P.runs), dim3(kSymThreads), 0, ctx->stream, src, \
                       P, ctx->eps2, ctx->partial)
        if (order == 1) {
            if (skip) H6_SYM(1, true); else H6_SYM(1, false);
        } else if (order == 2) {
            if (skip) H6_SYM(2, true); else H6_SYM(2, false);
        } else {
            if (skip) H6_SYM(3, true); else H6_SYM(3, false);
        }
#undef H6_SYM
        hipError_t e = hipGetLastError();
        if (e == hipSuccess)
            e = launch_sym_reduce(ctx, P, ncomp, out0, out, P.d0 > 0 ? (1u << ncomp) - 1u : 0u);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace h6
