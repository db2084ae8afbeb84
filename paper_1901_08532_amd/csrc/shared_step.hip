// Shared steps in one or two kernels a step: small systems in one
// (shared_step_body.h), larger ones that the third-law evaluation takes in one
// batch with its slot sums, corrector and next prediction in the second.
#include "shared_step_body.h"
#include "sym_plan.h"

namespace h6 {
namespace {

using namespace stepbody;

// Sums of a third-law evaluation's slots (as k_sym_reduce), corrector, and the
// prediction of the next step, or after the last one the forces: one component
// of one particle per thread. Bound by memory latency and the slots' traffic;
// as three kernels (reduce, correct, predict) 9.2 + 4.8 + 4.7 us at n = 16384,
// in one 11 us.
__global__ __launch_bounds__(256) void k_sym_step(const double *__restrict__ partial, SymPlan P,
                                                  h6_state st, double h, bool predict, h6_pred out,
                                                  h6_force f, int32_t *flags) {
    const int n = P.n;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)3 * n) return;
    const int c = (int)(idx / n), k = (int)(idx - (int64_t)c * n);
    const double x0 = st.x[c][k], v0 = st.v[c][k], a0 = st.a[c][k], j0 = st.j[c][k],
                 s0 = st.s[c][k];
    double F[3];
    sym_sums<3>(partial, P, 9, c, k, F);  // components c, 3 + c, 6 + c: a, j, s
    const double hinv = 1.0 / h;
    double x1, v1, c1;
    correct_comp(h, h * h, hinv * hinv * hinv, x0, v0, a0, j0, s0, F[0], F[1], F[2], x1, v1, c1);
    if (!(isfinite(x1) && isfinite(v1) && isfinite(c1))) atomicOr(flags, kFlagNonFinite);
    st.x[c][k] = x1;
    st.v[c][k] = v1;
    st.a[c][k] = F[0];
    st.j[c][k] = F[1];
    st.s[c][k] = F[2];
    st.c[c][k] = c1;
    if (predict) {
        double xp, vp, ap;
        predict_comp(x1, v1, F[0], F[1], F[2], c1, h, xp, vp, ap);
        out.x[c][k] = xp;
        out.v[c][k] = vp;
        out.a[c][k] = ap;
    } else {
        f.a[c][k] = F[0];
        f.j[c][k] = F[1];
        f.s[c][k] = F[2];
    }
}

}  // namespace

int shared_step_targets(h6_ctx ctx, int n) {
    int tgt = 1;
    while (tgt < kWgMaxTgt && tgt * ctx->n_cu < n) tgt *= 2;
    return tgt;
}

hipError_t launch_shared_step(h6_ctx ctx, h6_state *st, int n, int precision, const SrcPtrs &src,
                              double dt, bool predict, const h6_pred *out, const h6_force *f) {
    if (precision == H6_MIXED)
        return launch_mixed_shared_step(ctx, st, n, src, dt, predict, out, f);
    return self_pair_masked(ctx->eps2, H6_FP64)
               ? launch_shared_step_ops(ctx, EvalOps<2, true>{src, ctx->eps2}, st, n, dt, predict,
                                        out, f)
               : launch_shared_step_ops(ctx, EvalOps<2, false>{src, ctx->eps2}, st, n, dt, predict,
                                        out, f);
}

hipError_t launch_sym_step(h6_ctx ctx, const SymPlan &P, h6_state *st, double dt, bool predict,
                           const h6_pred *out, const h6_force *f) {
    hipLaunchKernelGGL(k_sym_step, dim3((unsigned)(((int64_t)3 * P.n + 255) / 256)), dim3(256), 0,
                       ctx->stream, ctx->partial, P, *st, dt, predict, *out, *f, ctx->flags);
    return hipGetLastError();
}

}  // namespace h6
