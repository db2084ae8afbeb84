// One shared step of a small system in one kernel: evaluation, corrector and
// the prediction to the next step.
//
// Bound by latency at these sizes: as separate kernels (predict, evaluate,
// reduce, correct) a step paid four launches and their memory round trips,
// 4.5 to 5 us each, beside 62 us of evaluation on 32 waves at n = 1024
// (70 us a step; 9.2 us with this kernel). The mixed form: n = 32 11.1 -> 5.0 us
// a step, 256 46 -> 7.9, 1024 75 -> 14, 4096 82 -> 45. Here a workgroup sums its
// targets over all sources (eval_wg_body.h: no slice sums in memory), corrects
// them and predicts them to the next step. Other workgroups still read the sources' predicted
// arrays, so the predictions go to a second set; the caller alternates them.
#pragma once

#include "eval_wg_body.h"
#include "steps_body.h"

namespace h6 {
namespace stepbody {

using namespace evalbody;

// PREDICT: predict the next step into `out`; otherwise (the last step) write
// the forces to f.
template <int TGT, class OPS>
__global__ __launch_bounds__(kWgThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_shared_step(
    h6_state st, OPS ops, int n, double h, bool predict, h6_pred out, h6_force f, int32_t *flags) {
    constexpr int kOld = 15;  // x, v, a, j, s of each target
    __shared__ double2 pool[wg_pool_bytes<TGT, OPS>() / sizeof(double2)];
    __shared__ double fs[TGT * 9];
    __shared__ double old[kOld][TGT];
    const int tid = threadIdx.x, lane = tid & 63;
    const int k0 = (int)blockIdx.x * TGT;
    // the old state on its way while the sums run, a component per wave
    for (int q = __builtin_amdgcn_readfirstlane(tid >> 6); q < kOld; q += kWgThreads / 64) {
        const int c = q % 3;
        const double *p = q < 3 ? st.x[c] : q < 6 ? st.v[c] : q < 9 ? st.a[c] : q < 12 ? st.j[c] : st.s[c];
        if (lane < TGT && k0 + lane < n) old[q][lane] = p[k0 + lane];
    }
    wg_sums<TGT>(ops, nullptr, n, n, (int)blockIdx.x, 0, n, pool, fs);
    // one component of one target per thread
    const int t = tid % TGT, c = tid / TGT, i = k0 + t;
    if (c >= 3 || i >= n) return;
    const double a1 = fs[t * 9 + c], j1 = fs[t * 9 + 3 + c], s1 = fs[t * 9 + 6 + c];
    const double hinv = 1.0 / h;
    const double hinv3 = hinv * hinv * hinv;
    double x1, v1, c1;
    correct_comp(h, h * h, hinv3, old[c][t], old[3 + c][t], old[6 + c][t], old[9 + c][t],
                 old[12 + c][t], a1, j1, s1, x1, v1, c1);
    if (!(isfinite(x1) && isfinite(v1) && isfinite(c1))) atomicOr(flags, kFlagNonFinite);
    st.x[c][i] = x1;
    st.v[c][i] = v1;
    st.a[c][i] = a1;
    st.j[c][i] = j1;
    st.s[c][i] = s1;
    st.c[c][i] = c1;
    if (predict) {
        double xp, vp, ap;
        predict_comp(x1, v1, a1, j1, s1, c1, h, xp, vp, ap);
        out.x[c][i] = xp;
        out.v[c][i] = vp;
        out.a[c][i] = ap;
    } else {
        f.a[c][i] = a1;
        f.j[c][i] = j1;
        f.s[c][i] = s1;
    }
}

// Launch on ctx's stream; shared_step_targets gives the targets a workgroup.
template <class OPS>
hipError_t launch_shared_step_ops(h6_ctx ctx, const OPS &ops, h6_state *st, int n, double dt,
                                  bool predict, const h6_pred *out, const h6_force *f) {
    int tgt = shared_step_targets(ctx, n);
    if (tgt < OPS::kMinTgt) tgt = OPS::kMinTgt;
    auto launch = [&](auto t) {
        constexpr int T = decltype(t)::value;
        if constexpr (T >= OPS::kMinTgt) {
            if (tgt != T) return false;
            hipLaunchKernelGGL((k_shared_step<T, OPS>), dim3((n + T - 1) / T), dim3(kWgThreads), 0,
                               ctx->stream, *st, ops, n, dt, predict, *out, *f, ctx->flags);
            return true;
        }
        return false;
    };
    return for_each_tgt(launch) ? hipGetLastError() : hipErrorInvalidValue;
}

}  // namespace stepbody
}  // namespace h6
