// The FP64 particles and pairs of the evaluation (OPS of sym_body.h and
// eval_wg_body.h).
#pragma once

#include "eval_body.h"
#include "sym_body.h"

namespace h6 {
namespace evalbody {

using symbody::CompSum;
using symbody::Word2;

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

// Whole records from an OPS with one array per word.
template <class OPS>
__device__ __forceinline__ void rec_from_fields(const OPS &ops, int jj,
                                                Word2<typename OPS::Word> *rec) {
    auto *w = reinterpret_cast<typename OPS::Word *>(rec);
#pragma unroll
    for (int f = 0; f < 2 * OPS::NREC; ++f)
        w[f] = f < OPS::NF ? OPS::word(ops.field(f)[jj]) : typename OPS::Word{};
}
template <class OPS>
__device__ __forceinline__ void rec_padding(Word2<typename OPS::Word> *rec) {
    auto *w = reinterpret_cast<typename OPS::Word *>(rec);
#pragma unroll
    for (int f = 0; f < 2 * OPS::NREC; ++f) w[f] = f < OPS::NF ? OPS::pad(f) : typename OPS::Word{};
}

template <int ORDER, bool SKIPSELF>
struct EvalOps {
    using Word = double;
    using Acc = double;
    static constexpr int kRun = 1, kMinTgt = 1, kDirectMaxTgt = ORDER == 2 ? 2 : 0;
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
    __device__ __forceinline__ void load_rec(int jj, Word2<double> *rec) const {
        rec_from_fields(*this, jj, rec);
    }
    static __device__ __forceinline__ void pad_rec(Word2<double> *rec) {
        rec_padding<EvalOps>(rec);
    }
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

}  // namespace evalbody
}  // namespace h6
