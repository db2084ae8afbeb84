// Adjoint of the shared-step Hermite-6 path: vector-Jacobian products of
// the a/j/s evaluation (and of the start-up passes), and the transposes of
// the shared-step predictor and corrector.
//
// Pair VJP. Write the sum on target k as F_k = sum_j m_j Q(r, v, a, jr)
// with r = x_j - x_k, v = v_j - v_k, a = a_j - a_k, jr = j_j - j_k and Q the
// pair terms per unit source mass (A, J, S or S, C). Q is odd in the joint
// argument, so its Jacobian is even, and the contributions of k as target
// and as source combine into one gather over the same pairs as the forward
// sum: with cotangents g of the outputs,
//   xbar_k = sum_j (dQ/dr)^T (m_k g_j - m_j g_k)      (likewise v, a, jr)
//   mbar_k = -sum_j Q . g_j.
// (dQ/d.)^T is applied by the hand reversal of the forward pair code:
// the forward values of R^-3, alpha, beta, gamma, w, u, z are recomputed,
// then their adjoints are accumulated in reverse order. The self pair
// (whose terms cancel in exact arithmetic) is excluded explicitly.
//
// Over all pairs the VJP of a pair is taken once for both particles: swapping
// k and j changes the sign of r, v, a, jr and of m_k g_j - m_j g_k, so the
// gradient terms of j are those of k with the opposite sign; only the mass
// terms differ (Q . g_j for k, Q . g_k for j).
//
#include <algorithm>
#include <type_traits>

#include "device_math.h"
#include "sym_body.h"

namespace h6 {
namespace {

using namespace symbody;

template <int ORDER>
struct VTraits;
template <>  // start-up pass 1: outputs A, J; inputs x, v
struct VTraits<1> {
    static constexpr int NG = 6;    // output cotangent components
    static constexpr int NOUT = 7;  // xbar 3, vbar 3, mbar
    static constexpr int NF = 13;   // source record: x 3, v 3, m, g 6
};
template <>  // per step: outputs A, J, S; inputs x, v, a
struct VTraits<2> {
    static constexpr int NG = 9;
    static constexpr int NOUT = 10;  // xbar, vbar, abar, mbar
    static constexpr int NF = 19;    // x, v, a, m, g 9
};
template <>  // start-up pass 2: outputs S, C; inputs x, v, a, j
struct VTraits<3> {
    static constexpr int NG = 6;
    static constexpr int NOUT = 13;  // xbar, vbar, abar, jbar, mbar
    static constexpr int NF = 19;    // x, v, a, j, m, g 6
};

__device__ __forceinline__ double dot3(const double *p, const double *q) {
    return fma(p[2], q[2], fma(p[1], q[1], p[0] * q[0]));
}

// Reverse-mode pair of the start-up passes (orders 1 and 3): T = (dQ/dr)^T gh,
// (dQ/dv)^T gh, ... (3 components each, in the order x, v, a, jr), and the mass
// terms qj = Q . gj and qk = Q . gk.
template <int ORDER>
__device__ __forceinline__ void pair_vjp(const double *r, const double *v, const double *a,
                                         const double *jr, double r2, double mk, double mj,
                                         const double *gj, const double *gk, double *T, double &qj,
                                         double &qk) {
    constexpr int NG = VTraits<ORDER>::NG;
    double gh[NG];
#pragma unroll
    for (int p = 0; p < NG; ++p) gh[p] = fma(mk, gj[p], -mj * gk[p]);
    // ---- forward values
    const double rho = rsqrt_f64(r2);
    const double rho2 = rho * rho;
    const double q3 = rho * rho2;  // R^-3
    const double rv = dot3(r, v);
    const double alpha = rv * rho2;
    double w[3], u[3] = {0, 0, 0}, z[3] = {0, 0, 0};
#pragma unroll
    for (int c = 0; c < 3; ++c) w[c] = fma(-3.0 * alpha, r[c], v[c]);
    double vvra = 0, beta = 0, va = 0, rj = 0, gamma = 0;
    if constexpr (ORDER >= 2) {
        vvra = fma(v[2], v[2], fma(v[1], v[1], v[0] * v[0])) + dot3(r, a);
        beta = fma(alpha, alpha, vvra * rho2);
#pragma unroll
        for (int c = 0; c < 3; ++c) u[c] = fma(-6.0 * alpha, w[c], fma(-3.0 * beta, r[c], a[c]));
    }
    if constexpr (ORDER == 3) {
        va = dot3(v, a);
        rj = dot3(r, jr);
        gamma = fma(alpha, fma(-4.0 * alpha, alpha, 3.0 * beta), fma(3.0, va, rj) * rho2);
#pragma unroll
        for (int c = 0; c < 3; ++c)
            z[c] = fma(-9.0 * alpha, u[c], fma(-9.0 * beta, w[c], fma(-3.0 * gamma, r[c], jr[c])));
    }
    // ---- cotangent layout of the outputs
    const double zero3[3] = {0, 0, 0};
    const double *Ab = ORDER == 3 ? zero3 : gh;
    const double *Jb = ORDER == 3 ? zero3 : gh + 3;
    const double *Sb = ORDER == 3 ? gh : zero3;
    const double *Cb = ORDER == 3 ? gh + 3 : zero3;
    // mass: Q . g with Q = R^-3 (r, w, u, z) for (A, J, S, C)
    if constexpr (ORDER == 3) {
        qj = q3 * (dot3(u, gj) + dot3(z, gj + 3));
        qk = q3 * (dot3(u, gk) + dot3(z, gk + 3));
    } else {
        qj = q3 * (dot3(r, gj) + dot3(w, gj + 3));
        qk = q3 * (dot3(r, gk) + dot3(w, gk + 3));
    }
    // ---- reverse sweep
    double q3b = dot3(Ab, r) + dot3(Jb, w);
    if constexpr (ORDER >= 2) q3b += dot3(Sb, u);
    if constexpr (ORDER == 3) q3b += dot3(Cb, z);
    double rb[3], wb[3], ub[3], vbl[3] = {0, 0, 0}, abl[3] = {0, 0, 0}, jrb[3] = {0, 0, 0};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        rb[c] = q3 * Ab[c];
        wb[c] = q3 * Jb[c];
        ub[c] = q3 * Sb[c];
    }
    double alphab = 0, betab = 0, rho2b = 0;
    if constexpr (ORDER == 3) {
        double zb[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) zb[c] = q3 * Cb[c];
        // z = jr - 9 alpha u - 9 beta w - 3 gamma r
        const double gammab = -3.0 * dot3(r, zb);
        alphab = -9.0 * dot3(u, zb);
        betab = -9.0 * dot3(w, zb);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            jrb[c] = zb[c];
            ub[c] = fma(-9.0 * alpha, zb[c], ub[c]);
            wb[c] = fma(-9.0 * beta, zb[c], wb[c]);
            rb[c] = fma(-3.0 * gamma, zb[c], rb[c]);
        }
        // gamma = (3 v.a + r.jr) rho2 + alpha (3 beta - 4 alpha^2)
        const double gr = gammab * rho2;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            vbl[c] = fma(3.0 * gr, a[c], vbl[c]);
            abl[c] = fma(3.0 * gr, v[c], abl[c]);
            rb[c] = fma(gr, jr[c], rb[c]);
            jrb[c] = fma(gr, r[c], jrb[c]);
        }
        rho2b = gammab * fma(3.0, va, rj);
        alphab = fma(gammab, fma(-12.0 * alpha, alpha, 3.0 * beta), alphab);
        betab = fma(3.0 * alpha, gammab, betab);
    }
    if constexpr (ORDER >= 2) {
        // u = a - 6 alpha w - 3 beta r
        alphab = fma(-6.0, dot3(w, ub), alphab);
        betab = fma(-3.0, dot3(r, ub), betab);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            abl[c] += ub[c];
            wb[c] = fma(-6.0 * alpha, ub[c], wb[c]);
            rb[c] = fma(-3.0 * beta, ub[c], rb[c]);
        }
        // beta = (v.v + r.a) rho2 + alpha^2
        const double br = betab * rho2;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            vbl[c] = fma(2.0 * br, v[c], vbl[c]);
            rb[c] = fma(br, a[c], rb[c]);
            abl[c] = fma(br, r[c], abl[c]);
        }
        rho2b = fma(betab, vvra, rho2b);
        alphab = fma(2.0 * alpha, betab, alphab);
    }
    // w = v - 3 alpha r
    alphab = fma(-3.0, dot3(r, wb), alphab);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        vbl[c] += wb[c];
        rb[c] = fma(-3.0 * alpha, wb[c], rb[c]);
    }
    // alpha = (r.v) rho2
    const double ar = alphab * rho2;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        rb[c] = fma(ar, v[c], rb[c]);
        vbl[c] = fma(ar, r[c], vbl[c]);
    }
    rho2b = fma(alphab, rv, rho2b);
    // q3 = R2^(-3/2), rho2 = R2^(-1), R2 = r.r + eps^2
    const double r2b = -1.5 * q3b * q3 * rho2 - rho2b * rho2 * rho2;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        T[c] = fma(2.0 * r2b, r[c], rb[c]);
        T[3 + c] = vbl[c];
        if constexpr (ORDER >= 2) T[6 + c] = abl[c];
        if constexpr (ORDER == 3) T[9 + c] = jrb[c];
    }
}

constexpr double kPadPosVjp = 1.0e18;

struct CotPtrs {
    const double *g[9];
};



// Order-2 pair VJP, factored. With gh = m_k g_j - m_j g_k and
//   G(g)  = gA.r + gJ.w + gS.u
//         = gA.r + gJ.v - 3 alpha gJ.r + gS.a - 6 alpha gS.v + c18 gS.r,
//   c18   = 18 alpha^2 - 3 beta,
//   Ga(g) = -3 gJ.r - 6 gS.v + 30 alpha gS.r    (dG/dalpha, beta's alpha^2
//                                                included),
// the pair's contribution Q . gh = R^-3 G(gh) has the gradients
//   d/dr: R^-3 (gA - 3 alpha gJ + c18 gS) + sa v + sb a + cr r,
//   d/dv: R^-3 (gJ - 6 alpha gS) + sa r + 2 sb v,
//   d/da: R^-3 gS + sb r,
// with sa = R^-5 Ga(gh), sb = -3 R^-5 gS.r, cr = -3 R^-5 G(gh) - 2 alpha sa
// - 2 beta' sb, beta' = (v.v + r.a)/R^2. G, Ga and gS.r are linear in g, so
// they come from six dot products with each of g_j and g_k.
__device__ __forceinline__ void g_terms(const double *g, const double *r, const double *v,
                                        const double *a, double a3, double a6, double c18,
                                        double a30, double &G, double &Ga, double &dSr) {
    const double dAr = dot3(g, r), dJr = dot3(g + 3, r), dJv = dot3(g + 3, v);
    dSr = dot3(g + 6, r);
    const double dSv = dot3(g + 6, v), dSa = dot3(g + 6, a);
    G = fma(c18, dSr, fma(-a6, dSv, fma(-a3, dJr, dAr + dJv) + dSa));
    Ga = fma(a30, dSr, fma(-6.0, dSv, -3.0 * dJr));
}

// The pair's gradient terms T (x, v, a) and the mass terms qj = R^-3 G(g_j),
// qk = R^-3 G(g_k); with GK false g_k is zero (gh = m_k g_j, no qk).
template <bool GK>
__device__ __forceinline__ void pair_vjp2(const double *r, const double *v, const double *a,
                                          double r2, double mk, double mj, const double *gj,
                                          const double *gk, double *T, double &qj, double &qk) {
    const double rho = rsqrt_f64(r2);
    const double rho2 = rho * rho;
    const double q3 = rho * rho2;
    const double alpha = dot3(r, v) * rho2;
    const double bp = (fma(v[2], v[2], fma(v[1], v[1], v[0] * v[0])) + dot3(r, a)) * rho2;
    const double beta = fma(alpha, alpha, bp);
    const double a3 = 3.0 * alpha;
    const double a6 = a3 + a3;
    const double c18 = fma(6.0 * a3, alpha, -3.0 * beta);
    const double a30 = 10.0 * a3;
    double Gj, Gaj, dSj;
    g_terms(gj, r, v, a, a3, a6, c18, a30, Gj, Gaj, dSj);
    qj = q3 * Gj;
    double G = mk * Gj, Ga = mk * Gaj, dS = mk * dSj;
    if constexpr (GK) {
        double Gk, Gak, dSk;
        g_terms(gk, r, v, a, a3, a6, c18, a30, Gk, Gak, dSk);
        qk = q3 * Gk;
        G = fma(-mj, Gk, G);
        Ga = fma(-mj, Gak, Ga);
        dS = fma(-mj, dSk, dS);
    }
    const double qr = q3 * rho2;
    const double sa = qr * Ga;
    const double sb = (-3.0 * qr) * dS;
    const double cr = fma(-3.0 * qr, G, fma(-2.0 * alpha, sa, (-2.0 * bp) * sb));
    const double sb2 = sb + sb;
    const double mkq = mk * q3, mjq = mj * q3;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double hA = mkq * gj[c], hJ = mkq * gj[3 + c], hS = mkq * gj[6 + c];  // R^-3 gh
        if constexpr (GK) {
            hA = fma(-mjq, gk[c], hA);
            hJ = fma(-mjq, gk[3 + c], hJ);
            hS = fma(-mjq, gk[6 + c], hS);
        }
        T[c] = fma(sa, v[c], fma(sb, a[c], fma(cr, r[c], fma(-a3, hJ, fma(c18, hS, hA)))));
        T[3 + c] = fma(sa, r[c], fma(sb2, v[c], fma(-a6, hS, hJ)));
        T[6 + c] = fma(sb, r[c], hS);
    }
}

// Particles and pairs of the all-pairs VJP for sym_body.h's walk: the pair's
// terms T are added to the target's sums and subtracted from the source's.
// Bound by FP64 issue: at order 2 194 operations an unordered pair (20 of them
// the DPP moves of ten sums), against 2 x 153 in ordered form. All pairs of
// n = 16384: 1432 -> 870 us; of 420001: 0.92 -> 0.59 s.
template <int ORDER>
struct VjpOps {
    using Word = double;
    using Sum = CompSum;
    static constexpr int NG = VTraits<ORDER>::NG, NF = VTraits<ORDER>::NF;
    static constexpr int NREC = (NF + 1) / 2;
    static constexpr int NI = VTraits<ORDER>::NOUT, NJ = NI, K = 1, kUnroll = 1;
    static constexpr int kG = NF - NG;  // first cotangent word
    struct Target {
        double x[3], v[3], a[3], j[3], m, g[NG];
    };
    SrcPtrs src;
    CotPtrs cot;
    double eps2;
    // record order x0 x1 x2 m v0 v1 v2 (a.. (j..)) g..
    __device__ __forceinline__ const double *field(int f) const {
        return f < 3    ? src.x[f]
               : f == 3  ? src.m
               : f < 7   ? src.v[f - 4]
               : f >= kG ? cot.g[f - kG]
               : f < 10  ? src.a[f - 7]
                         : src.j[f - 10];
    }
    static __device__ __forceinline__ double word(double x) { return x; }
    static __device__ __forceinline__ double pad(int f) { return f < 3 ? kPadPosVjp : 0.0; }
    __device__ __forceinline__ void load(int k, int n, Target &t) const {
        const bool in = k < n;
        const int kc = in ? k : n - 1;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            t.x[c] = in ? src.x[c][kc] : -kPadPosVjp;
            t.v[c] = src.v[c][kc];
            if constexpr (ORDER >= 2) t.a[c] = src.a[c][kc];
            if constexpr (ORDER == 3) t.j[c] = src.j[c][kc];
        }
        t.m = in ? src.m[kc] : 0.0;
#pragma unroll
        for (int q = 0; q < NG; ++q) t.g[q] = in ? cot.g[q][kc] : 0.0;
    }
    // self: the self pair is left out explicitly: m_k g_k - m_k g_k is not
    // exactly zero once the first product is fused (fma keeps its rounding
    // error), and dQ/dr at r = 0 is of order eps^-3. With both masses zero gh
    // is exactly zero; r, v, a, jr are zero there, so Q and the mass term are
    // too (R^2 set to 1 keeps them finite when eps = 0).
    __device__ __forceinline__ void terms(const Word2<double> *e, const Target &t, bool self,
                                          double *T, double &qj, double &qk) const {
        auto f = [&](int q) { return q & 1 ? e[q >> 1].y : e[q >> 1].x; };
        double r[3], v[3], a[3] = {0, 0, 0}, jr[3] = {0, 0, 0}, gj[NG];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            r[c] = f(c) - t.x[c];
            v[c] = f(4 + c) - t.v[c];
            if constexpr (ORDER >= 2) a[c] = f(7 + c) - t.a[c];
            if constexpr (ORDER == 3) jr[c] = f(10 + c) - t.j[c];
        }
#pragma unroll
        for (int q = 0; q < NG; ++q) gj[q] = f(kG + q);
        double r2 = fma(r[2], r[2], fma(r[1], r[1], fma(r[0], r[0], eps2)));
        r2 = self ? 1.0 : r2;
        const double mj = self ? 0.0 : f(3), mk = self ? 0.0 : t.m;
        if constexpr (ORDER == 2)
            pair_vjp2<true>(r, v, a, r2, mk, mj, gj, t.g, T, qj, qk);
        else
            pair_vjp<ORDER>(r, v, a, jr, r2, mk, mj, gj, t.g, T, qj, qk);
    }
    __device__ __forceinline__ void both(const Word2<double> *e, const Target &t, double *acci,
                                         double *accj) const {
        double T[NI - 1], qj, qk;
        terms(e, t, false, T, qj, qk);
#pragma unroll
        for (int q = 0; q < NI - 1; ++q) {
            acci[q] += T[q];
            accj[q] -= T[q];
        }
        acci[NI - 1] -= qj;
        accj[NI - 1] += qk;
    }
    __device__ __forceinline__ void one(const Word2<double> *e, const Target &t, bool self,
                                        double *acci) const {
        double T[NI - 1], qj, qk;
        terms(e, t, self, T, qj, qk);
#pragma unroll
        for (int q = 0; q < NI - 1; ++q) acci[q] += T[q];
        acci[NI - 1] -= qj;
    }
    static __device__ __forceinline__ void add(Sum &s, double x) { two_sum_into(s.hi, s.lo, x); }
    static __device__ __forceinline__ double value(const Sum &s) { return s.hi + s.lo; }
    static __device__ __forceinline__ double value(double x) { return x; }
};

template <int ORDER>
__global__ __launch_bounds__(kSymThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_vjp_sym(
    SrcPtrs src, CotPtrs cot, SymPlan P, double eps2, double *__restrict__ partial) {
    sym_run(VjpOps<ORDER>{src, cot, eps2}, P, partial);
}

// ---------------------------------------------------------------- active sets
// VJP of the evaluation of an active set (block steps): the cotangents g are
// nonzero only on the active particles j, so the pair (k, j), k any particle
// and j an active one, has gh = m_k g_j. Its terms go to k with one sign and
// to j with the other, and the mass term -Q . g_j to k: every (k, j) pair is
// taken once (as two halves, the pairs of each active particle as source and
// as target, it was visited twice).
//
// A wave holds 64 particles k, one a lane; chunks of R active particles go
// round the lanes as in sym_body.h, in rings of R lanes (R = 4 or 16 for small
// blocks: a chunk of 64 would be mostly padding). The four waves of a
// workgroup take four tiles of k (WK = 4), or for small blocks the four
// quarters of a chunk's steps on one tile (WK = 1), so that the n / 64 tiles
// of a small system still fill the GPU. Workgroup (x, y) takes tile group x
// and the y-th part of the chunks. Sums of k are added to the outputs when
// one part covers all chunks, else they go through the partial sums, as the
// sums of j do (a slot per tile group; large lists in batches whose slots fit).
//
// Bound by latency for small blocks, by FP64 issue (150 operations a pair) for
// large ones. One h6_evaluate_vjp_active call, the two halves before and this:
// 4 active of 4096 190 -> 11 us, 300 of 4096 270 -> 26 us, 1000 of 16384 322 ->
// 111 us, 16000 of 65536 10.3 -> 5.8 ms.
constexpr int kActThreads = 256;

// The value of the next lane of a ring of R lanes.
template <int R>
__device__ __forceinline__ double ring_next(double v) {
    // wave rotate left by one; row rotate right by 15; quad permutation 1 2 3 0
    constexpr int kCtrl = R == 64 ? 0x134 : R == 16 ? 0x12F : 0x39;
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), kCtrl, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), kCtrl, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

template <int R, int WK>
__global__ __launch_bounds__(kActThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_vjp_active(
    SrcPtrs src, CotPtrs cot, int n, const int32_t *__restrict__ list, int n_act, double eps2,
    int part_chunks, double *__restrict__ part_j, double *__restrict__ part_k, OutPtrs out) {
    static_assert(R == 4 || R == 16 || R == 64, "ring of a quad, a row or a wave");
    constexpr int NW = 18;                            // words of a source: x, v, a, g
    constexpr int kSteps = WK == 4 ? R : R / 4;       // steps of a wave per chunk
    constexpr int NLOAD = (NW + 3) / 4;
    __shared__ double2 rec[NW / 2 * 2 * R];           // records twice over (no wrap)
    __shared__ double sums[4][10][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kt = ((int)blockIdx.x * WK + (WK == 4 ? wave : 0)) * 64;
    const int k = kt + lane, kc = k < n ? k : n - 1;
    const int sa = WK == 4 ? 0 : wave * kSteps, sb = sa + kSteps;
    // lane's place in its ring
    const int l = lane & (R - 1);
    double xk[3], vk[3], ak[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        xk[c] = k < n ? src.x[c][kc] : -kPadPosVjp;
        vk[c] = src.v[c][kc];
        ak[c] = src.a[c][kc];
    }
    const double mk = k < n ? src.m[kc] : 0.0;
    const double *field[NLOAD] = {};
    bool by_rank[NLOAD] = {};
#pragma unroll
    for (int f = 0; f < NW; ++f)
        if (f % 4 == wave) {
            field[f / 4] = f < 3 ? src.x[f] : f < 6 ? src.v[f - 3] : f < 9 ? src.a[f - 6] : cot.g[f - 9];
            by_rank[f / 4] = f >= 9;
        }
    double hi[10], lo[10];
#pragma unroll
    for (int q = 0; q < 10; ++q) hi[q] = lo[q] = 0.0;
    const int chunks = (n_act + R - 1) / R;
    const int c0 = (int)blockIdx.y * part_chunks, c1 = min(chunks, c0 + part_chunks);
    for (int c = c0; c < c1; ++c) {
        const int rank = c * R + l;
        const int id = rank < n_act ? list[rank] : -1;
        double *rd = reinterpret_cast<double *>(rec);
#pragma unroll
        for (int q = 0; q < NLOAD; ++q) {
            const int f = wave + 4 * q;
            if (f < NW && lane < R) {
                const double w = id < 0 ? (f < 3 ? kPadPosVjp : 0.0) : field[q][by_rank[q] ? rank : id];
                const int at = ((f >> 1) * 2 * R + lane) * 2 + (f & 1);
                rd[at] = w;
                rd[at + 2 * R] = w;
            }
        }
        __syncthreads();
        double acc[10], accj[9];
#pragma unroll
        for (int q = 0; q < 10; ++q) acc[q] = 0.0;
#pragma unroll
        for (int q = 0; q < 9; ++q) accj[q] = 0.0;
        auto steps = [&](auto test_self) {
            int idr = id;
            if constexpr (decltype(test_self)::value) {
                // the particle of step sa, one lane on each step
                idr = __shfl(id, (lane & ~(R - 1)) | ((l + sa) & (R - 1)), 64);
            }
#pragma unroll 1
            for (int s = sa; s < sb; ++s) {
                double f[NW];
#pragma unroll
                for (int q = 0; q < NW / 2; ++q) {
                    const double2 d = rec[q * 2 * R + l + s];
                    f[2 * q] = d.x;
                    f[2 * q + 1] = d.y;
                }
                double r[3], v[3], a[3], T[9], qj, qk;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    r[cc] = f[cc] - xk[cc];
                    v[cc] = f[3 + cc] - vk[cc];
                    a[cc] = f[6 + cc] - ak[cc];
                }
                double r2 = fma(r[2], r[2], fma(r[1], r[1], fma(r[0], r[0], eps2)));
                double m = mk;
                if constexpr (decltype(test_self)::value) {
                    // the self pair left out: a zero mass makes every term an
                    // exact zero (r, v, a vanish in qj)
                    const bool self = idr == k;
                    r2 = self ? 1.0 : r2;
                    m = self ? 0.0 : m;
                    idr = __shfl(idr, (lane & ~(R - 1)) | ((l + 1) & (R - 1)), 64);
                }
                pair_vjp2<false>(r, v, a, r2, m, 0.0, f + 9, nullptr, T, qj, qk);
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    acc[q] += T[q];
                    accj[q] = ring_next<R>(accj[q] - T[q]);
                }
                acc[9] -= qj;
            }
        };
        if (__any(id >= kt && id < kt + 64))
            steps(std::true_type{});
        else
            steps(std::false_type{});
#pragma unroll
        for (int q = 0; q < 10; ++q) two_sum_into(hi[q], lo[q], acc[q]);
#pragma unroll
        for (int q = 0; q < 9; ++q) sums[wave][q][(lane & ~(R - 1)) | ((l + sb) & (R - 1))] = accj[q];
        __syncthreads();
        // the chunk's sums over the waves and rings, in order
        for (int e = tid; e < 9 * R; e += kActThreads) {
            const int q = e / R, i = e % R;
            double hs = 0.0, hc = 0.0;
#pragma unroll
            for (int w = 0; w < 4; ++w)
#pragma unroll
                for (int g = 0; g < 64 / R; ++g) two_sum_into(hs, hc, sums[w][q][g * R + i]);
            if (c * R + i < n_act)
                part_j[((int64_t)blockIdx.x * 9 + q) * n_act + c * R + i] = hs + hc;
        }
    }
    auto put = [&](int q, int kk, double val) {
        if (part_k)
            part_k[((int64_t)blockIdx.y * 10 + q) * n + kk] = val;
        else
            out.p[q][kk] += val;
    };
    if constexpr (WK == 4) {
        if (k < n)
#pragma unroll
            for (int q = 0; q < 10; ++q) put(q, k, hi[q] + lo[q]);
    } else {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 10; ++q) sums[wave][q][lane] = hi[q] + lo[q];
        __syncthreads();
        for (int e = tid; e < 640; e += kActThreads) {
            const int q = e / 64, i = e % 64;
            double hs = 0.0, hc = 0.0;
#pragma unroll
            for (int w = 0; w < 4; ++w) two_sum_into(hs, hc, sums[w][q][i]);
            if (kt + i < n) put(q, kt + i, hs + hc);
        }
    }
}

// Transpose of the shared-step corrector. Forward (step h, per component):
//   v1 = v + h/2 (a + A1) - h^2/10 (J1 - j) + h^3/120 (s + S1)
//   x1 = x + h/2 (v + v1) - h^2/10 (A1 - a) + h^3/120 (j + J1)
//   c1 = [60 (A1 - a) - h (24 j + 36 J1) + h^2 (9 S1 - 3 s)] / h^3
//   a1 = A1, j1 = J1, s1 = S1.
// In: cotangents of (x1, v1, a1, j1, s1, c1) in cot. Out: cotangents of the
// old (x, v, a, j, s) in cot (c's set to zero: the old crackle enters only
// the predictor), and of the evaluated (A1, J1, S1) in cf.
__global__ __launch_bounds__(256) void k_correct_shared_vjp(h6_state cot, int n, h6_force cf,
                                                            double h) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double h2 = h * h, h3 = h2 * h;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double X = cot.x[c][i], V = cot.v[c][i], Ab = cot.a[c][i];
        const double Jb = cot.j[c][i], Sb = cot.s[c][i], Cb = cot.c[c][i];
        const double V1 = fma(0.5 * h, X, V);  // cotangent of v1 (x1 depends on it)
        const double xo = X;
        const double vo = fma(0.5 * h, X, V1);
        const double ao = fma(0.1 * h2, X, fma(0.5 * h, V1, -60.0 / h3 * Cb));
        const double jo = fma(h3 / 120.0, X, fma(0.1 * h2, V1, -24.0 / h2 * Cb));
        const double so = fma(h3 / 120.0, V1, -3.0 / h * Cb);
        const double A1 = Ab + fma(-0.1 * h2, X, fma(0.5 * h, V1, 60.0 / h3 * Cb));
        const double J1 = Jb + fma(h3 / 120.0, X, fma(-0.1 * h2, V1, -36.0 / h2 * Cb));
        const double S1 = Sb + fma(h3 / 120.0, V1, 9.0 / h * Cb);
        cot.x[c][i] = xo;
        cot.v[c][i] = vo;
        cot.a[c][i] = ao;
        cot.j[c][i] = jo;
        cot.s[c][i] = so;
        cot.c[c][i] = 0.0;
        cf.a[c][i] = A1;
        cf.j[c][i] = J1;
        cf.s[c][i] = S1;
    }
}

// Transpose of the shared-step predictor (Taylor series over h), added to
// the state cotangents:
//   xbar += xpb; vbar += h xpb + vpb; abar += h^2/2 xpb + h vpb + apb;
//   jbar += h^3/6 xpb + h^2/2 vpb + h apb; sbar += h^4/24 xpb + h^3/6 vpb
//   + h^2/2 apb; cbar += h^5/120 xpb + h^4/24 vpb + h^3/6 apb.
__global__ __launch_bounds__(256) void k_predict_dt_vjp(h6_state cot, int n, h6_pred cp, double h) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double h2 = h * h, h3 = h2 * h, h4 = h3 * h, h5 = h4 * h;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double X = cp.x[c][i], V = cp.v[c][i], A = cp.a[c][i];
        cot.x[c][i] += X;
        cot.v[c][i] += fma(h, X, V);
        cot.a[c][i] += fma(0.5 * h2, X, fma(h, V, A));
        cot.j[c][i] += fma(h3 / 6.0, X, fma(0.5 * h2, V, h * A));
        cot.s[c][i] += fma(h4 / 24.0, X, fma(h3 / 6.0, V, 0.5 * h2 * A));
        cot.c[c][i] += fma(h5 / 120.0, X, fma(h4 / 24.0, V, h3 / 6.0 * A));
    }
}

int ceil_div_i(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// VJP of the sums over all pairs, each unordered pair once; in ordered form
// where the partial sums hold too few slots for that.
template <int ORDER>
hipError_t launch_vjp_order(h6_ctx ctx, const SrcPtrs &src, const CotPtrs &cot, int n,
                            const OutPtrs &out, unsigned acc_mask) {
    constexpr int NOUT = VTraits<ORDER>::NOUT, kBlock = kSymThreads * VjpOps<ORDER>::K;
    auto launch = [&](const SymPlan &P) {
        hipLaunchKernelGGL((k_vjp_sym<ORDER>), dim3(P.runs), dim3(kSymThreads), 0, ctx->stream, src,
                           cot, P, ctx->eps2, ctx->partial);
        return hipGetLastError();
    };
    bool done = false;
    hipError_t e = sym_batches(ctx, n, kBlock, NOUT, SymCost{48.0f, 3.0f}, 0, out, acc_mask, &done, launch);
    if (e != hipSuccess || done) return e;
    SymPlan P;
    for (int d = 0; e == hipSuccess && (d == 0 || d < P.nsb); d = P.d1) {
        P = sym_plan_ordered(n, kBlock, d);
        e = launch(P);
        if (e == hipSuccess) e = launch_sym_reduce(ctx, P, NOUT, 0, out, d > 0 ? (1u << NOUT) - 1u : acc_mask);
    }
    return e;
}

// Transpose of the block-step corrector for the active particles, each over
// its own step (dt_old, ticks): the shared-step transpose with h per
// particle; cf by rank.
__global__ __launch_bounds__(256) void k_correct_block_vjp(h6_state cot,
                                                           const int32_t *__restrict__ active,
                                                           int n_act,
                                                           const int64_t *__restrict__ dt_old,
                                                           h6_force cf) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_act) return;
    const int i = active[k];
    const double h = (double)dt_old[i] * (1.0 / (double)((int64_t)1 << kTickBits));
    const double h2 = h * h, h3 = h2 * h;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double X = cot.x[c][i], V = cot.v[c][i], Ab = cot.a[c][i];
        const double Jb = cot.j[c][i], Sb = cot.s[c][i], Cb = cot.c[c][i];
        const double V1 = fma(0.5 * h, X, V);
        cot.x[c][i] = X;
        cot.v[c][i] = fma(0.5 * h, X, V1);
        cot.a[c][i] = fma(0.1 * h2, X, fma(0.5 * h, V1, -60.0 / h3 * Cb));
        cot.j[c][i] = fma(h3 / 120.0, X, fma(0.1 * h2, V1, -24.0 / h2 * Cb));
        cot.s[c][i] = fma(h3 / 120.0, V1, -3.0 / h * Cb);
        cot.c[c][i] = 0.0;
        cf.a[c][k] = Ab + fma(-0.1 * h2, X, fma(0.5 * h, V1, 60.0 / h3 * Cb));
        cf.j[c][k] = Jb + fma(h3 / 120.0, X, fma(-0.1 * h2, V1, -36.0 / h2 * Cb));
        cf.s[c][k] = Sb + fma(h3 / 120.0, V1, 9.0 / h * Cb);
    }
}

// Transpose of the block-step predictor: the shared-step transpose with the
// interval of each particle, d = (t_tick - t_old[i]) ticks.
__global__ __launch_bounds__(256) void k_predict_block_vjp(h6_state cot, int n,
                                                           const int64_t *__restrict__ t_old,
                                                           int64_t t_tick, h6_pred cp) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double h = (double)(t_tick - t_old[i]) * (1.0 / (double)((int64_t)1 << kTickBits));
    const double h2 = h * h, h3 = h2 * h, h4 = h3 * h, h5 = h4 * h;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double X = cp.x[c][i], V = cp.v[c][i], A = cp.a[c][i];
        cot.x[c][i] += X;
        cot.v[c][i] += fma(h, X, V);
        cot.a[c][i] += fma(0.5 * h2, X, fma(h, V, A));
        cot.j[c][i] += fma(h3 / 6.0, X, fma(0.5 * h2, V, h * A));
        cot.s[c][i] += fma(h4 / 24.0, X, fma(h3 / 6.0, V, 0.5 * h2 * A));
        cot.c[c][i] += fma(h5 / 120.0, X, fma(h4 / 24.0, V, h3 / 6.0 * A));
    }
}

// Potential of each particle, phi_i = -sum_{j != i} m_j / sqrt(r^2 + eps^2),
// and with GRAD the gradient of the total energy E = sum_i m_i |v_i|^2 / 2 -
// sum_{i<j} m_i m_j (r_ij^2 + eps^2)^(-1/2) scaled by its cotangent g (one
// device double; NULL: 1): dE/dx_i = -m_i a_i with a_i the softened
// acceleration, dE/dv_i = m_i v_i, dE/dm_i = |v_i|^2 / 2 + phi_i; phi and a
// share each pair's r^2 and 1/sqrt.
//
// Bound by FP64 issue (about 20 operations a pair). A workgroup of 512
// threads takes 2 TG targets, two a thread, with 512 / TG strands over the
// sources of each LDS tile, so that a small system fills the GPU (one target
// per thread over all sources left 192 of 256 CUs idle at n = 16384) and two
// pairs share an LDS record. The self test is made only in the tiles that
// hold targets of the group. With
// GRAD, n = 16384: 986 -> 205 us (24 TFLOP/s at 18 operations a pair, FMA 2).
constexpr int kPotThreads = 512;
constexpr int kPotPerSum = 16;  // strand sums one thread adds in the final reduction
template <int TG, bool GRAD>
__global__ __launch_bounds__(kPotThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_potential(
    h6_state st, int n, double eps2, const double *__restrict__ cot, double *__restrict__ phi,
    h6_state out) {
    constexpr int NACC = GRAD ? 4 : 1;  // phi, a
    constexpr int STR = kPotThreads / TG;
    constexpr int LD = STR + 1;
    constexpr int kTileLen = 2 * kPotThreads + 64;  // double2: (x, y), (z, m); the sums need a little more
    static_assert(NACC * TG * LD <= 2 * kTileLen, "strand sums fit the tile");
    __shared__ double2 tile[kTileLen];
    __shared__ double fs[2 * TG][NACC];
    const int tid = threadIdx.x, t = tid % TG, s = tid / TG;
    const int k0 = (int)blockIdx.x * 2 * TG;
    int id[2];
    double xi[2][3], acc[2][NACC], hi[2][NACC], lo[2][NACC];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int k = k0 + u * TG + t;
        id[u] = k < n ? k : n - 1;
#pragma unroll
        for (int c = 0; c < 3; ++c) xi[u][c] = st.x[c][id[u]];
#pragma unroll
        for (int q = 0; q < NACC; ++q) acc[u][q] = hi[u][q] = lo[u][q] = 0.0;
    }
    auto flush = [&]() {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < NACC; ++q) {
                two_sum_into(hi[u][q], lo[u][q], acc[u][q]);
                acc[u][q] = 0.0;
            }
    };
    int since = 0;
    for (int jt = 0; jt < n; jt += kPotThreads) {
        if (jt) __syncthreads();
        const int jj = jt + tid;
        const bool in = jj < n;
        tile[tid] = in ? make_double2(st.x[0][jj], st.x[1][jj]) : make_double2(kPadPosVjp, kPadPosVjp);
        tile[kPotThreads + tid] =
            in ? make_double2(st.x[2][jj], st.m[jj]) : make_double2(kPadPosVjp, 0.0);
        __syncthreads();
        const int steps = (min(kPotThreads, n - jt) + STR - 1) / STR;
        auto pairs = [&](auto test_self) {
#pragma unroll 2
            for (int i = 0; i < steps; ++i) {
                const int e = i * STR + s;
                const double2 xy = tile[e], zm = tile[kPotThreads + e];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const double dx = xy.x - xi[u][0], dy = xy.y - xi[u][1], dz = zm.x - xi[u][2];
                    double r2 = fma(dz, dz, fma(dy, dy, fma(dx, dx, eps2)));
                    double mj = zm.y;
                    if (decltype(test_self)::value) {
                        // (the padding too: a lone particle may be at infinity)
                        const bool none = jt + e == id[u] || jt + e >= n;
                        r2 = none ? 1.0 : r2;
                        mj = none ? 0.0 : mj;
                    }
                    const double rinv = rsqrt_f64(r2);
                    if constexpr (GRAD) {
                        const double mr = mj * rinv;
                        const double mr3 = mr * (rinv * rinv);
                        acc[u][0] += mr;
                        acc[u][1] = fma(mr3, dx, acc[u][1]);
                        acc[u][2] = fma(mr3, dy, acc[u][2]);
                        acc[u][3] = fma(mr3, dz, acc[u][3]);
                    } else {
                        acc[u][0] = fma(mj, rinv, acc[u][0]);
                    }
                }
            }
        };
        // targets past the end repeat particle n - 1
        if (jt < k0 + 2 * TG && (jt + kPotThreads > k0 || jt + kPotThreads >= n))
            pairs(std::true_type{});
        else
            pairs(std::false_type{});
        since += TG;
        if (since >= 64) {
            since = 0;
            flush();
        }
    }
    flush();
    double *red = reinterpret_cast<double *>(tile);
    constexpr int G = STR / kPotPerSum;  // threads per sum
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NACC; ++q) red[(q * TG + t) * LD + s] = hi[u][q] + lo[u][q];
        __syncthreads();
        const int o = tid / G, gl = tid % G;
        const bool mine = o < NACC * TG;
        double hs = 0.0, hc = 0.0;
        if (mine) {
#pragma unroll
            for (int i = 0; i < kPotPerSum; ++i) two_sum_into(hs, hc, red[o * LD + gl + i * G]);
        }
        seg_comp_reduce_n<1>(&hs, &hc, G);
        if (mine && gl == G - 1) fs[u * TG + o % TG][o / TG] = hs + hc;
    }
    __syncthreads();
    const int i = k0 + tid;
    if (tid >= 2 * TG || i >= n) return;
    if constexpr (GRAD) {
        const double g = cot ? *cot : 1.0;
        const double mi = st.m[i];
        double vv = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double vc = st.v[c][i];
            vv = fma(vc, vc, vv);
            out.x[c][i] = -g * (mi * fs[tid][1 + c]);
            out.v[c][i] = g * (mi * vc);
        }
        out.m[i] = g * fma(0.5, vv, -fs[tid][0]);
    } else {
        phi[i] = -fs[tid][0];
    }
}

// Particles and pairs of the third-law form for sym_body.h's walk: sums m/R (the
// potential's negative) and, with GRAD, a. Bound by FP64 issue: 24 operations an
// unordered pair and 8 / K DPP moves, against 2 x 19 in ordered form. Ordered
// form and this, GRAD: n = 16384 205 -> 161 us, 65536 2819 -> 1903 us; potential
// alone: 141 -> 100 and 1962 -> 1212 us. With GRAD four targets a lane (16384
// with two 165 us, 65536 2182 us), without two (105 and 1114 us with four).
template <bool GRAD>
struct PotOps {
    using Word = double;
    using Sum = CompSum;
    static constexpr int NF = 4, NREC = 2, NI = GRAD ? 4 : 1, NJ = NI, K = GRAD ? 4 : 2, kUnroll = 2;
    struct Target {
        double x[3], m;
    };
    h6_state st;
    double eps2;
    __device__ __forceinline__ const double *field(int f) const { return f < 3 ? st.x[f] : st.m; }
    static __device__ __forceinline__ double word(double x) { return x; }
    static __device__ __forceinline__ double pad(int f) { return f < 3 ? kPadPosVjp : 0.0; }
    __device__ __forceinline__ void load(int k, int n, Target &t) const {
        const bool in = k < n;
        const int kc = in ? k : n - 1;
#pragma unroll
        for (int c = 0; c < 3; ++c) t.x[c] = in ? st.x[c][kc] : -kPadPosVjp;
        t.m = in ? st.m[kc] : 0.0;
    }
    template <bool BOTH>
    __device__ __forceinline__ void terms(const Word2<double> *e, const Target &t, bool self,
                                          double *acci, double *accj) const {
        const double r[3] = {e[0].x - t.x[0], e[0].y - t.x[1], e[1].x - t.x[2]};
        double r2 = fma(r[2], r[2], fma(r[1], r[1], fma(r[0], r[0], eps2)));
        double mj = e[1].y;
        if (!BOTH) {
            r2 = self ? 1.0 : r2;
            mj = self ? 0.0 : mj;
        }
        const double rinv = rsqrt_f64(r2);
        if constexpr (GRAD) {
            const double rinv2 = rinv * rinv;
            const double pj = mj * rinv, fj = pj * rinv2;
            acci[0] += pj;
#pragma unroll
            for (int c = 0; c < 3; ++c) acci[1 + c] = fma(fj, r[c], acci[1 + c]);
            if (BOTH) {
                const double pi = t.m * rinv, fi = pi * rinv2;
                accj[0] += pi;
#pragma unroll
                for (int c = 0; c < 3; ++c) accj[1 + c] = fma(-fi, r[c], accj[1 + c]);
            }
        } else {
            acci[0] = fma(mj, rinv, acci[0]);
            if (BOTH) accj[0] = fma(t.m, rinv, accj[0]);
        }
    }
    __device__ __forceinline__ void both(const Word2<double> *e, const Target &t, double *acci,
                                         double *accj) const {
        terms<true>(e, t, false, acci, accj);
    }
    __device__ __forceinline__ void one(const Word2<double> *e, const Target &t, bool self,
                                        double *acci) const {
        terms<false>(e, t, self, acci, nullptr);
    }
    static __device__ __forceinline__ void add(Sum &s, double x) { two_sum_into(s.hi, s.lo, x); }
    static __device__ __forceinline__ double value(const Sum &s) { return s.hi + s.lo; }
    static __device__ __forceinline__ double value(double x) { return x; }
};

template <bool GRAD>
__global__ __launch_bounds__(kSymThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_pot_sym(
    h6_state st, SymPlan P, double eps2, double *__restrict__ partial) {
    sym_run(PotOps<GRAD>{st, eps2}, P, partial);
}

// The slots' sums and, with GRAD, the gradient's components from them: one sum
// of one particle per thread.
template <bool GRAD>
__global__ __launch_bounds__(256) void k_pot_sums(const double *__restrict__ partial, SymPlan P,
                                                  h6_state st, const double *__restrict__ cot,
                                                  double *__restrict__ phi, h6_state out) {
    const int n = P.n;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)PotOps<GRAD>::NI * n) return;
    const int q = (int)(idx / n), i = (int)(idx - (int64_t)q * n);
    double s;
    sym_sums<1>(partial, P, PotOps<GRAD>::NI, q, i, &s);
    if constexpr (GRAD) {
        const double g = cot ? *cot : 1.0;
        if (q == 0) {
            double vv = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) vv = fma(st.v[c][i], st.v[c][i], vv);
            out.m[i] = g * fma(0.5, vv, -s);
        } else {
            const int c = q - 1;
            const double mi = st.m[i];
            out.x[c][i] = -g * (mi * s);
            out.v[c][i] = g * (mi * st.v[c][i]);
        }
    } else {
        phi[i] = -s;
    }
}

// From this size on each pair once, where one batch of slots holds the sums: up to
// 91136 particles with GRAD, 137728 without (256 CUs, the scratch of a small
// context), ordered beyond. The ordered and the third-law form, us: GRAD n = 4096
// 23 and 34, 6000 48 and 47, 8192 67 and 64; potential 4096 18 and 22, 6000 33 and
// 30. Either side of the end: GRAD 90000 3520, 95000 6000; potential 130000 4820,
// 140000 9190.
constexpr int kPotSymMin = 6000;

// Thread targets TG (a power of two): the rounds of workgroups a CU takes
// times the length of one, which per target is longer with few targets (more
// distinct LDS records a wave reads, kShare, measured at n = 65536 in units
// of TG = 16: 7212, 4759, 3562, 3063, 2790, 2710 us for TG 1 .. 32). The
// choice is the fastest TG at n = 1024 to 100000 (ten sizes), or within 3%.
template <bool GRAD>
hipError_t launch_pot(h6_ctx ctx, const h6_state *st, int n, const double *cot, double *phi,
                      h6_state *out) {
    static const float kShare[6] = {2.6f, 1.71f, 1.28f, 1.10f, 1.0f, 0.97f};
    const h6_state none = {};
    if (n >= kPotSymMin) {
        using Ops = PotOps<GRAD>;
        constexpr int kBlock = kSymThreads * Ops::K;
        SymPlan P;
        if (sym_plan(ctx, n, kBlock, Ops::NI, GRAD ? SymCost{28.0f, 3.0f} : SymCost{20.0f, 3.0f}, 0, &P) &&
            P.d1 == P.nsb / 2 + 1) {
            hipLaunchKernelGGL((k_pot_sym<GRAD>), dim3(P.runs), dim3(kSymThreads), 0, ctx->stream,
                               *st, P, ctx->eps2, ctx->partial);
            hipLaunchKernelGGL((k_pot_sums<GRAD>),
                               dim3((unsigned)(((int64_t)Ops::NI * n + 255) / 256)), dim3(256), 0,
                               ctx->stream, ctx->partial, P, *st, cot, phi, out ? *out : none);
            return hipGetLastError();
        }
    }
    int tg = 1;
    float best = 3.0e38f;
    for (int l = 0; l < 6; ++l) {
        const int rounds = ceil_div_i(ceil_div_i(n, 2 << l), ctx->n_cu);
        const float cost = (float)rounds * (float)(1 << l) * kShare[l] * (rounds == 1 ? 1.08f : 1.0f);
        if (cost < best) {
            best = cost;
            tg = 1 << l;
        }
    }
    const dim3 grid((n + 2 * tg - 1) / (2 * tg));
#define H6_POT(T)                                                                             \
    if (tg == T)                                                                              \
        hipLaunchKernelGGL((k_potential<T, GRAD>), grid, dim3(kPotThreads), 0, ctx->stream,   \
                           *st, n, ctx->eps2, cot, phi, out ? *out : none);
    H6_POT(1)
    H6_POT(2)
    H6_POT(4)
    H6_POT(8)
    H6_POT(16)
    H6_POT(32)
#undef H6_POT
    return hipGetLastError();
}

}  // namespace

hipError_t launch_energy_vjp(h6_ctx ctx, const h6_state *st, int n, const double *cot,
                             h6_state *out) {
    return launch_pot<true>(ctx, st, n, cot, nullptr, out);
}

hipError_t launch_eval_vjp(h6_ctx ctx, int order, const SrcPtrs &src, const double *const *cot,
                           int n, const OutPtrs &out, unsigned acc_mask) {
    CotPtrs cp;
    const int ng = order == 2 ? 9 : 6;
    for (int q = 0; q < 9; ++q) cp.g[q] = q < ng ? cot[q] : nullptr;
    if (order == 1) return launch_vjp_order<1>(ctx, src, cp, n, out, acc_mask);
    if (order == 2) return launch_vjp_order<2>(ctx, src, cp, n, out, acc_mask);
    return launch_vjp_order<3>(ctx, src, cp, n, out, acc_mask);
}

hipError_t launch_correct_shared_vjp(h6_ctx ctx, h6_state *cot, int n, const h6_force *cf,
                                     double dt) {
    hipLaunchKernelGGL(k_correct_shared_vjp, dim3((n + 255) / 256), dim3(256), 0, ctx->stream, *cot,
                       n, *cf, dt);
    return hipGetLastError();
}

hipError_t launch_predict_dt_vjp(h6_ctx ctx, h6_state *cot, int n, const h6_pred *cp, double dt) {
    hipLaunchKernelGGL(k_predict_dt_vjp, dim3((n + 255) / 256), dim3(256), 0, ctx->stream, *cot, n,
                       *cp, dt);
    return hipGetLastError();
}

hipError_t launch_eval_vjp_active(h6_ctx ctx, const SrcPtrs &src, const double *const *cot, int n,
                                  const int32_t *active, int n_act, const OutPtrs &out) {
    // ring: the least padding that does not multiply the chunks' fixed cost
    const int ring = n_act <= 4 ? 4 : n_act <= 48 ? 16 : 64;
    const int chunks = ceil_div_i(n_act, ring);
    const int64_t cu = ctx->n_cu;
    // four tiles a workgroup once they fill the GPU twice over
    const int wk = ring == 64 && (int64_t)ceil_div_i(n, 256) * chunks >= 4 * cu ? 4 : 1;
    const int groups = ceil_div_i(n, 64 * wk);
    // The active particles go in batches, each over all tile groups, whose sums
    // of j (a slot per group) fit the scratch: the list is cut, never the groups,
    // which fill the GPU (groups in batches left 8 workgroups to all of 262144
    // particles, 8.5 s; the list in batches 0.35 s). One part of a batch's chunks
    // per workgroup, or more parts to fill the GPU at the price of a reduction.
    // Times in us: a step 0.27 alone on its SIMD, 0.9 a chunk for staging and
    // sums, 5 a reduction and 1 per 3 MB it reads.
    const double tc = 0.27 * (wk == 4 ? ring : ring / 4) + 0.9;
    int parts = 1, batch = 0;  // chunks a batch
    double best = 1e300;
    for (int p = 1; p <= chunks && p <= 64; p *= 2) {
        const int64_t left = ctx->partial_cap - (p > 1 ? (int64_t)p * 10 * n : 0);
        const int64_t fit = left / ((int64_t)9 * groups * ring);
        if (fit < 1) break;
        const int bt = (int)std::min<int64_t>(chunks, fit);
        const double one = (double)ceil_div_i((int64_t)groups * p, cu) * ceil_div_i(bt, p) * tc + 5.0 +
                           2.4e-5 * groups * (double)bt * ring + (p > 1 ? 5.0 + 2.7e-5 * p * (double)n : 0.0);
        const double t = ceil_div_i(chunks, bt) * one;
        if (t < best) {
            best = t;
            parts = p;
            batch = bt;
        }
    }
    if (batch < 1) return hipErrorInvalidValue;  // not with the scratch of a context (9 n doubles for one chunk)
    for (int c0 = 0; c0 < chunks; c0 += batch) {
        const int a0 = c0 * ring, an = std::min(n_act - a0, batch * ring);
        const int32_t *list = active + a0;
        CotPtrs cp;
        for (int q = 0; q < 9; ++q) cp.g[q] = cot[q] + a0;
        const int bc = ceil_div_i(an, ring);
        const int part_chunks = ceil_div_i(bc, parts);
        const int bp = ceil_div_i(bc, part_chunks);
        double *part_k = bp > 1 ? ctx->partial : nullptr;
        double *part_j = ctx->partial + (bp > 1 ? (int64_t)bp * 10 * n : 0);
        const dim3 grid(groups, bp);
#define H6_ACT(R, W)                                                                            \
    if (ring == R && wk == W)                                                                   \
        hipLaunchKernelGGL((k_vjp_active<R, W>), grid, dim3(kActThreads), 0, ctx->stream, src,  \
                           cp, n, list, an, ctx->eps2, part_chunks, part_j, part_k, out);
        H6_ACT(4, 1)
        H6_ACT(16, 1)
        H6_ACT(64, 1)
        H6_ACT(64, 4)
#undef H6_ACT
        hipError_t e = hipGetLastError();
        // the sums of j, added to the active particles
        if (e == hipSuccess) e = launch_reduce(ctx, part_j, groups, 9, 0, an, out, 0x1ffu, list);
        if (e == hipSuccess && bp > 1) e = launch_reduce(ctx, part_k, bp, 10, 0, n, out, 0x3ffu, nullptr);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_correct_block_vjp(h6_ctx ctx, h6_state *cot, const int32_t *active, int n_act,
                                    const int64_t *dt_old, const h6_force *cf) {
    if (n_act <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_correct_block_vjp, dim3((n_act + 255) / 256), dim3(256), 0, ctx->stream,
                       *cot, active, n_act, dt_old, *cf);
    return hipGetLastError();
}

hipError_t launch_predict_block_vjp(h6_ctx ctx, h6_state *cot, int n, const int64_t *t_old,
                                    int64_t t_tick, const h6_pred *cp) {
    hipLaunchKernelGGL(k_predict_block_vjp, dim3((n + 255) / 256), dim3(256), 0, ctx->stream,
                       *cot, n, t_old, t_tick, *cp);
    return hipGetLastError();
}

hipError_t launch_potential(h6_ctx ctx, const h6_state *st, int n, double *phi) {
    return launch_pot<false>(ctx, st, n, nullptr, phi, nullptr);
}

}  // namespace h6
