// Extended-precision (EX) and single-precision (SP) evaluation of
// acceleration, jerk and snap (order 2).
//
// Sec. 3 item 6 of the paper lets the whole evaluation run in one of three
// arithmetics: IEEE double (DP), an extended type of about 48 significand
// bits with the single-precision exponent range (EX), or plain single
// precision (SP); its accuracy study compares the three by the drift of
// energy and angular momentum. These kernels are the EX and SP forms of the
// pair sum; the predictor, corrector and step rule stay FP64.
//
// EX is double-single ("float-float") arithmetic: a value is an unevaluated
// sum h + l of two floats with |l| <= ulp(h)/2, and every operation is built
// from error-free transformations of float operations:
//   TwoSum (Knuth): s = fl(a + b) and the exact error of that addition;
//   Fast2Sum (Dekker): the same when |a| >= |b|, in three operations;
//   TwoProd: p = fl(a b) and its exact error fma(a, b, -p).
// The differences of nearby coordinates use the accurate addition (TwoSum
// on both the high and the low parts, then two renormalisations), so that
// they keep their full double-single precision; the other sums (of
// products, and the accumulations) the sloppy one, whose operand-relative
// error is that of the terms it adds. Multiplication adds the two cross
// products into the error of the high product. The reciprocal square root
// starts from the hardware single-precision estimate and takes one
// third-order Newton step in double-single. Only float operations are used
// in the pair loop; FP64 inputs are split into (h, l) once when staged
// (h = fl32(x), l = fl32(x - h)) and the per-slice double-single sums leave
// the kernel as the exact double h + l. Contraction of a * b + c into one
// fused operation is switched off in the helpers: the error terms depend on
// each operation being rounded on its own.
//
// SP rounds the staged inputs to float and does every operation of the pair
// terms and the per-slice sums in float.
//
// EX runs in the FP64 evaluation's kernels with its own particles and pairs:
// all particles by the third law (sym_body.h), active sets by whole workgroups
// (eval_wg_body.h). Its sums are double-single within a slice: 64 sources of a
// strand, the steps of a cell, the targets a travelling source
// meets in a wave; slices are combined in FP64. SP keeps one target per lane
// over LDS tiles, its slices combined by the common FP64 reduction.
#include "eval_wg_body.h"

namespace h6 {
namespace {

using namespace evalbody;
using namespace symbody;

// ---------------------------------------------------------------- EX
struct fpair {
    float h, l;
};

__device__ __forceinline__ fpair two_sum(float a, float b) {
#pragma clang fp contract(off)
    const float s = a + b;
    const float bb = s - a;
    const float e = (a - (s - bb)) + (b - bb);
    return {s, e};
}

__device__ __forceinline__ fpair fast_two_sum(float a, float b) {  // needs |a| >= |b| or a == 0
#pragma clang fp contract(off)
    const float s = a + b;
    const float e = b - (s - a);
    return {s, e};
}

__device__ __forceinline__ fpair two_prod(float a, float b) {
#pragma clang fp contract(off)
    const float p = a * b;
    return {p, fmaf(a, b, -p)};
}

__device__ __forceinline__ fpair ds_add(fpair x, fpair y) {
#pragma clang fp contract(off)
    fpair s = two_sum(x.h, y.h);
    const fpair t = two_sum(x.l, y.l);
    s.l += t.h;
    s = fast_two_sum(s.h, s.l);
    s.l += t.l;
    return fast_two_sum(s.h, s.l);
}

// The sum without the error-free addition of the low parts (the "sloppy"
// form, 11 operations against 20): exact sum of the high parts, the low
// parts and its error added in float, renormalised. Its error is about
// 2u^2 (|x| + |y|), u = 2^-24: relative to the result when x and y have
// the same sign, to the operands' size when they cancel. The pair terms
// carry operand-relative errors of that size anyway (every product, sum of
// products and accumulation is rounded relative to its operands), so it is
// used for those; the differences of nearby coordinates, whose relative
// precision the pair terms need, keep the accurate form.
__device__ __forceinline__ fpair ds_add_sloppy(fpair x, fpair y) {
#pragma clang fp contract(off)
    fpair s = two_sum(x.h, y.h);
    s.l += x.l + y.l;
    return fast_two_sum(s.h, s.l);
}

__device__ __forceinline__ fpair ds_neg(fpair x) { return {-x.h, -x.l}; }

__device__ __forceinline__ fpair ds_sub_sloppy(fpair x, fpair y) {
    return ds_add_sloppy(x, ds_neg(y));
}

__device__ __forceinline__ fpair ds_sub(fpair x, fpair y) { return ds_add(x, ds_neg(y)); }

__device__ __forceinline__ fpair ds_add_f(fpair x, float b) {
#pragma clang fp contract(off)
    fpair s = two_sum(x.h, b);
    s.l += x.l;
    return fast_two_sum(s.h, s.l);
}

__device__ __forceinline__ fpair ds_mul(fpair x, fpair y) {
#pragma clang fp contract(off)
    fpair p = two_prod(x.h, y.h);
    p.l = fmaf(x.h, y.l, fmaf(x.l, y.h, p.l));
    return fast_two_sum(p.h, p.l);
}

// Products that only feed a sloppy sum skip the final renormalisation: the
// sum adds the low parts in float and renormalises itself, so a low part a
// few ulp of the high one larger costs nothing measurable.
__device__ __forceinline__ fpair ds_mul_raw(fpair x, fpair y) {
#pragma clang fp contract(off)
    fpair p = two_prod(x.h, y.h);
    p.l = fmaf(x.h, y.l, fmaf(x.l, y.h, p.l));
    return p;
}

__device__ __forceinline__ fpair ds_sqr_raw(fpair x) {
#pragma clang fp contract(off)
    fpair p = two_prod(x.h, x.h);
    p.l = fmaf(x.h + x.h, x.l, p.l);
    return p;
}

__device__ __forceinline__ fpair ds_mul_f(fpair x, float b) {
#pragma clang fp contract(off)
    fpair p = two_prod(x.h, b);
    p.l = fmaf(x.l, b, p.l);
    return fast_two_sum(p.h, p.l);
}

__device__ __forceinline__ fpair ds_sqr(fpair x) {
#pragma clang fp contract(off)
    fpair p = two_prod(x.h, x.h);
    p.l = fmaf(x.h + x.h, x.l, p.l);
    return fast_two_sum(p.h, p.l);
}

// x times a power of two: exact
__device__ __forceinline__ fpair ds_scale2(fpair x, float p2) { return {x.h * p2, x.l * p2}; }

__device__ __forceinline__ fpair ds_from(double d) {
    const float h = (float)d;
    return {h, (float)(d - (double)h)};
}

// 1/sqrt(r2): single-precision estimate y0 (relative error d of a few
// 2^-24), then y = y0 (1 + e/2 + 3 e^2/8) with e = 1 - r2 y0^2 formed in
// double-single; the step leaves a relative error of about (5/2) d^3, below
// the double-single rounding. e^2 needs only float precision (it is of
// order d^2).
__device__ __forceinline__ fpair ds_rsqrt(fpair r2) {
#pragma clang fp contract(off)
    const float y0 = __builtin_amdgcn_rsqf(r2.h);
    const fpair y2 = two_prod(y0, y0);
    const fpair e = ds_add_f(ds_neg(ds_mul(r2, y2)), 1.0f);
    const float e2 = e.h * e.h * 0.375f;
    const fpair p = ds_add_f(ds_scale2(e, 0.5f), e2);
    return ds_add_f(ds_mul_f(p, y0), y0);
}

__device__ __forceinline__ fpair ds_dot3(const fpair *p, const fpair *q) {
    return ds_add_sloppy(ds_add_sloppy(ds_mul_raw(p[0], q[0]), ds_mul_raw(p[1], q[1])),
                         ds_mul_raw(p[2], q[2]));
}

// The vectors of an order-2 pair in double-single: w, u, 1/R and 1/R^2, with
// R^2 = |r|^2 + eps^2, alpha = r.v/R^2, beta = (v.v + r.a)/R^2 + alpha^2,
// w = v - 3 alpha r, u = a - 6 alpha w - 3 beta r: A = m r/R^3, J = m w/R^3,
// S = m u/R^3.
__device__ __forceinline__ void pair_ex(const fpair *r, const fpair *v, const fpair *a, fpair r2,
                                        fpair *w, fpair *u, fpair &rinv, fpair &rinv2) {
    rinv = ds_rsqrt(r2);
    rinv2 = ds_sqr(rinv);
    const fpair alpha = ds_mul(ds_dot3(r, v), rinv2);
    const fpair a3 = ds_mul_f(alpha, 3.0f);
#pragma unroll
    for (int c = 0; c < 3; ++c) w[c] = ds_sub_sloppy(v[c], ds_mul_raw(a3, r[c]));
    const fpair vvra = ds_add_sloppy(ds_dot3(v, v), ds_dot3(r, a));
    const fpair beta = ds_add_sloppy(ds_sqr_raw(alpha), ds_mul_raw(vvra, rinv2));
    const fpair b3 = ds_mul_f(beta, 3.0f);
    const fpair a6 = ds_scale2(a3, 2.0f);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        u[c] = ds_sub_sloppy(ds_sub_sloppy(a[c], ds_mul_raw(a6, w[c])), ds_mul_raw(b3, r[c]));
}

// Far, massless padding source: contributes exactly zero.
constexpr float kPadPosF = 1.0e18f;

// Particles and pairs of the EX evaluation (sym_body.h, eval_wg_body.h).
// Bound by FP32 issue: about 720 operations for the terms of one particle and
// 160 more for both. All particles of n = 4096: 335 -> 200 us
// (155 registers: three waves per SIMD).
template <bool SKIPSELF>
struct ExOps {
    using Word = float2;  // high and low part
    using Acc = float2;
    static constexpr int kRun = 1, kMinTgt = 1, kDirectMaxTgt = 0;
    using Sum = CompSum;  // slices: FP64
    static constexpr int NF = 10, NREC = 5, NI = 9, NJ = 9, K = 1, kUnroll = 1;
    struct Target {
        fpair x[3], v[3], a[3], m;
    };
    SrcPtrs src;
    double eps2;
    // record order x0 x1 | x2 m | v0 v1 | v2 a0 | a1 a2
    __device__ __forceinline__ const double *field(int f) const {
        return f < 3 ? src.x[f] : f == 3 ? src.m : f < 7 ? src.v[f - 4] : src.a[f - 7];
    }
    static __device__ __forceinline__ float2 word(double d) {
        const fpair p = ds_from(d);
        return make_float2(p.h, p.l);
    }
    static __device__ __forceinline__ float2 pad(int f) {
        return make_float2(f < 3 ? kPadPosF : 0.0f, 0.0f);
    }
    __device__ __forceinline__ void load_rec(int jj, Word2<float2> *rec) const {
        rec_from_fields(*this, jj, rec);
    }
    static __device__ __forceinline__ void pad_rec(Word2<float2> *rec) { rec_padding<ExOps>(rec); }
    __device__ __forceinline__ void load(int k, int n, Target &t) const {
        const bool in = k < n;
        const int kc = in ? k : n - 1;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            t.x[c] = in ? ds_from(src.x[c][kc]) : fpair{-kPadPosF, 0.0f};
            t.v[c] = ds_from(src.v[c][kc]);
            t.a[c] = ds_from(src.a[c][kc]);
        }
        t.m = in ? ds_from(src.m[kc]) : fpair{0.0f, 0.0f};
    }
    // the pair's r, w, u, 1/R and 1/R^2
    __device__ __forceinline__ void pair(const Word2<float2> *e, const Target &t, bool self,
                                         fpair *r, fpair *w, fpair *u, fpair &mj, fpair &rinv,
                                         fpair &rinv2) const {
        auto f = [&](int q) {
            const float2 d = q & 1 ? e[q >> 1].y : e[q >> 1].x;
            return fpair{d.x, d.y};
        };
        fpair v[3], a[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            r[c] = ds_sub(f(c), t.x[c]);
            v[c] = ds_sub(f(4 + c), t.v[c]);
            a[c] = ds_sub(f(7 + c), t.a[c]);
        }
        fpair r2 = ds_add_sloppy(
            ds_add_sloppy(ds_add_sloppy(ds_from(eps2), ds_sqr_raw(r[0])), ds_sqr_raw(r[1])),
            ds_sqr_raw(r[2]));
        mj = f(3);
        if (self) {  // r, v, a are zero: mask the 1/0
            r2 = {1.0f, 0.0f};
            mj = {0.0f, 0.0f};
        }
        pair_ex(r, v, a, r2, w, u, rinv, rinv2);
    }
    // m / R^3, the mass first: R^-3 alone leaves the floats' range for R above
    // 2^34 (its low part) to 2^49 (all of it), where a large m keeps m / R and the
    // product within it (coordinates in metres, G m as masses). For both particles
    // of a pair one product more than with a common R^-3, under 1% of the pair's
    // operations.
    static __device__ __forceinline__ fpair m_r3(fpair m, fpair rinv, fpair rinv2) {
        return ds_mul(ds_mul(m, rinv), rinv2);
    }
    static __device__ __forceinline__ void accumulate(float2 *acc, fpair p, const fpair *r,
                                                      const fpair *w, const fpair *u) {
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const fpair x = q < 3 ? r[q] : q < 6 ? w[q - 3] : u[q - 6];
            const fpair s = ds_add_sloppy({acc[q].x, acc[q].y}, ds_mul_raw(p, x));
            acc[q] = make_float2(s.h, s.l);
        }
    }
    __device__ __forceinline__ void both(const Word2<float2> *e, const Target &t, float2 *acci,
                                         float2 *accj) const {
        fpair r[3], w[3], u[3], mj, rinv, rinv2;
        pair(e, t, false, r, w, u, mj, rinv, rinv2);
        accumulate(acci, m_r3(mj, rinv, rinv2), r, w, u);
        accumulate(accj, ds_neg(m_r3(t.m, rinv, rinv2)), r, w, u);
    }
    __device__ __forceinline__ void one(const Word2<float2> *e, const Target &t, bool self,
                                        float2 *acci) const {
        fpair r[3], w[3], u[3], mj, rinv, rinv2;
        pair(e, t, SKIPSELF && self, r, w, u, mj, rinv, rinv2);
        accumulate(acci, m_r3(mj, rinv, rinv2), r, w, u);
    }
    // the pair's ten numbers m/R^3, r, w, u as a chain adds them
    __device__ __forceinline__ void terms(const Word2<float2> *e, const Target &t, bool self,
                                          float2 *out) const {
        fpair r[3], w[3], u[3], mj, rinv, rinv2;
        pair(e, t, SKIPSELF && self, r, w, u, mj, rinv, rinv2);
        const fpair p = m_r3(mj, rinv, rinv2);
        out[0] = make_float2(p.h, p.l);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            out[1 + c] = make_float2(r[c].h, r[c].l);
            out[4 + c] = make_float2(w[c].h, w[c].l);
            out[7 + c] = make_float2(u[c].h, u[c].l);
        }
    }
    static __device__ __forceinline__ double value(float2 x) { return (double)x.x + (double)x.y; }
    static __device__ __forceinline__ void add(Sum &s, float2 x) {
        two_sum_into(s.hi, s.lo, value(x));
    }
    static __device__ __forceinline__ double value(const Sum &s) { return s.hi + s.lo; }
};

template <bool SKIPSELF>
__global__ __launch_bounds__(kSymThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_ex_sym(
    SrcPtrs src, SymPlan P, double eps2, double *__restrict__ partial) {
    sym_run(ExOps<SKIPSELF>{src, eps2}, P, partial);
}

// A target's sums over a slice as one serial chain of double-single additions,
// for shared steps: the interpolated crackle divides a difference of a by h^3 /
// 60, so that another order of these additions (1e-14 of a) shows in it, by more
// the fewer the particles. A workgroup takes one chain of 64 targets: of each 8
// sources every wave computes one's terms, which go to LDS, and then adds one or
// two of the nine components of all eight, in source order. Bound by FP32 issue,
// 740 operations a pair; one wave a chain, with the same additions, left three of
// four SIMDs idle at n = 1024 (256 chains), and one wave alone issues at 4.8
// clocks an operation. A shared step, one wave a chain and this: n = 256 92 -> 33
// us, 1024 96 -> 35, 2048 135 -> 76, 2999 290 -> 152. (Two sets of terms, so that a
// batch needs one barrier, leave one workgroup a CU: 1024 32, 2048 95 us.)
constexpr int kChainWaves = 8, kChainTile = 64;
template <bool SKIPSELF>
__global__ __launch_bounds__(64 * kChainWaves) void k_ex_chain(SrcPtrs src, int n, double eps2,
                                                               int slice_len, OutPtrs out,
                                                               int64_t slice_stride) {
    using Ops = ExOps<SKIPSELF>;
    const Ops ops{src, eps2};
    __shared__ Word2<float2> tile[2][kChainTile][Ops::NREC];
    __shared__ float2 terms[kChainWaves][10][64];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int k = (int)blockIdx.x * 64 + lane, kc = k < n ? k : n - 1;
    typename Ops::Target t;
    ops.load(kc, n, t);
    fpair acc[2] = {{0.0f, 0.0f}, {0.0f, 0.0f}};  // component w, and 8 (wave 7)
    const int jb = (int)blockIdx.y * slice_len, je = min(n, jb + slice_len);
    // word w (and 8 + w) of source lane of the tile at jt
    const double *f0 = nullptr, *f1 = nullptr;
#pragma unroll
    for (int f = 0; f < Ops::NF; ++f) {
        if (f == w) f0 = ops.field(f);
        if (f == w + 8) f1 = ops.field(f);
    }
    float2 pre[2];
    auto fetch = [&](int jt) {
        const int j = jt + lane;
        pre[0] = j < je ? Ops::word(f0[j]) : Ops::pad(w);
        if (f1) pre[1] = j < je ? Ops::word(f1[j]) : Ops::pad(w + 8);
    };
    auto stage = [&](int b) {
        float2 *rec = reinterpret_cast<float2 *>(&tile[b][lane][0]);
        rec[w] = pre[0];
        if (f1) rec[w + 8] = pre[1];
    };
    if (jb < je) {
        fetch(jb);
        stage(0);
    }
    __syncthreads();
    int buf = 0;
    for (int jt = jb; jt < je; jt += kChainTile, buf ^= 1) {
        const bool more = jt + kChainTile < je;
        if (more) fetch(jt + kChainTile);
#pragma unroll 1
        for (int b = 0; b < kChainTile / kChainWaves; ++b) {
            const int q = b * kChainWaves + w;
            float2 x[10];
            ops.terms(&tile[buf][q][0], t, jt + q == kc, x);
#pragma unroll
            for (int f = 0; f < 10; ++f) terms[w][f][lane] = x[f];
            if (more && b == kChainTile / kChainWaves - 1) stage(buf ^ 1);
            __syncthreads();
#pragma unroll
            for (int s = 0; s < kChainWaves; ++s) {
                const float2 p = terms[s][0][lane];
                auto add = [&](fpair &sum, int f) {
                    const float2 y = terms[s][f][lane];
                    sum = ds_add_sloppy(sum, ds_mul_raw({p.x, p.y}, {y.x, y.y}));
                };
                add(acc[0], 1 + w);
                if (w == 7) add(acc[1], 9);
            }
            __syncthreads();
        }
    }
    if (k < n) {
        const int64_t soff = (int64_t)blockIdx.y * slice_stride;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            if (q == w) out.p[q][soff + k] = (double)acc[0].h + (double)acc[0].l;
            if (q == 8 && w == 7) out.p[q][soff + k] = (double)acc[1].h + (double)acc[1].l;
        }
    }
}

// ---------------------------------------------------------------- SP
// Bound by FP32 issue (54 operations a pair). A target's sum over a slice is one
// serial chain, so a small set has about one chain a SIMD, and one wave alone
// issues an operation in 4.8 clocks where two take 3.05 each.
struct SpTarget {
    float x[3], v[3], a[3];
    int id;
};
// What a pair adds to its target: m / R^3 times r, w and u.
struct SpTerms {
    float m, r[3], w[3], u[3];
};

__device__ __forceinline__ SpTarget sp_target(const SrcPtrs &src, int p) {
    SpTarget t;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        t.x[c] = (float)src.x[c][p];
        t.v[c] = (float)src.v[c][p];
        t.a[c] = (float)src.a[c][p];
    }
    t.id = p;
    return t;
}

// LDS record of source jj: x, m, v, a as floats (plus padding), three float4;
// far, massless padding from je on.
struct SpSource {
    double x[3], v[3], a[3], m;
};
__device__ __forceinline__ SpSource sp_load(const SrcPtrs &src, int jj, int je) {
    SpSource s;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        s.x[c] = jj < je ? src.x[c][jj] : (double)kPadPosF;
        s.v[c] = jj < je ? src.v[c][jj] : 0.0;
        s.a[c] = jj < je ? src.a[c][jj] : 0.0;
    }
    s.m = jj < je ? src.m[jj] : 0.0;
    return s;
}
__device__ __forceinline__ void sp_store(const SpSource &s, float4 *rec) {
    rec[0] = make_float4((float)s.x[0], (float)s.x[1], (float)s.x[2], (float)s.m);
    rec[1] = make_float4((float)s.v[0], (float)s.v[1], (float)s.v[2], (float)s.a[0]);
    rec[2] = make_float4((float)s.a[1], (float)s.a[2], 0.0f, 0.0f);
}

template <bool SKIPSELF>
__device__ __forceinline__ SpTerms sp_pair(const float4 *rec, const SpTarget &t, float eps2,
                                           int j) {
    const float4 r0 = rec[0], r1 = rec[1], r2v = rec[2];
    const float dx = r0.x - t.x[0], dy = r0.y - t.x[1], dz = r0.z - t.x[2];
    const float dvx = r1.x - t.v[0], dvy = r1.y - t.v[1], dvz = r1.z - t.v[2];
    const float dax = r1.w - t.a[0], day = r2v.x - t.a[1], daz = r2v.y - t.a[2];
    float r2 = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, eps2)));
    float mj = r0.w;
    if (SKIPSELF && j == t.id) {
        r2 = 1.0f;
        mj = 0.0f;
    }
    // hardware estimate refined by one Newton step
    const float y0 = __builtin_amdgcn_rsqf(r2);
    const float rinv = y0 * fmaf(-0.5f * r2 * y0, y0, 1.5f);
    const float rinv2 = rinv * rinv;
    const float mr3 = mj * rinv * rinv2;
    const float alpha = fmaf(dz, dvz, fmaf(dy, dvy, dx * dvx)) * rinv2;
    const float a3 = 3.0f * alpha;
    const float wx = fmaf(-a3, dx, dvx), wy = fmaf(-a3, dy, dvy), wz = fmaf(-a3, dz, dvz);
    const float vvra =
        fmaf(dz, daz, fmaf(dy, day, fmaf(dx, dax, fmaf(dvz, dvz, fmaf(dvy, dvy, dvx * dvx)))));
    const float beta = fmaf(alpha, alpha, vvra * rinv2);
    const float b3 = 3.0f * beta, a6 = a3 + a3;
    return {mr3,
            {dx, dy, dz},
            {wx, wy, wz},
            {fmaf(-a6, wx, fmaf(-b3, dx, dax)), fmaf(-a6, wy, fmaf(-b3, dy, day)),
             fmaf(-a6, wz, fmaf(-b3, dz, daz))}};
}
__device__ __forceinline__ void sp_add(float *acc, const SpTerms &s) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        acc[c] = fmaf(s.m, s.r[c], acc[c]);
        acc[3 + c] = fmaf(s.m, s.w[c], acc[3 + c]);
        acc[6 + c] = fmaf(s.m, s.u[c], acc[6 + c]);
    }
}

template <int BLOCK, bool SKIPSELF>
__global__ __launch_bounds__(BLOCK) void k_eval_sp(SrcPtrs src, const int32_t *__restrict__ active,
                                                   int n, int n_act, double eps2_d, int slice_len,
                                                   OutPtrs out, int64_t slice_stride) {
    __shared__ float4 tile[BLOCK * 3];
    const int tid = threadIdx.x;
    const int k = (int)blockIdx.x * BLOCK + tid;
    const int kc = k < n_act ? k : n_act - 1;
    const SpTarget t = sp_target(src, active ? active[kc] : kc);
    const float eps2 = (float)eps2_d;
    float acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) acc[q] = 0.0f;

    const int jb = (int)blockIdx.y * slice_len;
    const int je = min(n, jb + slice_len);
    for (int jt = jb; jt < je; jt += BLOCK) {
        __syncthreads();
        sp_store(sp_load(src, jt + tid, je), &tile[tid * 3]);
        __syncthreads();
        // by four, so that a record's LDS reads overlap the previous pairs (the
        // lone wave of a small set waited for each: 2048 of 2048 targets 23.8
        // -> 14.5 us, 1000 of 10007 41.5 -> 30.8 us, 10007 of 10007 unchanged)
#pragma unroll 4
        for (int q = 0; q < BLOCK; ++q) sp_add(acc, sp_pair<SKIPSELF>(&tile[q * 3], t, eps2, jt + q));
    }
    if (k < n_act) {
        const int64_t soff = (int64_t)blockIdx.y * slice_stride;
#pragma unroll
        for (int q = 0; q < 9; ++q) out.p[q][soff + k] = (double)acc[q];
    }
}

// The same chains by two waves: of every 8 sources the first wave takes 4 from
// record to sum, and the other's four, whose terms come through LDS a batch
// later. The sums' operations and their order are the one-wave kernel's; 57
// issued a pair instead of 54, but by two waves, and the CUs' shares are even
// where 1099 lone waves on 1024 SIMDs were not. Bound by LDS now: 40 clocks of
// its reads and writes a source and chain, four or five chains a CU. One wave and
// this: n = 8192 142 -> 126 us, 10007 212 -> 191, 16384 509 -> 437, 65536 8.17 ->
// 6.45 ms (22 to 30 TFLOP/s at 42 operations a pair). Three or five of eight by
// the second wave: 10007 197 and 208 us; batches of four 199, of sixteen 271.
// While all chains are resident, six workgroups a CU: 1536 chains (n = 98304)
// 15.0 -> 13.4 ms, 2048 20.1 -> 27.6 ms.
constexpr int kSpPairPerCu = 6;
constexpr int kSpBatch = 8, kSpHalf = 4, kSpOwn = kSpBatch - kSpHalf, kSpTile = 64;
template <bool SKIPSELF>
__global__ __launch_bounds__(128) void k_eval_sp_pair(SrcPtrs src,
                                                      const int32_t *__restrict__ active, int n,
                                                      int n_act, double eps2_d, int slice_len,
                                                      OutPtrs out, int64_t slice_stride) {
    __shared__ float4 tile[2][kSpTile * 3];
    __shared__ float4 ring4[2][kSpHalf][2][64];  // m r | w u0
    __shared__ float2 ring2[2][kSpHalf][64];     // u1 u2
    const int lane = threadIdx.x & 63;
    const bool adds = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) == 0;
    const int k = (int)blockIdx.x * 64 + lane;
    const int kc = k < n_act ? k : n_act - 1;
    const SpTarget t = sp_target(src, active ? active[kc] : kc);
    const float eps2 = (float)eps2_d;
    float acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) acc[q] = 0.0f;
    const int jb = (int)blockIdx.y * slice_len;
    const int je = min(n, jb + slice_len);
    auto add_ring = [&](int par) {
#pragma unroll
        for (int q = 0; q < kSpHalf; ++q) {
            const float4 a = ring4[par][q][0][lane], b = ring4[par][q][1][lane];
            const float2 c = ring2[par][q][lane];
            sp_add(acc, {a.x, {a.y, a.z, a.w}, {b.x, b.y, b.z}, {b.w, c.x, c.y}});
        }
    };
    SpSource next;
    if (!adds && jb < je) sp_store(sp_load(src, jb + lane, je), &tile[0][lane * 3]);
    __syncthreads();
    int buf = 0;
    for (int jt = jb; jt < je; jt += kSpTile, buf ^= 1) {
        if (!adds && jt + kSpTile < je) next = sp_load(src, jt + kSpTile + lane, je);
#pragma unroll 2
        for (int b = 0; b < kSpTile / kSpBatch; ++b) {
            const int j0 = b * kSpBatch;
            if (adds) {
                if (b > 0 || jt > jb) add_ring((b + 1) & 1);
#pragma unroll
                for (int q = 0; q < kSpOwn; ++q)
                    sp_add(acc, sp_pair<SKIPSELF>(&tile[buf][(j0 + q) * 3], t, eps2, jt + j0 + q));
            } else {
#pragma unroll
                for (int q = 0; q < kSpHalf; ++q) {
                    const int j = j0 + kSpOwn + q;
                    const SpTerms s = sp_pair<SKIPSELF>(&tile[buf][j * 3], t, eps2, jt + j);
                    ring4[b & 1][q][0][lane] = make_float4(s.m, s.r[0], s.r[1], s.r[2]);
                    ring4[b & 1][q][1][lane] = make_float4(s.w[0], s.w[1], s.w[2], s.u[0]);
                    ring2[b & 1][q][lane] = make_float2(s.u[1], s.u[2]);
                }
                if (b == kSpTile / kSpBatch - 1 && jt + kSpTile < je)
                    sp_store(next, &tile[buf ^ 1][lane * 3]);
            }
            __syncthreads();
        }
    }
    if (adds) {
        if (jb < je) add_ring((kSpTile / kSpBatch - 1) & 1);
        if (k < n_act) {
            const int64_t soff = (int64_t)blockIdx.y * slice_stride;
#pragma unroll
            for (int q = 0; q < 9; ++q) out.p[q][soff + k] = (double)acc[q];
        }
    }
}

}  // namespace

void launch_ex_sym_pairs(h6_ctx ctx, const SrcPtrs &src, const SymPlan &P) {
    static_assert(ExOps<false>::K == 1, "superblocks of kSymThreads particles");
    if (self_pair_masked(ctx->eps2, H6_EX))
        hipLaunchKernelGGL((k_ex_sym<true>), dim3(P.runs), dim3(kSymThreads), 0, ctx->stream, src,
                           P, ctx->eps2, ctx->partial);
    else
        hipLaunchKernelGGL((k_ex_sym<false>), dim3(P.runs), dim3(kSymThreads), 0, ctx->stream, src,
                           P, ctx->eps2, ctx->partial);
}

hipError_t dispatch_ex_chain(bool skipself, dim3 grid, hipStream_t st, const SrcPtrs &src, int n,
                             double eps2, int slice_len, const OutPtrs &out, int64_t slice_stride) {
    auto launch = [&](auto skip) {
        hipLaunchKernelGGL((k_ex_chain<decltype(skip)::value>), grid, dim3(64 * kChainWaves), 0, st,
                           src, n, eps2, slice_len, out, slice_stride);
    };
    if (skipself) launch(std::true_type{}); else launch(std::false_type{});
    return hipGetLastError();
}

hipError_t dispatch_ex_wg(int tgt, bool skipself, dim3 grid, hipStream_t st, const SrcPtrs &src,
                          const int32_t *active, int n, int n_act, double eps2, int slice_len,
                          const OutPtrs &out, int64_t slice_stride) {
    return skipself ? launch_wg(tgt, grid, st, ExOps<true>{src, eps2}, active, n, n_act, slice_len,
                                0, out, slice_stride)
                    : launch_wg(tgt, grid, st, ExOps<false>{src, eps2}, active, n, n_act, slice_len,
                                0, out, slice_stride);
}

hipError_t dispatch_sp(int n_cu, bool skipself, dim3 grid, hipStream_t st, const SrcPtrs &src,
                       const int32_t *active, int n, int n_act, double eps2, int slice_len,
                       const OutPtrs &out, int64_t slice_stride) {
    auto launch = [&](auto skip) {
        constexpr bool S = decltype(skip)::value;
        if ((int64_t)grid.x * grid.y <= (int64_t)kSpPairPerCu * n_cu)
            hipLaunchKernelGGL((k_eval_sp_pair<S>), grid, dim3(128), 0, st, src, active, n, n_act,
                               eps2, slice_len, out, slice_stride);
        else
            hipLaunchKernelGGL((k_eval_sp<kSpBlock, S>), grid, dim3(kSpBlock), 0, st, src, active, n,
                               n_act, eps2, slice_len, out, slice_stride);
    };
    if (skipself) launch(std::true_type{}); else launch(std::false_type{});
    return hipGetLastError();
}

}  // namespace h6
