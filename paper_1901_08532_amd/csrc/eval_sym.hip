// Evaluation over all particles with each unordered pair taken once
// (sym_plan.h): the a, j, s terms of a pair serve both particles, by Newton's
// third law.
//
// A wave holds 2 x 64 targets in registers, two per lane. The sources of a
// chunk go round the lanes: at step s lane l takes source (l + s) mod 64, read
// from LDS, against its targets, and the source's sums, which start and end
// at the source's home lane, move on one lane a step (18 DPP moves for 128
// pairs). Per unordered pair that is 63 + 9 VALU operations at order 2
// against 2 x 54 in ordered form; the bound stays FP64 issue. Evaluation of
// all particles, ordered form and this: n = 8192 139 -> 116 us, 16384 493 ->
// 364 us, 32768 1902 -> 1335 us, 65536 7585 -> 5200 us (64 TFLOP/s at 78
// operations an ordered pair, 82% of the FP64 vector peak). Both start-up passes: n = 32768 3999 -> 2510 us.
#include <algorithm>

#include "eval_body.h"
#include "sym_plan.h"

namespace h6 {
namespace {

using namespace evalbody;

constexpr int kSymWaves = 4;
constexpr int kSymIpl = 2;
constexpr int kSymThreads = 64 * kSymWaves;
constexpr int kSymBlock = kSymThreads * kSymIpl;

// A double from the next lane (wave rotate left by one).
__device__ __forceinline__ double rotate_lane(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x134, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x134, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

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
__global__ __launch_bounds__(kSymThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_eval_sym(
    SrcPtrs src, SymPlan P, double eps2, double *__restrict__ partial) {
    using T = Traits<ORDER>;
    constexpr int NACC = T::NACC, NREC = T::NREC, K = kSymIpl;
    constexpr int NF = ORDER == 1 ? 7 : ORDER == 2 ? 10 : 13;  // doubles of a source: x, m, v, a, j
    constexpr int NLOAD = (NF + kSymWaves - 1) / kSymWaves;
    // a chunk's records twice over, so that a rotated index needs no wrap
    __shared__ double2 rec[NREC * 2 * kSymChunk];
    __shared__ double jsum[kSymWaves][NACC][kSymChunk];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = P.n, per_d = P.per_d(), part_steps = kSymChunk / P.sub;
    const int64_t x0 = (int64_t)blockIdx.x * P.cells / P.runs;
    const int64_t x1 = (int64_t)(blockIdx.x + 1) * P.cells / P.runs;
    // the superblock, offset and chunk of the first cell
    int I;
    {
        const int64_t full = (int64_t)(P.d1 - P.d0) * per_d;
        const int h = P.nsb / 2;
        if (P.half && x0 >= P.first_cell(h)) {
            const int64_t part = full - per_d;
            I = h + (part > 0 ? (int)((x0 - P.first_cell(h)) / part) : 0);
        } else {
            I = (int)(x0 / full);
        }
    }
    int local = (int)(x0 - P.first_cell(I));
    const PredSrc S{src, nullptr};

    double xi[K][3], vi[K][3], ai[K][3], ji[K][3], mi[K];
    int ki[K];
    double hi[K][NACC], lo[K][NACC];
    auto load_targets = [&]() {
#pragma unroll
        for (int u = 0; u < K; ++u) {
            ki[u] = I * kSymBlock + (wave * K + u) * 64 + lane;
            const bool in = ki[u] < n;
            S.template get<ORDER>(in ? ki[u] : n - 1, xi[u], vi[u], ai[u], ji[u]);
            // past the end: far and massless (no term for any source)
            mi[u] = in ? src.m[ki[u]] : 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) xi[u][c] = in ? xi[u][c] : -kPadPos;
#pragma unroll
            for (int q = 0; q < NACC; ++q) hi[u][q] = lo[u][q] = 0.0;
        }
    };
    auto store_targets = [&]() {
        const int slot = P.slots_j + ((int)blockIdx.x - P.first_run(I));
#pragma unroll
        for (int u = 0; u < K; ++u)
            if (ki[u] < n)
#pragma unroll
                for (int q = 0; q < NACC; ++q)
                    partial[((int64_t)slot * NACC + q) * n + ki[u]] = hi[u][q] + lo[u][q];
    };
    // double `f` of source jj in record order (x0 x1 x2 m v0 v1 v2 a.. j..)
    auto field = [&](int f) {
        const int c = f < 3 ? f : (f - 4) % 3;
        return f == 3 ? src.m : f < 3 ? src.x[c] : f < 7 ? src.v[c] : f < 10 ? src.a[c] : src.j[c];
    };
    double pre[NLOAD];
    auto fetch = [&](int Jc) {  // this thread's doubles of the chunk at particle Jc
#pragma unroll
        for (int q = 0; q < NLOAD; ++q) {
            const int f = wave + q * kSymWaves;
            const int jj = Jc + lane;
            pre[q] = 0.0;
            if (f < NF) pre[q] = jj < n ? field(f)[jj] : f < 3 ? kPadPos : 0.0;
        }
    };
    auto chunk_of = [&](int local_cell) {
        const int d = P.d0 + local_cell / per_d;
        int J = I + d;
        J = J >= P.nsb ? J - P.nsb : J;
        return J * kSymBlock + (local_cell % per_d) / P.sub * kSymChunk;
    };
    if (x0 < x1) {
        load_targets();
        fetch(chunk_of(local));
    }
    for (int64_t x = x0; x < x1; ++x) {
        const int d = P.d0 + local / per_d;
        const int part = local % per_d % P.sub;
        const int sa = part * part_steps, sb = sa + part_steps;  // this part's steps
        const int Jc = chunk_of(local);
        double *rd = reinterpret_cast<double *>(rec);
#pragma unroll
        for (int q = 0; q < NLOAD; ++q) {
            const int f = wave + q * kSymWaves;
            if (f < NF) {
                const int at = ((f >> 1) * 2 * kSymChunk + lane) * 2 + (f & 1);
                rd[at] = pre[q];
                rd[at + 2 * kSymChunk] = pre[q];
            }
        }
        __syncthreads();
        // the next cell: its sources on their way during this one
        const bool last_of_I = x + 1 < x1 && x + 1 == P.first_cell(I + 1);
        if (x + 1 < x1) {
            if (!last_of_I) fetch(chunk_of(local + 1));
        }
        const bool live = Jc < n;
        double acc[K][NACC], accj[NACC];
#pragma unroll
        for (int q = 0; q < NACC; ++q) {
            accj[q] = 0.0;
#pragma unroll
            for (int u = 0; u < K; ++u) acc[u][q] = 0.0;
        }
        auto steps = [&](auto both) {
            constexpr bool BOTH = decltype(both)::value;
            const double2 *p = rec + lane;
#pragma unroll 2
            for (int s = sa; s < sb; ++s) {
                double2 e[NREC];
#pragma unroll
                for (int q = 0; q < NREC; ++q) e[q] = p[q * 2 * kSymChunk + s];
                // order 1's last record holds v2 alone; the others v2, a0
#pragma unroll
                for (int u = 0; u < K; ++u) {
                    if constexpr (BOTH) {
                        const double r[3] = {e[0].x - xi[u][0], e[0].y - xi[u][1], e[1].x - xi[u][2]};
                        const double v[3] = {e[2].x - vi[u][0], e[2].y - vi[u][1], e[3].x - vi[u][2]};
                        double a[3] = {0, 0, 0}, jr[3] = {0, 0, 0};
                        if constexpr (ORDER >= 2) {
                            a[0] = e[3].y - ai[u][0];
                            a[1] = e[4].x - ai[u][1];
                            a[2] = e[4].y - ai[u][2];
                        }
                        if constexpr (ORDER == 3) {
                            jr[0] = e[5].x - ji[u][0];
                            jr[1] = e[5].y - ji[u][1];
                            jr[2] = e[6].x - ji[u][2];
                        }
                        const double r2 = fma(r[2], r[2], fma(r[1], r[1], fma(r[0], r[0], eps2)));
                        pair_both<ORDER>(r, v, a, jr, r2, mi[u], e[1].y, acc[u], accj);
                    } else {
                        const int j = Jc + ((lane + s) & (kSymChunk - 1));
                        pair_terms<ORDER, SKIPSELF>(e, xi[u], vi[u], ai[u], ji[u], eps2, j == ki[u],
                                                    acc[u]);
                    }
                }
                if constexpr (BOTH) {
#pragma unroll
                    for (int q = 0; q < NACC; ++q) accj[q] = rotate_lane(accj[q]);
                }
            }
        };
        if (live) {
            if (d > 0)
                steps(std::true_type{});
            else
                steps(std::false_type{});
#pragma unroll
            for (int u = 0; u < K; ++u)
#pragma unroll
                for (int q = 0; q < NACC; ++q) two_sum_into(hi[u][q], lo[u][q], acc[u][q]);
            if (d > 0) {
#pragma unroll
                for (int q = 0; q < NACC; ++q)
                    jsum[wave][q][(lane + sb) & (kSymChunk - 1)] = accj[q];
            }
        }
        __syncthreads();
        if (live && d > 0) {
            const int slot = (d - (P.d0 > 0 ? P.d0 : 1)) * P.sub + part;
            for (int e = tid; e < NACC * kSymChunk; e += kSymThreads) {
                const int q = e / kSymChunk, l = e % kSymChunk;
                double hs = jsum[0][q][l], hc = 0.0;
#pragma unroll
                for (int w = 1; w < kSymWaves; ++w) two_sum_into(hs, hc, jsum[w][q][l]);
                if (Jc + l < n) partial[((int64_t)slot * NACC + q) * n + Jc + l] = hs + hc;
            }
        }
        ++local;
        if (last_of_I) {
            store_targets();
            ++I;
            local = 0;
            load_targets();
            fetch(chunk_of(0));
        }
    }
    if (x0 < x1) store_targets();
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
    const int nd = P.nsb / 2 + 1, dj = d0 > 0 ? d0 : 1;
    const int64_t slots = ctx->partial_cap / ((int64_t)ncomp * n);
    // target-side slots: the runs a superblock's cells can span (it holds at
    // most 2 / nsb of a batch's cells, when the batch is d = nsb / 2 alone)
    const int64_t span = (2 * (int64_t)runs + P.nsb - 1) / P.nsb + 2;
    const int64_t room = slots - span;
    if (room < 1 || d0 >= nd) return false;
    P.d1 = (int)std::min<int64_t>(nd, dj + room);
    P.half = P.nsb % 2 == 0 && P.nsb > 1 && P.d1 == nd;
    // parts: the longest run in chunk times (a part costs about 1/12 more for
    // its staging and sums: n = 16384 in 9 whole chunks a run 352 us, in 17
    // halves 358; n = 8192 in 3 chunks 116 us, in 5 halves 105), where the slots allow
    float best = 3.0e38f;
    SymPlan Q = P;
    for (int sub = 1; sub <= kSymMaxSub; sub *= 2) {
        if (sub > 1 && (int64_t)(P.d1 - dj) * sub > room) break;
        Q.sub = sub;
        Q.runs = 1;
        Q.cells = 1;
        Q.cells = Q.first_cell(Q.nsb);
        Q.runs = (int)std::min<int64_t>(runs, Q.cells);
        Q.slots_j = (P.d1 - dj) * sub;
        const float longest = (float)((Q.cells + Q.runs - 1) / Q.runs);
        const float cost = longest * (1.0f / (float)sub + 1.0f / 12.0f);
        if (cost < best) {
            best = cost;
            *plan = Q;
        }
    }
    return true;
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
    const int runs = 2 * ctx->n_cu;  // two workgroups of four waves a CU (two waves a SIMD)
    SymPlan P;
    *done = sym_plan(ctx, n, kSymBlock, runs, ncomp, 0, &P);
    if (!*done) return hipSuccess;
    const bool skip = self_pair_masked(ctx->eps2, H6_FP64);
    for (bool more = true; more; more = sym_plan(ctx, n, kSymBlock, runs, ncomp, P.d1, &P)) {
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
