// Work split of the all-pairs kernels that take each unordered pair once
// (evaluation over all particles, start-up passes and their gradients).
//
// The particles form nsb superblocks of `block` (a wave of the workgroup
// holds block / waves targets in registers). Superblock I meets the
// superblocks J = I + d (mod nsb), d = 0 .. nsb / 2: d = 0 in ordered form,
// the others in third-law form (both particles of a pair get its terms), and
// for even nsb the last d only from I < nsb / 2, so that every unordered pair
// of superblocks comes once. A cell is (I, d, 64-source chunk of J, part): the
// chunk's sources go round the lanes of a wave in 64 steps, of which a part
// takes 64 / sub. The cells of a batch, I-major, are cut into equal runs, one
// per workgroup, all resident at once: no round of workgroups is left
// part-filled, whatever n.
//
// Sums leave through slots of the context's partial sums, [slot][component]
// [particle]: `sub` slots per d >= 1 of the batch for the source side (each
// cell writes its chunk once), then one per workgroup that touches I for the
// target side. Batches take as many d as the slots hold; very large systems,
// whose scratch holds no more than a slot or two, take the ordered form, one
// workgroup a superblock.
#pragma once

#include "device_math.h"
#include "h6_internal.h"

namespace h6 {

constexpr int kSymChunk = 64;  // sources of a cell
constexpr int kSymMaxSub = 16;

struct SymPlan {
    int n;
    int block;      // particles of a superblock
    int nsb;        // superblocks
    int sub;        // parts of a chunk's 64 steps
    int d0, d1;     // offsets d of this batch
    int ordered;    // 1: offsets up to nsb - 1 in ordered form, no source-side sums
    int half;       // 1: the batch holds d = nsb / 2 of an even nsb
    int runs;       // workgroups
    int slots_j;    // source-side slots (sub for each d >= 1 of the batch)
    int64_t cells;  // cells of the batch

    // cells of a superblock and offset
    __host__ __device__ int per_d() const { return block / kSymChunk * sub; }
    // cells before superblock I's first
    __host__ __device__ int64_t first_cell(int I) const {
        const int64_t full = (int64_t)(d1 - d0) * per_d();
        const int h = nsb / 2;
        const int64_t less = half && I > h ? (int64_t)(I - h) * per_d() : 0;
        return (int64_t)I * full - less;
    }
    // run holding cell x: runs are [r * cells / runs, (r + 1) * cells / runs)
    __host__ __device__ int run_of(int64_t x) const {
        return (int)(((x + 1) * runs - 1) / cells);
    }
    // first run of superblock I, and how many touch it
    __host__ __device__ int first_run(int I) const { return run_of(first_cell(I)); }
    __host__ __device__ int run_count(int I) const {
        const int64_t a = first_cell(I), b = first_cell(I + 1);
        return b > a ? run_of(b - 1) - run_of(a) + 1 : 0;
    }
    // whether superblock J has a source-side sum for offset d (>= 1)
    __host__ __device__ bool has_source_sum(int J, int d) const {
        return !(2 * d == nsb && J < nsb / 2);
    }
};

// Price of a cell in microseconds, two workgroups on a CU: a whole chunk's
// steps, and the fixed part (staging, barriers, sums); chunk3: the steps with
// three on a CU (0: the kernel's registers allow two).
struct SymCost {
    float chunk, part, chunk3 = 0.0f;
};

// Sums of a batch's slots for particle k, components c, c + ncomp / N, ... (N of
// them): the source-side slots that its superblock has, then the target-side
// ones of the runs that touched it (compensated).
template <int N>
__device__ __forceinline__ void sym_sums(const double *__restrict__ partial, const SymPlan &P,
                                         int ncomp, int c, int k, double *out) {
    const int J = k / P.block;
    const int64_t ld = (int64_t)ncomp * P.n;
    const int64_t cs = (int64_t)(ncomp / N) * P.n;
    const double *__restrict__ p = partial + (int64_t)c * P.n + k;
    int nj = P.slots_j;
    // the batch's last slots are d = nsb / 2, which only half the superblocks have
    if (P.half && nj > 0 && !P.has_source_sum(J, P.nsb / 2)) nj -= P.sub;
    const int ni = P.run_count(J);
    double s[N], comp[N];
#pragma unroll
    for (int q = 0; q < N; ++q) s[q] = comp[q] = 0.0;
    constexpr int U = N == 1 ? 8 : 4;  // slots whose loads are in flight together
    for (int part = 0; part < 2; ++part) {
        const int cnt = part ? ni : nj;
        const double *__restrict__ b = p + (part ? P.slots_j * ld : 0);
        for (int s0 = 0; s0 < cnt; s0 += U) {
            double x[U][N];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < N; ++q)
                    x[u][q] = s0 + u < cnt ? b[(int64_t)(s0 + u) * ld + q * cs] : 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < N; ++q) two_sum_into(s[q], comp[q], x[u][q]);
        }
    }
#pragma unroll
    for (int q = 0; q < N; ++q) out[q] = s[q] + comp[q];
}

// The next batch from offset d0 on, for ncomp sums a particle; false at the
// end, or at d0 = 0 where the slots do not suffice.
bool sym_plan(h6_ctx ctx, int n, int block, int ncomp, SymCost cost, int d0, SymPlan *plan);
// The ordered form (one slot) from offset d0 on, kOrderedMax offsets at most: a run is
// a superblock there, and cells * runs stays within 64 bits at every size.
constexpr int kOrderedMax = 1024;
SymPlan sym_plan_ordered(int n, int block, int d0);
hipError_t launch_sym_reduce(h6_ctx ctx, const SymPlan &P, int ncomp, int out0, const OutPtrs &out,
                             unsigned acc_mask);

// An order-2 evaluation over all particles (FP64 or EX) whose sums fit one
// batch: the plan (false: more than one, or none), the pair kernel, and a
// shared step's remainder on its slots.
bool eval_sym_single(h6_ctx ctx, int precision, int n, SymPlan *plan);
hipError_t launch_eval_sym_pairs(h6_ctx ctx, int order, int precision, const SrcPtrs &src,
                                 const SymPlan &P);
void launch_ex_sym_pairs(h6_ctx ctx, const SrcPtrs &src, const SymPlan &P);
hipError_t launch_sym_step(h6_ctx ctx, const SymPlan &P, h6_state *st, double dt, bool predict,
                           const h6_pred *out, const h6_force *f);

// All batches of a third-law sum over n particles: launch(plan) enqueues the
// pair kernel, the slots are then summed into (bits of acc_mask: added to)
// out.p[out0 ..]. *done is false, and nothing launched, where the slots do not
// suffice.
template <class LAUNCH>
hipError_t sym_batches(h6_ctx ctx, int n, int block, int ncomp, SymCost cost, int out0,
                       const OutPtrs &out, unsigned acc_mask, bool *done, LAUNCH launch) {
    SymPlan P;
    *done = sym_plan(ctx, n, block, ncomp, cost, 0, &P);
    for (bool more = *done; more; more = sym_plan(ctx, n, block, ncomp, cost, P.d1, &P)) {
        hipError_t e = launch(P);
        if (e == hipSuccess)
            e = launch_sym_reduce(ctx, P, ncomp, out0, out, P.d0 > 0 ? (1u << ncomp) - 1u : acc_mask);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace h6
