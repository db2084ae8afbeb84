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

#include "h6_internal.h"

namespace h6 {

constexpr int kSymChunk = 64;  // sources of a cell
constexpr int kSymMaxSub = 4;

struct SymPlan {
    int n;
    int block;      // particles of a superblock
    int nsb;        // superblocks
    int sub;        // parts of a chunk's 64 steps
    int d0, d1;     // offsets d of this batch
    int ordered;    // 1: d = 0 .. nsb - 1 in ordered form, no source-side sums
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

// The next batch from offset d0 on, for `runs` workgroups and ncomp sums a
// particle; false at the end, or at d0 = 0 where the slots do not suffice.
bool sym_plan(h6_ctx ctx, int n, int block, int runs, int ncomp, int d0, SymPlan *plan);
// The ordered form (one slot).
SymPlan sym_plan_ordered(int n, int block);
hipError_t launch_sym_reduce(h6_ctx ctx, const SymPlan &P, int ncomp, int out0, const OutPtrs &out,
                             unsigned acc_mask);

}  // namespace h6
