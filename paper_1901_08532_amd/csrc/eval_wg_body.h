// Evaluation by whole workgroups (FP64): a workgroup sums a few targets over
// a range of sources, so that no slice sums go through memory.
//
// 512 threads are TGT targets x 512 / TGT strands: thread t serves target
// t % TGT and every (512 / TGT)-th source of each 512-source tile staged in
// LDS. The strands' sums are then combined in LDS, compensated. Two such
// workgroups fit a CU (four waves per SIMD, 40 KiB of LDS each at order 2),
// so one computes while the other waits for its tile or a barrier.
//
// Bound by FP64 issue for large sets and by launch and memory latency for
// small ones. The one-wave tile kernel it replaces there needs a slice of at
// least four 64-source tiles per wave, which left most SIMDs idle (32 of 1024
// busy at n = n_act = 1024). h6_evaluate, this kernel and any slice
// reduction, before and after: n = n_act = 1024 63 -> 7.8 us, 40 of 4096
// 41.7 -> 8.6 us, 4096 of 4096 67 -> 40 us, 300 of 65536 73 -> 53 us, 1000 of
// 65536 137 -> 134 us, 7 of 1024 8.3 -> 6.2 us.
#pragma once

#include "eval_body.h"

namespace h6 {
namespace evalbody {

constexpr int kWgThreads = kWgBlock;
constexpr int kWgMaxTgt = 32;
constexpr int kWgFlush = 64;   // sources per strand between compensated flushes
constexpr int kWgPerSum = 16;  // strand sums one thread adds in the final reduction

// Workgroup memory of wg_sums, in double2: a tile, or the strand sums.
template <int ORDER>
constexpr int wg_pool() {
    return Traits<ORDER>::NREC * kWgThreads;
}

// Sums of the targets g * TGT .. g * TGT + TGT - 1 over the sources
// [jb, je), into fs[t * NACC + q] (workgroup memory, TGT * NACC doubles).
// Every thread of the workgroup calls it; it ends with a barrier.
template <int ORDER, int TGT, bool SKIPSELF, class SRC>
__device__ __forceinline__ void wg_sums(const SRC &S, int n_act, double eps2, int g, int jb, int je,
                                        double2 *pool, double *fs) {
    using T = Traits<ORDER>;
    constexpr int NREC = T::NREC, NACC = T::NACC;
    constexpr int STR = kWgThreads / TGT;  // strands
    const int tid = threadIdx.x;
    const int t = tid % TGT, s = tid / TGT;
    const int k = g * TGT + t;
    const int pid = S.target(k < n_act ? k : n_act - 1);
    double xi[3], vi[3], ai[3], ji[3];
    S.template get<ORDER>(pid, xi, vi, ai, ji);
    double acc[NACC], hi[NACC], lo[NACC];
#pragma unroll
    for (int q = 0; q < NACC; ++q) acc[q] = hi[q] = lo[q] = 0.0;

    int since = 0;
    for (int jt = jb; jt < je; jt += kWgThreads) {
        const int cnt = min(kWgThreads, je - jt);
        if (jt != jb) __syncthreads();  // previous tile fully consumed
        {
            double2 rec[NREC];
            if (tid < cnt) {
                load_rec<ORDER>(S, jt + tid, rec);
            } else {
                pad_rec<ORDER>(rec);
            }
#pragma unroll
            for (int q = 0; q < NREC; ++q) pool[q * kWgThreads + tid] = rec[q];
        }
        __syncthreads();
        const int steps = (cnt + STR - 1) / STR;
#pragma unroll 2
        for (int i = 0; i < steps; ++i) {
            const int e = i * STR + s;
            double2 rec[NREC];
#pragma unroll
            for (int q = 0; q < NREC; ++q) rec[q] = pool[q * kWgThreads + e];
            pair_terms<ORDER, SKIPSELF>(rec, xi, vi, ai, ji, eps2, jt + e == pid, acc);
        }
        since += TGT;
        if (since >= kWgFlush) {
            since = 0;
#pragma unroll
            for (int q = 0; q < NACC; ++q) {
                two_sum_into(hi[q], lo[q], acc[q]);
                acc[q] = 0.0;
            }
        }
    }
    __syncthreads();
    // strand sums, [q][target][strand], rows padded by one double so that a
    // wave's rows fall on different banks
    double *red = reinterpret_cast<double *>(pool);
    constexpr int LD = STR + 1;
    static_assert(NACC * TGT * LD <= 2 * wg_pool<ORDER>(), "strand sums fit the tile");
#pragma unroll
    for (int q = 0; q < NACC; ++q) {
        two_sum_into(hi[q], lo[q], acc[q]);
        red[(q * TGT + t) * LD + s] = hi[q] + lo[q];
    }
    __syncthreads();
    // G threads per sum, kWgPerSum strands each, merged within the segment
    constexpr int G = STR / kWgPerSum;
    static_assert(G >= 1 && G <= 64 && NACC * TGT * G <= kWgThreads, "one pass of threads");
    const int o = tid / G, gl = tid % G;
    const bool mine = o < NACC * TGT;
    double hs = 0.0, hc = 0.0;
    if (mine) {
#pragma unroll
        for (int i = 0; i < kWgPerSum; ++i) two_sum_into(hs, hc, red[o * LD + gl + i * G]);
    }
    seg_comp_reduce_n<1>(&hs, &hc, G);  // valid in the segment's last lane
    if (mine && gl == G - 1) fs[(o % TGT) * NACC + o / TGT] = hs + hc;
    __syncthreads();
}

}  // namespace evalbody
}  // namespace h6
