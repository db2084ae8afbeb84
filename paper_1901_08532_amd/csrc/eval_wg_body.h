// Evaluation by whole workgroups: a workgroup sums a few targets over
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

#include "eval_ops.h"

namespace h6 {
namespace evalbody {

constexpr int kWgThreads = kWgBlock;
constexpr int kWgMaxTgt = 32;
constexpr int kWgFlush = 64;   // sources per strand between compensated flushes
constexpr int kWgPerSum = 16;  // strand sums one thread adds in the final reduction

// Workgroup memory of wg_sums, in bytes: a tile, or the strand sums.
template <class OPS>
constexpr int wg_pool_bytes() {
    return OPS::NREC * kWgThreads * (int)sizeof(Word2<typename OPS::Word>);
}

// Sums of the targets g * TGT .. g * TGT + TGT - 1 (of list; NULL: particles)
// over the sources [jb, je), into fs[t * NI + q] (workgroup memory, TGT * NI
// doubles). OPS as in sym_body.h (one(), add(), value()). Every thread of the
// workgroup calls it; it ends with a barrier.
template <int TGT, class OPS>
__device__ __forceinline__ void wg_sums(const OPS &ops, const int32_t *__restrict__ list, int n,
                                        int n_act, int g, int jb, int je, void *pool, double *fs) {
    using W = typename OPS::Word;
    constexpr int NREC = OPS::NREC, NF = OPS::NF, NACC = OPS::NI;
    constexpr int STR = kWgThreads / TGT;  // strands
    const int tid = threadIdx.x;
    const int t = tid % TGT, s = tid / TGT;
    const int k = g * TGT + t, kc = k < n_act ? k : n_act - 1;
    const int pid = list ? list[kc] : kc;
    typename OPS::Target tgt;
    ops.load(pid, n, tgt);
    W acc[NACC];
    typename OPS::Sum sum[NACC];
#pragma unroll
    for (int q = 0; q < NACC; ++q) {
        acc[q] = W{};
        sum[q] = {};
    }
    auto *tile = static_cast<Word2<W> *>(pool);

    int since = 0;
    for (int jt = jb; jt < je; jt += kWgThreads) {
        const int cnt = min(kWgThreads, je - jt);
        if (jt != jb) __syncthreads();  // previous tile fully consumed
        {
            Word2<W> rec[NREC];
            W *w = reinterpret_cast<W *>(rec);
#pragma unroll
            for (int f = 0; f < 2 * NREC; ++f)
                w[f] = f >= NF ? W{} : tid < cnt ? OPS::word(ops.field(f)[jt + tid]) : OPS::pad(f);
#pragma unroll
            for (int q = 0; q < NREC; ++q) tile[q * kWgThreads + tid] = rec[q];
        }
        __syncthreads();
        const int steps = (cnt + STR - 1) / STR;
#pragma unroll OPS::kUnroll
        for (int i = 0; i < steps; ++i) {
            const int e = i * STR + s;
            Word2<W> rec[NREC];
#pragma unroll
            for (int q = 0; q < NREC; ++q) rec[q] = tile[q * kWgThreads + e];
            ops.one(rec, tgt, jt + e == pid, acc);
        }
        since += TGT;
        if (since >= kWgFlush) {
            since = 0;
#pragma unroll
            for (int q = 0; q < NACC; ++q) {
                OPS::add(sum[q], acc[q]);
                acc[q] = W{};
            }
        }
    }
    __syncthreads();
    // strand sums, [q][target][strand], rows padded by one double so that a
    // wave's rows fall on different banks
    double *red = static_cast<double *>(pool);
    constexpr int LD = STR + 1;
    static_assert(NACC * TGT * LD * (int)sizeof(double) <= wg_pool_bytes<OPS>(),
                  "strand sums fit the tile");
#pragma unroll
    for (int q = 0; q < NACC; ++q) {
        OPS::add(sum[q], acc[q]);
        red[(q * TGT + t) * LD + s] = OPS::value(sum[q]);
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

// Evaluation by whole workgroups: target group blockIdx.x, source slice
// blockIdx.y.
template <int TGT, class OPS>
__global__ __launch_bounds__(kWgThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_wg(
    OPS ops, const int32_t *__restrict__ active, int n, int n_act, int slice_len, int out0,
    OutPtrs out, int64_t slice_stride) {
    constexpr int NACC = OPS::NI;
    __shared__ double2 pool[wg_pool_bytes<OPS>() / sizeof(double2)];
    __shared__ double fs[TGT * NACC];
    const int g = blockIdx.x, jb = (int)blockIdx.y * slice_len;
    wg_sums<TGT>(ops, active, n, n_act, g, jb, min(n, jb + slice_len), pool, fs);
    const int k = g * TGT + (int)threadIdx.x;
    if ((int)threadIdx.x < TGT && k < n_act) {
#pragma unroll
        for (int q = 0; q < NACC; ++q)
            out.p[out0 + q][(int64_t)blockIdx.y * slice_stride + k] = fs[threadIdx.x * NACC + q];
    }
}

// Launch for tgt targets a workgroup (a power of two up to kWgMaxTgt).
template <class OPS>
hipError_t launch_wg(int tgt, dim3 grid, hipStream_t st, const OPS &ops, const int32_t *active,
                     int n, int n_act, int slice_len, int out0, const OutPtrs &out,
                     int64_t slice_stride) {
#define H6_WG(T)                                                                              \
    if (tgt == T) {                                                                           \
        hipLaunchKernelGGL((k_eval_wg<T, OPS>), grid, dim3(kWgThreads), 0, st, ops, active, n, \
                           n_act, slice_len, out0, out, slice_stride);                        \
        return hipGetLastError();                                                             \
    }
    H6_WG(1)
    H6_WG(2)
    H6_WG(4)
    H6_WG(8)
    H6_WG(16)
    H6_WG(32)
#undef H6_WG
    return hipErrorInvalidValue;
}

}  // namespace evalbody
}  // namespace h6
