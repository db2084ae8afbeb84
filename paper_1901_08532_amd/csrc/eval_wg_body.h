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
// 65536 137 -> 134 us, 7 of 1024 8.3 -> 5.1 us. The mixed form: 33 of 1024
// 41 -> 9.2 us, 1024 of 1024 67 -> 9.8 us, 4096 of 4096 75 -> 37 us, 1000 of
// 65536 168 -> 128 us.
#pragma once

#include "eval_ops.h"

namespace h6 {
namespace evalbody {

constexpr int kWgThreads = kWgBlock;
constexpr int kWgMaxTgt = 32;
constexpr int kWgFlush = 64;   // sources per strand between compensated flushes
constexpr int kWgPerSum = 16;  // strand sums one thread adds in the final reduction

// Workgroup memory of wg_sums, in bytes: a tile, or the strand sums.
template <int TGT, class OPS>
constexpr int wg_pool_bytes() {
    constexpr int tile = OPS::NREC * kWgThreads * (int)sizeof(Word2<typename OPS::Word>);
    constexpr int sums = OPS::NI * (kWgThreads + TGT) * (int)sizeof(double);
    return tile > sums ? tile : sums;
}

// Sums of the targets g * TGT .. g * TGT + TGT - 1 (of list; NULL: particles)
// over the sources [jb, je), into fs[t * NI + q] (workgroup memory, TGT * NI
// doubles). OPS as in sym_body.h (one(), add(), value()), with load_rec() and
// pad_rec() for whole records, kDirectMaxTgt the largest TGT that goes without
// LDS tiles, Acc the type of a strand's running sums, and
// kRun: a strand takes kRun consecutive sources in a row (1, or 8 for the mixed
// form, whose FP32 sums cover 8 consecutive sources). Every thread of the
// workgroup calls it; it ends with a barrier.
template <int TGT, class OPS>
__device__ __forceinline__ void wg_sums(const OPS &ops, const int32_t *__restrict__ list, int n,
                                        int n_act, int g, int jb, int je, void *pool, double *fs) {
    using W = typename OPS::Word;
    using A = typename OPS::Acc;
    constexpr int NREC = OPS::NREC, NACC = OPS::NI, RUN = OPS::kRun;
    constexpr int STR = kWgThreads / TGT;  // strands
    const int tid = threadIdx.x;
    const int t = tid % TGT, s = tid / TGT;
    const int k = g * TGT + t, kc = k < n_act ? k : n_act - 1;
    const int pid = list ? list[kc] : kc;
    typename OPS::Target tgt;
    ops.load(pid, n, tgt);
    A acc[NACC];
    typename OPS::Sum sum[NACC];
#pragma unroll
    for (int q = 0; q < NACC; ++q) {
        acc[q] = A{};
        sum[q] = {};
    }
    auto flush = [&]() {
#pragma unroll
        for (int q = 0; q < NACC; ++q) {
            OPS::add(sum[q], acc[q]);
            acc[q] = A{};
        }
    };
    // one or two targets: each thread loads its strand's sources itself, the next
    // one ahead. A tile of 512 through LDS costs 0.9 us there, two barriers and
    // the LDS round trip for one or two pairs a thread; with and without: 7 of
    // 1024 5.7 / 5.1 us, 7 of 1500 7.0 / 5.7, 40 of 2048 7.4 / 6.2, 100 of 4096
    // 9.4 / 8.6 (fewer slices pay now). With four targets no further gain.
    constexpr bool kDirect = TGT <= OPS::kDirectMaxTgt;
    if constexpr (kDirect) {
        Word2<W> rec[NREC], next[NREC];
        auto fetch = [&](int j, Word2<W> *r) {
            if (j < je)
                ops.load_rec(j, r);
            else
                OPS::pad_rec(r);
        };
        fetch(jb + s, next);
        int since = 0;
#pragma unroll 1
        for (int j0 = jb; j0 < je; j0 += STR) {
#pragma unroll
            for (int q = 0; q < NREC; ++q) rec[q] = next[q];
            fetch(j0 + STR + s, next);
            ops.one(rec, tgt, j0 + s == pid, acc);
            if (++since == kWgFlush) {
                since = 0;
                flush();
            }
        }
    }
    auto *tile = static_cast<Word2<W> *>(pool);
    int since = 0;
    for (int jt = jb; !kDirect && jt < je; jt += kWgThreads) {
        const int cnt = min(kWgThreads, je - jt);
        // the target's own entry (never the padding past a slice's end: a mixed
        // term overflows where a mask makes the radius of 1e15 one)
        const int own = pid - jt < cnt ? pid - jt : -1;
        if (jt != jb) __syncthreads();  // previous tile fully consumed
        {
            Word2<W> rec[NREC];
            if (tid < cnt)
                ops.load_rec(jt + tid, rec);
            else
                OPS::pad_rec(rec);
            // slots in the order the strands read them: step by step, the
            // strands of a step side by side
            const int run = tid / RUN;
            const int slot = (run / STR * RUN + tid % RUN) * STR + run % STR;
#pragma unroll
            for (int q = 0; q < NREC; ++q) tile[q * kWgThreads + slot] = rec[q];
        }
        __syncthreads();
        const int steps = (cnt + STR * RUN - 1) / (STR * RUN) * RUN;
        auto step = [&](int i) {
            Word2<W> rec[NREC];
#pragma unroll
            for (int q = 0; q < NREC; ++q) rec[q] = tile[q * kWgThreads + i * STR + s];
            const int e = RUN == 1 ? i * STR + s : (i / RUN * STR + s) * RUN + i % RUN;
            ops.one(rec, tgt, e == own, acc);
        };
        if constexpr (RUN == 1) {
#pragma unroll OPS::kUnroll
            for (int i = 0; i < steps; ++i) step(i);
            since += TGT;
            if (since >= kWgFlush) {
                since = 0;
                flush();
            }
        } else {
#pragma unroll 1
            for (int i = 0; i < steps; i += RUN) {
#pragma unroll
                for (int r = 0; r < RUN; ++r) step(i + r);
                flush();
            }
        }
    }
    __syncthreads();
    // strand sums, [q][target][strand], rows padded by one double so that a
    // wave's rows fall on different banks
    double *red = static_cast<double *>(pool);
    constexpr int LD = STR + 1;
#pragma unroll
    for (int q = 0; q < NACC; ++q) {
        if constexpr (RUN == 1) OPS::add(sum[q], acc[q]);
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

// f(integral_constant of 1, 2, .. kWgMaxTgt) until one returns true.
template <class F>
bool for_each_tgt(F f) {
    static_assert(kWgMaxTgt == 32, "the list below");
    return f(std::integral_constant<int, 1>{}) || f(std::integral_constant<int, 2>{}) ||
           f(std::integral_constant<int, 4>{}) || f(std::integral_constant<int, 8>{}) ||
           f(std::integral_constant<int, 16>{}) || f(std::integral_constant<int, 32>{});
}

// Evaluation by whole workgroups: target group blockIdx.x, source slice
// blockIdx.y.
template <int TGT, class OPS>
__global__ __launch_bounds__(kWgThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_wg(
    OPS ops, const int32_t *__restrict__ active, int n, int n_act, int slice_len, int out0,
    OutPtrs out, int64_t slice_stride) {
    constexpr int NACC = OPS::NI;
    __shared__ double2 pool[wg_pool_bytes<TGT, OPS>() / sizeof(double2)];
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

// Launch for tgt targets a workgroup (a power of two from OPS::kMinTgt to
// kWgMaxTgt).
template <class OPS>
hipError_t launch_wg(int tgt, dim3 grid, hipStream_t st, const OPS &ops, const int32_t *active,
                     int n, int n_act, int slice_len, int out0, const OutPtrs &out,
                     int64_t slice_stride) {
    auto launch = [&](auto t) {
        constexpr int T = decltype(t)::value;
        if constexpr (T >= OPS::kMinTgt) {
            if (tgt != T) return false;
            hipLaunchKernelGGL((k_eval_wg<T, OPS>), grid, dim3(kWgThreads), 0, st, ops, active, n,
                               n_act, slice_len, out0, out, slice_stride);
            return true;
        }
        return false;
    };
    return for_each_tgt(launch) ? hipGetLastError() : hipErrorInvalidValue;
}

}  // namespace evalbody
}  // namespace h6
