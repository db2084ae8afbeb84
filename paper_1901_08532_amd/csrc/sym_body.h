// Body of the all-pairs kernels that take each unordered pair once: the walk
// of one workgroup through its run of cells (sym_plan.h), common to the
// evaluation, its gradient and the double-single evaluation.
//
// A wave holds K x 64 targets in registers, K per lane. The sources of a
// chunk go round the lanes: at step s lane l takes source (l + s) mod 64, read
// from LDS, against its targets; the source's sums, which start and end at
// the source's home lane, move on one lane a step.
//
// OPS describes the particles and the pair:
//   Word            an 8-byte number (double, or a float pair)
//   NF, NREC        words of a source record, and its double2-sized planes
//   NI, NJ          sums of a target and of a source
//   K, kUnroll      targets per lane, steps unrolled
//   Target, Sum     a target's data; a target's running sum over cells
//   const double *field(f)  the array word f of a source comes from (f known
//                           when compiled); Word word(x) its stored form
//   Word pad(f)             word f of the far, massless padding source
//   load(k, n, t)           target k (padding from n on)
//   both(rec, t, acci, accj)  the pair's terms added to both particles
//   one(rec, t, self, acci)   the pair's terms added to the target only
//   add(sum, acci), value(sum), value(word)
#pragma once

#include <type_traits>

#include "device_math.h"
#include "sym_plan.h"

namespace h6 {
namespace symbody {

constexpr int kSymWaves = 4;
constexpr int kSymThreads = 64 * kSymWaves;

// The value of the next lane (wave rotate left by one).
__device__ __forceinline__ double rotate_lane(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x134, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x134, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float2 rotate_lane(float2 v) {
    const int x = __builtin_amdgcn_mov_dpp(__float_as_int(v.x), 0x134, 0xF, 0xF, true);
    const int y = __builtin_amdgcn_mov_dpp(__float_as_int(v.y), 0x134, 0xF, 0xF, true);
    return make_float2(__int_as_float(x), __int_as_float(y));
}

// FP64 sums of a target over cells: compensated.
struct CompSum {
    double hi, lo;
};

template <class W>
struct alignas(16) Word2 {
    W x, y;
};

template <class OPS>
__device__ __forceinline__ void sym_run(const OPS &ops, const SymPlan &P,
                                        double *__restrict__ partial) {
    using W = typename OPS::Word;
    constexpr int NF = OPS::NF, NREC = OPS::NREC, NI = OPS::NI, NJ = OPS::NJ, K = OPS::K;
    constexpr int NLOAD = (NF + kSymWaves - 1) / kSymWaves;
    constexpr int kBlock = kSymThreads * K;
    static_assert(2 * NREC >= NF && NJ <= NI, "record planes; slots are sized by the target's sums");
    // a chunk's records twice over, so that a rotated index needs no wrap
    __shared__ Word2<W> rec[NREC * 2 * kSymChunk];
    __shared__ double jsum[kSymWaves][NJ][kSymChunk];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = P.n, per_d = P.per_d(), part_steps = kSymChunk / P.sub;
    const int64_t x0 = (int64_t)blockIdx.x * P.cells / P.runs;
    const int64_t x1 = (int64_t)(blockIdx.x + 1) * P.cells / P.runs;
    if (x0 >= x1) return;  // the whole workgroup
    // the superblock of the first cell
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

    typename OPS::Target tgt[K];
    typename OPS::Sum sum[K][NI];
    auto target_index = [&](int u) { return I * kBlock + (wave * K + u) * 64 + lane; };
    auto load_targets = [&]() {
#pragma unroll
        for (int u = 0; u < K; ++u) {
            ops.load(target_index(u), n, tgt[u]);
#pragma unroll
            for (int q = 0; q < NI; ++q) sum[u][q] = {};
        }
    };
    auto store_targets = [&]() {
        const int slot = P.slots_j + ((int)blockIdx.x - P.first_run(I));
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const int k = target_index(u);
            if (k < n)
#pragma unroll
                for (int q = 0; q < NI; ++q)
                    partial[((int64_t)slot * NI + q) * n + k] = OPS::value(sum[u][q]);
        }
    };
    // the arrays this wave stages (every kSymWaves-th word)
    const double *field[NLOAD] = {};
#pragma unroll
    for (int f = 0; f < NF; ++f)
        if (f % kSymWaves == wave) field[f / kSymWaves] = ops.field(f);
    W pre[NLOAD];
    auto fetch = [&](int Jc) {  // this thread's words of the chunk at particle Jc
#pragma unroll
        for (int q = 0; q < NLOAD; ++q) {
            const int f = wave + q * kSymWaves;
            const int jj = Jc + lane;
            if (f < NF) pre[q] = jj < n ? OPS::word(field[q][jj]) : OPS::pad(f);
        }
    };
    auto chunk_of = [&](int cell) {
        const int d = P.d0 + cell / per_d;
        int J = I + d;
        J = J >= P.nsb ? J - P.nsb : J;
        return J * kBlock + cell % per_d / P.sub * kSymChunk;
    };
    load_targets();
    fetch(chunk_of(local));
    for (int64_t x = x0; x < x1; ++x) {
        const int d = P.d0 + local / per_d;
        const int part = local % per_d % P.sub;
        const int sa = part * part_steps, sb = sa + part_steps;  // this part's steps
        const int Jc = chunk_of(local);
        const bool both_ways = d > 0 && !P.ordered;
        W *rd = reinterpret_cast<W *>(rec);
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
        if (x + 1 < x1 && !last_of_I) fetch(chunk_of(local + 1));
        const bool live = Jc < n;
        if (live) {
            W acc[K][NI], accj[NJ];
#pragma unroll
            for (int q = 0; q < NJ; ++q) accj[q] = W{};
#pragma unroll
            for (int u = 0; u < K; ++u)
#pragma unroll
                for (int q = 0; q < NI; ++q) acc[u][q] = W{};
            auto steps = [&](auto both) {
                constexpr bool BOTH = decltype(both)::value;
                const Word2<W> *p = rec + lane;
#pragma unroll 1
                for (int s2 = sa; s2 < sb; s2 += OPS::kUnroll) {  // parts are whole multiples
#pragma unroll
                    for (int s = s2; s < s2 + OPS::kUnroll; ++s) {
                        Word2<W> e[NREC];
#pragma unroll
                        for (int q = 0; q < NREC; ++q) e[q] = p[q * 2 * kSymChunk + s];
#pragma unroll
                        for (int u = 0; u < K; ++u) {
                            if constexpr (BOTH) {
                                ops.both(e, tgt[u], acc[u], accj);
                            } else {
                                const int j = Jc + ((lane + s) & (kSymChunk - 1));
                                ops.one(e, tgt[u], j == target_index(u), acc[u]);
                            }
                        }
                        if constexpr (BOTH) {
#pragma unroll
                            for (int q = 0; q < NJ; ++q) accj[q] = rotate_lane(accj[q]);
                        }
                    }
                }
            };
            if (both_ways)
                steps(std::true_type{});
            else
                steps(std::false_type{});
#pragma unroll
            for (int u = 0; u < K; ++u)
#pragma unroll
                for (int q = 0; q < NI; ++q) OPS::add(sum[u][q], acc[u][q]);
            if (both_ways) {
#pragma unroll
                for (int q = 0; q < NJ; ++q)
                    jsum[wave][q][(lane + sb) & (kSymChunk - 1)] = OPS::value(accj[q]);
            }
        }
        __syncthreads();
        if (live && both_ways) {
            const int slot = (d - (P.d0 > 0 ? P.d0 : 1)) * P.sub + part;
            for (int e = tid; e < NJ * kSymChunk; e += kSymThreads) {
                const int q = e / kSymChunk, l = e % kSymChunk;
                double hs = jsum[0][q][l], hc = 0.0;
#pragma unroll
                for (int w = 1; w < kSymWaves; ++w) two_sum_into(hs, hc, jsum[w][q][l]);
                if (Jc + l < n) partial[((int64_t)slot * NI + q) * n + Jc + l] = hs + hc;
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
    store_targets();
}

}  // namespace symbody
}  // namespace h6
