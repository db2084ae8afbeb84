// Integrator steps around the evaluation: predictor, corrector with
// interpolation and time-step assignment, start-up steps, the block
// scheduler, and the energy / angular momentum diagnostic.
//
// All of these are bandwidth- or latency-bound elementwise passes over
// structure-of-arrays FP64 data: one particle per lane, coalesced loads
// and stores, no LDS except for block-level reductions.
#include <algorithm>

#include "steps_body.h"

namespace h6 {
namespace {

using namespace stepbody;

__global__ __launch_bounds__(256) void k_predict(h6_state st, int n, int64_t t_tick, double dt,
                                                 int shared, h6_pred out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double d = shared ? dt : (double)(t_tick - st.t[i]) * kTick;
    predict_one(st, i, d, out);
}

template <bool SHARED>
__global__ __launch_bounds__(256) void k_correct(h6_state st, const int32_t *__restrict__ active,
                                                 int n_act, h6_force f, int64_t t_next, double dt_sh,
                                                 double eta6, int lev_min, int lev_max,
                                                 int32_t *flags) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_act) return;
    const int i = SHARED ? k : active[k];
    double fa[3], fj[3], fs[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        fa[c] = f.a[c][k];
        fj[c] = f.j[c][k];
        fs[c] = f.s[c][k];
    }
    correct_one<SHARED>(st, i, fa, fj, fs, t_next, dt_sh, eta6, lev_min, lev_max, flags);
}

// ---------------------------------------------------------------- start-up steps
// dt^2 = eta_s^2 (|a||s| + |j|^2) / (|j||c| + |s|^2)  (4th-order criterion)
__global__ __launch_bounds__(256) void k_initial_steps(h6_state st, int n, double eta2, int lev_min,
                                                       int lev_max, int32_t *flags) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double a0 = st.a[0][i], a1 = st.a[1][i], a2 = st.a[2][i];
    const double j0 = st.j[0][i], j1 = st.j[1][i], j2 = st.j[2][i];
    const double s0 = st.s[0][i], s1 = st.s[1][i], s2 = st.s[2][i];
    const double c0 = st.c[0][i], c1 = st.c[1][i], c2 = st.c[2][i];
    const double num = fma(norm3(a0, a1, a2), norm3(s0, s1, s2), fma(j0, j0, fma(j1, j1, j2 * j2)));
    const double den = fma(norm3(j0, j1, j2), norm3(c0, c1, c2), fma(s0, s0, fma(s1, s1, s2 * s2)));
    int L = level_from_power((num / den) * eta2, 2, lev_min, lev_max + 1);
    if (L > lev_max) {
        atomicOr(flags, kFlagDtMin);
        L = lev_max;
    }
    st.t[i] = 0;
    st.dt[i] = (int64_t)1 << (kTickBits - L);
}

// ---------------------------------------------------------------- scheduler
// Up to kSchedSmall particles, one workgroup finds the earliest due time
// t + dt and writes the particles due then, in index order. Beyond, two passes
// over fixed chunks of kSchedChunk particles per workgroup:
//   1. each chunk finds its minimum due time and how many of its particles
//      are due then; the last workgroup to finish takes the
//      global minimum t_next, gives every chunk whose minimum equals t_next
//      an offset (exclusive scan of their counts, in chunk order) and
//      publishes t_next and n_act;
//   2. each such chunk writes its due particles, in index order, at its
//      offset.
// Both are bound by latency: due times are read once and held in registers,
// and the scan over chunks is parallel (n = 4096: 15 -> 7 us for both).
constexpr int kSchedThreads = 256;
constexpr int kSchedPer = 16;  // particles of a chunk per thread
constexpr int kSchedChunk = kSchedThreads * kSchedPer;
constexpr int kSchedSmallThreads = 1024;
constexpr int kSchedSmallPer = 8;
constexpr int kSchedSmall = kSchedSmallThreads * kSchedSmallPer;

// Ordered hand-off between workgroups of one launch: every workgroup
// publishes its result, then increments the counter with a device-scope
// release; the one that sees count == nblocks - 1 is the last, acquires,
// and may read all published results. It resets the counter for the next
// launch.
__device__ __forceinline__ bool last_workgroup(unsigned *counter, unsigned nblocks) {
    __shared__ bool is_last;
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        const unsigned prev =
            __hip_atomic_fetch_add(counter, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        is_last = (prev == nblocks - 1);
        if (is_last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (is_last) __threadfence();
    return is_last;
}

template <typename T>
__device__ __forceinline__ T load_agent(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int64_t wave_min_i64(int64_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int64_t o = __shfl_xor(v, off, 64);
        v = o < v ? o : v;
    }
    return v;
}

template <int THREADS>
__device__ __forceinline__ int64_t block_min_i64(int64_t v) {
    __shared__ int64_t wmin[THREADS / 64];
    v = wave_min_i64(v);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) wmin[w] = v;
    __syncthreads();
    int64_t r = wmin[0];
#pragma unroll
    for (int q = 1; q < THREADS / 64; ++q) r = wmin[q] < r ? wmin[q] : r;
    __syncthreads();
    return r;
}

__device__ __forceinline__ int block_sum_i32(int v) {
    __shared__ int wsum[kSchedThreads / 64];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
    __syncthreads();
    int r = 0;
#pragma unroll
    for (int q = 0; q < kSchedThreads / 64; ++q) r += wsum[q];
    __syncthreads();
    return r;
}

// out[0] = t_next, out[1] = n_act; host_out (pinned host memory) the same
__global__ __launch_bounds__(kSchedThreads) void k_sched_select(const int64_t *__restrict__ t,
                                                                const int64_t *__restrict__ dt,
                                                                int n, int64_t *chunk_min,
                                                                int32_t *chunk_cnt,
                                                                int32_t *chunk_off,
                                                                unsigned *counter, int64_t *out,
                                                                int64_t *host_out) {
    const int base = blockIdx.x * kSchedChunk;
    int64_t due[kSchedPer], v = INT64_MAX;
#pragma unroll
    for (int r = 0; r < kSchedPer; ++r) {
        const int i = base + r * kSchedThreads + threadIdx.x;
        due[r] = i < n ? t[i] + dt[i] : INT64_MAX;
        v = due[r] < v ? due[r] : v;
    }
    const int64_t cmin = block_min_i64<kSchedThreads>(v);
    int cnt = 0;
#pragma unroll
    for (int r = 0; r < kSchedPer; ++r)
        cnt += (base + r * kSchedThreads + (int)threadIdx.x < n && due[r] == cmin);
    cnt = block_sum_i32(cnt);
    if (threadIdx.x == 0) {
        chunk_min[blockIdx.x] = cmin;
        chunk_cnt[blockIdx.x] = cnt;
    }
    if (!last_workgroup(counter, gridDim.x)) return;
    int64_t r = INT64_MAX;
    for (int b = threadIdx.x; b < (int)gridDim.x; b += kSchedThreads) {
        const int64_t x = load_agent(&chunk_min[b]);
        r = x < r ? x : r;
    }
    r = block_min_i64<kSchedThreads>(r);
    // exclusive scan over the chunks that hold t_next, kSchedThreads at a time
    __shared__ int wtot[kSchedThreads / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int run = 0;
    for (int b0 = 0; b0 < (int)gridDim.x; b0 += kSchedThreads) {
        const int b = b0 + threadIdx.x;
        const bool has = b < (int)gridDim.x && load_agent(&chunk_min[b]) == r;
        const int c = has ? load_agent(&chunk_cnt[b]) : 0;
        int incl = c;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(incl, off, 64);
            incl += lane >= off ? o : 0;
        }
        if (lane == 63) wtot[w] = incl;
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int q = 0; q < kSchedThreads / 64; ++q) {
            before += q < w ? wtot[q] : 0;
            total += wtot[q];
        }
        if (b < (int)gridDim.x) chunk_off[b] = has ? run + before + incl - c : -1;
        run += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = host_out[0] = r;
        out[1] = host_out[1] = run;
    }
}

// Select and compact in one workgroup (n <= kSchedSmall).
__global__ __launch_bounds__(kSchedSmallThreads) void k_sched_small(const int64_t *__restrict__ t,
                                                                    const int64_t *__restrict__ dt,
                                                                    int n, int32_t *active,
                                                                    int64_t *host_out) {
    constexpr int kWaves = kSchedSmallThreads / 64, kCounts = kSchedSmallPer * kWaves;
    static_assert(kCounts == 128, "two counts per lane of the scanning wave");
    __shared__ int count[kCounts];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int64_t due[kSchedSmallPer], v = INT64_MAX;
#pragma unroll
    for (int r = 0; r < kSchedSmallPer; ++r) {
        const int i = r * kSchedSmallThreads + tid;
        due[r] = i < n ? t[i] + dt[i] : INT64_MAX;
        v = due[r] < v ? due[r] : v;
    }
    const int64_t tn = block_min_i64<kSchedSmallThreads>(v);
    // counts in index order (round, wave), then their exclusive scan
    int before[kSchedSmallPer];
#pragma unroll
    for (int r = 0; r < kSchedSmallPer; ++r) {
        const bool is = r * kSchedSmallThreads + tid < n && due[r] == tn;
        const unsigned long long mask = __ballot(is);
        before[r] = is ? __popcll(mask & ((1ull << lane) - 1ull)) : -1;
        if (lane == 0) count[r * kWaves + w] = __popcll(mask);
    }
    __syncthreads();
    if (w == 0) {
        const int c0 = count[2 * lane], c1 = count[2 * lane + 1];
        int incl = c0 + c1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(incl, off, 64);
            incl += lane >= off ? o : 0;
        }
        count[2 * lane] = incl - c0 - c1;
        count[2 * lane + 1] = incl - c1;
        if (lane == 63) {
            host_out[0] = tn;
            host_out[1] = incl;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSchedSmallPer; ++r)
        if (before[r] >= 0) active[count[r * kWaves + w] + before[r]] = r * kSchedSmallThreads + tid;
}

__global__ __launch_bounds__(kSchedThreads) void k_sched_compact(const int64_t *__restrict__ t,
                                                                 const int64_t *__restrict__ dt,
                                                                 int n, const int64_t *sel,
                                                                 const int32_t *chunk_off,
                                                                 int32_t *active) {
    __shared__ int wcnt[kSchedThreads / 64];
    const int off0 = chunk_off[blockIdx.x];
    if (off0 < 0) return;  // no particle of this chunk is due
    const int64_t tn = sel[0];
    const int base = blockIdx.x * kSchedChunk;
    const int end = min(n, base + kSchedChunk);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int run = off0;
    for (int r = base; r < end; r += kSchedThreads) {
        const int i = r + threadIdx.x;
        const bool due = i < end && (t[i] + dt[i] == tn);
        const unsigned long long mask = __ballot(due);
        const int before = __popcll(mask & ((1ull << lane) - 1ull));
        if (lane == 0) wcnt[w] = __popcll(mask);
        __syncthreads();
        int woff = 0, tot = 0;
#pragma unroll
        for (int q = 0; q < kSchedThreads / 64; ++q) {
            woff += q < w ? wcnt[q] : 0;
            tot += wcnt[q];
        }
        if (due) active[run + woff + before] = i;
        run += tot;
        __syncthreads();
    }
}

// ---------------------------------------------------------------- energy
constexpr int kEnergyThreads = 256;
constexpr int kEnergyBlock = 2 * kEnergyThreads;  // targets of a block, two a thread
constexpr int kEnergyUnit = 64;                   // sources a slice boundary falls on
constexpr int kEnergyMaxSplit = 64;               // source slices per pair of blocks

__device__ __forceinline__ void two_sum(double a, double b, double &s, double &e) {
    s = a + b;
    const double bp = s - a;
    e = (a - (s - bp)) + (b - bp);
}

// Potential energy W = -sum over pairs i < j of m_i m_j / sqrt(r^2+eps^2),
// each pair once: target block b (kEnergyBlock particles, two per thread)
// meets the sources from its own first one on, and among its own only the
// sources j > i. Blocks b and nb-1-b share a workgroup, so that every
// workgroup has about as many sources; these are cut into gridDim.y slices
// of whole units of kEnergyUnit. Sums over a tile are plain, over tiles
// compensated. Kinetic m v^2/2 and angular momentum m x cross v of the
// workgroup's particles are taken by the first slice. Workgroup sums as
// compensated (hi, lo) trees; the last workgroup adds them in order.
// Bound by FP64 issue (about 13 operations a pair); with one target a thread
// the two LDS reads a pair bounded it instead (n = 65536: 1063 -> 938 us; the
// call at n = 16384 134 -> 116 us, at 1024 54 -> 39 us).
__global__ __launch_bounds__(kEnergyThreads) void k_energy(h6_state st, int n, double eps2,
                                                           double *partial, unsigned *counter,
                                                           double *out) {
    __shared__ double4 tile[kEnergyThreads];  // x, y, z, m
    __shared__ double red_hi[5][kEnergyThreads];
    __shared__ double red_lo[5][kEnergyThreads];
    const int tid = threadIdx.x;
    const int nb = (n + kEnergyBlock - 1) / kEnergyBlock;
    constexpr int kBlockUnits = kEnergyBlock / kEnergyUnit;
    const int nu = (n + kEnergyUnit - 1) / kEnergyUnit;
    const int b0 = (int)blockIdx.x, b1 = nb - 1 - (int)blockIdx.x;
    const bool two = b1 > b0;
    // units from each block's first source on, and this slice's part of both
    const int nu0 = nu - b0 * kBlockUnits, nut = nu0 + (two ? nu - b1 * kBlockUnits : 0);
    const int vu0 = (int)(((int64_t)blockIdx.y * nut) / gridDim.y);
    const int vu1 = (int)(((int64_t)(blockIdx.y + 1) * nut) / gridDim.y);
    double v[5] = {0, 0, 0, 0, 0};
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {  // the slice's sources of block b0, then of b1
        if (half == 1 && !two) break;
        const int b = half ? b1 : b0;
        const int ja = b * kEnergyBlock + kEnergyUnit * (half ? max(vu0 - nu0, 0) : vu0);
        const int je = b * kEnergyBlock + kEnergyUnit * (half ? vu1 - nu0 : min(vu1, nu0));
        int id[2];
        double xi[2][3], hi[2] = {0, 0}, lo[2] = {0, 0};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            id[u] = b * kEnergyBlock + u * kEnergyThreads + tid;
            const int c = id[u] < n ? id[u] : n - 1;
#pragma unroll
            for (int q = 0; q < 3; ++q) xi[u][q] = st.x[q][c];
        }
        for (int jt = ja; jt < je; jt += kEnergyThreads) {
            const int cnt = min(kEnergyThreads, je - jt);  // whole units
            __syncthreads();
            const int jj = jt + tid;
            tile[tid] = jj < n ? make_double4(st.x[0][jj], st.x[1][jj], st.x[2][jj], st.m[jj])
                               : make_double4(1.0e18, 1.0e18, 1.0e18, 0.0);
            __syncthreads();
            double acc[2] = {0.0, 0.0};
            if (jt < (b + 1) * kEnergyBlock) {  // the block's own: sources after the target only
#pragma unroll 4
                for (int q = 0; q < cnt; ++q) {
                    const double4 r = tile[q];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const double dx = r.x - xi[u][0], dy = r.y - xi[u][1], dz = r.z - xi[u][2];
                        double r2 = fma(dz, dz, fma(dy, dy, fma(dx, dx, eps2)));
                        const bool take = jt + q > id[u];
                        r2 = take ? r2 : 1.0;
                        acc[u] = fma(take ? r.w : 0.0, rsqrt_f64(r2), acc[u]);
                    }
                }
            } else {
#pragma unroll 4
                for (int q = 0; q < cnt; ++q) {
                    const double4 r = tile[q];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const double dx = r.x - xi[u][0], dy = r.y - xi[u][1], dz = r.z - xi[u][2];
                        const double r2 = fma(dz, dz, fma(dy, dy, fma(dx, dx, eps2)));
                        acc[u] = fma(r.w, rsqrt_f64(r2), acc[u]);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                double s, e;
                two_sum(hi[u], acc[u], s, e);
                hi[u] = s;
                lo[u] += e;
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (id[u] >= n) continue;
            const double m = st.m[id[u]];
            v[1] = fma(-m, hi[u] + lo[u], v[1]);
            if (blockIdx.y == 0) {
                const double vx = st.v[0][id[u]], vy = st.v[1][id[u]], vz = st.v[2][id[u]];
                v[0] += 0.5 * m * fma(vx, vx, fma(vy, vy, vz * vz));
                v[2] += m * (xi[u][1] * vz - xi[u][2] * vy);
                v[3] += m * (xi[u][2] * vx - xi[u][0] * vz);
                v[4] += m * (xi[u][0] * vy - xi[u][1] * vx);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        red_hi[q][tid] = v[q];
        red_lo[q][tid] = 0.0;
    }
    __syncthreads();
    for (int w = kEnergyThreads / 2; w >= 1; w >>= 1) {
        if (tid < w) {
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                double s, e;
                two_sum(red_hi[q][tid], red_hi[q][tid + w], s, e);
                red_hi[q][tid] = s;
                red_lo[q][tid] += red_lo[q][tid + w] + e;
            }
        }
        __syncthreads();
    }
    const int wg = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    const int n_wg = (int)(gridDim.x * gridDim.y);
    if (tid < 5) {
        partial[2 * (wg * 5 + tid)] = red_hi[tid][0];
        partial[2 * (wg * 5 + tid) + 1] = red_lo[tid][0];
    }
    if (!last_workgroup(counter, n_wg)) return;
    // the last workgroup: every thread takes every 256th workgroup sum, then
    // the same fixed tree (deterministic for a launch shape)
    double hi[5] = {0, 0, 0, 0, 0}, lo[5] = {0, 0, 0, 0, 0};
    for (int b = tid; b < n_wg; b += kEnergyThreads) {
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            double s, e;
            two_sum(hi[q], load_agent(&partial[2 * (b * 5 + q)]), s, e);
            hi[q] = s;
            lo[q] += e + load_agent(&partial[2 * (b * 5 + q) + 1]);
        }
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        red_hi[q][tid] = hi[q];
        red_lo[q][tid] = lo[q];
    }
    __syncthreads();
    for (int w = kEnergyThreads / 2; w >= 1; w >>= 1) {
        if (tid < w) {
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                double s, e;
                two_sum(red_hi[q][tid], red_hi[q][tid + w], s, e);
                red_hi[q][tid] = s;
                red_lo[q][tid] += red_lo[q][tid + w] + e;
            }
        }
        __syncthreads();
    }
    if (tid < 5) out[tid] = red_hi[tid][0] + red_lo[tid][0];  // pinned host memory
}

}  // namespace

int sched_blocks_for(int64_t n) { return (int)((n + kSchedChunk - 1) / kSchedChunk); }
// workgroup partial slots for n particles (target blocks x the most slices)
int energy_blocks_for(int64_t n) {
    const int64_t nb = (n + kEnergyBlock - 1) / kEnergyBlock;
    return (int)((nb + 1) / 2) * kEnergyMaxSplit;
}

hipError_t launch_predict(h6_ctx ctx, const h6_state *st, int n, int64_t t_tick, double dt,
                          bool shared, const h6_pred *out) {
    hipLaunchKernelGGL(k_predict, dim3((n + 255) / 256), dim3(256), 0, ctx->stream, *st, n, t_tick,
                       dt, shared ? 1 : 0, *out);
    return hipGetLastError();
}

hipError_t launch_correct(h6_ctx ctx, h6_state *st, const int32_t *active, int n_act,
                          const h6_force *f, int64_t t_next, double dt, const h6_params *prm,
                          bool shared) {
    if (n_act <= 0) return hipSuccess;
    dim3 grid((n_act + 255) / 256);
    if (shared) {
        hipLaunchKernelGGL(k_correct<true>, grid, dim3(256), 0, ctx->stream, *st, active, n_act, *f,
                           (int64_t)0, dt, 0.0, 0, 0, ctx->flags);
    } else {
        const double e = prm->eta, e2 = e * e;
        hipLaunchKernelGGL(k_correct<false>, grid, dim3(256), 0, ctx->stream, *st, active, n_act,
                           *f, t_next, 0.0, e2 * e2 * e2, prm->lev_min, prm->lev_max, ctx->flags);
    }
    return hipGetLastError();
}

hipError_t launch_initial_steps(h6_ctx ctx, h6_state *st, int n, double eta_s, int lev_min,
                                int lev_max) {
    hipLaunchKernelGGL(k_initial_steps, dim3((n + 255) / 256), dim3(256), 0, ctx->stream, *st, n,
                       eta_s * eta_s, lev_min, lev_max, ctx->flags);
    return hipGetLastError();
}

// Scratch layout: ctx->sched64[0..1] = {t_next, n_act} (also written to
// the pinned host buffer), ctx->sched64[2..] chunk minima; ctx->sched32[0..nb) chunk counts,
// [nb..2nb) chunk offsets; counters[0] is the hand-off counter.
hipError_t launch_next_block(h6_ctx ctx, const h6_state *st, int n, int32_t *active) {
    int64_t *host_out = (int64_t *)((char *)ctx->host_dev + kHostBlock);
    if (n <= kSchedSmall) {
        hipLaunchKernelGGL(k_sched_small, dim3(1), dim3(kSchedSmallThreads), 0, ctx->stream, st->t,
                           st->dt, n, active, host_out);
        return hipGetLastError();
    }
    const int nb = sched_blocks_for(n);
    int64_t *sel = ctx->sched64;
    int64_t *cmin = ctx->sched64 + 2;
    int32_t *ccnt = ctx->sched32;
    int32_t *coff = ctx->sched32 + nb;
    hipLaunchKernelGGL(k_sched_select, dim3(nb), dim3(kSchedThreads), 0, ctx->stream, st->t, st->dt,
                       n, cmin, ccnt, coff, ctx->counters, sel, host_out);
    hipLaunchKernelGGL(k_sched_compact, dim3(nb), dim3(kSchedThreads), 0, ctx->stream, st->t,
                       st->dt, n, (const int64_t *)sel, (const int32_t *)coff, active);
    return hipGetLastError();
}

hipError_t launch_energy(h6_ctx ctx, const h6_state *st, int n) {
    const int nb = (n + kEnergyBlock - 1) / kEnergyBlock;
    const int pairs = (nb + 1) / 2;  // workgroups per slice: blocks b and nb-1-b together
    // about four workgroups of four waves per compute unit, at most one slice
    // per unit of a workgroup's sources (the middle block has the fewest)
    int split = std::max(1, std::min(kEnergyMaxSplit, (4 * ctx->n_cu + pairs - 1) / pairs));
    split = std::min(split, std::max(1, nb / 2 * (kEnergyBlock / kEnergyUnit)));
    hipLaunchKernelGGL(k_energy, dim3(pairs, split), dim3(kEnergyThreads), 0, ctx->stream, *st, n,
                       ctx->eps2, ctx->ered, ctx->counters + 2, (double *)((char *)ctx->host_dev + kHostEnergy));
    return hipGetLastError();
}

}  // namespace h6
