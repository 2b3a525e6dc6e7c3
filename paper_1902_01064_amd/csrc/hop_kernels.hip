// HIP kernels of the Hop hot path for gfx950 (CDNA4, 64-wide wavefronts, 256 CUs in 8 XCDs).
//
// About half a flop per byte, so none uses MFMA: the kernels of one wave are bound by HBM (small ones by their launch
// and their chain of dependent loads) and do coalesced 128-bit streaming, wavefront reductions and LDS staging of small
// tables; the generator of synthetic gradients and the whole pass in one launch are bound by instruction issue.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "hop_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kXcd = 8;                 // workgroups are dealt round-robin to the 8 XCDs

typedef float vf4 __attribute__((ext_vector_type(4)));
// Every vector handed to these kernels is device (global) memory, but the pointers come out of job
// descriptors, where the compiler only knows them as generic: without the address-space cast it emits
// flat_load / flat_store, which also count on the LDS counter, so every wait for a scalar load (the next
// pointer, the next weight) would wait for the vector loads in flight too.
#ifndef HOP_FLAT_ACCESS
#define HOP_GLOBAL __attribute__((address_space(1)))
#else
#define HOP_GLOBAL
#endif
typedef const HOP_GLOBAL vf4* gvec_in;
typedef HOP_GLOBAL vf4* gvec_out;
__device__ __forceinline__ float4 ld4(const float* p, int64_t i4) {
    vf4 v = ((gvec_in)p)[i4];
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st4(float* p, int64_t i4, float4 v) {
    vf4 t = {v.x, v.y, v.z, v.w};
    ((gvec_out)p)[i4] = t;
}
// Four columns from column c on of a vector that need not be 16-byte aligned (the rows of a dense data set when d is no
// multiple of 4): global memory takes 128-bit accesses at any multiple of 4 bytes.  `n`: columns that exist, at least 1.
typedef float vf4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 ldu4(const float* p, int64_t c) {
    const vf4u v = *(const HOP_GLOBAL vf4u*)(p + c);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float4 ldu4_stream(const float* p, int64_t c) {
    const vf4u v = __builtin_nontemporal_load((const HOP_GLOBAL vf4u*)(p + c));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float4 ldu4(const float* p, int64_t c, int n) {
    if (n >= 4) return ldu4(p, c);
    return make_float4(p[c], n > 1 ? p[c + 1] : 0.f, n > 2 ? p[c + 2] : 0.f, 0.f);
}
__device__ __forceinline__ void stu4(float* p, int64_t c, int n, float4 v) {
    if (n >= 4) {
        const vf4u t = {v.x, v.y, v.z, v.w};
        *(HOP_GLOBAL vf4u*)(p + c) = t;
        return;
    }
    p[c] = v.x;
    if (n > 1) p[c + 1] = v.y;
    if (n > 2) p[c + 2] = v.z;
}
__device__ __forceinline__ float4 fma4(float a, float4 x, float4 y) {
    return make_float4(fmaf(a, x.x, y.x), fmaf(a, x.y, y.y), fmaf(a, x.z, y.z), fmaf(a, x.w, y.w));
}
// streaming (non-temporal) 128-bit accesses for data touched once
__device__ __forceinline__ float4 ld4_stream(const float* p, int64_t i4) {
    vf4 v = __builtin_nontemporal_load((gvec_in)p + i4);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st4_stream(float* p, int64_t i4, float4 v) {
    vf4 t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, (gvec_out)p + i4);
}
// NEAR: see hop_stays_near (a template argument: of a run-time choice the compiler makes one store, without the hint)
template <bool NEAR>
__device__ __forceinline__ void st4_once(float* p, int64_t i4, float4 v) {
    if (NEAR) st4(p, i4, v);
    else st4_stream(p, i4, v);
}

// A launch's grid over jobs and column chunks is (chunks of one round, jobs, rounds), so a workgroup's job and chunk are its
// block index: worked out from one number they took up to four divisions, 100 to 200 scalar instructions in front of the first
// load of every workgroup (us per pass: 4 workers x 1024 columns, dense, 316 -> 308; 8 x 30 011 2085 -> 2022; 16 x 65536
// 3544 -> 3480; external gradients 16 x 4 M 2983 -> 2933; 16 x 2^20 sparse 6921 -> 6870).  Workgroups are dealt out in the order x, y, z, one to each of the 8 XCDs in turn, and a round is a
// multiple of 8 chunks: those dealt out at the same moment work on 8 different chunks, and one XCD sees the same chunk for
// all jobs of a wave back to back, so a source vector read by several jobs (a worker and its neighbours all average it) is
// fetched from HBM once per XCD-local L2 instead of once per job.
constexpr int64_t kMaxGridYZ = 65535;

// (8, jobs, chunks / 8), wider rounds where a grid has no room for as many; false: too many workgroups
inline bool chunk_grid(int n_jobs, int64_t n_chunks, dim3* grid) {
    int64_t width = kXcd;
    while ((n_chunks + width - 1) / width > kMaxGridYZ) width *= 2;
    const int64_t rounds = (n_chunks + width - 1) / width;
    if (width * n_jobs * rounds > 0x7FFFFFFFll) return false;
    *grid = dim3((unsigned)width, (unsigned)n_jobs, (unsigned)rounds);
    return true;
}
// chunk of this workgroup of such a grid (`width`: its x); it may lie past the last one
__device__ __forceinline__ int64_t grid_chunk(int width) { return (int64_t)blockIdx.z * width + blockIdx.x; }

// Rounds in which every XCD takes a run of consecutive chunks: longer contiguous pieces of every stream are in flight at a
// time.  The last, partly filled round is dealt out evenly (shorter runs on all XCDs, not full runs on the first few).
struct Runs {
    int n_chunks, run, whole, tail;         // chunks, length of a run, whole rounds, length of a run in the round behind them
    int front;                              // rounds of other workgroups in front
};
// its members as arguments of a kernel: one by one, so that they are in scalar registers when a wavefront starts
#define HOP_RUNS_IN int n_chunks, int run, int whole, int tail
#define HOP_RUNS Runs{n_chunks, run, whole, tail, 0}
#define HOP_RUNS_OF(r) r.n_chunks, r.run, r.whole, r.tail
// grid.z: `front` workgroups for something else, filled up to whole rounds, then the rounds; false: too many workgroups
inline bool run_grid(int n_jobs, int64_t n_chunks, int run, int64_t front, Runs* r, dim3* grid) {
    for (;; run *= 2) {
        const int64_t span = (int64_t)kXcd * run, round = span * n_jobs;
        const int64_t ahead = (front + round - 1) / round, z = ahead + (n_chunks + span - 1) / span;
        if (z * round > 0x7FFFFFFFll) return false;
        if (z > kMaxGridYZ) continue;
        *r = Runs{(int)n_chunks, run, (int)(n_chunks / span), (int)((n_chunks % span + kXcd - 1) / kXcd), (int)ahead};
        *grid = dim3((unsigned)span, (unsigned)n_jobs, (unsigned)z);
        return true;
    }
}
// index of this workgroup in the order in which they are dealt out
__device__ __forceinline__ unsigned grid_index(const Runs& r, int n_jobs) {
    return (blockIdx.z * n_jobs + blockIdx.y) * (unsigned)(kXcd * r.run) + blockIdx.x;
}
// chunk of this workgroup in round `round`; -1: none
__device__ __forceinline__ int run_chunk(const Runs& r, int round) {
    const int xcd = blockIdx.x % kXcd, sub = blockIdx.x / kXcd;
    if (round < r.whole) return (round * kXcd + xcd) * r.run + sub;
    const int chunk = r.whole * kXcd * r.run + xcd * r.tail + sub;
    return sub < r.tail && chunk < r.n_chunks ? chunk : -1;
}

// ------------------------------------------------------------------------ Reduce + Apply ----
// out[c] = sum_a w_a src_a[c] - eta g[c]   (Figure "Standard Decentralized Training", steps 2-3;
// weights from Eq. 2 times the mixing matrix, already normalised on the host).
//
// A thread takes one float4 of every vector, a workgroup 4 KB: few registers, so many workgroups at a time, is what counts
// (records with a velocity, us per pass with 4, 2 and 1: 64 workers x 50 000 columns, external gradients, 290 / 242 / 215;
// 16 x 300 000 256 / 229 / 215; 32 x 4 M 5160 / 5020 / 4970; 16 x 2^20, sparse, 935 / 858 / 813).  g, velocity and result
// non-temporal (each touched once).  Measured on 32 jobs x 25 M columns with ~7.6 shared sources each: job-major workgroups
// are 2.3x slower than the grid above and chunk-major ones that ignore the XCDs 1.45x slower.
template <int A, bool MOM, bool NEAR>
__device__ __forceinline__ void mix_tile(const HopMixJob* __restrict__ job, int64_t i) {
    const float* g = job->g;
    const float neg_eta = -job->eta;
    float* vel = job->vel;
    const float4 x0 = ld4(job->src[0], i);
    const float w0 = job->w[0];
    float4 acc = make_float4(w0 * x0.x, w0 * x0.y, w0 * x0.z, w0 * x0.w);
#pragma unroll
    for (int a = 1; a < A; ++a) acc = fma4(job->w[a], ld4(job->src[a], i), acc);
    if (MOM) {
        // v <- mu v + g (a missing g counts as zero), Apply with the new velocity
        float4 v = ld4_stream(vel, i);
        float4 gg = g != nullptr ? ld4_stream(g, i) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (job->lam_fold != 0.f) gg = fma4(job->lam_fold, x0, gg);    // lambda w of a gradient whose sparse part is scattered later
        v = fma4(job->mu, v, gg);
        st4_stream(vel, i, v);
        acc = fma4(neg_eta, v, acc);
    } else if (g != nullptr) {
        acc = fma4(neg_eta, ld4_stream(g, i), acc);
    }
    st4_once<NEAR>(job->out, i, acc);
}

// more than 12 sources: a loop over the sources instead of an unrolled chain
template <bool NEAR>
__device__ __forceinline__ void mix_tile_any(const HopMixJob* __restrict__ job, int64_t i) {
    const int A = job->A;
    const float* g = job->g;
    const float neg_eta = -job->eta;
    const float4 x0 = ld4(job->src[0], i);
    const float w0 = job->w[0];
    float4 acc = make_float4(w0 * x0.x, w0 * x0.y, w0 * x0.z, w0 * x0.w);
    for (int a = 1; a < A; ++a) acc = fma4(job->w[a], ld4(job->src[a], i), acc);
    if (job->vel != nullptr) {
        float4 gg = g != nullptr ? ld4_stream(g, i) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (job->lam_fold != 0.f) gg = fma4(job->lam_fold, x0, gg);
        const float4 v = fma4(job->mu, ld4_stream(job->vel, i), gg);
        st4_stream(job->vel, i, v);
        acc = fma4(neg_eta, v, acc);
    } else if (g != nullptr) {
        acc = fma4(neg_eta, ld4_stream(g, i), acc);
    }
    st4_once<NEAR>(job->out, i, acc);
}

// Work of one workgroup of the mix in round `round` of the chunks (the launch may hold other workgroups in front of them).
template <bool NEAR>
__device__ __forceinline__ void mix_block(const HopMixJob* __restrict__ jobs, int64_t d, const Runs& runs, int round) {
    const int chunk = run_chunk(runs, round);
    if (chunk < 0) return;
    const HopMixJob* job = jobs + blockIdx.y;
    const int64_t n4 = d >> 2, i = (int64_t)chunk * kThreads + threadIdx.x;
    if (i < n4) {
#define HOP_MIX_CASE(AA)                                           \
    case AA:                                                       \
        if (job->vel != nullptr) mix_tile<AA, true, NEAR>(job, i); \
        else mix_tile<AA, false, NEAR>(job, i);                    \
        break;
        switch (job->A) {
            HOP_MIX_CASE(1) HOP_MIX_CASE(2) HOP_MIX_CASE(3) HOP_MIX_CASE(4) HOP_MIX_CASE(5) HOP_MIX_CASE(6)
            HOP_MIX_CASE(7) HOP_MIX_CASE(8) HOP_MIX_CASE(9) HOP_MIX_CASE(10) HOP_MIX_CASE(11) HOP_MIX_CASE(12)
            default: mix_tile_any<NEAR>(job, i); break;
        }
#undef HOP_MIX_CASE
    }
    // the d mod 4 trailing columns, one thread each, by the workgroup of the last chunk
    if (chunk == runs.n_chunks - 1) {
        int64_t c = (n4 << 2) + threadIdx.x;
        if (threadIdx.x < 4 && c < d) {
            float acc = job->w[0] * job->src[0][c];
            for (int a = 1; a < job->A; ++a) acc = fmaf(job->w[a], job->src[a][c], acc);
            if (job->vel != nullptr) {
                float v = fmaf(job->mu, job->vel[c],
                               fmaf(job->lam_fold, job->src[0][c], job->g != nullptr ? job->g[c] : 0.f));
                job->vel[c] = v;
                acc = fmaf(-job->eta, v, acc);
            } else if (job->g != nullptr) {
                acc = fmaf(-job->eta, job->g[c], acc);
            }
            job->out[c] = acc;
        }
    }
}

// Runs of its 4 KB chunks: 32 on vectors of 16 MB and more (against 16: 32 workers x 8 M columns 7714 -> 7645 us per pass, 16 x
// 12 M 4912 -> 4868), 4 on shorter ones (8: 32 x 50 000 columns 170.5 -> 171.9)
inline bool mix_grid(int n_jobs, int64_t d, int64_t front, Runs* runs, dim3* grid) {
    const int64_t n4 = d >> 2, n_chunks = n4 > kThreads ? (n4 + kThreads - 1) / kThreads : 1;
    return run_grid(n_jobs, n_chunks, hop_stays_near(n_jobs, d, 3) ? 1 : n4 >= (1 << 20) ? 32 : 4, front, runs, grid);
}

template <bool NEAR>
__global__ __launch_bounds__(kThreads) void mix_kernel(const HopMixJob* __restrict__ jobs, int64_t d, HOP_RUNS_IN) {
    mix_block<NEAR>(jobs, d, HOP_RUNS, (int)blockIdx.z);
}

// ---------------------------------------------------------- Reduce + Apply, records in pairs ----
// The plain path (no velocity).  Neighbouring workers average almost the same vectors (on a ring i and
// i + 1 share x_i and x_{i+1}), so the host packs a wave's records two by two where their source sets
// overlap and the union has at most kPairU vectors.  One workgroup loads the union for a column chunk (16 KB
// in long launches, pair_vec)
// once into registers and forms both sums from there; a source shared inside the pair then costs one L2
// request instead of two.  Against the record-by-record kernel above this also changes how the work is issued:
//  - the union size is a compile-time constant (switch over U), every pointer and weight is read by one batch
//    of scalar loads ahead of the first vector load, and interior chunks take a path without bounds checks,
//    so a wavefront has all its 128-bit loads in flight after one scalar wait instead of one per source;
//  - every XCD walks `run` consecutive chunks per job group (run chosen by the host so that run x 16 KB x
//    distinct sources of the wave stays near 3 MB of the XCD's 4 MB L2).
// Measured on the 134 waves of the 32-worker, 25 M-parameter workload: 1.51 ms -> 1.41 ms per launch.
// Terms are added in the order of the union (the first record's own order; the second record's sources fall
// where the union has them), in fp32 FMAs starting from zero.
constexpr int kPairU = HOP_PAIR_U;

template <int VEC, int U, bool FULL, bool NEAR, class Job>
__device__ __forceinline__ void pair_tile(Job job, int64_t first4, int64_t n4) {
    const int G = job->G;
    const float* src[U];
#pragma unroll
    for (int u = 0; u < U; ++u) src[u] = job->src[u];
    const float* gp[2];
    float* op[2];
    uint32_t mk[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) { gp[r] = job->g[r]; op[r] = job->out[r]; mk[r] = job->mask[r]; }
    const float neg_eta = -job->eta;
    const int64_t i0 = first4 + threadIdx.x;
    float4 x[U][VEC];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            x[u][v] = (FULL || i0 + v * kThreads < n4) ? ld4(src[u], i0 + v * kThreads) : make_float4(0.f, 0.f, 0.f, 0.f);
    float4 gv[2][VEC];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        if (r < G && gp[r] != nullptr) {
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                gv[r][v] = (FULL || i0 + v * kThreads < n4) ? ld4_stream(gp[r], i0 + v * kThreads)
                                                            : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        if (r < G) {
            float wr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) wr[u] = job->w[r][u];
            float4 acc[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if ((mk[r] >> u) & 1u) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        acc[v].x = fmaf(wr[u], x[u][v].x, acc[v].x);
                        acc[v].y = fmaf(wr[u], x[u][v].y, acc[v].y);
                        acc[v].z = fmaf(wr[u], x[u][v].z, acc[v].z);
                        acc[v].w = fmaf(wr[u], x[u][v].w, acc[v].w);
                    }
                }
            }
            if (gp[r] != nullptr) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    acc[v].x = fmaf(neg_eta, gv[r][v].x, acc[v].x);
                    acc[v].y = fmaf(neg_eta, gv[r][v].y, acc[v].y);
                    acc[v].z = fmaf(neg_eta, gv[r][v].z, acc[v].z);
                    acc[v].w = fmaf(neg_eta, gv[r][v].w, acc[v].w);
                }
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                if (FULL || i0 + v * kThreads < n4) st4_once<NEAR>(op[r], i0 + v * kThreads, acc[v]);
        }
    }
}

// a single record with more than kPairU sources: a loop over the sources
template <int VEC, bool NEAR, class Job>
__device__ __forceinline__ void pair_tile_wide(Job job, int64_t first4, int64_t n4) {
    const int U = job->U;
    const float* g = job->g[0];
    const float neg_eta = -job->eta;
    for (int v = 0; v < VEC; ++v) {
        const int64_t i = first4 + (int64_t)v * kThreads + threadIdx.x;
        if (i >= n4) continue;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int u = 0; u < U; ++u) {
            const float4 xv = ld4(job->src[u], i);
            const float w = job->w[0][u];
            acc.x = fmaf(w, xv.x, acc.x);
            acc.y = fmaf(w, xv.y, acc.y);
            acc.z = fmaf(w, xv.z, acc.z);
            acc.w = fmaf(w, xv.w, acc.w);
        }
        if (g != nullptr) {
            const float4 gv = ld4_stream(g, i);
            acc.x = fmaf(neg_eta, gv.x, acc.x);
            acc.y = fmaf(neg_eta, gv.y, acc.y);
            acc.z = fmaf(neg_eta, gv.z, acc.z);
            acc.w = fmaf(neg_eta, gv.w, acc.w);
        }
        st4_once<NEAR>(job->out[0], i, acc);
    }
}

// One chunk of a job.  Job: const HopPairJob*, or HopPairArg in the kernel's argument segment.
template <int VEC, bool NEAR, class Job>
__device__ __forceinline__ void pair_chunk(Job job, int64_t d, int n_chunks, int chunk) {
    const int64_t n4 = d >> 2;
    const int64_t first4 = (int64_t)chunk * (kThreads * VEC);
    const bool full = first4 + kThreads * VEC <= n4;
    static_assert(kPairU == 12, "the switch below unrolls unions of 1..12 vectors");
#define HOP_PAIR_CASE(UU)                                            \
    case UU:                                                         \
        if (full) pair_tile<VEC, UU, true, NEAR>(job, first4, n4);   \
        else pair_tile<VEC, UU, false, NEAR>(job, first4, n4);       \
        break;
    switch (job->U) {
        HOP_PAIR_CASE(1) HOP_PAIR_CASE(2) HOP_PAIR_CASE(3) HOP_PAIR_CASE(4) HOP_PAIR_CASE(5) HOP_PAIR_CASE(6)
        HOP_PAIR_CASE(7) HOP_PAIR_CASE(8) HOP_PAIR_CASE(9) HOP_PAIR_CASE(10) HOP_PAIR_CASE(11) HOP_PAIR_CASE(12)
        default: pair_tile_wide<VEC, NEAR>(job, first4, n4); break;
    }
#undef HOP_PAIR_CASE
    // the d mod 4 trailing columns, one thread each, by the workgroup of the last chunk
    if (chunk == n_chunks - 1) {
        const int64_t c = (n4 << 2) + (threadIdx.x & 3);
        const int r = threadIdx.x >> 2;
        if (threadIdx.x < 8 && r < job->G && c < d) {
            float acc = 0.f;
            for (int u = 0; u < job->U; ++u)
                if ((job->mask[r] >> u) & 1u) acc = fmaf(job->w[r][u], job->src[u][c], acc);
            if (job->g[r] != nullptr) acc = fmaf(-job->eta, job->g[r][c], acc);
            job->out[r][c] = acc;
        }
    }
}

// Work of one workgroup in round `round` of the chunks.
template <int VEC, bool NEAR, class Job>
__device__ __forceinline__ void pair_block(Job jobs, int64_t d, const Runs& runs, int reverse, int round) {
    const int ahead = run_chunk(runs, round);
    if (ahead < 0) return;
    // consecutive launches walk the vectors in opposite directions: what the previous kernels wrote or read last
    // is still in the memory-side cache when the next launch begins there (1453 -> 1430 us per launch with the
    // gradient generator in between, 386 -> 381 us between launches of small waves)
    pair_chunk<VEC, NEAR>(jobs + blockIdx.y, d, runs.n_chunks, reverse ? runs.n_chunks - 1 - ahead : ahead);
}

template <int VEC, bool NEAR>
__global__ __launch_bounds__(kThreads) void pair_mix_kernel(const HopPairJob* __restrict__ jobs, int64_t d, int reverse,
                                                            HOP_RUNS_IN) {
    pair_block<VEC, NEAR>(jobs, d, HOP_RUNS, reverse, (int)blockIdx.z);
}

// The same for a stand-alone call: its descriptors travel as the kernel's argument, so the call allocates and copies
// nothing (16 jobs of 5 sources and a gradient on 1 M columns, through the
// Python binding: 76.8 -> 56.3 us a call, 34.8 us of them this kernel).
struct HopPairArgs {
    HopPairArg job[kPairArgs];
};
typedef const __attribute__((address_space(4))) HopPairArg* pair_args_in;

template <int VEC>
__global__ __launch_bounds__(kThreads) void pair_mix_args_kernel(HopPairArgs, int64_t d, HOP_RUNS_IN) {
    // the first argument where it lies: a copy indexed by job would go through scratch memory
    pair_block<VEC, false>((pair_args_in)__builtin_amdgcn_kernarg_segment_ptr(), d, HOP_RUNS, 0, (int)blockIdx.z);
}

// float4 per thread and vector, and with it the columns of a chunk.  Long launches: 4, 16 KB of every vector per workgroup
// (25 M columns: 8 and 32 KB are 1 to 3 % slower).  Short ones finish in one or two turns of the 2 workgroups per CU that
// the registers of that form allow, so they take smaller workgroups, more of them at a time: 16 workers x 4 M columns
// 36.5 -> 35.6 us per launch with 2, 16 x 1 M columns with CSR margins beside 12.3 -> 11.8 with 2 and 11.4 with 1; waves of
// 7 records of 2^24 columns: no difference.
// Plain launches that fit one turn stay (64 records in 32 pairs, 32768 columns: 6.9 us per wave against 7.5 with 2).
constexpr int64_t kPairShort = 8192, kPairTurn = 512;  // workgroups of 16 KB chunks
constexpr int kPairPlain = 2, kPairMargin = 1;         // the short width alone, and with margins beside
// Long launches with sparse margins beside single records: 1 too, in runs twice as long (64 workers x 2^24 columns 75.1 ->
// 73.9 ms, 64 x 2^23 10.18 -> 9.96); in pairs a source shared in registers is what counts (32 workers x 3 M columns, lock-step,
// 1.88 -> 2.24).
inline int pair_vec(int n_jobs, int64_t d, bool margins, bool single = false) {
    const int64_t blocks = n_jobs * ((d + 4095) / 4096);
    if (blocks >= kPairShort) return single ? kPairMargin : 4;
    return margins ? kPairMargin : blocks <= kPairTurn ? 4 : kPairPlain;
}

inline int64_t pair_chunks(int64_t d, int vec) {
    const int64_t per = (int64_t)kThreads * vec;
    const int64_t n = ((d >> 2) + per - 1) / per;
    return n < 1 ? 1 : n;
}

// chunks an XCD walks per job group: run x chunk x distinct sources near 3 MB of its 4 MB L2 (measured on 32
// sources: runs of 5 to 7 equal, 4 and 8 1.3 % slower, 12 10 % slower), never more than the vector has
inline int pair_run(int n_sources, int64_t n_chunks, int vec) {
    int run = (192 * 4 / vec + n_sources / 2) / (n_sources < 1 ? 1 : n_sources);
    if (run > 8 * 4 / vec) run = 8 * 4 / vec;
    const int64_t room = n_chunks / kXcd;
    if (run > room) run = (int)room;
    return run < 1 ? 1 : run;
}

// A launch over pairs.  `may_near`: whether the results may stay in the L2s (a few jobs as an argument are a call by itself, which waits
// for them to get out: 16 x 400 000 columns 34.0 -> 34.9 us); margins: `front` workgroups of them in front; single: sparse margins
// beside single records.
struct PairShape {
    int vec;
    bool near;
    Runs runs;
    dim3 grid;
};
inline bool pair_shape(PairShape* p, int n_jobs, int n_sources, int64_t d, bool may_near, bool margins = false, int64_t front = 0,
                       bool single = false) {
    p->vec = pair_vec(n_jobs, d, margins, single);
    p->near = may_near && hop_stays_near(n_jobs, d);
    const int64_t n_chunks = pair_chunks(d, p->vec);
    int run = p->near ? 1 : pair_run(n_sources, n_chunks, p->vec);
    if (!p->near && p->vec != pair_vec(n_jobs, d, margins)) run *= 2;
    return run_grid(n_jobs, n_chunks, run, front, &p->runs, &p->grid);
}

// ------------------------------------------------------------------- synthetic gradient ----
// g[c] = (sum of the 12 bytes of a = h32(c ^ k0), b = h32(c ^ k1), (a + rotl(b, 16)) ^ k2  - 1530) * scale:
// integer work and one correctly rounded multiply, so any implementation agrees bit for bit.
// x ^ (x >> 16), the first step of the 32-bit hash below, is linear over xor: of a column and a key it is taken once each,
// and a hash starts from the xor of the two
__device__ __forceinline__ uint32_t fold16(uint32_t x) { return x ^ (x >> 16); }
__device__ __forceinline__ uint32_t h32_folded(uint32_t x) {
    x *= 0x7FEB352Du;
    x ^= x >> 15;
    x *= 0x846CA68Bu;
    x ^= x >> 16;
    return x;
}
__device__ __forceinline__ uint32_t byte_sum(uint32_t x, uint32_t acc) {
    return __builtin_amdgcn_sad_u8(x, 0u, acc);       // acc + sum of the four bytes of x
}
// cf, f0, f1: fold16 of the column, k0 and k1
__device__ __forceinline__ float synth_one(uint32_t cf, uint32_t f0, uint32_t f1, uint32_t k2, float scale) {
    // two hashed words and a third made of both: a + rotl(b, 16) is uniform and independent of a and of
    // b taken one at a time, so the twelve bytes are pairwise independent and the variance is exact,
    // at two thirds of the integer multiplies (32-bit multiplies are the slow instruction here)
    const uint32_t a = h32_folded(cf ^ f0), b = h32_folded(cf ^ f1);
    const uint32_t t = (a + ((b << 16) | (b >> 16))) ^ k2;
    uint32_t s = byte_sum(a, (uint32_t)-1530);
    s = byte_sum(b, s);
    s = byte_sum(t, s);
    return (float)(int)s * scale;
}

constexpr int kSynthVec = 2;
constexpr int kSynthChunk4 = kThreads * kSynthVec;

// `reverse`: walk the vectors from their end, so that the launch finishes where the Reduce + Apply that consumes
// these gradients starts and finds their last-written part still in the memory-side cache.
__device__ __forceinline__ void synth_chunk(const HopGradJob* __restrict__ job, int64_t d, int64_t n_chunks, int64_t chunk) {
    const uint32_t f0 = fold16(job->k0), f1 = fold16(job->k1), k2 = job->k2;
    const float scale = job->scale;
    float* g = job->g;
    const int64_t n4 = d >> 2;
#pragma unroll
    for (int u = 0; u < kSynthVec; ++u) {
        int64_t i = chunk * kSynthChunk4 + (int64_t)u * kThreads + threadIdx.x;
        if (i < n4) {
            uint32_t c = (uint32_t)(i << 2);
            float4 v;
            v.x = synth_one(fold16(c), f0, f1, k2, scale);
            v.y = synth_one(fold16(c + 1), f0, f1, k2, scale);
            v.z = synth_one(fold16(c + 2), f0, f1, k2, scale);
            v.w = synth_one(fold16(c + 3), f0, f1, k2, scale);
            st4(g, i, v);
        }
    }
    if (chunk == n_chunks - 1) {
        int64_t c = (n4 << 2) + threadIdx.x;
        if (threadIdx.x < 4 && c < d) g[c] = synth_one(fold16((uint32_t)c), f0, f1, k2, scale);
    }
}

__global__ __launch_bounds__(kThreads) void synth_kernel(const HopGradJob* __restrict__ jobs, int width, int reverse, int64_t d,
                                                         int64_t n_chunks) {
    const int64_t chunk = grid_chunk(width);
    if (chunk < n_chunks) synth_chunk(jobs + blockIdx.y, d, n_chunks, reverse ? n_chunks - 1 - chunk : chunk);
}

__global__ __launch_bounds__(kThreads) void synth_one_kernel(const HopGradJob job, int64_t d, int64_t n_chunks) {
    synth_chunk(&job, d, n_chunks, blockIdx.x);
}

// ------------------------------------------------------------- a whole pass, column by column ----
// Reduce, Apply and the synthetic (external, absent) gradient act on every column by itself, so a wavefront can run ALL
// records of a pass on its own 64 columns: no launch, no barrier and no trip to HBM between two waves of the schedule.
// The values that later records still read live in vector registers (the host hands out the local slots by live range:
// about 1.6 vectors per worker, whatever the ring depth); a ring slot is read once if its old content is used and written
// once if its content survives the pass.  Lanes never exchange data.
// Bound by the vector unit's issue rate: per record one instruction per source, 18 for a synthetic gradient (worked out beside
// every record) and one to apply it, each 4.1 to 4.4 cycles.  In index mode every vector instruction takes that, the multiplies
// among the 18 no more than a v_xor; outside it v_xor, shifts, adds and v_fma take 2.2 to 2.4 on a full SIMD, v_mul_lo, v_dot4,
// v_alignbit and sdwa forms 4.1.  That is why the body is written out:
//  - a record names its sources, and registers can only be named by number: the index mode of the vector unit (M0, set by
//    the scalar unit beside the arithmetic) lets v_fmac read a local slot where it is.  With the local slots in LDS a source
//    took an address, a load and the v_fmac;
//  - the number of sources is a jump into a chain of twelve, so records of different kinds need no sorting and no tests;
//  - the centred byte sum of a gradient times the scale is one of 3061 numbers, in LDS: three v_dot4 give the address, in
//    place of three v_sad_u8, a conversion and a multiplication.  Four wavefronts share the table, and nothing else.
// 32 workers x 25 M columns x 3136 records (52 local slots): 242 ms wave by wave, 83.7 with local slots in LDS, 60.5 with them
// in registers, 57.0 with the table, 54.1 with a scalar unit that only sets indexes (records count themselves, the jump
// is one s_or): 25.7 vector instructions a record, 95 % of the launch at 4 cycles; 16 workers x 2 M columns x 640 records with
// momentum: 7.7, 1.57, 0.98, 0.94, 0.90 ms.  Without a gradient
// the words of the records count (128 B each through the scalar cache): short records of up to five sources are one
// load, 16 workers x 3 M columns, 240 records of three sources: 336 -> 290 us.
// Index mode stays on all along; which operand is relative, if any, is said anew by s_set_gpr_idx_on, which writes M0 as any
// scalar instruction writes its result and holds for the next vector instruction.  (A first form that turned the mode off
// between the chains gave wrong velocities now and then, and its cause is not known: on a full GPU, 6e9 rounds of three changes
// each by off and on, with 0 to 8 scalar instructions between, ran no vector instruction in a wrong mode, nor did as many
// rounds of the changes made here.)  M0 is reserved, so no clobber: the compiler sets it before each use of its own.
// The instructions between the last v_dot4 and the ds_read of its result are needed: inside an asm block no compiler fills
// up wait states.
#define HOP_REGS_2(x, t) x #t "0", x #t "1"
#define HOP_REGS_4(x, t) HOP_REGS_2(x, t), x #t "2", x #t "3"
#define HOP_REGS_6(x, t) HOP_REGS_4(x, t), x #t "4", x #t "5"
#define HOP_REGS(x, t) HOP_REGS_6(x, t), x #t "6", x #t "7", x #t "8", x #t "9"
#define HOP_SWEEP_V64                                                                                                    \
    "v8", "v9", HOP_REGS("v", 1), HOP_REGS("v", 2), HOP_REGS("v", 3), HOP_REGS("v", 4), HOP_REGS("v", 5), HOP_REGS_4("v", 6)
#define HOP_SWEEP_V96                                                                                                    \
    HOP_SWEEP_V64, "v64", "v65", "v66", "v67", "v68", "v69", HOP_REGS("v", 7), HOP_REGS("v", 8), HOP_REGS_6("v", 9)
#define HOP_SWEEP_V128                                                                                                   \
    HOP_SWEEP_V96, "v96", "v97", "v98", "v99", HOP_REGS("v", 10), HOP_REGS("v", 11), HOP_REGS_6("v", 12), "v126", "v127"
#define HOP_SWEEP_V184                                                                                                   \
    HOP_SWEEP_V128, "v128", "v129", HOP_REGS("v", 13), HOP_REGS("v", 14), HOP_REGS("v", 15), HOP_REGS("v", 16),          \
        HOP_REGS("v", 17), HOP_REGS_4("v", 18)
#define HOP_SWEEP_S                                                                                                      \
    "s16", "s17", "s18", "s19", HOP_REGS("s", 2), "s30", "s31", "s34", "s35", "s36", "s37", "s38", "s39", HOP_REGS("s", 4), \
        HOP_REGS("s", 5), HOP_REGS("s", 6), HOP_REGS("s", 7), HOP_REGS("s", 8), HOP_REGS("s", 9)

// v8..v15 work, v16.. the local slots; s[36:67] and s[68:99] the words of the record at work and of the next one;
//   s[16:17] records  s[18:19] list  s[20:21] byte offset of the workgroup's columns  s23 list groups left  s24 -eta  s25 mu
//   s26 the chains' low address  s27 s28 the hash's factors  s29 four bytes of 4  s[30:31] an address  s[34:35] a jump
#define HOP_SWEEP_TEXT                                                                                                \
    /* eight vectors of the list at s[18:19] */                                                                       \
    ".macro hop_list_words\n"                                                                                         \
    "  s_load_dwordx16 s[68:83], s[18:19], 0\n"                                                                       \
    "  s_load_dwordx16 s[84:99], s[18:19], 64\n"                                                                      \
    "  s_add_u32 s18, s18, 128\n"                                                                                     \
    "  s_addc_u32 s19, s19, 0\n"                                                                                      \
    "  s_waitcnt lgkmcnt(0)\n"                                                                                        \
    ".endm\n"                                                                                                         \
    /* s[30:31]: the address at s[w:w+1] for the columns of this workgroup */                                         \
    ".macro hop_columns w\n"                                                                                          \
    "  s_add_u32 s30, s[\\w], s20\n"                                                                                  \
    "  s_addc_u32 s31, s[\\w+1], s21\n"                                                                               \
    ".endm\n"                                                                                                         \
    ".macro hop_list_load q\n"                                                                                        \
    "  s_cmp_eq_u64 s[68+4*\\q:69+4*\\q], 0\n"                                                                        \
    "  s_cbranch_scc1 .Lhop_wait_%=\n"                                                                                \
    "  hop_columns 68+4*\\q\n"                                                                                        \
    "  global_load_dword v[8+\\q], %[lane], s[30:31] nt\n"                                                            \
    ".endm\n"                                                                                                         \
    ".macro hop_list_put q\n"                                                                                         \
    "  s_cmp_eq_u64 s[68+4*\\q:69+4*\\q], 0\n"                                                                        \
    "  s_cbranch_scc1 .Lhop_loaded_%=\n"                                                                              \
    "  s_set_gpr_idx_on s[70+4*\\q], 8\n"                                                                             \
    "  v_mov_b32_e32 v16, v[8+\\q]\n"                                                                                 \
    ".endm\n"                                                                                                         \
    ".macro hop_list_store q\n"                                                                                       \
    "  s_cmp_eq_u64 s[68+4*\\q:69+4*\\q], 0\n"                                                                        \
    "  s_cbranch_scc1 .Lhop_out_%=\n"                                                                                 \
    "  s_set_gpr_idx_on s[70+4*\\q], 1\n"                                                                             \
    "  v_mov_b32_e32 v[8+\\q], v16\n"                                                                                 \
    "  hop_columns 68+4*\\q\n"                                                                                        \
    "  global_store_dword %[lane], v[8+\\q], s[30:31] nt\n"                                                           \
    ".endm\n"                                                                                                         \
    /* v11: where the synthetic gradient of the keys at s[w+2] is in the table */                                     \
    ".macro hop_generate w\n"                                                                                         \
    "  v_xor_b32_e32 v8, s[\\w+2], %[folded]\n"                                                                       \
    "  v_xor_b32_e32 v9, s[\\w+3], %[folded]\n"                                                                       \
    "  v_mul_lo_u32 v8, v8, s27\n"                                                                                    \
    "  v_mul_lo_u32 v9, v9, s27\n"                                                                                    \
    "  v_lshrrev_b32_e32 v10, 15, v8\n"                                                                               \
    "  v_lshrrev_b32_e32 v11, 15, v9\n"                                                                               \
    "  v_xor_b32_e32 v8, v8, v10\n"                                                                                   \
    "  v_xor_b32_e32 v9, v9, v11\n"                                                                                   \
    "  v_mul_lo_u32 v8, v8, s28\n"                                                                                    \
    "  v_mul_lo_u32 v9, v9, s28\n"                                                                                    \
    "  v_xor_b32_sdwa v8, v8, v8 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD\n"                \
    "  v_xor_b32_sdwa v9, v9, v9 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD\n"                \
    "  v_alignbit_b32 v10, v9, v9, 16\n"                                                                              \
    "  v_dot4_u32_u8 v11, v8, s29, %[table]\n"                                                                        \
    "  v_add_u32_e32 v10, v8, v10\n"                                                                                  \
    "  v_dot4_u32_u8 v11, v9, s29, v11\n"                                                                             \
    "  v_xor_b32_e32 v10, s[\\w+4], v10\n"                                                                            \
    "  v_dot4_u32_u8 v11, v10, s29, v11\n"                                                                            \
    ".endm\n"                                                                                                         \
    /* v13: the external gradient that the next record with one takes */                                              \
    ".macro hop_external w\n"                                                                                         \
    "  hop_columns \\w+2\n"                                                                                           \
    "  global_load_dword v13, %[lane], s[30:31]\n"                                                                    \
    ".endm\n"                                                                                                         \
    /* the gradient (with a velocity the velocity, which stays in its local slot too) applied to the sum; */          \
    /* dst 8: into the local slot, 0: left in v12 */                                                                  \
    ".macro hop_apply w, dst\n"                                                                                       \
    "  .if %[mode] == %[external]\n"                                                                                  \
    "  s_waitcnt vmcnt(0)\n"                                                                                          \
    "  .else\n"                                                                                                       \
    "  s_waitcnt lgkmcnt(0)\n"                                                                                        \
    "  .endif\n"                                                                                                      \
    "  .if %[mom]\n"                                                                                                  \
    "  s_set_gpr_idx_on s[\\w+15], 2\n"                                                                               \
    "  v_fma_f32 v11, s25, v16, v[11+2*(%[mode]/%[external])]\n"                                                      \
    "  s_set_gpr_idx_on s[\\w+15], 8\n"                                                                               \
    "  v_mov_b32_e32 v16, v11\n"                                                                                      \
    "  s_set_gpr_idx_on s[\\w+1], \\dst\n"                                                                            \
    "  v_fma_f32 v[12+\\dst/2], s24, v11, v12\n"                                                                      \
    "  .else\n"                                                                                                       \
    "  s_set_gpr_idx_on s[\\w+1], \\dst\n"                                                                            \
    "  v_fma_f32 v[12+\\dst/2], s24, v[11+2*(%[mode]/%[external])], v12\n"                                            \
    "  .endif\n"                                                                                                      \
    "  .if %[mode] == %[external]\n"                                                                                  \
    "  hop_external \\w\n"                                                                                            \
    "  .endif\n"                                                                                                      \
    ".endm\n"                                                                                                         \
    /* sources 2 to 12 of a record; a jump to the first entry ends the pass */                                        \
    ".macro hop_chain w\n"                                                                                            \
    "  .p2align 8\n"                                                                                                  \
    "  s_branch .Lhop_end_%=\n"                                                                                       \
    "  s_nop 0\n"                                                                                                     \
    "  .irp k, 28, 26, 24, 22, 20, 18, 16, 13, 11, 9, 7\n"                                                            \
    "  s_set_gpr_idx_idx s[\\w+\\k]\n"                                                                                \
    "  v_fmac_f32_e32 v12, s[\\w+1+\\k], v16\n"                                                                       \
    "  .endr\n"                                                                                                       \
    ".endm\n"                                                                                                         \
    /* a record as most are: with the gradient of the pass, if it has any, and its result to a local slot only */     \
    ".macro hop_short w, n\n"                                                                                         \
    "  hop_chain \\w\n"                                                                                               \
    "  .if %[mode] == %[zero]\n"                                                                                      \
    "  s_set_gpr_idx_on s[\\w+1], 8\n"                                                                                \
    "  v_mov_b32_e32 v16, v12\n"                                                                                      \
    "  .else\n"                                                                                                       \
    "  hop_apply \\w, 8\n"                                                                                            \
    "  .endif\n"                                                                                                      \
    "  .if %[mode] == %[synth]\n"                                                                                     \
    "  s_set_gpr_idx_on s29, 0\n"                                                                                     \
    "  .endif\n"                                                                                                      \
    "  s_waitcnt lgkmcnt(0)\n"                                                                                        \
    "  s_branch .Lhop_record\\n\\()_%=\n"                                                                             \
    ".endm\n"                                                                                                         \
    ".macro hop_long w\n"                                                                                             \
    "  hop_chain \\w\n"                                                                                               \
    "  s_branch .Lhop_rest\\w\\()_%=\n"                                                                               \
    ".endm\n"                                                                                                         \
    ".macro hop_rest w, n\n"                                                                                          \
    ".Lhop_rest\\w\\()_%=:\n"                                                                                         \
    "  .if %[mode] != %[zero]\n"                                                                                      \
    "  s_bitcmp1_b32 s[\\w+1], 9\n"                                                                                   \
    "  s_cbranch_scc0 .Lhop_plain\\w\\()_%=\n"                                                                        \
    "  hop_apply \\w, 0\n"                                                                                            \
    ".Lhop_plain\\w\\()_%=:\n"                                                                                        \
    "  .endif\n"                                                                                                      \
    "  s_bitcmp1_b32 s[\\w+1], 10\n"                                                                                  \
    "  s_cbranch_scc0 .Lhop_store\\w\\()_%=\n"                                                                        \
    "  s_set_gpr_idx_on s[\\w+1], 8\n"                                                                                \
    "  v_mov_b32_e32 v16, v12\n"                                                                                      \
    ".Lhop_store\\w\\()_%=:\n"                                                                                        \
    "  s_set_gpr_idx_on s29, 0\n"                                                                                     \
    "  s_bitcmp1_b32 s[\\w+1], 11\n"                                                                                  \
    "  s_cbranch_scc0 .Lhop_stored\\w\\()_%=\n"                                                                       \
    "  hop_columns \\w+30\n"                                                                                          \
    "  global_store_dword %[lane], v12, s[30:31] nt\n"                                                                \
    ".Lhop_stored\\w\\()_%=:\n"                                                                                       \
    "  s_waitcnt lgkmcnt(0)\n"                                                                                        \
    "  s_branch .Lhop_record\\n\\()_%=\n"                                                                             \
    ".endm\n"                                                                                                         \
    /* the record whose words are at s[w..], while those of the next are loaded to s[n..]; from the start of a line of the */ \
    /* instruction cache on: 25 M columns 54.3 -> 54.0 ms against 4 lines touched instead of 3 */                     \
    ".macro hop_record w, n, at\n"                                                                                    \
    "  .p2align 6\n"                                                                                                  \
    ".Lhop_record\\w\\()_%=:\n"                                                                                       \
    "  s_load_dwordx16 s[\\n:\\n+15], s[16:17], \\at\n"                                                               \
    "  .if %[mode] != %[synth]\n"                                                                                     \
    "  s_bitcmp1_b32 s[\\w+1], 12\n"                                                                                  \
    "  s_cbranch_scc0 .Lhop_half\\w\\()_%=\n"                                                                         \
    "  .endif\n"                                                                                                      \
    "  s_load_dwordx16 s[\\n+16:\\n+31], s[16:17], \\at+64\n"                                                         \
    ".Lhop_half\\w\\()_%=:\n"                                                                                         \
    "  .if %[mode] == %[synth]\n"                                                                                     \
    "  hop_generate \\w\n"                                                                                            \
    "  .endif\n"                                                                                                      \
    "  s_or_b32 s34, s26, s[\\w]\n"                                                                                   \
    "  s_set_gpr_idx_on s[\\w+5], 2\n"                                                                                \
    "  .if %[mom]\n"                                                                                                  \
    "  v_mul_f32_e32 v12, s[\\w+6], v16\n"                                                                            \
    "  .else\n"                                                                                                       \
    "  v_fma_f32 v12, s[\\w+6], v16, 0\n"                                                                             \
    "  .endif\n"                                                                                                      \
    "  .if %[mode] == %[synth]\n"                                                                                     \
    "  ds_read_b32 v11, v11\n"                                                                                        \
    "  .endif\n"                                                                                                      \
    ".endm\n"                                                                                                         \
    "  s_mov_b64 s[16:17], %[records]\n"                                                                              \
    /* the first record's words, under the lists */                                                                   \
    "  s_load_dwordx16 s[36:51], s[16:17], 0\n"                                                                       \
    "  s_load_dwordx16 s[52:67], s[16:17], 64\n"                                                                      \
    "  s_mov_b64 s[18:19], %[lists]\n"                                                                                \
    "  s_mov_b64 s[20:21], %[columns]\n"                                                                              \
    "  s_mov_b32 s23, %[loads]\n"                                                                                     \
    "  s_mov_b32 s24, %[neg_eta]\n"                                                                                   \
    "  s_mov_b32 s25, %[mu]\n"                                                                                        \
    "  s_mov_b32 s27, 0x7FEB352D\n"                                                                                   \
    "  s_mov_b32 s28, 0x846CA68B\n"                                                                                   \
    "  s_mov_b32 s29, 0x04040404\n"                                                                                   \
    "  s_set_gpr_idx_on s29, 0\n"                                                                                     \
    "  s_nop 7\n"                                                                                                     \
    ".Lhop_load_%=:\n"                                                                                                \
    "  s_sub_u32 s23, s23, 1\n"                                                                                       \
    "  s_cbranch_scc1 .Lhop_loaded_%=\n"                                                                              \
    "  hop_list_words\n"                                                                                              \
    "  .irp q, 0, 1, 2, 3, 4, 5, 6, 7\n"                                                                              \
    "  hop_list_load \\q\n"                                                                                           \
    "  .endr\n"                                                                                                       \
    ".Lhop_wait_%=:\n"                                                                                                \
    "  s_waitcnt vmcnt(0)\n"                                                                                          \
    "  .irp q, 0, 1, 2, 3, 4, 5, 6, 7\n"                                                                              \
    "  hop_list_put \\q\n"                                                                                            \
    "  .endr\n"                                                                                                       \
    "  s_branch .Lhop_load_%=\n"                                                                                      \
    ".Lhop_loaded_%=:\n"                                                                                              \
    "  s_set_gpr_idx_on s29, 0\n"                                                                                     \
    "  .if %[mode] == %[external]\n"                                                                                  \
    "  s_mov_b64 s[70:71], %[first]\n"                                                                                \
    "  hop_external 68\n"                                                                                             \
    "  .endif\n"                                                                                                      \
    "  s_getpc_b64 s[34:35]\n"                                                                                        \
    ".Lhop_here_%=:\n"                                                                                                \
    "  s_add_u32 s26, s34, .Lhop_chains_%=-.Lhop_here_%=\n"                                                           \
    "  s_addc_u32 s35, s35, 0\n"                                                                                      \
    "  s_waitcnt lgkmcnt(0)\n"                                                                                        \
    "  hop_record 36, 68, 128\n"                                                                                      \
    "  s_setpc_b64 s[34:35]\n"                                                                                        \
    "  hop_record 68, 36, 256\n"                                                                                      \
    "  s_add_u32 s16, s16, 256\n"                                                                                     \
    "  s_addc_u32 s17, s17, 0\n"                                                                                      \
    "  s_setpc_b64 s[34:35]\n"                                                                                        \
    /* four chains, 256 bytes apart, in a block that no address crosses a carry in: a record names its own */         \
    "  .p2align 10\n"                                                                                                 \
    ".Lhop_chains_%=:\n"                                                                                              \
    "  hop_short 36, 68\n"                                                                                            \
    "  hop_long 36\n"                                                                                                 \
    "  hop_short 68, 36\n"                                                                                            \
    "  hop_long 68\n"                                                                                                 \
    "  hop_rest 36, 68\n"                                                                                             \
    "  hop_rest 68, 36\n"                                                                                             \
    ".Lhop_end_%=:\n"                                                                                                 \
    /* what the last record had loaded ahead is not used, but its registers are */                                    \
    "  s_waitcnt vmcnt(0) lgkmcnt(0)\n"                                                                               \
    "  .if %[mom]\n"                                                                                                  \
    "  s_mov_b32 s23, %[velocities]\n"                                                                                \
    ".Lhop_back_%=:\n"                                                                                                \
    "  s_sub_u32 s23, s23, 1\n"                                                                                       \
    "  s_cbranch_scc1 .Lhop_out_%=\n"                                                                                 \
    "  hop_list_words\n"                                                                                              \
    "  .irp q, 0, 1, 2, 3, 4, 5, 6, 7\n"                                                                              \
    "  hop_list_store \\q\n"                                                                                          \
    "  .endr\n"                                                                                                       \
    "  s_branch .Lhop_back_%=\n"                                                                                      \
    ".Lhop_out_%=:\n"                                                                                                 \
    "  .endif\n"                                                                                                      \
    "  s_waitcnt vmcnt(0) lgkmcnt(0)\n"                                                                               \
    "  s_nop 7\n"                                                                                                     \
    "  s_set_gpr_idx_off\n"                                                                                           \
    "  s_nop 7\n"                                                                                                     \
    ".purgem hop_list_words\n"                                                                                        \
    ".purgem hop_columns\n"                                                                                           \
    ".purgem hop_list_load\n"                                                                                         \
    ".purgem hop_list_put\n"                                                                                          \
    ".purgem hop_list_store\n"                                                                                        \
    ".purgem hop_generate\n"                                                                                          \
    ".purgem hop_external\n"                                                                                          \
    ".purgem hop_apply\n"                                                                                             \
    ".purgem hop_chain\n"                                                                                             \
    ".purgem hop_short\n"                                                                                             \
    ".purgem hop_long\n"                                                                                              \
    ".purgem hop_rest\n"                                                                                              \
    ".purgem hop_record\n"

#define HOP_SWEEP_ASM(...)                                                                                            \
    asm volatile(HOP_SWEEP_TEXT                                                                                       \
                 :                                                                                                    \
                 : [records] "s"(a.program), [lists] "s"(a.program + a.first_list), [columns] "s"(columns),           \
                   [loads] "s"(a.n_load_groups), [velocities] "s"(a.n_store_groups),    \
                   [neg_eta] "s"(-a.eta), [mu] "s"(a.mu), [first] "s"(a.first_external), [lane] "v"(lane),            \
                   [folded] "v"(folded), [table] "v"(table), [mode] "n"(MODE), [mom] "n"((int)MOM),                   \
                   [zero] "n"(HOP_GRAD_ZERO), [synth] "n"(HOP_GRAD_SYNTH), [external] "n"(HOP_GRAD_EXTERNAL)          \
                 : "memory", "scc", "vcc", HOP_SWEEP_S, __VA_ARGS__)

constexpr int kSweepThreads = 256;
constexpr int kSynthSums = 12 * 255 + 1;               // values of a sum of 12 bytes
// Of each thread, the table filled up: written out it is three instructions an entry.  As a loop up to the last sum it was a
// tenth of a short pass (2 workers x 3 M columns, 30 records: 65.9 -> 60.6 us; 16 workers, 240 records: 497 -> 492).
constexpr int kSynthEach = (kSynthSums + kSweepThreads - 1) / kSweepThreads;

// LOCAL: local slots there are registers for.  64, 96, 128 and 184 registers: 8, 5, 4 and 2 wavefronts per SIMD.
template <int MODE, bool MOM, int LOCAL>
__global__ __launch_bounds__(kSweepThreads) void sweep_kernel(const HopSweepArgs a) {
    __shared__ float tableS[MODE == HOP_GRAD_SYNTH ? kSynthEach * kSweepThreads : 1];
    if (MODE == HOP_GRAD_SYNTH) {
        const float sum = (float)((int)threadIdx.x - 1530);
#pragma unroll
        for (int k = 0; k < kSynthEach; ++k) tableS[threadIdx.x + k * kSweepThreads] = (sum + (float)(k * kSweepThreads)) * a.scale;
        __syncthreads();
    }
    const uint32_t table = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)tableS;
    const int64_t c = (int64_t)blockIdx.x * kSweepThreads + threadIdx.x;
    if (c >= a.d) return;                              // the wavefront at the end of the vectors: fewer lanes, the same way
    const uint32_t lane = threadIdx.x * (uint32_t)sizeof(float), folded = fold16((uint32_t)c);
    const uint64_t columns = (uint64_t)blockIdx.x * kSweepThreads * sizeof(float);
    static_assert(LOCAL == 48 || LOCAL == 80 || LOCAL == 112 || LOCAL == kSweepRegisters, "16 registers beside the local slots");
    if constexpr (LOCAL == 48) HOP_SWEEP_ASM(HOP_SWEEP_V64);
    else if constexpr (LOCAL == 80) HOP_SWEEP_ASM(HOP_SWEEP_V96);
    else if constexpr (LOCAL == 112) HOP_SWEEP_ASM(HOP_SWEEP_V128);
    else HOP_SWEEP_ASM(HOP_SWEEP_V184);
}

// ------------------------------------------------------------------ wavefront reductions ----
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;                                          // lane 0 holds the sum
}

// c_m of g = lambda w - sum_m c_m x_m: hinge y/B where y <x, w> < 1, log loss y / (B (1 + e^{y <x, w>}))
__device__ __forceinline__ float loss_coef(float y, float dot, float invB, int loss) {
    const float m = y * dot;
    if (loss == HOP_LOSS_LOG) return y * invB / (1.0f + expf(m));
    return m < 1.0f ? y * invB : 0.f;
}

// ------------------------------------------------------------- dense SVM: margins ("Compute") ----
// One workgroup per (job, minibatch row, column segment): partial <x_r, w> over 16384 columns.
constexpr int kSegVec = 16;
constexpr int kSeg4 = kThreads * kSegVec;             // float4 per segment
constexpr int64_t kSegCols = (int64_t)kSeg4 * 4;

// ROWS minibatch rows from m0 on against one load of w; thread t < ROWS of the workgroup writes the partial of row m0 + t,
// or, where a row has one segment only, its coefficient: the gradient kernel then has that to load and nothing to work out
// (the label's load under the row's; see dense_grad_chunk).  Each row is summed in the same order whatever ROWS is.
// How a row is cut up: segments of kSegCols columns, one such segment, or a slice for each XCD (hop_wave_slices), whose margins
// and gradient run there: the gradient finds in that XCD's L2 what the margins have read, as much as fits.
enum class Cut { segments, one, slices };
// first of n_chunks chunks that belong to slice s
__device__ __forceinline__ int slice_begin(int n_chunks, int s) { return n_chunks * s / kXcd; }

template <int ROWS, bool STREAM, Cut CUT>
__device__ __forceinline__ void dense_margin_rows(const HopGradJob* __restrict__ job, int B, int64_t d, int nseg, int seg,
                                                  int m0, float (*red)[kThreads / 64]) {
    constexpr bool ONE = CUT == Cut::one;
    const float* w = job->w;
    const float* x[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) x[r] = job->X + (int64_t)job->rows[min(m0 + r, B - 1)] * d;
    const int mine = m0 + (int)threadIdx.x;
    const bool writes = threadIdx.x < ROWS && mine < B;
    float y = 0.f;
    if (ONE && writes) y = job->y[job->rows[mine]];
    const int chunks = (int)((d + 255) / 256);
    const int64_t lo = CUT == Cut::slices ? slice_begin(chunks, seg) * 256 : (int64_t)seg * kSegCols;
    const int64_t hi = min(d, CUT == Cut::slices ? slice_begin(chunks, seg + 1) * (int64_t)256 : lo + kSegCols);
    float a[ROWS][4];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) a[r][0] = a[r][1] = a[r][2] = a[r][3] = 0.f;
    const int64_t hi4 = hi >> 2;
    int64_t i = (lo >> 2) + threadIdx.x;
    auto piece = [&](int64_t k) {
        const float4 wv = ldu4(w, k << 2);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const float4 xv = STREAM ? ldu4_stream(x[r], k << 2) : ldu4(x[r], k << 2);
            a[r][0] = fmaf(xv.x, wv.x, a[r][0]);
            a[r][1] = fmaf(xv.y, wv.y, a[r][1]);
            a[r][2] = fmaf(xv.z, wv.z, a[r][2]);
            a[r][3] = fmaf(xv.w, wv.w, a[r][3]);
        }
    };
    if (ROWS == 1) {                                               // eight pieces in flight; what is left by fours, not singly
        for (; i + 7 * kThreads < hi4; i += 8 * kThreads) {
#pragma unroll
            for (int u = 0; u < 8; ++u) piece(i + u * kThreads);
        }
    }
#pragma unroll 4
    for (; i < hi4; i += kThreads) piece(i);
    if (const int64_t c = (hi4 << 2) + threadIdx.x; c < hi) {      // the d mod 4 last columns
#pragma unroll
        for (int r = 0; r < ROWS; ++r) a[r][0] = fmaf(x[r][c], w[c], a[r][0]);
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const float v = wave_sum((a[r][0] + a[r][1]) + (a[r][2] + a[r][3]));
        if (lane == 0) red[r][wv] = v;
    }
    __syncthreads();
    if (writes) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < kThreads / 64; ++k) t += red[threadIdx.x][k];
        if (ONE) job->coef[mine] = loss_coef(y, t, 1.0f / (float)B, (int)job->k0);
        else job->partial[(int64_t)mine * nseg + seg] = t;
    }
}

// Small minibatches keep to one XCD (hop_one_xcd): all margins of a record run on XCD (record mod 8) and so does its gradient, which
// finds rows and coefficients in that XCD's L2.
static_assert(kOneXcdCols <= kSegCols, "rows of one segment");

// one workgroup per (job, minibatch row), the job on one XCD; b: its index, in launches with other workgroups
__device__ __forceinline__ void dense_margin_near(const HopGradJob* __restrict__ jobs, unsigned n_jobs, int B, int64_t d, unsigned b,
                                                  float (*red)[kThreads / 64]) {
    const unsigned rest = b / kXcd, job = rest / (unsigned)B * kXcd + b % kXcd;
    if (job < n_jobs) dense_margin_rows<1, false, Cut::one>(jobs + job, B, d, 1, 0, (int)(rest % (unsigned)B), red);
}

// one workgroup per (job, minibatch row, column segment), b its index, in launches with other workgroups
__device__ __forceinline__ void dense_margin_block(const HopGradJob* __restrict__ jobs, int B, int64_t d, int nseg,
                                                   unsigned b, float (*red)[kThreads / 64]) {
    if (nseg == 1) {
        dense_margin_rows<1, false, Cut::one>(jobs + b / (unsigned)B, B, d, nseg, 0, (int)(b % (unsigned)B), red);
        return;
    }
    const unsigned row = b / (unsigned)nseg;
    dense_margin_rows<1, false, Cut::segments>(jobs + row / (unsigned)B, B, d, nseg, (int)(b % (unsigned)nseg), (int)(row % (unsigned)B), red);
}

// The margin pass as a launch of its own: four minibatch rows per workgroup share every load of w (the L2 sees
// 5 requests per 4 row pieces instead of 8); with few workgroups (kMarginFew) one row each, so that all CUs have rows in
// flight (one minibatch of 128 x 65536: 14.1 -> 8.9 us; 3 records of 100 x 30 011: 36 -> 14 us, scalar loads before).
// The line: 16 workers x 65536 columns, B = 128 (128 workgroups of four rows per record) 3627 us per pass with one row
// up to 767 workgroups, 3529 up to 383; 16 x 400 000, B = 16, momentum 1587 and 1486 us.
// Rows by non-temporal loads: a wave's rows are new to every cache, and a cold stream
// runs faster without allocating in the memory-side cache (6.9 against 5.5 TB/s stand-alone).  Leaving
// them there for the gradient pass with ordinary loads was measured on 16 workers x 65536 columns, B = 128, 6.6 records:
// margins 37.4 -> 42.5 us, gradient 23.8 -> 21.5 us per wave, nothing gained; where a launch of few workgroups reads no
// more than half of that cache (kMarginNear) ordinary loads pay: 3 to 4 records of 100 x 30 011 2.20 -> 2.12 ms per pass.
constexpr int kMarginRows = 4;
// Slices are an eighth of a row, at most a segment: two rows per workgroup (geometric mean over 33 sizes 3.6 % ahead of four).
constexpr int kSliceRows = 2;
constexpr int64_t kMarginFew = 384;
constexpr int64_t kMarginNear = 128ll << 20;           // bytes of rows in a launch up to which they are left in the caches
static_assert(kMarginFew * kMarginRows * kSegCols * 4 <= kMarginNear, "a launch of few workgroups by segments always is");

template <int ROWS, bool STREAM, Cut CUT>
__global__ __launch_bounds__(kThreads) void dense_margin_kernel(const HopGradJob* __restrict__ jobs, int B, int64_t d,
                                                                int nseg) {
    __shared__ float red[ROWS][kThreads / 64];
    dense_margin_rows<ROWS, STREAM, CUT>(jobs + blockIdx.z, B, d, nseg, (int)blockIdx.x, (int)blockIdx.y * ROWS, red);
}

// The kernels whose name ends in _one are for stand-alone calls: the descriptor is the kernel's argument, nothing is
// allocated, copied or staged.  Per call: 128 x 65536 dense 42.5 -> 28.4 us, 64 x 1024 without allocation 10.4 -> 7.7 us
// (one launch fewer), 256 samples of 64 non-zeros on 2^20 columns 33.0 -> 18.6 us (margins beside the dense part).
// every eighth workgroup: the call keeps to one XCD (hop_one_xcd_alone)
__global__ __launch_bounds__(kThreads) void dense_margin_near_one(const HopGradJob job, int B, int64_t d) {
    __shared__ float red[1][kThreads / 64];
    if (blockIdx.x == 0) dense_margin_rows<1, false, Cut::one>(&job, B, d, 1, 0, (int)blockIdx.y, red);
}

template <int ROWS, bool STREAM, bool ONE>
__global__ __launch_bounds__(kThreads) void dense_margin_one(const HopGradJob job, int B, int64_t d, int nseg) {
    __shared__ float red[ROWS][kThreads / 64];
    dense_margin_rows<ROWS, STREAM, ONE ? Cut::one : Cut::segments>(&job, B, d, nseg, (int)(blockIdx.x % nseg), (int)(blockIdx.x / nseg) * ROWS, red);
}

// The partial margins of a wave's STEP records and the wave's Reduce in one launch: both only read x_k
// (the parallel approach of Section 3.2 runs Compute beside Reduce).  The Reduce leaves sum_a w'_a x_a
// in the result slot; dense_grad_kernel then applies -eta g to it.
// (ONE: each record on one XCD, n their number; else n the segments of a row.  NEAR: hop_in_place_near)
template <bool ONE, bool NEAR>
__global__ __launch_bounds__(kThreads) void mix_dense_margin_kernel(const HopMixJob* __restrict__ mix_jobs, int64_t d, int front,
                                                                    HOP_RUNS_IN, unsigned margins, int n_mix,
                                                                    const HopGradJob* __restrict__ grad_jobs, int B,
                                                                    int n) {
    __shared__ float red[1][kThreads / 64];
    if ((int)blockIdx.z >= front) {
        mix_block<NEAR>(mix_jobs, d, HOP_RUNS, (int)blockIdx.z - front);
        return;
    }
    const unsigned b = grid_index(HOP_RUNS, n_mix);
    if (b >= margins) return;
    if (ONE) dense_margin_near(grad_jobs, (unsigned)n, B, d, b, red);
    else dense_margin_block(grad_jobs, B, d, n, b, red);
}

// ----------------------------------------------------- dense SVM: g = lambda w - sum_m c_m x_m ----
// One workgroup per (job, column chunk).  The hinge coefficients c_m = y_m / B if
// y_m <x_m, w> < 1 else 0 are rebuilt by every workgroup from the partial dot products (B values,
// cheap) and the active rows are compacted in LDS in minibatch order.  Three endings: write g; apply -eta g to
// a vector the wave's Reduce has already left in the result slot; or do the record's Reduce here as well
// (steps 2-3 of the standard-training figure on the freshly computed gradient), which saves the launch of a
// separate mix and the round trip of g through memory when the minibatch is large.
constexpr int kMaxB = 1024;
constexpr int kRowUnroll = 8;

// A column chunk is 256 columns times WIDE wavefronts side by side; SPLIT such groups share it and take alternate groups
// of 8 active rows, their sums joined through LDS in a fixed order.
// Up to a few chunks of 256 columns per CU the time is the chain of dependent row loads, so a chunk is as narrow as a
// wavefront's 1 KB of a row and its rows are split.  Per pass, chunks of 1024 columns with one group of 256 threads (four
// in launches of up to 128 workgroups) -> this: 8 workers x 30 011 columns, B = 100 (rows not 16-byte aligned, scalar
// loads before): 6.91 -> 2.20 ms; 16 x 65536, B = 128: 3.86 -> 3.75 ms; 4 x 1024, B = 64: 392 -> 360 us; one gradient of
// 128 x 65536: 14.4 -> 8.8 us.  4 against 8 wavefronts per chunk, log loss (all rows active), 4 x 1024 columns, B = 64
// and 128: 164 / 162, 186 / 174 us; 16 x 16384, B = 128: 703 / 682; 16 x 65536, B = 16: 601 / 636 us.
// With more chunks the row loads of other workgroups fill the wait, and what counts is that every workgroup sums up the
// coefficients of all rows again, from a partial product per 16384 columns: four times as many of them cost more than
// the split gives.  SPLIT = WIDE = 4, 1 against 1, 4: one gradient of 2^20 columns, B = 128: 238 / 210 us, 4 M columns
// 1564 / 962, 2^24 columns and B = 64 10.8 / 3.2 ms; a pass of 16 workers x 400 000 columns, B = 16: 1943 / 1487 us; of
// 64 x 65536, B = 128, 13 records a wave: 3973 / 3813 us; the other way round 64 x 16384, B = 128: 1461 / 1543 us.
// kGradFew: chunks of 256 columns up to which a launch takes 8 wavefronts for each
constexpr int64_t kGradMany = 2048;                    // over that many, or
constexpr int kGradSegs = 16;                          // from that many partial products per row on: 1024 columns, rows whole
// From 65 partial products per row on a wavefront sums them up, not a thread: 4 M columns, B = 1 and 128: 54 -> 20,
// 962 -> 842 us; 2^24 columns, B = 1 and 64: 635 -> 89 us, 3.2 -> 1.95 ms (2^20 columns, 64 of them, B = 8 and 128:
// 20.5 -> 17.3, 211 -> 216).
constexpr int kSegThread = 64;

// (Loading a wavefront's 8 rows at once, active or not, while the coefficients are still being worked out - one chain of
// loads instead of two, for minibatches of up to 8 SPLIT rows - was slower: 4 x 1024, B = 64: 364 -> 460 us per pass.)
// ONE: a row has one segment, and the margins have left the coefficients themselves: one round of loads less in the chain to
// the rows (4 workers x 1024 columns, B = 64: 360 -> 338 us a pass).
// LAST: rows by non-temporal loads, so that of what the margins left in the L2s what is yet to be read stays longest (hop_rows_again).
template <int SPLIT, int WIDE, bool ONE, bool LAST>
__device__ __forceinline__ void dense_grad_chunk(const HopGradJob* __restrict__ job, int B, int64_t d, int nseg, float lambda,
                                                 int loss, int64_t chunk) {
    __shared__ float coefS[kMaxB];
    __shared__ int rowS[kMaxB + kRowUnroll];
    __shared__ float allC[ONE ? 1 : kMaxB];
    __shared__ int nactS;
    constexpr int kCols = 64 * WIDE;                   // threads side by side
    __shared__ float4 joinS[SPLIT > 1 ? (SPLIT - 1) * kCols : 1];
    const float invB = 1.0f / (float)B;
    const int part = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kCols);  // which share of the rows
    const int col = (int)threadIdx.x % kCols;
    const float* X = job->X;
    const float* w = job->w;
    float* out = job->out;                             // set: apply -eta g (or -eta v) to it instead of writing g
    const HopMixJob* red = job->reduce;                // set (with out): out = sum_a w'_a x_a - eta g, the Reduce done here
    const int64_t c = (chunk * kCols + col) * 4;       // first of this thread's columns
    const int n = (int)min((int64_t)4, d - c);         // how many of them exist
    // what the ending needs beside the sum, loaded ahead of the rows
    float4 wv = make_float4(0.f, 0.f, 0.f, 0.f), o = wv;
    if (part == 0 && n > 0) {
        wv = ldu4(w, c, n);
        if (red != nullptr) {                          // the record's Reduce, in the order the mix kernels sum
            const int A = red->A;
            const float4 x0 = ldu4(red->src[0], c, n);
            const float wa = red->w[0];
            o = make_float4(wa * x0.x, wa * x0.y, wa * x0.z, wa * x0.w);
            for (int a = 1; a < A; ++a) o = fma4(red->w[a], ldu4(red->src[a], c, n), o);
        } else if (out != nullptr) {                   // already reduced into the result slot
            o = ldu4(out, c, n);
        }
    }
    if (!ONE) {
        auto put_coef = [&](int m, float dot) {
            const float cm = loss_coef(job->y[job->rows[m]], dot, invB, loss);
            allC[m] = cm;
            if (chunk == 0) job->coef[m] = cm;
        };
        if (WIDE == 1 || nseg <= kSegThread) {
            for (int m = threadIdx.x; m < B; m += kCols * SPLIT) {
                float dot = 0.f;
                for (int sg = 0; sg < nseg; ++sg) dot += job->partial[(int64_t)m * nseg + sg];
                put_coef(m, dot);
            }
        } else {                                           // a wavefront per row
            for (int m = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64); m < B; m += WIDE * SPLIT) {
                float dot = 0.f;
                for (int sg = (int)threadIdx.x % 64; sg < nseg; sg += 64) dot += job->partial[(int64_t)m * nseg + sg];
                dot = wave_sum(dot);
                if (threadIdx.x % 64 == 0) put_coef(m, dot);
            }
        }
        __syncthreads();
    }
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (threadIdx.x < 64) {                        // first wavefront compacts the active rows, keeping order
        int count = 0, any = 0;
        for (int base = 0; base < B; base += 64) {
            const int m = base + threadIdx.x;
            const float cm = m < B ? ONE ? job->coef[m] : allC[m] : 0.f;
            const int id = ONE && m < B ? job->rows[m] : 0;
            const bool act = cm != 0.f;
            const unsigned long long mask = __ballot(act);
            const int pos = count + __popcll(mask & ((1ull << threadIdx.x) - 1ull));
            const int row = act ? ONE ? id : job->rows[m] : 0;
            if (act) {
                coefS[pos] = cm;
                rowS[pos] = row;
            }
            if (mask) any = __builtin_amdgcn_readlane(row, __ffsll(mask) - 1);
            count += __popcll(mask);
        }
        if (threadIdx.x < kRowUnroll) rowS[count + threadIdx.x] = any;     // loaded with the last rows, not added
        if (threadIdx.x == 0) nactS = count;
    }
    __syncthreads();
    const int nact = __builtin_amdgcn_readfirstlane(nactS);
    // active rows only, each once: a zero times an infinity in a row that takes no part would be a NaN in the sum
    auto add_rows = [&](auto row_at) {
        for (int q = part * kRowUnroll; q < nact; q += kRowUnroll * SPLIT) {
            float4 v[kRowUnroll];
#pragma unroll
            for (int u = 0; u < kRowUnroll; ++u) v[u] = row_at(X + (int64_t)rowS[q + u] * d);
            if (q + kRowUnroll <= nact) {
#pragma unroll
                for (int u = 0; u < kRowUnroll; ++u) acc = fma4(coefS[q + u], v[u], acc);
            } else {
#pragma unroll
                for (int u = 0; u < kRowUnroll - 1; ++u)
                    if (q + u < nact) acc = fma4(coefS[q + u], v[u], acc);
            }
        }
    };
    // The thread at the end of a vector, with d mod 4 columns left, reads the last four like any other and keeps its own: a pass over
    // the rows for itself made its wavefront's chain twice as long.  us per pass, log loss, 12 iterations: 16 workers x 14 columns, B = 120
    // 160 -> 121, 566 460 -> 276; 8 x 255, B = 566 376 -> 211; 32 x 1023, B = 120 198 -> 174.
    const auto at = [&](int64_t i) { return [=](const float* x) { return LAST ? ldu4_stream(x, i) : ldu4(x, i); }; };
    if (d % 4 == 0) {
        if (n == 4) add_rows(at(c));
    } else if (d > 4) {
        if (n > 0) add_rows(at(min(c, d - 4)));
        if (n == 3) acc = make_float4(acc.y, acc.z, acc.w, 0.f);
        else if (n == 2) acc = make_float4(acc.z, acc.w, 0.f, 0.f);
        else if (n == 1) acc = make_float4(acc.w, 0.f, 0.f, 0.f);
    } else if (n > 0) {
        add_rows([&](const float* x) { return ldu4(x, c, n); });
    }
    if constexpr (SPLIT > 1) {                     // join the shares: ((part 0 + part 1) + part 2) + ...
        if (part > 0) joinS[(part - 1) * kCols + col] = acc;
        __syncthreads();
#pragma unroll
        for (int q = 1; q < SPLIT; ++q) {
            if (part != 0) break;
            const float4 t = joinS[(q - 1) * kCols + col];
            acc = make_float4(acc.x + t.x, acc.y + t.y, acc.z + t.z, acc.w + t.w);
        }
    }
    if (n <= 0 || part != 0) return;
    float4 gv = make_float4(fmaf(lambda, wv.x, -acc.x), fmaf(lambda, wv.y, -acc.y), fmaf(lambda, wv.z, -acc.z),
                            fmaf(lambda, wv.w, -acc.w));
    if (out == nullptr) {
        stu4(job->g, c, n, gv);
        return;
    }
    float* vel = job->vel;
    if (vel != nullptr) {
        gv = fma4(job->mu, ldu4(vel, c, n), gv);
        stu4(vel, c, n, gv);
    }
    stu4(out, c, n, fma4(-job->eta, gv, o));
}

template <int SPLIT, int WIDE, bool ONE>
__global__ __launch_bounds__(64 * SPLIT * WIDE) void dense_grad_kernel(const HopGradJob* __restrict__ jobs, int width, int B,
                                                                int64_t d, int nseg, float lambda, int loss,
                                                                int64_t n_chunks) {
    const int64_t chunk = grid_chunk(width);
    if (chunk < n_chunks) dense_grad_chunk<SPLIT, WIDE, ONE, false>(jobs + blockIdx.y, B, d, nseg, lambda, loss, chunk);
}

// each XCD a slice of the columns: a grid of (8, jobs, chunks of the longest slice)
template <int SPLIT, int WIDE, bool LAST>
__global__ __launch_bounds__(64 * SPLIT * WIDE) void dense_grad_slice_kernel(const HopGradJob* __restrict__ jobs, int n_chunks, int B,
                                                                             int64_t d, float lambda, int loss) {
    const int chunk = slice_begin(n_chunks, (int)blockIdx.x) + (int)blockIdx.z;
    if (chunk < slice_begin(n_chunks, (int)blockIdx.x + 1))
        dense_grad_chunk<SPLIT, WIDE, false, LAST>(jobs + blockIdx.y, B, d, kXcd, lambda, loss, chunk);
}

// each job on one XCD: a grid of (8, chunks, jobs / 8)
__global__ __launch_bounds__(512) void dense_grad_near_kernel(const HopGradJob* __restrict__ jobs, int n_jobs, int B, int64_t d,
                                                              float lambda, int loss) {
    const int job = (int)(blockIdx.z * kXcd + blockIdx.x);
    if (job < n_jobs) dense_grad_chunk<8, 1, true, false>(jobs + job, B, d, 1, lambda, loss, blockIdx.y);
}

__global__ __launch_bounds__(512) void dense_grad_near_one(const HopGradJob job, int B, int64_t d, float lambda, int loss) {
    if (blockIdx.x == 0) dense_grad_chunk<8, 1, true, false>(&job, B, d, 1, lambda, loss, blockIdx.y);
}

template <int SPLIT, int WIDE, bool ONE>
__global__ __launch_bounds__(64 * SPLIT * WIDE) void dense_grad_one(const HopGradJob job, int B, int64_t d, int nseg, float lambda,
                                                             int loss) {
    dense_grad_chunk<SPLIT, WIDE, ONE, false>(&job, B, d, nseg, lambda, loss, blockIdx.x);
}

// ------------------------------------------------------------------- CSR SVM: margins ----
// One wavefront per (job, minibatch row): gather w[col], reduce across the 64 lanes.  Workgroups are dealt out to the XCDs one
// by one: the four blocks of rows that one workgroup of the scatter takes run on the XCD where it will run, so it finds their
// row pointers, columns and values in that XCD's L2, or some of them (16 workers x 2^20 columns, B = 256: 6870 -> 6761 us per
// pass).  Workgroup b of the margins belongs to workgroup csr_margin_group(b) of the scatter, counted over all records.  In waves of
// few records each has whole turns of the XCDs (its first rows on the XCD whose L2 holds what the last wave wrote of the first
// columns, which nearly every row reads); filled up like that beyond kCsrTurns workgroups, idle ones cost more than it brings.  us
// per pass, filled up and not, 20 000 columns: 16 workers, Exp(1), B = 1 176 / 191, with a velocity 173 / 189; lock-step, B = 8, 16
// workers 57.6 / 58.2, 32 (256 workgroups) 64.3 / 62.3, 40 71.6 / 64.0, 64 95.5 / 73.2, 64 with B = 64 110 / 86.
constexpr int64_t kCsrTurns = 256;      // workgroups of the scatter
__device__ __forceinline__ unsigned csr_margin_group(unsigned b) { return b / (4 * kXcd) * kXcd + b % kXcd; }

// its rows: of the scatter's workgroup `group` of this record; b / 8 mod 4 says which of its four blocks
__device__ __forceinline__ void csr_margin_rows(const HopGradJob* __restrict__ job, int B, int loss, int group, unsigned b) {
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m = (group * 4 + (int)(b / kXcd % 4)) * (kThreads / 64) + wv;
    if (m >= B) return;
    const int r = job->rows[m];
    const int64_t lo = job->rowptr[r], hi = job->rowptr[r + 1];
    const float* w = job->w;
    float acc = 0.f;
    for (int64_t p = lo + lane; p < hi; p += 64) acc = fmaf(job->val[p], w[job->col[p]], acc);
    acc = wave_sum(acc);
    if (lane == 0) job->coef[m] = loss_coef(job->y[r], acc, 1.0f / (float)B, loss);
}

// Margins and the dense part lambda w of a gradient that is wanted as a dense vector, side by side (the sparse part is
// scattered into g afterwards).  The margins' workgroups in the order of their rows and no more than there are: in turns of the XCDs
// a call of few rows waits for idle ones and larger ones gain nothing (us, in turns -> in order, medians of 6 processes each: 600 columns, B = 1
// 15.97 -> 15.18, 256 17.91 -> 17.73; 200 000, B = 1 16.09 -> 15.82, 40 17.16 -> 16.91, 512 17.69 -> 17.67; 2^20, B = 2 16.51 -> 16.31, 256 17.69 ->
// 17.81; 3 M, B = 40 19.50 -> 19.92, 512 20.93 -> 21.01).
__global__ __launch_bounds__(kThreads) void csr_margin_dense_one(const HopGradJob job, int B, int64_t d, float lambda,
                                                                 int loss, int margin_blocks) {
    if ((int)blockIdx.x < margin_blocks) {
        csr_margin_rows(&job, B, loss, (int)(blockIdx.x / 4), blockIdx.x % 4 * kXcd);
        return;
    }
    const int64_t c = ((int64_t)(blockIdx.x - margin_blocks) * kThreads + threadIdx.x) * 4;
    const int n = (int)min((int64_t)4, d - c);
    if (n > 0) {
        const float4 w = ldu4(job.w, c, n);
        stu4(job.out, c, n, make_float4(lambda * w.x, lambda * w.y, lambda * w.z, lambda * w.w));
    }
}

// workgroup b of the margins of n_jobs records, `per` workgroups of the scatter each
__device__ __forceinline__ void csr_margin_block(const HopGradJob* __restrict__ jobs, unsigned n_jobs, int B, unsigned per, int loss,
                                                 unsigned b) {
    const unsigned at = csr_margin_group(b), job = at / per;
    if (job < n_jobs) csr_margin_rows(jobs + job, B, loss, (int)(at % per), b);
}

__global__ __launch_bounds__(kThreads) void csr_margin_kernel(const HopGradJob* __restrict__ jobs, int n_jobs, int B, unsigned per,
                                                              int loss) {
    csr_margin_block(jobs, (unsigned)n_jobs, B, per, loss, blockIdx.x);
}

// The margins of a wave's STEP records and the wave's Reduce + Apply in one launch: both only read
// x_k, and nothing a wave writes is read inside it, so they need no order between them.  The few
// latency-bound margin workgroups come first and run under the streaming ones.
// (n_grad records of `per` workgroups of the scatter)
template <bool NEAR>
__global__ __launch_bounds__(kThreads) void mix_csr_margin_kernel(const HopMixJob* __restrict__ mix_jobs, int64_t d, int front,
                                                                  HOP_RUNS_IN, unsigned margins, int n_mix,
                                                                  const HopGradJob* __restrict__ grad_jobs, int n_grad, int B,
                                                                  unsigned per, int loss) {
    if ((int)blockIdx.z >= front) {
        mix_block<NEAR>(mix_jobs, d, HOP_RUNS, (int)blockIdx.z - front);
        return;
    }
    const unsigned b = grid_index(HOP_RUNS, n_mix);
    if (b < margins) csr_margin_block(grad_jobs, (unsigned)n_grad, B, per, loss, b);
}

// the same two fusions for the paired Reduce + Apply
template <int VEC, bool NEAR>
__global__ __launch_bounds__(kThreads) void pair_csr_margin_kernel(const HopPairJob* __restrict__ mix_jobs, int64_t d, int front,
                                                                   HOP_RUNS_IN, int reverse, unsigned margins, int n_mix,
                                                                   const HopGradJob* __restrict__ grad_jobs, int n_grad, int B,
                                                                   unsigned per, int loss) {
    if ((int)blockIdx.z >= front) {
        pair_block<VEC, NEAR>(mix_jobs, d, HOP_RUNS, reverse, (int)blockIdx.z - front);
        return;
    }
    const unsigned b = grid_index(HOP_RUNS, n_mix);
    if (b < margins) csr_margin_block(grad_jobs, (unsigned)n_grad, B, per, loss, b);
}

template <int VEC, bool ONE, bool NEAR>
__global__ __launch_bounds__(kThreads) void pair_dense_margin_kernel(const HopPairJob* __restrict__ mix_jobs, int64_t d, int front,
                                                                     HOP_RUNS_IN, int reverse, unsigned margins, int n_mix,
                                                                     const HopGradJob* __restrict__ grad_jobs, int B,
                                                                    int n) {
    __shared__ float red[1][kThreads / 64];
    if ((int)blockIdx.z >= front) {
        pair_block<VEC, NEAR>(mix_jobs, d, HOP_RUNS, reverse, (int)blockIdx.z - front);
        return;
    }
    const unsigned b = grid_index(HOP_RUNS, n_mix);
    if (b >= margins) return;
    if (ONE) dense_margin_near(grad_jobs, (unsigned)n, B, d, b, red);
    else dense_margin_block(grad_jobs, B, d, n, b, red);
}

// Margins in slices and the Reduce of the wave's records without a gradient (jumps) behind them in one launch (us per pass
// with skipping, jumps in a launch of their own before: 16 workers x 12 000 columns, B = 32, 621 -> 566, 16 x 65536, B = 128, 3331 ->
// 3288).  grid: (8, groups of rows, records, then what the chunks need).
template <int ROWS, bool STREAM>
__global__ __launch_bounds__(kThreads) void pair_dense_slice_kernel(const HopGradJob* __restrict__ grad_jobs, int64_t d, int B, int n_grad,
                                                                    int groups, int n_chunks, int n_mix,
                                                                    const HopPairJob* __restrict__ mix_jobs) {
    __shared__ float red[ROWS][kThreads / 64];
    if ((int)blockIdx.z < n_grad) {
        dense_margin_rows<ROWS, STREAM, Cut::slices>(grad_jobs + blockIdx.z, B, d, kXcd, (int)blockIdx.x, (int)blockIdx.y * ROWS, red);
        return;
    }
    const unsigned b = ((blockIdx.z - n_grad) * groups + blockIdx.y) * kXcd + blockIdx.x, job = b / (unsigned)n_chunks;
    if (job < (unsigned)n_mix) pair_chunk<kPairMargin, false>(mix_jobs + job, d, n_chunks, (int)(b % (unsigned)n_chunks));
}

// target[col] += factor * c_m * val for the active rows (the sparse part of -eta g, or of g).
// One wavefront per minibatch row, 16 rows per workgroup, all in flight together.  Sparse features
// are heavy-tailed (a few columns occur in almost every row) and fp32 atomics on one address
// serialise in L2: B atomics in a chain on the hottest column would set the kernel's duration.
// Contributions to the first kHotCols columns are therefore added up in LDS first and leave the
// workgroup as one global atomic per column touched (16 times fewer on the hot ones).
constexpr int kScatterThreads = 1024;
constexpr int kScatterRows = kScatterThreads / 64;
constexpr int kHotCols = 1024;

// All loads of a row are under way before the workgroup has cleared its sums, the coefficient's beside the row's chain
// (id -> row pointers -> columns and values).  BOTH: into the velocity as well, with factor -1 (g itself), in the same
// pass over the rows: with momentum 16 workers x 2^20 columns, B = 256: 5.33 -> 4.86 ms, 4 x 50 000, B = 64: 0.99 -> 0.76 ms.
// 512 and 256 threads per workgroup, which sum fewer rows' hot columns before they leave: 7.17 -> 7.20, 7.66 ms per run of
// 16 x 2^20; 256 hot columns 7.39 ms.
template <bool BOTH>
__device__ __forceinline__ void csr_scatter_rows(const HopGradJob* __restrict__ job, int B, float factor, int block) {
    __shared__ float hot[BOTH ? 2 : 1][kHotCols];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m = block * kScatterRows + wv;
    float* out = job->out;
    float* vel = BOTH ? job->vel : nullptr;
    float c = 0.f, val = 0.f;
    int col = 0;
    int64_t p = 0, hi = 0;
    if (m < B) {
        c = job->coef[m];
        const int r = job->rows[m];
        p = job->rowptr[r] + lane;
        hi = job->rowptr[r + 1];
        if (p < hi) {
            col = job->col[p];
            val = job->val[p];
        }
    }
    for (int i = threadIdx.x; i < kHotCols; i += kScatterThreads) {
        hot[0][i] = 0.f;
        if (BOTH) hot[BOTH ? 1 : 0][i] = 0.f;
    }
    __syncthreads();
    if (c != 0.f) {
        const float f = factor * c;
        while (p < hi) {
            const float v = f * val, g = -c * val;
            if (col < kHotCols) {
                atomicAdd(&hot[0][col], v);
                if (BOTH) atomicAdd(&hot[BOTH ? 1 : 0][col], g);
            } else {
                unsafeAtomicAdd(out + col, v);
                if (BOTH) unsafeAtomicAdd(vel + col, g);
            }
            p += 64;
            if (p < hi) {
                col = job->col[p];
                val = job->val[p];
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kHotCols; i += kScatterThreads) {
        const float v = hot[0][i];
        if (v != 0.f) unsafeAtomicAdd(out + i, v);
        if (BOTH) {
            const float g = hot[BOTH ? 1 : 0][i];
            if (g != 0.f) unsafeAtomicAdd(vel + i, g);
        }
    }
}

template <bool BOTH>
__global__ __launch_bounds__(kScatterThreads) void csr_scatter_kernel(const HopGradJob* __restrict__ jobs, int B, float factor) {
    csr_scatter_rows<BOTH>(jobs + blockIdx.y, B, factor, (int)blockIdx.x);
}

__global__ __launch_bounds__(kScatterThreads) void csr_scatter_one(const HopGradJob job, int B, float factor) {
    csr_scatter_rows<false>(&job, B, factor, blockIdx.x);
}

// Input check for CSR data: rowptr non-decreasing over [0, rows], every column id inside [0, d).
// flag[0] becomes 1 on any violation.
__global__ __launch_bounds__(kThreads) void csr_check_kernel(const int64_t* __restrict__ rowptr,
                                                             const int32_t* __restrict__ col, int64_t rows,
                                                             int64_t first, int64_t nnz, int64_t d, int* flag) {
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    bool bad = false;
    if (t < rows) bad = rowptr[t] > rowptr[t + 1] || rowptr[t] < first;
    if (t < nnz) {
        const int32_t c = col[first + t];
        bad = bad || c < 0 || (int64_t)c >= d;
    }
    if (bad) atomicExch(flag, 1);
}

__global__ __launch_bounds__(kThreads) void copy_kernel(float4* __restrict__ dst, const float4* __restrict__ src,
                                                        int64_t n16) {
    int64_t i = (int64_t)blockIdx.x * (kThreads * 4) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < 4; ++u, i += kThreads)
        if (i < n16) dst[i] = src[i];
}

inline int launch_status() { return (int)hipGetLastError(); }

// workgroups of the scatter of a sparse minibatch, and of the margins of n of them
static_assert(kScatterRows == 4 * (kThreads / 64), "four blocks of margins are one of the scatter");
inline int csr_scatter_blocks(int n_jobs, int B) {
    const int rows = (B + kScatterRows - 1) / kScatterRows, turns = (rows + kXcd - 1) / kXcd * kXcd;
    return (int64_t)n_jobs * turns <= kCsrTurns ? turns : rows;
}
inline int64_t csr_margin_blocks(int n_jobs, int B) {
    return 4 * (((int64_t)n_jobs * csr_scatter_blocks(n_jobs, B) + kXcd - 1) / kXcd * kXcd);
}

}  // namespace

// More jobs than a grid has rows (kMaxGridYZ) go in several launches: the records of a launch need no order between them.
template <class Job, class F>
static int in_parts(const Job* jobs, int n_jobs, F launch) {
    for (int64_t at = 0; at < n_jobs; at += kMaxGridYZ)
        if (const int rc = launch(jobs + at, (int)std::min<int64_t>(n_jobs - at, kMaxGridYZ))) return rc;
    return 0;
}

int hopk_mix(const HopMixJob* jobs_dev, int n_jobs, int64_t d, void* stream) {
    return in_parts(jobs_dev, n_jobs, [&](const HopMixJob* jobs, int n) {
        Runs runs;
        dim3 grid;
        if (!mix_grid(n, d, 0, &runs, &grid)) return (int)hipErrorInvalidConfiguration;
        const auto kernel = hop_stays_near(n, d, 3) ? mix_kernel<true> : mix_kernel<false>;
        hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, (hipStream_t)stream, jobs, d, HOP_RUNS_OF(runs));
        return launch_status();
    });
}

int hopk_synth(const HopGradJob* jobs_dev, int n_jobs, int reverse, int64_t d, void* stream) {
    const int64_t n = ((d >> 2) + kSynthChunk4 - 1) / kSynthChunk4, n_chunks = n < 1 ? 1 : n;
    return in_parts(jobs_dev, n_jobs, [&](const HopGradJob* jobs, int n_part) {
        dim3 grid;
        if (!chunk_grid(n_part, n_chunks, &grid)) return (int)hipErrorInvalidConfiguration;
        hipLaunchKernelGGL(synth_kernel, grid, dim3(kThreads), 0, (hipStream_t)stream, jobs, (int)grid.x, reverse, d, n_chunks);
        return launch_status();
    });
}

template <int MODE, bool MOM>
static void launch_sweep(const HopSweepArgs& a, unsigned grid, void* stream) {
    const dim3 blocks(grid), threads(kSweepThreads);
    const hipStream_t st = (hipStream_t)stream;
    if (a.n_local <= 48) hipLaunchKernelGGL((sweep_kernel<MODE, MOM, 48>), blocks, threads, 0, st, a);
    else if (a.n_local <= 80) hipLaunchKernelGGL((sweep_kernel<MODE, MOM, 80>), blocks, threads, 0, st, a);
    else if (a.n_local <= 112) hipLaunchKernelGGL((sweep_kernel<MODE, MOM, 112>), blocks, threads, 0, st, a);
    else hipLaunchKernelGGL((sweep_kernel<MODE, MOM, kSweepRegisters>), blocks, threads, 0, st, a);
}
template <int MODE>
static void launch_sweep(const HopSweepArgs& a, unsigned grid, void* stream) {
    if (a.velocities) launch_sweep<MODE, true>(a, grid, stream);
    else launch_sweep<MODE, false>(a, grid, stream);
}

int hopk_sweep(const HopSweepArgs& a, void* stream) {
    if (a.n_records <= 0) return 0;
    if (a.n_local > kSweepRegisters) return (int)hipErrorInvalidValue;
    const int64_t grid = (a.d + kSweepThreads - 1) / kSweepThreads;
    if (grid > 0x7FFFFFFFll) return (int)hipErrorInvalidConfiguration;
    if (a.mode == HOP_GRAD_SYNTH) launch_sweep<HOP_GRAD_SYNTH>(a, (unsigned)grid, stream);
    else if (a.mode == HOP_GRAD_EXTERNAL) launch_sweep<HOP_GRAD_EXTERNAL>(a, (unsigned)grid, stream);
    else launch_sweep<HOP_GRAD_ZERO>(a, (unsigned)grid, stream);
    return launch_status();
}

int hopk_dense_nseg(int64_t d) {
    int64_t n = (d + kSegCols - 1) / kSegCols;
    return (int)(n < 1 ? 1 : n);
}

int hopk_dense_margin(const HopGradJob* jobs_dev, int n_jobs, int B, int64_t d, void* stream) {
    if (n_jobs <= 0 || B <= 0) return 0;
    const int nseg = hopk_dense_nseg(d), groups = (B + kMarginRows - 1) / kMarginRows;
    const int64_t blocks = (int64_t)n_jobs * groups * nseg;
    if (blocks > 0x7FFFFFFFll || B > kMaxB) return (int)hipErrorInvalidConfiguration;
    const bool near = (int64_t)n_jobs * B * d * 4 <= kMarginNear;
    if (hop_wave_slices(n_jobs, B, d))
        return in_parts(jobs_dev, n_jobs, [&](const HopGradJob* jobs, int n) {
            const dim3 rows(kXcd, (unsigned)B, (unsigned)n), pairs(kXcd, (unsigned)((B + kSliceRows - 1) / kSliceRows), (unsigned)n);
#define HOP_SLICES(GRID, ROWS, STREAM)                                                                                      \
    hipLaunchKernelGGL((dense_margin_kernel<ROWS, STREAM, Cut::slices>), GRID, dim3(kThreads), 0, (hipStream_t)stream, jobs, \
                       B, d, kXcd)
            if ((int64_t)n * groups * kXcd < kMarginFew) HOP_SLICES(rows, 1, false);
            else if (near) HOP_SLICES(pairs, kSliceRows, false);
            else HOP_SLICES(pairs, kSliceRows, true);
#undef HOP_SLICES
            return launch_status();
        });
    return in_parts(jobs_dev, n_jobs, [&](const HopGradJob* jobs, int n) {
        const dim3 rows((unsigned)nseg, (unsigned)B, (unsigned)n), fours((unsigned)nseg, (unsigned)groups, (unsigned)n);
#define HOP_MARGINS(GRID, ROWS, STREAM, ONE)                                                                                \
    hipLaunchKernelGGL((dense_margin_kernel<ROWS, STREAM, ONE>), GRID, dim3(kThreads), 0, (hipStream_t)stream, jobs, B, d, nseg)
        if (blocks < kMarginFew && nseg == 1) HOP_MARGINS(rows, 1, false, Cut::one);
        else if (blocks < kMarginFew) HOP_MARGINS(rows, 1, false, Cut::segments);
        else if (nseg == 1) HOP_MARGINS(fours, kMarginRows, true, Cut::one);
        else HOP_MARGINS(fours, kMarginRows, true, Cut::segments);
#undef HOP_MARGINS
        return launch_status();
    });
}

enum class GradShape { few, some, many };
static GradShape grad_shape(int n_jobs, int64_t d, int nseg) {
    const int64_t chunks = n_jobs * ((d + 255) / 256);
    return chunks > kGradMany || nseg >= kGradSegs ? GradShape::many : chunks > kGradFew ? GradShape::some : GradShape::few;
}

int hopk_dense_grad(const HopGradJob* jobs_dev, int n_jobs, int B, int64_t d, float lambda, int loss, bool rows_again, void* stream) {
    if (n_jobs <= 0 || B <= 0) return 0;
    if (B > kMaxB) return (int)hipErrorInvalidValue;
    const int nseg = hopk_dense_nseg(d);
    const GradShape shape = grad_shape(n_jobs, d, nseg);
    if (hop_one_xcd(n_jobs, B, d)) {
        const dim3 grid(kXcd, (unsigned)((d + 255) / 256), (unsigned)((n_jobs + kXcd - 1) / kXcd));
        hipLaunchKernelGGL(dense_grad_near_kernel, grid, dim3(512), 0, (hipStream_t)stream, jobs_dev, n_jobs, B, d, lambda, loss);
        return launch_status();
    }
    if (hop_wave_slices(n_jobs, B, d))
        return in_parts(jobs_dev, n_jobs, [&](const HopGradJob* jobs, int n) {
            const int cols = shape == GradShape::many ? 1024 : 256, n_chunks = (int)((d + cols - 1) / cols);
            const dim3 grid(kXcd, (unsigned)n, (unsigned)((n_chunks + kXcd - 1) / kXcd));
            const bool cached = rows_again && (int64_t)n_jobs * B * d * 4 > kRowsNear;
            const auto kernel = shape == GradShape::few    ? cached ? dense_grad_slice_kernel<8, 1, false> : dense_grad_slice_kernel<8, 1, true>
                                : shape == GradShape::some ? cached ? dense_grad_slice_kernel<4, 1, false> : dense_grad_slice_kernel<4, 1, true>
                                                           : cached ? dense_grad_slice_kernel<1, 4, false> : dense_grad_slice_kernel<1, 4, true>;
            hipLaunchKernelGGL(kernel, grid, dim3(shape == GradShape::few ? 512 : 256), 0, (hipStream_t)stream, jobs, n_chunks, B, d, lambda,
                               loss);
            return launch_status();
        });
    const int64_t cols = shape == GradShape::many ? 1024 : 256, n_chunks = (d + cols - 1) / cols;
    return in_parts(jobs_dev, n_jobs, [&](const HopGradJob* jobs, int n) {
        dim3 grid;
        if (!chunk_grid(n, n_chunks, &grid)) return (int)hipErrorInvalidConfiguration;
#define HOP_GRADS(SPLIT, WIDE, ONE)                                                                                         \
    hipLaunchKernelGGL((dense_grad_kernel<SPLIT, WIDE, ONE>), grid, dim3(64 * SPLIT * WIDE), 0, (hipStream_t)stream, jobs,   \
                       (int)grid.x, B, d, nseg, lambda, loss, n_chunks)
        if (shape == GradShape::few && nseg == 1) HOP_GRADS(8, 1, true);
        else if (shape == GradShape::few) HOP_GRADS(8, 1, false);
        else if (shape == GradShape::some && nseg == 1) HOP_GRADS(4, 1, true);
        else if (shape == GradShape::some) HOP_GRADS(4, 1, false);
        else if (nseg == 1) HOP_GRADS(1, 4, true);
        else HOP_GRADS(1, 4, false);
#undef HOP_GRADS
        return launch_status();
    });
}

int hopk_csr_margin(const HopGradJob* jobs_dev, int n_jobs, int B, int loss, void* stream) {
    if (n_jobs <= 0 || B <= 0) return 0;
    const int64_t blocks = csr_margin_blocks(n_jobs, B);
    if (blocks > 0x7FFFFFFFll) return (int)hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(csr_margin_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, (hipStream_t)stream, jobs_dev, n_jobs, B,
                       (unsigned)csr_scatter_blocks(n_jobs, B), loss);
    return launch_status();
}

// workgroups of margins that keep to one XCD a record
static int64_t near_margins(int n_grad, int B) { return (int64_t)(n_grad + kXcd - 1) / kXcd * kXcd * B; }

// Margins in front of a Reduce over at most kMaxGridYZ jobs; the rest of a longer one behind it, by itself.
int hopk_mix_dense_margin(const HopMixJob* mix_dev, int n_mix, int64_t d, const HopGradJob* grad_dev, int n_grad, int B,
                          void* stream) {
    if (n_grad <= 0 || B <= 0) return hopk_mix(mix_dev, n_mix, d, stream);
    if (n_mix <= 0) return hopk_dense_margin(grad_dev, n_grad, B, d, stream);
    const int nseg = hopk_dense_nseg(d), n = (int)std::min<int64_t>(n_mix, kMaxGridYZ);
    const bool one = hop_one_xcd(n_grad, B, d);
    const int64_t margins = one ? near_margins(n_grad, B) : (int64_t)n_grad * B * nseg;
    Runs runs;
    dim3 grid;
    if (!mix_grid(n, d, margins, &runs, &grid)) return (int)hipErrorInvalidConfiguration;
    const auto kernel = one                            ? mix_dense_margin_kernel<true, true>
                        : hop_in_place_near(n_grad, d) ? mix_dense_margin_kernel<false, true>
                                                       : mix_dense_margin_kernel<false, false>;
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, (hipStream_t)stream, mix_dev, d, runs.front, HOP_RUNS_OF(runs),
                       (unsigned)margins, n, grad_dev, B, one ? n_grad : nseg);
    if (const int rc = launch_status()) return rc;
    return hopk_mix(mix_dev + n, n_mix - n, d, stream);
}

int hopk_mix_csr_margin(const HopMixJob* mix_dev, int n_mix, int64_t d, const HopGradJob* grad_dev, int n_grad, int B,
                        int loss, void* stream) {
    if (n_grad <= 0 || B <= 0) return hopk_mix(mix_dev, n_mix, d, stream);
    if (n_mix <= 0) return hopk_csr_margin(grad_dev, n_grad, B, loss, stream);
    const int n = (int)std::min<int64_t>(n_mix, kMaxGridYZ);
    const int64_t margins = csr_margin_blocks(n_grad, B);
    Runs runs;
    dim3 grid;
    if (!mix_grid(n, d, margins, &runs, &grid)) return (int)hipErrorInvalidConfiguration;
    const auto kernel = hop_stays_near(n, d, 3) ? mix_csr_margin_kernel<true> : mix_csr_margin_kernel<false>;
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, (hipStream_t)stream, mix_dev, d,
                       runs.front, HOP_RUNS_OF(runs), (unsigned)margins, n, grad_dev, n_grad, B, (unsigned)csr_scatter_blocks(n_grad, B), loss);
    if (const int rc = launch_status()) return rc;
    return hopk_mix(mix_dev + n, n_mix - n, d, stream);
}

static int launch_pairs(const HopPairJob* jobs_dev, int n_jobs, int n_sources, int reverse, int64_t d, bool may_near, void* stream) {
    return in_parts(jobs_dev, n_jobs, [&](const HopPairJob* jobs, int n) {
        PairShape p;
        if (!pair_shape(&p, n, n_sources, d, may_near)) return (int)hipErrorInvalidConfiguration;
        const auto kernel = p.vec == 4 ? p.near ? pair_mix_kernel<4, true> : pair_mix_kernel<4, false>
                                       : p.near ? pair_mix_kernel<kPairPlain, true> : pair_mix_kernel<kPairPlain, false>;
        hipLaunchKernelGGL(kernel, p.grid, dim3(kThreads), 0, (hipStream_t)stream, jobs, d, p.near ? 0 : reverse, HOP_RUNS_OF(p.runs));
        return launch_status();
    });
}

int hopk_pair(const HopPairJob* jobs_dev, int n_jobs, int n_sources, int reverse, int64_t d, void* stream) {
    return launch_pairs(jobs_dev, n_jobs, n_sources, reverse, d, true, stream);
}

int hopk_pair_alone(const HopPairJob* jobs_dev, int n_jobs, int n_results, int n_sources, int64_t d, void* stream) {
    return launch_pairs(jobs_dev, n_jobs, n_sources, 0, d, hop_near_alone(n_jobs, n_results, d), stream);
}

int hopk_pair_csr_margin(const HopPairJob* mix_dev, int n_mix, int n_results, int n_sources, int reverse, int64_t d,
                         const HopGradJob* grad_dev, int n_grad, int B, int loss, void* stream) {
    if (n_grad <= 0 || B <= 0) return hopk_pair(mix_dev, n_mix, n_sources, reverse, d, stream);
    if (n_mix <= 0) return hopk_csr_margin(grad_dev, n_grad, B, loss, stream);
    const int n = (int)std::min<int64_t>(n_mix, kMaxGridYZ);
    const int64_t margins = csr_margin_blocks(n_grad, B);
    PairShape p;
    if (!pair_shape(&p, n, n_sources, d, true, true, margins, n_mix == n_results)) return (int)hipErrorInvalidConfiguration;
    const auto kernel = p.vec == 4 ? pair_csr_margin_kernel<4, false>
                        : p.near   ? pair_csr_margin_kernel<kPairMargin, true>
                                   : pair_csr_margin_kernel<kPairMargin, false>;
    hipLaunchKernelGGL(kernel, p.grid, dim3(kThreads), 0, (hipStream_t)stream, mix_dev, d, p.runs.front, HOP_RUNS_OF(p.runs),
                       p.near ? 0 : reverse, (unsigned)margins, n, grad_dev, n_grad, B, (unsigned)csr_scatter_blocks(n_grad, B), loss);
    if (const int rc = launch_status()) return rc;
    return hopk_pair(mix_dev + n, n_mix - n, n_sources, reverse, d, stream);
}

int hopk_pair_dense_margin(const HopPairJob* mix_dev, int n_mix, int n_sources, int reverse, int64_t d,
                           const HopGradJob* grad_dev, int n_grad, int B, void* stream) {
    if (n_grad <= 0 || B <= 0) return hopk_pair(mix_dev, n_mix, n_sources, reverse, d, stream);
    if (n_mix <= 0) return hopk_dense_margin(grad_dev, n_grad, B, d, stream);
    if (hop_dense_slices(B, d)) {                      // large minibatches: the records without a gradient
        const bool few = (int64_t)n_grad * ((B + kMarginRows - 1) / kMarginRows) * kXcd < kMarginFew;
        const int groups = few ? B : (B + kSliceRows - 1) / kSliceRows;
        const int64_t n_chunks = pair_chunks(d, kPairMargin), round = (int64_t)groups * kXcd;
        const int64_t z = n_grad + (n_mix * n_chunks + round - 1) / round;
        if (!hop_wave_slices(n_grad, B, d) || z > kMaxGridYZ || z * round > 0x7FFFFFFFll) {
            const int rc = hopk_dense_margin(grad_dev, n_grad, B, d, stream);
            return rc ? rc : hopk_pair(mix_dev, n_mix, n_sources, reverse, d, stream);
        }
        const bool near = (int64_t)n_grad * B * d * 4 <= kMarginNear;
        const auto kernel = few    ? pair_dense_slice_kernel<1, false>
                            : near ? pair_dense_slice_kernel<kSliceRows, false>
                                   : pair_dense_slice_kernel<kSliceRows, true>;
        hipLaunchKernelGGL(kernel, dim3(kXcd, (unsigned)groups, (unsigned)z), dim3(kThreads), 0, (hipStream_t)stream, grad_dev, d, B, n_grad,
                           groups, (int)n_chunks, n_mix, mix_dev);
        return launch_status();
    }
    const int nseg = hopk_dense_nseg(d), n = (int)std::min<int64_t>(n_mix, kMaxGridYZ);
    const bool one = hop_one_xcd(n_grad, B, d) && pair_vec(n, d, true) == kPairMargin;
    const int64_t margins = one ? near_margins(n_grad, B) : (int64_t)n_grad * B * nseg;
    PairShape p;
    if (!pair_shape(&p, n, n_sources, d, true, true, margins)) return (int)hipErrorInvalidConfiguration;
    const auto kernel = p.vec == 4                     ? pair_dense_margin_kernel<4, false, false>       // 128 MB of jobs and more
                        : one                          ? pair_dense_margin_kernel<kPairMargin, true, true>
                        : hop_in_place_near(n_grad, d) ? pair_dense_margin_kernel<kPairMargin, false, true>
                                                       : pair_dense_margin_kernel<kPairMargin, false, false>;
    hipLaunchKernelGGL(kernel, p.grid, dim3(kThreads), 0, (hipStream_t)stream, mix_dev, d, p.runs.front, HOP_RUNS_OF(p.runs),
                       p.near ? 0 : reverse, (unsigned)margins, n, grad_dev, B, one ? n_grad : nseg);
    if (const int rc = launch_status()) return rc;
    return hopk_pair(mix_dev + n, n_mix - n, n_sources, reverse, d, stream);
}

int hopk_csr_scatter(const HopGradJob* jobs_dev, int n_jobs, int B, float factor, int into_velocity, void* stream) {
    if (n_jobs <= 0 || B <= 0) return 0;
    const int per = csr_scatter_blocks(n_jobs, B);
    if ((int64_t)n_jobs * per > 0x7FFFFFFFll) return (int)hipErrorInvalidConfiguration;
    return in_parts(jobs_dev, n_jobs, [&](const HopGradJob* jobs, int n) {
        const dim3 grid((unsigned)per, (unsigned)n), threads(kScatterThreads);
        if (into_velocity)
            hipLaunchKernelGGL(csr_scatter_kernel<true>, grid, threads, 0, (hipStream_t)stream, jobs, B, factor);
        else
            hipLaunchKernelGGL(csr_scatter_kernel<false>, grid, threads, 0, (hipStream_t)stream, jobs, B, factor);
        return launch_status();
    });
}

int hopk_one_grad(const HopGradJob& given, int mode, int B, int64_t d, float lambda, int loss, void* stream) {
    const hipStream_t st = (hipStream_t)stream;
    HopGradJob job = given;
    if (mode == HOP_GRAD_SVM_DENSE) {
        job.k0 = (uint32_t)loss;
        const int nseg = hopk_dense_nseg(d);
        const int64_t few = (int64_t)B * nseg, grid = (int64_t)((B + kMarginRows - 1) / kMarginRows) * nseg;
        if (B > kMaxB) return (int)hipErrorInvalidValue;
        if (grid > 0x7FFFFFFFll || (d + 255) / 256 > 0x7FFFFFFFll) return (int)hipErrorInvalidConfiguration;
        const dim3 threads(kThreads), rows((unsigned)few), groups((unsigned)grid);
        if (hop_one_xcd_alone(B, d)) {
            hipLaunchKernelGGL(dense_margin_near_one, dim3(kXcd, (unsigned)B), threads, 0, st, job, B, d);
            if (const int rc = launch_status()) return rc;
            hipLaunchKernelGGL(dense_grad_near_one, dim3(kXcd, (unsigned)((d + 255) / 256)), dim3(512), 0, st, job, B, d, lambda, loss);
            return launch_status();
        }
        if (nseg == 1 && grid < kMarginFew)
            hipLaunchKernelGGL((dense_margin_one<1, false, true>), rows, threads, 0, st, job, B, d, nseg);
        else if (grid < kMarginFew)
            hipLaunchKernelGGL((dense_margin_one<1, false, false>), rows, threads, 0, st, job, B, d, nseg);
        else
            hipLaunchKernelGGL((dense_margin_one<kMarginRows, true, false>), groups, threads, 0, st, job, B, d, nseg);
        if (const int rc = launch_status()) return rc;
        const GradShape shape = grad_shape(1, d, nseg);
        const unsigned chunks = (unsigned)((d + 255) / 256);
        static_assert((kMaxB + kMarginRows - 1) / kMarginRows < kMarginFew && kSegCols / 256 <= kGradFew, "one segment: few of both");
        if (nseg == 1)
            hipLaunchKernelGGL((dense_grad_one<8, 1, true>), dim3(chunks), dim3(512), 0, st, job, B, d, nseg, lambda, loss);
        else if (shape == GradShape::few)
            hipLaunchKernelGGL((dense_grad_one<8, 1, false>), dim3(chunks), dim3(512), 0, st, job, B, d, nseg, lambda, loss);
        else if (shape == GradShape::some)
            hipLaunchKernelGGL((dense_grad_one<4, 1, false>), dim3(chunks), dim3(256), 0, st, job, B, d, nseg, lambda, loss);
        else
            hipLaunchKernelGGL((dense_grad_one<1, 4, false>), dim3((chunks + 3) / 4), dim3(256), 0, st, job, B, d, nseg, lambda, loss);
    } else if (mode == HOP_GRAD_SVM_CSR) {
        const int margin_blocks = (B + kThreads / 64 - 1) / (kThreads / 64);
        const int64_t dense_blocks = (d + 4 * kThreads - 1) / (4 * kThreads), grid = margin_blocks + dense_blocks;
        if (grid > 0x7FFFFFFFll) return (int)hipErrorInvalidConfiguration;
        const uintptr_t w0 = (uintptr_t)job.w, g0 = (uintptr_t)job.out, bytes = (uintptr_t)d * sizeof(float);
        if (w0 < g0 + bytes && g0 < w0 + bytes) {          // g over w: the margins read w first
            hipLaunchKernelGGL(csr_margin_dense_one, dim3((unsigned)margin_blocks), dim3(kThreads), 0, st, job, B, d, lambda,
                               loss, margin_blocks);
            hipLaunchKernelGGL(csr_margin_dense_one, dim3((unsigned)dense_blocks), dim3(kThreads), 0, st, job, B, d, lambda,
                               loss, 0);
        } else {
            hipLaunchKernelGGL(csr_margin_dense_one, dim3((unsigned)grid), dim3(kThreads), 0, st, job, B, d, lambda, loss,
                               margin_blocks);
        }
        if (const int rc = launch_status()) return rc;
        hipLaunchKernelGGL(csr_scatter_one, dim3((unsigned)((B + kScatterRows - 1) / kScatterRows)), dim3(kScatterThreads), 0,
                           st, job, B, -1.0f);
    } else {
        const int64_t n = ((d >> 2) + kSynthChunk4 - 1) / kSynthChunk4, n_chunks = n < 1 ? 1 : n;
        if (n_chunks > 0x7FFFFFFFll) return (int)hipErrorInvalidConfiguration;
        hipLaunchKernelGGL(synth_one_kernel, dim3((unsigned)n_chunks), dim3(kThreads), 0, st, job, d, n_chunks);
    }
    return launch_status();
}

int hopk_pair_args(const HopPairArg* jobs, int n_jobs, int n_sources, int64_t d, void* stream) {
    if (n_jobs <= 0) return 0;
    if (n_jobs > kPairArgs) return (int)hipErrorInvalidValue;
    HopPairArgs args;
    memcpy(args.job, jobs, (size_t)n_jobs * sizeof(HopPairArg));
    PairShape p;
    if (!pair_shape(&p, n_jobs, n_sources, d, false)) return (int)hipErrorInvalidConfiguration;
    const auto kernel = p.vec == 4 ? pair_mix_args_kernel<4> : pair_mix_args_kernel<kPairPlain>;
    hipLaunchKernelGGL(kernel, p.grid, dim3(kThreads), 0, (hipStream_t)stream, args, d, HOP_RUNS_OF(p.runs));
    return launch_status();
}

int hopk_csr_check(const int64_t* rowptr, const int32_t* col, int64_t rows, int64_t first, int64_t nnz, int64_t d,
                   int* flag_dev, void* stream) {
    int64_t n = rows > nnz ? rows : nnz;
    if (n <= 0) return 0;
    int64_t grid = (n + kThreads - 1) / kThreads;
    if (grid > 0x7FFFFFFFll) return (int)hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(csr_check_kernel, dim3((unsigned)grid), dim3(kThreads), 0, (hipStream_t)stream, rowptr, col,
                       rows, first, nnz, d, flag_dev);
    return launch_status();
}

int hopk_copy(void* dst, const void* src, size_t bytes, void* stream) {
    int64_t n16 = (int64_t)(bytes / 16);
    if (n16 <= 0) return 0;
    int64_t grid = (n16 + kThreads * 4 - 1) / (kThreads * 4);
    if (grid > 0x7FFFFFFFll) return (int)hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)grid), dim3(kThreads), 0, (hipStream_t)stream, (float4*)dst,
                       (const float4*)src, n16);
    return launch_status();
}

// ------------------------------------------- dense SVM gradient without any allocation ----
// For callers that cannot allocate (a stream being captured, a tight serving loop, a harness that forbids
// hipMalloc): the partial dot products, which hop_svm_grad_dense keeps in the caller's scratch argument, live in a fixed
// array in device memory instead.
namespace {

constexpr int64_t kStaticPartials = 65536;                 // most B x column segments (16384 columns each)
static __device__ __align__(256) unsigned char scratch[kStaticPartials * sizeof(float)];

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];                          // device address of `scratch` on each GPU, once known
int g_scratch_state[kMaxDevices];                          // 0 unknown, 1 known

}  // namespace

extern "C" int hop_svm_grad_dense_static(const float* X, const float* y, const float* w, const int32_t* rows_dev,
                                         int32_t B, int64_t d, float lambda, int32_t loss, float* g, float* coef,
                                         void* hip_stream) {
    if (!X || !y || !w || !rows_dev || !g || !coef || B < 1 || B > kMaxB || d < 1 ||
        (loss != HOP_LOSS_HINGE && loss != HOP_LOSS_LOG))
        return HOP_ERR_INVALID_ARG;
    if (d % 4 == 0 && ((((uintptr_t)X | (uintptr_t)w | (uintptr_t)g) & 15u) != 0)) return HOP_ERR_INVALID_ARG;
    const int nseg = hopk_dense_nseg(d);
    if ((int64_t)B * nseg > kStaticPartials) {
        fprintf(stderr, "libhop: hop_svm_grad_dense_static: B x ceil(d / 16384) = %lld exceeds the fixed scratch of %lld "
                        "partial sums\n", (long long)B * nseg, (long long)kStaticPartials);
        return HOP_ERR_ARENA_TOO_SMALL;
    }
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return HOP_ERR_HIP;
    if (!g_scratch_state[dev]) {
        // each GPU holds its own copy of the array at its own address: ask once per device, with it current
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) {
            fprintf(stderr, "libhop: hipGetSymbolAddress(scratch): %s\n", hipGetErrorString(e));
            return HOP_ERR_HIP;
        }
        g_scratch_ptr[dev] = p;
        g_scratch_state[dev] = 1;
    }
    unsigned char* base = (unsigned char*)g_scratch_ptr[dev];
    HopGradJob gj;
    memset(&gj, 0, sizeof(gj));
    gj.X = X; gj.y = y; gj.w = w; gj.rows = rows_dev; gj.g = g; gj.coef = coef;
    gj.partial = (float*)base;                             // every entry is written by the margin pass before it is read
    const int rc = hopk_one_grad(gj, HOP_GRAD_SVM_DENSE, B, d, lambda, loss, hip_stream);
    if (rc) {
        fprintf(stderr, "libhop: hop_svm_grad_dense_static launch: %s\n", hipGetErrorString((hipError_t)rc));
        return HOP_ERR_HIP;
    }
    return HOP_OK;
}
