// fwi_device.h -- device helpers shared by the kernel files: stencil weights,
// job lookup, level addressing, the sponge update and global-memory accesses.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fwi_internal.h"

namespace fwi {

// ----------------------------------------------------------------- weights
// Maximal-order central second-derivative weights:
//   c_m = 2 (-1)^{m+1} (M!)^2 / (m^2 (M-m)! (M+m)!)   (difference form: c_0 unused)
__host__ __device__ constexpr double factd(int n) { return n <= 1 ? 1.0 : double(n) * factd(n - 1); }
__host__ __device__ constexpr double weightd(int M, int m)
{
    return 2.0 * ((m & 1) ? 1.0 : -1.0) * factd(M) * factd(M) /
           (double(m) * double(m) * factd(M - m) * factd(M + m));
}
template <int M>
struct Weights {
    float c[M + 1];
    float t3[M + 1], t2[M + 1];   // -6 resp. -4 times sum_{m > k} c_m
    __host__ __device__ constexpr Weights() : c(), t3(), t2()
    {
        for (int m = 1; m <= M; ++m) c[m] = float(weightd(M, m));
        for (int k = 0; k <= M; ++k) {
            double t = 0.0;
            for (int m = k + 1; m <= M; ++m) t += weightd(M, m);
            t3[k] = float(-6.0 * t);
            t2[k] = float(-4.0 * t);
        }
    }
};

// Radius 1, which carries most of the weight (c_1 = 1.6 of sum |c_m| = 1.83
// at 8th order), is summed in difference form (p_{+1} - p) + (p_{-1} - p),
// exact for neighbouring values of similar size.  The outer radii add plain
// neighbour sums and one -2 D (sum_{m>1} c_m) p term: half the arithmetic,
// and their rounding (about 6 eps |p| times their small weights) stays below
// that of radius 1.  Measured against the FP64 oracle, every parity case
// keeps its error within a factor of two of the all-difference form, and
// the 16th-order step runs 19 % faster.  FWI_DIFF_RADII at build time sets
// another number of difference-form radii (99: all).
#ifndef FWI_DIFF_RADII
#define FWI_DIFF_RADII 1
#endif
constexpr int kDiffRadii = FWI_DIFF_RADII;

// ----------------------------------------------------------------- helpers
__device__ __forceinline__ int sponge_depth(int i, int n, int nb)
{
    // cells into the sponge along one axis: max(nb - i, i - (n - 1 - nb), 0)
    return max(max(nb - i, i - (n - 1 - nb)), 0);
}

__device__ __forceinline__ int find_job(const int *__restrict__ prefix, int njobs, int b)
{
    int lo = 0, hi = njobs;   // prefix[lo] <= b < prefix[hi]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (prefix[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

// Blocks are dealt round-robin to the 8 XCDs; give XCD k the k-th contiguous
// eighth of the tile range instead (a bijection on [0, T)).
__device__ __forceinline__ int xcd_remap(int b, int T)
{
    const int q = T >> 3, r = T & 7, k = b & 7, i = b >> 3;
    return k * q + min(k, r) + i;
}

__device__ __forceinline__ int mod_pos(int a, int R) { int m = a % R; return m < 0 ? m + R : m; }

// Time level a launch's step updates for job J: n0 + step (forward) or
// k0 - step (adjoint), or, for jobs that change direction within a chunk
// (binomial checkpointing in the serving path), the step's entry of the job's
// level list (kNoLevel: no step of this launch's direction in that round).
__device__ __forceinline__ int step_level(const Job *__restrict__ J, int step, bool adj)
{
    // The list entry is block-uniform, but the compiler cannot see that through
    // a global load; without readfirstlane every plane base and buffer
    // resource derived from it would be built lane by lane (waterfall loops,
    // 20 % slower steps).
    if (J->lev) return __builtin_amdgcn_readfirstlane(J->lev[step]);
    return adj ? J->k0 - step : J->n0 + step;
}

// Field of forward level L: the ring slot L mod R, or a snapshot field the
// level map names (block-uniform, scalar).
__device__ __forceinline__ float *level_ptr(const Job *__restrict__ J, const LevelMap &lm, int L)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (lm.lev[i] == L) return J->snap + (int64_t)lm.fld[i] * J->fstride;
    return J->ring + (int64_t)mod_pos(L, J->R) * J->fstride;
}

// Receiver sampling: traces[n-1][r] = p^n[rec_r] (level n is read-only here).
__device__ __forceinline__ void gather_block(const Job *__restrict__ J, const LevelMap &lm, int r,
                                             int n)
{
    if (!J->record || n < 1 || n > J->nt || r >= J->nrec) return;
    const float *cur = level_ptr(J, lm, n);
    J->traces[(int64_t)(n - 1) * J->nrec + r] = cur[J->rec_off[r]];
}

// Adjoint source at receiver r (the first of its cell): the sum of
// res[k-1] over the receivers sharing the cell, in index order, so the
// result is deterministic.  psi'^k gains kappa' times it (alpha = 1 on the
// model grid, where every receiver sits).
__device__ __forceinline__ float adj_source(const Job *__restrict__ J, int k, int r)
{
    const float *res = J->res + (int64_t)(k - 1) * J->nrec;
    float s = res[r];
    for (int q = J->rec_next[r]; q >= 0; q = J->rec_next[q]) s += res[q];
    return s;
}

// Sponge factors from the squared depth d2 = sum_a d_a^2 into the sponge:
// eta dt = eta_dt * d2, alpha = 1/(1 + eta dt), beta = (1 - eta dt) alpha.
// out = alpha * val - beta * prev, written as alpha * (val - (1 - e) prev).
__device__ __forceinline__ float leapfrog(float val, float prev, int d2, float eta_dt)
{
    if (d2 == 0) return val - prev;
    return __builtin_amdgcn_rcpf(fmaf(eta_dt, (float)d2, 1.f)) *
           fmaf(-fmaf(-eta_dt, (float)d2, 1.f), prev, val);
}

// Field pointers come from the job table, so the compiler cannot see that
// they address global memory; without the cast every access would be a
// flat load (64-bit address arithmetic per access, and flat loads also hold
// the LDS counter, so each LDS wait would wait for the prefetches too).
#define GMEM __attribute__((address_space(1)))
typedef GMEM float gfloat;

__device__ __forceinline__ const gfloat *gptr(const float *p) { return (const gfloat *)p; }
__device__ __forceinline__ gfloat *gptr(float *p) { return (gfloat *)p; }

// Plane accesses go through a buffer resource (base and size of one plane in
// scalar registers) and a 32-bit per-lane byte offset: no per-lane address
// arithmetic, and an offset past the plane reads zero instead of faulting.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int kRsrcWord3 = 0x00020000;   // raw 32-bit buffer, CDNA
constexpr int kCacheNT = 2;              // non-temporal cache policy
// Streams read or written once per launch (kappa', the previous level, the
// new level, the gradient accumulator) are non-temporal, leaving L2 to the
// rows that neighbouring tiles share (+4 % on the 3-D forward step; keeping
// kappa' or the new level cached instead, for reuse by the next step from the
// Infinity Cache, measured no faster).  FWI_STREAM_CACHED at build time
// restores ordinary accesses.
#ifdef FWI_STREAM_CACHED
constexpr int kStreamPolicy = 0;
#else
constexpr int kStreamPolicy = kCacheNT;
#endif

__device__ __forceinline__ rsrc_t plane_rsrc(const gfloat *f, int zmem, int64_t plane,
                                             int pbytes)
{
    const float *p = (const float *)(f + (int64_t)zmem * plane);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, pbytes, kRsrcWord3);
}
__device__ __forceinline__ float ldb(rsrc_t r, uint32_t boff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)boff, 0, 0));
}
__device__ __forceinline__ float ldb_stream(rsrc_t r, uint32_t boff)
{
    return __builtin_bit_cast(float,
                              __builtin_amdgcn_raw_buffer_load_b32(r, (int)boff, 0, kStreamPolicy));
}
__device__ __forceinline__ void stb_stream(rsrc_t r, uint32_t boff, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)boff, 0,
                                          kStreamPolicy);
}

// Compile-time loop: f(Int<I>{}) for I = B .. E-1, fully unrolled, so an
// index derived from I can select a register.
template <int V>
struct Int {
    static constexpr int value = V;
};
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (B < E) {
        f(Int<B>{});
        static_for<B + 1, E>(f);
    }
}

// Byte offset past every plane: a buffer store to it is dropped by the
// hardware's range check, so masked lanes need no branch around a store.
constexpr uint32_t kDropOffset = 0x7ffffff0u;

// Block barrier for LDS traffic only.  __syncthreads() is a workgroup fence
// over all memory, so each wave first waits for every global load it has in
// flight; a step kernel's prefetches for the next plane would then have to
// arrive within the current plane.  The step kernels share nothing through
// global memory within a launch (a cell's previous level, output and
// gradient are read and written by the thread that owns it), so ordering
// the LDS staging is enough.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace fwi
