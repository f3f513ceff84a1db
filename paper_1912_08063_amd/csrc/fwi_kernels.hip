// fwi_kernels.hip -- gfx950 kernels of the acoustic FWI hot path.
//
// One launch of a step kernel advances every job of a job table by one time
// step (Eq. 3 of the paper with a sponge; star Laplacian of Fig. 3):
//     out = alpha * (2 p + kappa' * L'p + src) - beta * p_prev
// with L'p = sum_m c_m [(p_{+m} - p) + (p_{-m} - p)] summed over the axes
// (the Laplacian times dx^2; radius 1 evaluated in this difference form for
// fp32 accuracy, the outer radii as plain sums) and kappa' = (v dt / dx)^2.  The adjoint launch applies the same operator to
// the scaled adjoint field psi' (psi = kappa*alpha*lambda, divided by dx^2),
// for which the discrete adjoint recurrence IS the forward recurrence, and
// accumulates the imaging condition g += psi'^{k+1} * L'p^k.  The adjoint
// source enters at the receiver cells, inside the step.
//
// Design for CDNA4 (the paper's MXU band-matrix formulation does not apply:
// the star stencil is banded, not a dense contraction, and the step is HBM
// bound at 16 algorithmic bytes per cell-update):
//  * 3-D: 256-thread blocks own a 64 (x) x 16 (y) column of the grid over a
//    chunk of z planes.  Each thread keeps a register queue of 2M+2 planes of
//    four columns for the z-derivative (z marching), and the current xy plane
//    with its M-cell halo is staged in LDS for the x and y derivatives.  Small
//    grids take blocks of 64 x 16 x 2 cells instead (fwi_step3d.hip).
//  * 2-D: one wavefront per block, 64 columns marching down a chunk of rows;
//    runs of consecutive steps take several steps per launch (fwi_step2d.hip).
//  * Wavefronts read and write whole aligned 256-byte row segments.
//  * Blocks are remapped so that each XCD (one L2 each) gets a contiguous
//    range of tiles: neighbouring tiles share their halos in the same L2.
//  * Receiver sampling of level n is done by extra blocks of the launch that
//    computes level n+1 (level n is read-only there), so it costs no launch.
//  * Forward level L is field L mod R of the job's ring unless the launch's
//    level map places it in a snapshot field: binomial checkpointing then
//    reads restored states and writes snapshot states in place, without
//    copies.
#include <algorithm>
#include <mutex>

#include "fwi_device.h"

namespace fwi {

// ------------------------------------------------------------ side kernels
// kappa' = (v dt/dx)^2 on the padded grid (edge-replicated model), 0 on the frame.
// One wavefront per row, so the plane, row and their clamps are found once per
// row.
__global__ __launch_bounds__(256) void k_prep_kappa(const float *__restrict__ v,
                                                    float *__restrict__ kappa, int M, int gy,
                                                    int nz, int ny, int nx, int pitch, int nya,
                                                    int nb, int nzm, int nym, int nxm, int64_t rows,
                                                    float dt_dx)
{
    const int lane = threadIdx.x & 63;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; r < rows; r += nw) {
        const int zi = (int)(r / nya), z = zi - M, y = (int)(r - (int64_t)zi * nya) - gy;
        const bool in = z >= 0 && z < nz && y >= 0 && y < ny;
        const int zm = min(max(z - nb, 0), nzm - 1), ym = min(max(y - nb, 0), nym - 1);
        const float *src = v + ((int64_t)zm * nym + ym) * nxm;
        float *dst = kappa + r * pitch;
        for (int c = lane; c < pitch; c += 64) {
            const int x = c - M;
            float out = 0.f;
            if (in && x >= 0 && x < nx) {
                const float t = src[min(max(x - nb, 0), nxm - 1)] * dt_dx;
                out = t * t;
            }
            dst[c] = out;
        }
    }
}

__global__ void k_fill(float4 *__restrict__ p, int64_t n4, float val)
{
    const float4 w = make_float4(val, val, val, val);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = w;
}

// Snapshots of a leapfrog state (levels t and t-1) for every job of the table.
// dir 0: level -> snap[slot] (the level where the map puts it); 1: snap[slot]
// -> ring; 2: zero the two levels in the ring (t = 0).  mask bit w selects
// level t - w.
__global__ void k_snapshot(const Job *__restrict__ jobs, int slot, int time, int dir, int mask,
                           LevelMap lm)
{
    const Job *J = jobs + (blockIdx.y >> 1);
    const int which = blockIdx.y & 1;
    if (!((mask >> which) & 1)) return;
    float4 *r = reinterpret_cast<float4 *>(
        dir == 0 ? level_ptr(J, lm, time - which)
                 : J->ring + (int64_t)mod_pos(time - which, J->R) * J->fstride);
    float4 *s = reinterpret_cast<float4 *>(J->snap + (int64_t)(2 * slot + which) * J->fstride);
    if (r == s) return;
    typedef float vf4 __attribute__((ext_vector_type(4)));
    const vf4 *from = reinterpret_cast<const vf4 *>(dir == 0 ? r : s);
    vf4 *to = reinterpret_cast<vf4 *>(dir == 0 ? s : r);
    const int64_t n4 = J->fstride / 4, stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // (the fields are distinct.  Four loads in flight, and nothing kept in the caches,
    // where the next step's fields are: the copies of a binomial gradient on 560 x
    // 560 x 304 cells take 127 us instead of 135, and the call 48.8 ms instead of 49.7)
    for (; dir != 2 && i + 3 * stride < n4; i += 4 * stride) {
        vf4 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = __builtin_nontemporal_load(from + i + u * stride);
#pragma unroll
        for (int u = 0; u < 4; ++u) __builtin_nontemporal_store(t[u], to + i + u * stride);
    }
    for (; i < n4; i += stride) to[i] = dir == 2 ? vf4{0.f, 0.f, 0.f, 0.f} : from[i];
}
// Final receiver sampling (level n = n0 + step).
__global__ void k_gather(const Job *__restrict__ jobs, const int *__restrict__ gprefix,
                         int njobs, int step, LevelMap lm)
{
    const int j = find_job(gprefix, njobs, blockIdx.x);
    const Job *J = jobs + j;
    gather_block(J, lm, (blockIdx.x - gprefix[j]) * blockDim.x + threadIdx.x, J->n0 + step);
}

// Misfit (Eq. 1) and adjoint source: res = 2 (d - obs); per-block partial sums
// of (d - obs)^2 in fp64, reduced in a fixed order (deterministic).
// d and res may be the same array (traces recorded into the residual
// buffer): each element is read and then written by the same thread, and
// neither pointer is declared restrict.
__global__ __launch_bounds__(256) void k_misfit(const float *d, const float *__restrict__ obs,
                                                float *res, int64_t n,
                                                double *__restrict__ partial)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double e = (double)d[i] - (double)obs[i];
        res[i] = (float)(2.0 * e);
        acc += e * e;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void k_sum_partials(const double *__restrict__ partial,
                                                      int n, double *__restrict__ out)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) acc += partial[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

// Transpose of the edge padding, one axis at a time: padded index i of an
// axis of padded length np maps to model index clamp(i - nb, 0, nm - 1).
__device__ __forceinline__ void fold_range(int im, int nm, int np, int nb, int &lo, int &hi)
{
    lo = im == 0 ? 0 : im + nb;
    hi = im == nm - 1 ? np - 1 : im + nb;
}

// The passes go by tasks of one wave: kFoldCols columns of a row of the result.
constexpr int kFoldCols = 256;

// Adds n rows, `stride` apart, to columns c, c + 64, ... of a row of nc, in
// their order.  16 loads in flight per lane: the cells at the edges sum nb + 1
// rows, and with one load after the other these set the time of a pass.
__device__ __forceinline__ void fold_rows(const float *__restrict__ p, int64_t stride, int n,
                                          int c, int nc, float (&s)[kFoldCols / 64])
{
    constexpr int Q = kFoldCols / 64;
    int col[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) col[q] = min(c + 64 * q, nc - 1);
    for (; n >= 4; n -= 4, p += 4 * stride) {
        float t[4][Q];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < Q; ++q) t[u][q] = p[u * stride + col[q]];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < Q; ++q) s[q] += t[u][q];
    }
    for (; n > 0; --n, p += stride)
#pragma unroll
        for (int q = 0; q < Q; ++q) s[q] += p[col[q]];
}

// Sum of g[lo .. hi], added to s in order: 64 values are loaded at once and then
// added by the whole wave.
__device__ __forceinline__ float fold_run(const float *__restrict__ g, int lo, int hi, float s)
{
    const int lane = threadIdx.x & 63;
    for (; lo <= hi; lo += 64) {
        const int n = min(hi - lo + 1, 64);
        const float t = lane < n ? g[lo + lane] : 0.f;
        for (int i = 0; i < n; ++i) s += __shfl(t, i);
    }
    return s;
}

// x pass: out1[z][y][xm] = sum_shots sum_{x -> xm} g_s(z, y, x).  The last task
// of a row sums its two edges.  Bound by the read of the gradient fields and the
// write of out1: 512 x 512 x 256 with a sponge of 24 takes 237 us; a thread per
// cell, the edges one load after the other, took 638 us.
__global__ __launch_bounds__(256) void k_fold_x(const Job *__restrict__ jobs, int njobs, int M,
                                                int gy, int nxm, int nseg,
                                                float *__restrict__ out1)
{
    const Job *J0 = jobs;
    const int ny = J0->ny, nx = J0->nx, nb = J0->nb, pitch = J0->pitch;
    const int64_t plane = J0->plane, rows = (int64_t)J0->nz * ny, tasks = rows * (nseg + 1);
    const int lane = threadIdx.x & 63;
    for (int64_t task = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
         task < tasks; task += (int64_t)gridDim.x * 4) {
        const int64_t row = task / (nseg + 1);
        const int seg = (int)(task - row * (nseg + 1));
        const int z = (int)(row / ny), y = (int)(row - (int64_t)z * ny);
        const int64_t base = (int64_t)(z + M) * plane + (int64_t)(y + gy) * pitch + M;
        float *o = out1 + row * nxm;
        if (seg == nseg) {
            for (int e = 0; e < (nxm > 1 ? 2 : 1); ++e) {
                const int xm = e ? nxm - 1 : 0;
                int lo, hi;
                fold_range(xm, nxm, nx, nb, lo, hi);
                float s = 0.f;
                for (int jb = 0; jb < njobs; ++jb) s = fold_run(jobs[jb].grad + base, lo, hi, s);
                if (lane == 0) o[xm] = s;
            }
        } else {
            const int c = seg * kFoldCols + lane;
            float s[kFoldCols / 64] = {};
#pragma unroll 4
            for (int jb = 0; jb < njobs; ++jb)
                fold_rows(jobs[jb].grad + base + nb, 0, 1, c, nxm, s);
#pragma unroll
            for (int q = 0; q < kFoldCols / 64; ++q) {
                const int xm = c + 64 * q;
                if (xm > 0 && xm < nxm - 1) o[xm] = s[q];
            }
        }
    }
}

// y pass (3-D): out2[z][ym][xm] = sum_{y -> ym} in[z][y][xm].  As the x pass:
// 138 us for 274.
__global__ __launch_bounds__(256) void k_fold_y(const float *__restrict__ in, int nz, int ny,
                                                int nym, int nxm, int nb, int nseg,
                                                float *__restrict__ out2)
{
    const int64_t tasks = (int64_t)nz * nym * nseg;
    for (int64_t task = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
         task < tasks; task += (int64_t)gridDim.x * 4) {
        const int64_t row = task / nseg;
        const int c = (int)(task - row * nseg) * kFoldCols + (threadIdx.x & 63);
        const int z = (int)(row / nym), ym = (int)(row - (int64_t)z * nym);
        int lo, hi;
        fold_range(ym, nym, ny, nb, lo, hi);
        float s[kFoldCols / 64] = {};
        fold_rows(in + ((int64_t)z * ny + lo) * nxm, nxm, hi - lo + 1, c, nxm, s);
#pragma unroll
        for (int q = 0; q < kFoldCols / 64; ++q)
            if (c + 64 * q < nxm) out2[row * nxm + c + 64 * q] = s[q];
    }
}

// z pass and chain rule: dv[m] = (2 / v[m]) * sum_{z -> zm} in[z][ym][xm]
// (d kappa / d v = 2 kappa / v; the kappa cancels against psi = kappa*alpha*lambda).
// As the x pass: 175 us for 234.
__global__ __launch_bounds__(256) void k_fold_z(const float *__restrict__ in,
                                                const float *__restrict__ v, int nz, int nzm,
                                                int nym, int nxm, int nb, int nseg,
                                                float *__restrict__ dv)
{
    const int64_t per = (int64_t)nym * nxm, tasks = (int64_t)nzm * nym * nseg;
    for (int64_t task = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
         task < tasks; task += (int64_t)gridDim.x * 4) {
        const int64_t row = task / nseg;
        const int c = (int)(task - row * nseg) * kFoldCols + (threadIdx.x & 63);
        const int zm = (int)(row / nym), ym = (int)(row - (int64_t)zm * nym);
        int lo, hi;
        fold_range(zm, nzm, nz, nb, lo, hi);
        float s[kFoldCols / 64] = {};
        fold_rows(in + (int64_t)lo * per + (int64_t)ym * nxm, per, hi - lo + 1, c, nxm, s);
#pragma unroll
        for (int q = 0; q < kFoldCols / 64; ++q) {
            const int64_t idx = row * nxm + c + 64 * q;
            if (c + 64 * q < nxm) dv[idx] = 2.f * s[q] / v[idx];
        }
    }
}

// Model statistics for host validation: block b of B writes the min, max and
// count of non-finite values of its part (partial[b], [B + b], [2B + b]).  Four
// loads in flight per thread and 1024 blocks within a call: 256 blocks with one
// each took 430 us over a 512 x 512 x 256 model (0.6 TB/s), now 60 us (4.5 TB/s).
__device__ __forceinline__ void block_stats(const float *__restrict__ v, int64_t n, int b, int B,
                                            float *__restrict__ partial)
{
    __shared__ float smin[256], smax[256], sbad[256];
    float lo = INFINITY, hi = -INFINITY, bad = 0.f;
    const int64_t stride = (int64_t)B * 256;
    auto take = [&](float a) __attribute__((always_inline)) {
        if (!isfinite(a)) bad += 1.f;
        else { lo = fminf(lo, a); hi = fmaxf(hi, a); }
    };
    int64_t i = (int64_t)b * 256 + threadIdx.x;
    for (; i + 3 * stride < n; i += 4 * stride) {
        const float a0 = v[i], a1 = v[i + stride], a2 = v[i + 2 * stride], a3 = v[i + 3 * stride];
        take(a0); take(a1); take(a2); take(a3);
    }
    for (; i < n; i += stride) take(v[i]);
    smin[threadIdx.x] = lo; smax[threadIdx.x] = hi; sbad[threadIdx.x] = bad;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            smin[threadIdx.x] = fminf(smin[threadIdx.x], smin[threadIdx.x + s]);
            smax[threadIdx.x] = fmaxf(smax[threadIdx.x], smax[threadIdx.x + s]);
            sbad[threadIdx.x] += sbad[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[b] = smin[0];
        partial[B + b] = smax[0];
        partial[2 * B + b] = sbad[0];
    }
}

__global__ __launch_bounds__(256) void k_vstats(const float *__restrict__ v, int64_t n,
                                                float *__restrict__ partial)
{
    block_stats(v, n, blockIdx.x, gridDim.x, partial);
}

// ------------------------------------------------------------ call staging
// A call's tables are built on the device from its position arrays: copying
// them to the host, sorting the receivers of each shot there and uploading the
// tables took 1.9 ms of a 256^3 call with 65536 receivers, 7.6 ms of a 512 x
// 512 x 256 one and 0.07 ms of a 128 x 128 one.  The host reads back one
// StageResult and checks it.

// Model statistics (as k_vstats), and the initial values of the kernels below.
__global__ __launch_bounds__(256) void k_stage_begin(StageArgs a)
{
    const int B = a.vblocks;
    if ((int)blockIdx.x >= B) {
        const int64_t n = (int64_t)(gridDim.x - B) * blockDim.x;
        const int64_t i0 = (int64_t)(blockIdx.x - B) * blockDim.x + threadIdx.x;
        if (i0 == 0) {
            a.result->bad_src = a.result->bad_rec = 0x7fffffffffffffffll;
            a.result->duplicates = 0;
            a.result->map_set = 0;
        }
        for (int64_t i = i0; i < (int64_t)a.S * a.bins; i += n) a.rt_start[i] = 0;
        for (int64_t i = i0; i < a.S; i += n) {
            a.zrange[2 * i] = a.nz;
            a.zrange[2 * i + 1] = 0;
        }
        return;
    }
    block_stats(a.v, a.ncells, blockIdx.x, B, a.partial);
}

// Bounds of every source and receiver (the first one outside the model) and
// receiver offsets (-1: outside); their map cells are set to "no receiver" here
// unless the map is an output.  Block 0 also reduces the model statistics.
__global__ __launch_bounds__(256) void k_stage_positions(StageArgs a)
{
    const int64_t n = (int64_t)a.S * a.R;
    auto inside = [&](const int32_t *q) {
        const int x = q[a.D - 1], y = a.D == 3 ? q[1] : 0;
        return q[0] >= 0 && q[0] < a.nzm && y >= 0 && y < a.nym && x >= 0 && x < a.nxm;
    };
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n + a.S;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (i >= n) {
            if (!inside(a.src_pos + (i - n) * a.D))
                atomicMin((unsigned long long *)&a.result->bad_src, (unsigned long long)(i - n));
            continue;
        }
        const int32_t *q = a.rec_pos + i * a.D;
        if (!inside(q)) {
            atomicMin((unsigned long long *)&a.result->bad_rec, (unsigned long long)i);
            a.rec_off[i] = -1;
            continue;
        }
        const int z = q[0] + a.nb, y = a.D == 3 ? q[1] + a.nb : 0, x = q[a.D - 1] + a.nb;
        const int64_t off = ((int64_t)(z + a.M) * a.nya + (y + a.gy)) * a.pitch + (x + a.M);
        a.rec_off[i] = off;
        if (!a.map_is_output) a.map[i / a.R * a.mstride + off] = 0x7fffffff;
    }
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        float lo = INFINITY, hi = -INFINITY, bad = 0.f;
        for (int i = threadIdx.x; i < a.vblocks; i += 64) {
            lo = fminf(lo, a.partial[i]);
            hi = fmaxf(hi, a.partial[a.vblocks + i]);
            bad += a.partial[2 * a.vblocks + i];
        }
        for (int o = 32; o > 0; o >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, o));
            hi = fmaxf(hi, __shfl_xor(hi, o));
            bad += __shfl_xor(bad, o);
        }
        if (threadIdx.x == 0) {
            a.result->vmin = lo;
            a.result->vmax = hi;
            a.result->bad_v = bad;
        }
    }
}

// Whether the map may be written (the host's checks in stage(), in its order).
__device__ __forceinline__ bool map_writable(const StageArgs &a)
{
    if (!a.map_is_output) return true;
    const StageResult &r = *a.result;
    return r.bad_src == 0x7fffffffffffffffll && r.bad_rec == 0x7fffffffffffffffll &&
           !(r.bad_v > 0.f) && r.vmin > 0.f && !((double)r.vmax * a.dt / a.dx > a.cfl_max);
}

// The receivers' map cells set to "no receiver", for a map that is an output: a
// refused call leaves it as it was.
__global__ __launch_bounds__(256) void k_stage_clear(StageArgs a)
{
    if (!map_writable(a)) return;
    const int64_t n = (int64_t)a.S * a.R;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.result->map_set = 1;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        a.map[i / a.R * a.mstride + a.rec_off[i]] = 0x7fffffff;
}

// The first receiver of every receiver cell.
__global__ __launch_bounds__(256) void k_stage_first(StageArgs a)
{
    if (!map_writable(a)) return;
    const int64_t n = (int64_t)a.S * a.R;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t off = a.rec_off[i], s = i / a.R;
        if (off >= 0) atomicMin(a.map + s * a.mstride + off, (int)(i - s * a.R));
    }
}

// List bin, z and key of the receiver cell at a field offset.
__device__ __forceinline__ int64_t list_bin(const StageArgs &a, int64_t off, int &z, int &key)
{
    const int64_t row = off / a.pitch;
    const int c = (int)(off - row * a.pitch), zi = (int)(row / a.nya);
    const int y = (int)(row - (int64_t)zi * a.nya) - a.gy;
    z = zi - a.M;
    key = a.D == 2 ? z << 6 | (c % kTileX)
                   : z << kKeyBits3d | (y % kTile3dRows) << 6 | (c % kTileX);
    return ((int64_t)(c / kTileX) * a.nty + (a.D == 2 ? 0 : y / kTile3dRows)) * a.nz + z;
}

// Lanes in a row with the same bin (the cells of one row come in that order
// from a surface array): the first lane of each run and the run's length, so that
// one lane adds for all: 262144 receivers on one plane took k_stage_heads 1.2 ms
// with an add each, 0.2 ms now.  The whole wave calls it; lanes without a bin
// pass -1.
__device__ __forceinline__ void bin_run(int64_t bin, int &first, int &len)
{
    const int lane = threadIdx.x & 63;
    const int64_t prev = __shfl_up((long long)bin, 1);
    const unsigned long long starts = __ballot(lane == 0 || prev != bin);
    const unsigned long long upto = starts & (~0ull >> (63 - lane));
    first = 63 - __clzll((long long)upto);
    const unsigned long long after = lane == 63 ? 0ull : starts >> (lane + 1);
    len = (after ? lane + __ffsll((long long)after) : 64) - first;
}

// Heads, and the receiver cells of each list bin.
__global__ __launch_bounds__(256) void k_stage_heads(StageArgs a)
{
    if (!map_writable(a)) return;
    const int64_t n = (int64_t)a.S * a.R;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x; i0 < n;
         i0 += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = i0 + threadIdx.x;
        int64_t bin = -1;
        int z = 0, key = 0;
        if (i < n) {
            const int64_t off = a.rec_off[i], s = i / a.R;
            const int r = (int)(i - s * a.R);
            const int first_r = off >= 0 ? a.map[s * a.mstride + off] : r;
            const bool head = off >= 0 && first_r == r;
            a.rec_head[i] = first_r;
            a.rec_next[i] = -1;
            if (off >= 0 && !head) a.result->duplicates = 1;
            if (a.bins > 0 && head) bin = s * a.bins + list_bin(a, off, z, key) + 1;
        }
        if (a.bins > 0) {
            int first, len;
            bin_run(bin, first, len);
            if (bin >= 0 && (int)(threadIdx.x & 63) == first) {
                // (a run has one z; most runs do not widen the range, and a bound
                // read too early only costs an atomic that changes nothing)
                int32_t *zr = a.zrange + 2 * (i / a.R);
                if (z < zr[0]) atomicMin(zr, z);
                if (z + 1 > zr[1]) atomicMax(zr + 1, z + 1);
                atomicAdd(a.rt_start + bin, len);
            }
        }
    }
}

// Exclusive prefix sums of a shot's bin counts (entry t + 1 becomes the
// start of bin t; k_stage_lists moves it to its end, the start of bin t + 1).
__global__ __launch_bounds__(1024) void k_stage_scan(StageArgs a)
{
    __shared__ int wsum[16];
    int32_t *st = a.rt_start + (int64_t)blockIdx.x * a.bins + 1;
    const int n = (int)a.bins - 1, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // a run of bins per thread: their sum, the sums before it, then the bins
    const int per = (n + 1023) / 1024, i0 = min((int)threadIdx.x * per, n), i1 = min(i0 + per, n);
    int c = 0;
#pragma unroll 8
    for (int i = i0; i < i1; ++i) c += st[i];
    int s = c;   // inclusive within the wave
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(s, o);
        if (lane >= o) s += t;
    }
    if (lane == 63) wsum[w] = s;
    __syncthreads();
    int before = s - c;
    for (int q = 0; q < w; ++q) before += wsum[q];
#pragma unroll 8
    for (int i = i0; i < i1; ++i) {
        const int x = st[i];
        st[i] = before;
        before += x;
    }
}

__global__ __launch_bounds__(256) void k_stage_lists(StageArgs a)
{
    const int64_t n = (int64_t)a.S * a.R;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x; i0 < n;
         i0 += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = i0 + threadIdx.x, s = i < n ? i / a.R : 0;
        int64_t bin = -1;
        int z = 0, key = 0, first, len, p = 0;
        if (i < n && a.rec_head[i] == (int)(i - s * a.R))
            bin = s * a.bins + list_bin(a, a.rec_off[i], z, key) + 1;
        bin_run(bin, first, len);
        const int lane = threadIdx.x & 63;
        // (the order within a bin does not matter: its cells are distinct)
        if (bin >= 0 && lane == first) p = atomicAdd(a.rt_start + bin, len);
        p = __shfl(p, first) + (lane - first);
        if (bin >= 0) {
            a.rt_rec[s * a.R + p] = (int)(i - s * a.R);
            a.rt_key[s * a.R + p] = key;
        }
    }
}

// The job table from shot 0's entry: each shot's fields, tables and source.
__global__ __launch_bounds__(64) void k_stage_jobs(StageArgs a, Job J, JobStrides d,
                                                   Job *__restrict__ jobs, int *__restrict__ prefix)
{
    const int s = blockIdx.x * 64 + threadIdx.x;
    if (s > a.S) return;
    prefix[s] = s * J.tile[0].ntiles;
    prefix[a.S + 1 + s] = s * J.ngather;
    prefix[2 * (a.S + 1) + s] = s * J.tile[1].ntiles;
    if (s == a.S) return;
    const int64_t r = (int64_t)s * a.R;
    J.ring += s * d.ring;
    if (J.adj) J.adj += s * d.adj;
    if (J.grad) J.grad += s * J.fstride;
    if (J.snap) J.snap += s * d.snap;
    if (J.wavelet) J.wavelet += (int64_t)s * J.nt;
    if (J.traces) J.traces += (int64_t)s * J.nt * a.R;
    if (J.res) J.res += (int64_t)s * J.nt * a.R;
    J.rec_off += r;
    J.rec_next += r;
    J.rec_head += r;
    if (a.bins > 0) {
        J.rt_start += s * a.bins;
        J.rt_rec += r;
        J.rt_key += r;
        J.rec_z0 = a.zrange[2 * s];
        J.rec_z1 = a.zrange[2 * s + 1];
    }
    const int32_t *q = a.src_pos + (int64_t)s * a.D;
    J.src_z = q[0] + a.nb;
    J.src_y = a.D == 3 ? q[1] + a.nb : 0;
    J.src_x = q[a.D - 1] + a.nb;
    jobs[s] = J;
}

// --------------------------------------------------- bandwidth ceiling probe
// A pointwise stream with the forward step's memory mix: three fields read,
// one written (out = a + b * c), each field touched once per launch.  Any
// step kernel that reads p, p_prev and kappa' and writes p_next moves at
// least these bytes, so the probe's rate bounds the step's on this chip.
typedef float vf2 __attribute__((ext_vector_type(2)));
typedef float vf4 __attribute__((ext_vector_type(4)));

template <typename V, bool NT>
__device__ __forceinline__ V ld_probe(const V *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <typename V, bool NT>
__device__ __forceinline__ void st_probe(V *p, V v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <typename V, bool NT>
__global__ __launch_bounds__(256) void k_stream3r1w(const V *__restrict__ a,
                                                    const V *__restrict__ b,
                                                    const V *__restrict__ c,
                                                    V *__restrict__ o, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * 256) {
        const V x = ld_probe<V, NT>(a + i), y = ld_probe<V, NT>(b + i), z = ld_probe<V, NT>(c + i);
        st_probe<V, NT>(o + i, x + y * z);
    }
}

template <typename V, bool NT>
static void launch_probe_t(const float *a, const float *b, const float *c, float *o, int64_t n,
                           bool persistent, hipStream_t st)
{
    constexpr int W = sizeof(V) / sizeof(float);
    const int64_t nv = n / W;
    const int64_t full = (nv + 255) / 256;
    const int grid = (int)(persistent ? std::min<int64_t>(full, 2048) : full);
    hipLaunchKernelGGL((k_stream3r1w<V, NT>), dim3(grid), dim3(256), 0, st,
                       reinterpret_cast<const V *>(a), reinterpret_cast<const V *>(b),
                       reinterpret_cast<const V *>(c), reinterpret_cast<V *>(o), nv);
}

// variant: bits 0-1 load width (0: 32-bit, 1: 64-bit, 2: 128-bit), bit 2
// non-temporal, bit 3 a grid of at most 2048 blocks striding over the fields
// (otherwise one lane per vector).  n is a multiple of 4.
void launch_stream_probe(const float *a, const float *b, const float *c, float *o, int64_t n,
                         int variant, hipStream_t st)
{
    const bool nt = (variant >> 2) & 1, pers = (variant >> 3) & 1;
    switch (variant & 3) {
    case 0:
        if (nt) launch_probe_t<float, true>(a, b, c, o, n, pers, st);
        else launch_probe_t<float, false>(a, b, c, o, n, pers, st);
        break;
    case 1:
        if (nt) launch_probe_t<vf2, true>(a, b, c, o, n, pers, st);
        else launch_probe_t<vf2, false>(a, b, c, o, n, pers, st);
        break;
    default:
        if (nt) launch_probe_t<vf4, true>(a, b, c, o, n, pers, st);
        else launch_probe_t<vf4, false>(a, b, c, o, n, pers, st);
        break;
    }
}

// ------------------------------------------------ tile-march pattern probe
// The memory pattern of an 8th-order marching step with one column per lane
// (k_step3d has four, in 16-byte accesses), with the stencil taken out:
// blocks of 4 wavefronts x 4 rows march 64 x 16 column tiles through z
// chunks in the step's block order (XCD-remapped), load cur, prv and kappa
// once per cell through buffer resources (prv and kappa non-temporal) one
// plane ahead, and write out = 2 cur + kappa prv.
// Mode bits add such a step's other traffic and synchronisation one at a
// time: 1 the halo rows and columns of cur (loaded one plane ahead),
// 2 the plane staged in LDS
// behind the LDS-only barrier (the written cur value then comes from LDS),
// 4 the 2M warm-up planes of cur each chunk reads around its own.  Halo and
// warm-up values enter only a sum scaled by `zero` (0 from the host), so
// the output stays 2 cur + kappa prv for finite inputs.
template <int MODE>
__global__ __launch_bounds__(256) void k_tile_probe(const float *cur, const float *prv,
                                                    const float *kap, float *out, int nz, int ny,
                                                    int nx, int pitch, int zc, int ntx, int nty,
                                                    int ttiles, float zero)
{
    constexpr int M = 4, TX = kTileX, RY = 4, NW = 4, TY = RY * NW, NT = 64 * NW;
    constexpr int LX = TX + 2 * M, LY = TY + 2 * M, LS = LX * LY;
    constexpr int NYH = (2 * M * TX + NT - 1) / NT, NXH = (TY * 2 * M + NT - 1) / NT;
    constexpr bool HALO = MODE & 1, LDS = MODE & 2, WARM = MODE & 4;
    __shared__ float sp[LDS ? 2 * LS : 1];
    const int tid = threadIdx.x;
    int b = xcd_remap(blockIdx.x, ttiles);
    const int tx = b % ntx;
    b /= ntx;
    const int ty = b % nty, tz = b / nty;
    const int z0 = tz * zc, z1 = min(z0 + zc, nz);
    const int64_t plane = (int64_t)(ny + 2 * M) * pitch;
    const int pbytes = (int)(plane * (int64_t)sizeof(float));
    const int lane = tid & 63, wv = tid >> 6;
    const int col = tx * TX + lane, x = col - M;
    const int last_row = ny + 2 * M - 1;
    uint32_t roff[RY], soff[RY];
    int lrow[RY];
#pragma unroll
    for (int i = 0; i < RY; ++i) {
        const int yy = ty * TY + wv * RY + i;
        roff[i] = 4u * (uint32_t)(min(yy + M, last_row) * pitch + col);
        soff[i] = x >= 0 && x < nx && yy < ny ? roff[i] : kDropOffset;
        lrow[i] = (M + wv * RY + i) * LX + M + lane;
    }
    uint32_t hyo[NYH], hxo[NXH];
    int hyl[NYH], hxl[NXH];
#pragma unroll
    for (int q = 0; q < NYH; ++q) {
        const int h = tid + NT * q;
        const int r = (h / TX) % (2 * M), c = h % TX;
        const int ly = r < M ? r : r + TY;
        const int yg = ty * TY - M + ly;
        hyo[q] = 4u * (uint32_t)(min(max(yg + M, 0), last_row) * pitch + tx * TX + c);
        hyl[q] = h < 2 * M * TX ? ly * LX + M + c : -1;
    }
#pragma unroll
    for (int q = 0; q < NXH; ++q) {
        const int h = tid + NT * q;
        const int r = (h / (2 * M)) % TY, c = h % (2 * M);
        const int lc = c < M ? c : c + TX;
        const int cm = min(max(tx * TX - M + lc, 0), pitch - 1);
        hxo[q] = 4u * (uint32_t)(min(ty * TY + r + M, last_row) * pitch + cm);
        hxl[q] = h < TY * 2 * M ? (M + r) * LX + lc : -1;
    }
    float acc = 0.f;
    if constexpr (WARM) {
        // memory planes z0 .. z0+M-1 and z1+M .. z1+2M-1: the M planes on
        // either side of the chunk that the step's z-queue reads
#pragma unroll
        for (int s = 0; s < 2 * M; ++s) {
            const int zm = s < M ? z0 + s : z1 + s;
            const rsrc_t pw = plane_rsrc(gptr(cur), zm, plane, pbytes);
#pragma unroll
            for (int i = 0; i < RY; ++i) acc += ldb(pw, roff[i]);
        }
    }
    // Three-slot rings, chunk plane j in slot j % 3: cur and its halos are
    // loaded two planes ahead, so the plane staged into LDS at the end of an
    // iteration was loaded one iteration earlier (as the step's queue front
    // and halo ring are); kappa and prv one plane ahead.
    float q[3][RY], kv[3][RY], pv[3][RY];
    float hy[3][HALO ? NYH : 1], hx[3][HALO ? NXH : 1];
    auto load_cur = [&](const int sl, const int z) __attribute__((always_inline)) {
        const rsrc_t pc = plane_rsrc(gptr(cur), z + M, plane, pbytes);
        if constexpr (HALO) {
#pragma unroll
            for (int h = 0; h < NYH; ++h) hy[sl][h] = ldb(pc, hyo[h]);
#pragma unroll
            for (int h = 0; h < NXH; ++h) hx[sl][h] = ldb(pc, hxo[h]);
        }
#pragma unroll
        for (int i = 0; i < RY; ++i) q[sl][i] = ldb(pc, roff[i]);
    };
    auto load_pw = [&](const int sl, const int z) __attribute__((always_inline)) {
        const rsrc_t pk = plane_rsrc(gptr(kap), z + M, plane, pbytes);
        const rsrc_t pp = plane_rsrc(gptr(prv), z + M, plane, pbytes);
#pragma unroll
        for (int i = 0; i < RY; ++i) {
            kv[sl][i] = ldb_stream(pk, roff[i]);
            pv[sl][i] = ldb_stream(pp, roff[i]);
        }
    };
    // plane z's cells (and halos) into LDS buffer z & 1, or its halos into
    // the sum
    auto stage = [&](const int sl, const int z) __attribute__((always_inline)) {
        if constexpr (LDS) {
            float *L = sp + (z & 1) * LS;
#pragma unroll
            for (int i = 0; i < RY; ++i) L[lrow[i]] = q[sl][i];
            if constexpr (HALO) {
#pragma unroll
                for (int h = 0; h < NYH; ++h)
                    if (hyl[h] >= 0) L[hyl[h]] = hy[sl][h];
#pragma unroll
                for (int h = 0; h < NXH; ++h)
                    if (hxl[h] >= 0) L[hxl[h]] = hx[sl][h];
            }
        } else if constexpr (HALO) {
#pragma unroll
            for (int h = 0; h < NYH; ++h) acc += hy[sl][h];
#pragma unroll
            for (int h = 0; h < NXH; ++h) acc += hx[sl][h];
        }
    };
    load_cur(0, z0);
    if (z0 + 1 < z1) load_cur(1, z0 + 1);
    load_pw(0, z0);
    stage(0, z0);
    if constexpr (LDS) lds_barrier();
    // plane z (chunk slot K): loads of z+2 (cur) and z+1 (kappa, prv), the
    // store of z, then plane z+1 staged
    auto step_plane = [&](auto K, const int z, const bool more1, const bool more2)
        __attribute__((always_inline)) {
        constexpr int c = decltype(K)::value, c1 = (c + 1) % 3, c2 = (c + 2) % 3;
        if (more2) load_cur(c2, z + 2);
        if (more1) load_pw(c1, z + 1);
        const rsrc_t po = plane_rsrc(gptr(out), z + M, plane, pbytes);
        const float extra = zero * acc;
        const float *L = sp + (z & 1) * LS;
#pragma unroll
        for (int i = 0; i < RY; ++i) {
            const float cv = LDS ? L[lrow[i]] : q[c][i];
            stb_stream(po, soff[i], fmaf(kv[c][i], pv[c][i], 2.f * cv) + extra);
        }
        if (more1) stage(c1, z + 1);
        if constexpr (LDS) lds_barrier();
    };
    int z = z0;
    for (; z + 5 <= z1; z += 3) {
        step_plane(Int<0>{}, z, true, true);
        step_plane(Int<1>{}, z + 1, true, true);
        step_plane(Int<2>{}, z + 2, true, true);
    }
    static_for<0, 4>([&](auto K) __attribute__((always_inline)) {
        const int zz = z + decltype(K)::value;
        if (zz < z1) step_plane(Int<decltype(K)::value % 3>{}, zz, zz + 1 < z1, zz + 2 < z1);
    });
}

// The bare march (with or without the halo loads) with 64-bit loads and
// stores: each lane owns two adjacent columns of two rows, so one wavefront
// instruction covers two 256-byte row segments.  Same tiles, chunks, block
// order and output as k_tile_probe; halo values enter the zero-scaled sum.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
template <bool HALO>
__global__ __launch_bounds__(256) void k_tile_probe64(const float *cur, const float *prv,
                                                      const float *kap, float *out, int nz,
                                                      int ny, int nx, int pitch, int zc, int ntx,
                                                      int nty, int ttiles, float zero)
{
    constexpr int M = 4, TX = kTileX, TY = 16;
    const int tid = threadIdx.x;
    int b = xcd_remap(blockIdx.x, ttiles);
    const int tx = b % ntx;
    b /= ntx;
    const int ty = b % nty, tz = b / nty;
    const int z0 = tz * zc, z1 = min(z0 + zc, nz);
    const int64_t plane = (int64_t)(ny + 2 * M) * pitch;
    const int pbytes = (int)(plane * (int64_t)sizeof(float));
    const int lane = tid & 63, wv = tid >> 6;
    const int col = tx * TX + 2 * (lane & 31);   // even: 8-byte aligned
    const int last_row = ny + 2 * M - 1;
    uint32_t roff[2], soff[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int yy = ty * TY + wv * 4 + (lane >> 5) + 2 * i;
        roff[i] = 4u * (uint32_t)(min(yy + M, last_row) * pitch + col);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int x = col + e - M;
            soff[i][e] = x >= 0 && x < nx && yy < ny ? roff[i] + 4u * e : kDropOffset;
        }
    }
    // halos: 8 rows of 64 columns (one pair per thread) and 16 rows of 4 + 4
    // columns (two pairs per row, threads 0..63)
    uint32_t hyo, hxo;
    {
        const int r = tid >> 5, c = 2 * (tid & 31);
        const int ly = r < M ? r : r + TY;
        hyo = 4u * (uint32_t)(min(ty * TY - M + ly + M, last_row) * pitch + tx * TX + c);
        const int xr = (tid >> 2) & 15, xp = tid & 3;
        const int xc = min(max(tx * TX - M + (xp < 2 ? 2 * xp : TX + 2 * xp), 0), pitch - 2);
        hxo = 4u * (uint32_t)(min(ty * TY + xr + M, last_row) * pitch + xc);
    }
    auto ld2 = [&](rsrc_t r, uint32_t off) __attribute__((always_inline)) {
        return __builtin_bit_cast(vf2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
    };
    auto ld2_stream = [&](rsrc_t r, uint32_t off) __attribute__((always_inline)) {
        return __builtin_bit_cast(vf2,
                                  __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, kCacheNT));
    };
    float acc = 0.f;
    vf2 q[2][2], kv[2][2], pv[2][2], hh[2][2];
    auto load = [&](const int sl, const int z) __attribute__((always_inline)) {
        const rsrc_t pc = plane_rsrc(gptr(cur), z + M, plane, pbytes);
        const rsrc_t pk = plane_rsrc(gptr(kap), z + M, plane, pbytes);
        const rsrc_t pp = plane_rsrc(gptr(prv), z + M, plane, pbytes);
        if constexpr (HALO) {
            hh[sl][0] = ld2(pc, hyo);
            hh[sl][1] = ld2(pc, hxo);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            q[sl][i] = ld2(pc, roff[i]);
            kv[sl][i] = ld2_stream(pk, roff[i]);
            pv[sl][i] = ld2_stream(pp, roff[i]);
        }
    };
    load(0, z0);
    auto step_plane = [&](auto K, const int z, const bool more) __attribute__((always_inline)) {
        constexpr int c = decltype(K)::value, cn = 1 - c;
        if (more) load(cn, z + 1);
        if constexpr (HALO) acc += hh[c][0].x + hh[c][0].y + hh[c][1].x + hh[c][1].y;
        const rsrc_t po = plane_rsrc(gptr(out), z + M, plane, pbytes);
        const float extra = zero * acc;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const vf2 o = {fmaf(kv[c][i].x, pv[c][i].x, 2.f * q[c][i].x) + extra,
                           fmaf(kv[c][i].y, pv[c][i].y, 2.f * q[c][i].y) + extra};
            if (soff[i][0] != kDropOffset && soff[i][1] != kDropOffset)
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, o), po,
                                                      (int)roff[i], 0, kCacheNT);
            else {
                stb_stream(po, soff[i][0], o.x);
                stb_stream(po, soff[i][1], o.y);
            }
        }
    };
    int z = z0;
    for (; z + 2 < z1; z += 2) {
        step_plane(Int<0>{}, z, true);
        step_plane(Int<1>{}, z + 1, true);
    }
    static_for<0, 2>([&](auto K) __attribute__((always_inline)) {
        const int zz = z + decltype(K)::value;
        if (zz < z1) step_plane(K, zz, zz + 1 < z1);
    });
}

// One launch of the tile-march probe over nz x ny x nx cells (8th-order
// frame, rows of `pitch` floats) in z chunks of zc planes.
void launch_tile_probe(const float *cur, const float *prv, const float *kap, float *out, int nz,
                       int ny, int nx, int pitch, int zc, int mode, hipStream_t st)
{
    const int ntx = (nx + 4 + kTileX - 1) / kTileX, nty = (ny + 15) / 16;
    const int nzc = (nz + zc - 1) / zc;
    const int T = ntx * nty * nzc;
    if (mode & 8) {
        if (mode & 1)
            hipLaunchKernelGGL(k_tile_probe64<true>, dim3(T), dim3(256), 0, st, cur, prv, kap,
                               out, nz, ny, nx, pitch, zc, ntx, nty, T, 0.f);
        else
            hipLaunchKernelGGL(k_tile_probe64<false>, dim3(T), dim3(256), 0, st, cur, prv, kap,
                               out, nz, ny, nx, pitch, zc, ntx, nty, T, 0.f);
        return;
    }
    switch (mode & 7) {
#define FWI_TILE_PROBE(m)                                                                     \
    case m:                                                                                   \
        hipLaunchKernelGGL(k_tile_probe<m>, dim3(T), dim3(256), 0, st, cur, prv, kap, out, nz, \
                           ny, nx, pitch, zc, ntx, nty, T, 0.f);                              \
        break;
        FWI_TILE_PROBE(0)
        FWI_TILE_PROBE(1)
        FWI_TILE_PROBE(2)
        FWI_TILE_PROBE(3)
        FWI_TILE_PROBE(4)
        FWI_TILE_PROBE(5)
        FWI_TILE_PROBE(6)
        FWI_TILE_PROBE(7)
#undef FWI_TILE_PROBE
    }
}

// Launch tables of a serving chunk (see AssembleArgs): block i copies entry
// i from the job's memory and patches its time window and level list; block
// 0 also writes the launch's slices of the prefix arrays and level lists.
__global__ __launch_bounds__(64) void k_assemble(AssembleArgs a, Job *__restrict__ table,
                                                 int *__restrict__ prefix,
                                                 int32_t *__restrict__ levels)
{
    const int i = blockIdx.x;
    if (i < a.count) {
        const uint32_t *src = reinterpret_cast<const uint32_t *>(a.src[i]);
        uint32_t *dst = reinterpret_cast<uint32_t *>(table + a.first + i);
        constexpr int words = sizeof(Job) / sizeof(uint32_t);
        for (int w = threadIdx.x; w < words; w += blockDim.x) dst[w] = src[w];
        __syncthreads();
        if (threadIdx.x == 0) {
            Job &J = table[a.first + i];
            J.n0 = a.win[i][0];
            J.k0 = a.win[i][1];
            J.fwd_lo = a.win[i][2];
            J.fwd_hi = a.win[i][3];
            J.adj_lo = a.win[i][4];
            J.adj_hi = a.win[i][5];
            J.record = a.win[i][6];
            J.lev = a.levoff[i] >= 0 ? levels + a.levoff[i] : nullptr;
        }
    }
    if (i == 0) {
        for (int p = threadIdx.x; p < a.nprefix; p += blockDim.x) prefix[a.pfirst + p] = a.prefix[p];
        for (int p = threadIdx.x; p < a.nlev; p += blockDim.x) levels[a.lfirst + p] = a.lev[p];
    }
}

// Non-finite cells of one ring field (slot) of every job:
// per-block counts, partial[0 .. gridDim.x), summed on the host.
__global__ __launch_bounds__(256) void k_nonfinite_level(const Job *__restrict__ jobs, int njobs,
                                                         int slot, float *__restrict__ partial)
{
    __shared__ float red[256];
    float bad = 0.f;
    for (int j = 0; j < njobs; ++j) {
        const Job *J = jobs + j;
        const float4 *f =
            reinterpret_cast<const float4 *>(J->ring + (int64_t)slot * J->fstride);
        const int64_t n4 = J->fstride / 4;
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
             i += (int64_t)gridDim.x * blockDim.x) {
            const float4 a = f[i];
            bad += (isfinite(a.x) ? 0.f : 1.f) + (isfinite(a.y) ? 0.f : 1.f) +
                   (isfinite(a.z) ? 0.f : 1.f) + (isfinite(a.w) ? 0.f : 1.f);
        }
    }
    red[threadIdx.x] = bad;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// ------------------------------------------------- fixed per-GPU workspace
// The workspace of fwi_forward_noalloc, for callers that cannot allocate
// device memory: one array per GPU the library runs on, held until the
// process ends.  Host code never passes the array's name to a kernel (on the
// host it is only a stand-in for the symbol): it looks up each device's own
// address once, with that device current, and passes that address.
static __device__ __align__(256) unsigned char scratch[kScratchBytes + kScratchSlack];

int scratch_address(void **ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return -1;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return -1;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return 0;
}

// ---------------------------------------------------------------- launchers
// Blocks of model statistics within a call, in fwi_velocity_range (whose
// workspace of 4096 bytes holds their partials), and of the non-finite check.
int vstats_blocks() { return 1024; }
int range_blocks() { return 256; }
int nonfinite_blocks() { return 768; }

void launch_assemble(const AssembleArgs &a, Job *table, int *prefix, int32_t *levels,
                     hipStream_t st)
{
    hipLaunchKernelGGL(k_assemble, dim3(a.count > 0 ? a.count : 1), dim3(64), 0, st, a, table,
                       prefix, levels);
}

// Everything up to the result that the host checks.
void launch_stage_check(const StageArgs &a, hipStream_t st)
{
    const int64_t n = (int64_t)a.S * a.R;
    auto blocks = [](int64_t m) { return (int)std::max<int64_t>(1, std::min<int64_t>((m + 255) / 256, 2048)); };
    hipLaunchKernelGGL(k_stage_begin, dim3(a.vblocks + blocks((int64_t)a.S * std::max<int64_t>(a.bins, 1))),
                       dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_stage_positions, dim3(blocks(n + a.S)), dim3(256), 0, st, a);
    if (n == 0) return;
    if (a.map_is_output) hipLaunchKernelGGL(k_stage_clear, dim3(blocks(n)), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_stage_first, dim3(blocks(n)), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_stage_heads, dim3(blocks(n)), dim3(256), 0, st, a);
}

void launch_stage_tables(const StageArgs &a, const Job &j0, const JobStrides &d, Job *jobs,
                         int *prefix, hipStream_t st)
{
    const int64_t n = (int64_t)a.S * a.R;
    if (a.bins > 0 && n > 0) {
        hipLaunchKernelGGL(k_stage_scan, dim3(a.S), dim3(1024), 0, st, a);
        hipLaunchKernelGGL(k_stage_lists, dim3((int)std::min<int64_t>((n + 255) / 256, 2048)),
                           dim3(256), 0, st, a);
    }
    hipLaunchKernelGGL(k_stage_jobs, dim3(a.S / 64 + 1), dim3(64), 0, st, a, j0, d, jobs, prefix);
}

void launch_nonfinite_level(const Job *jobs, int njobs, int slot, float *partial, hipStream_t st)
{
    hipLaunchKernelGGL(k_nonfinite_level, dim3(nonfinite_blocks()), dim3(256), 0, st, jobs, njobs,
                       slot, partial);
}

void launch_vstats(const float *v, int64_t n, float *partial, int blocks, hipStream_t st)
{
    hipLaunchKernelGGL(k_vstats, dim3(blocks), dim3(256), 0, st, v, n, partial);
}

// 3-D step launches, one definition per stencil radius (fwi_step3d.hip); 2-D
// ones in fwi_step2d.hip.
#define FWI_STEP3D_DECL(m)                                                                       \
    void launch_step3d_m##m(int nw, bool adj, const Job *jobs, const int *prefix, int njobs,     \
                            int step, int ttiles, int grid, int remap, const LevelMap &lm,       \
                            hipStream_t st);
FWI_STEP3D_DECL(1)
FWI_STEP3D_DECL(2)
FWI_STEP3D_DECL(4)
FWI_STEP3D_DECL(8)
#undef FWI_STEP3D_DECL
void launch_step2d(int M, int nw, bool adj, const Job *jobs, const int *prefix, int njobs,
                   int step, int ttiles, int grid, int remap, const LevelMap &lm, hipStream_t st);

void launch_step(int ndim, int M, int nw, bool adj, const Job *jobs, const int *prefix,
                 int njobs, int step, int ttiles, int gblocks, int remap, const LevelMap &lm,
                 hipStream_t st)
{
    const int grid = ttiles + (adj ? 0 : gblocks);
    if (grid <= 0) return;
    if (ndim == 2) {
        launch_step2d(M, nw, adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st);
        return;
    }
    switch (M) {
    case 1: launch_step3d_m1(nw, adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    case 2: launch_step3d_m2(nw, adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    case 4: launch_step3d_m4(nw, adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    case 8: launch_step3d_m8(nw, adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    default: break;
    }
}

static int grid_for(int64_t n, int threads, int cap)
{
    int64_t g = (n + threads - 1) / threads;
    if (g < 1) g = 1;
    return (int)(g > cap ? cap : g);
}

void launch_prep_kappa(const float *v, float *kappa, int M, int gy, int nz, int ny, int nx,
                       int pitch, int nya, int nb, int nzm, int nym, int nxm, int64_t rows,
                       float dt_dx, hipStream_t st)
{
    hipLaunchKernelGGL(k_prep_kappa, dim3(grid_for(rows * 64, 256, 16384)), dim3(256), 0, st, v,
                       kappa, M, gy, nz, ny, nx, pitch, nya, nb, nzm, nym, nxm, rows, dt_dx);
}

// Zero the frame and row padding of nf consecutive fields (fstride floats
// each: nzp planes of nya rows of pitch floats; grid cells are planes
// M .. M+nz-1, rows gy .. gy+ny-1, columns M .. M+nx-1).  One wavefront per
// row: frame rows are cleared whole, grid rows outside columns M .. M+nx-1.
__global__ __launch_bounds__(256) void k_zero_frames(float *__restrict__ f, int64_t nrows,
                                                     int64_t fstride, int nya, int pitch, int M,
                                                     int gy, int nz, int ny, int nx)
{
    const int lane = threadIdx.x & 63;
    const int64_t w0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int planes = (int)(fstride / ((int64_t)nya * pitch));
    for (int64_t r = w0; r < nrows; r += nw) {
        const int64_t fld = r / ((int64_t)planes * nya);
        const int rem = (int)(r - fld * planes * nya);
        const int z = rem / nya, y = rem - (rem / nya) * nya;
        float *row = f + fld * fstride + ((int64_t)z * nya + y) * pitch;
        const bool frame = z < M || z >= nz + M || y < gy || y >= ny + gy;
        if (frame) {
            float4 *row4 = reinterpret_cast<float4 *>(row);
            for (int c = lane; c < pitch / 4; c += 64) row4[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
            if (lane < M) row[lane] = 0.f;
            for (int c = nx + M + lane; c < pitch; c += 64) row[c] = 0.f;
        }
    }
}

void launch_zero_frames(float *p, int64_t nfields, int64_t fstride, int nya, int pitch, int M,
                        int gy, int nz, int ny, int nx, hipStream_t st)
{
    const int64_t nrows = nfields * (fstride / pitch);
    hipLaunchKernelGGL(k_zero_frames, dim3(grid_for(nrows * 64, 256, 8192)), dim3(256), 0, st, p,
                       nrows, fstride, nya, pitch, M, gy, nz, ny, nx);
}

void launch_fill(float *p, int64_t n, float val, hipStream_t st)
{
    // n is a multiple of 4 (fields are multiples of 64 floats)
    hipLaunchKernelGGL(k_fill, dim3(grid_for(n / 4, 256, 65536)), dim3(256), 0, st,
                       reinterpret_cast<float4 *>(p), n / 4, val);
}

void launch_snapshot(const Job *jobs, int njobs, int64_t fstride, int slot, int time, int dir,
                     int mask, const LevelMap &lm, hipStream_t st)
{
    hipLaunchKernelGGL(k_snapshot, dim3(grid_for(fstride / 4, 256, 4096), 2 * njobs), dim3(256),
                       0, st, jobs, slot, time, dir, mask, lm);
}
void launch_gather(const Job *jobs, const int *gprefix, int njobs, int gblocks, int threads,
                   int step, const LevelMap &lm, hipStream_t st)
{
    if (gblocks > 0)
        hipLaunchKernelGGL(k_gather, dim3(gblocks), dim3(threads), 0, st, jobs, gprefix, njobs,
                           step, lm);
}

int misfit_partials() { return 1024; }

void launch_misfit(const float *d, const float *obs, float *res, int64_t n, double *partial,
                   double *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_misfit, dim3(misfit_partials()), dim3(256), 0, st, d, obs, res, n,
                       partial);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, st, partial, misfit_partials(),
                       out);
}

void launch_fold(int ndim, const Job *jobs, int njobs, int M, int gy, int nz, int ny, int nx,
                 int nb, int nzm, int nym, int nxm, float *tmp1, float *tmp2, const float *v,
                 float *dv, hipStream_t st)
{
    (void)nx;
    const int nseg = (nxm + kFoldCols - 1) / kFoldCols;
    // a wave per task
    const int64_t n1 = (int64_t)nz * ny * (nseg + 1) * 64;
    hipLaunchKernelGGL(k_fold_x, dim3(grid_for(n1, 256, 65536)), dim3(256), 0, st, jobs, njobs,
                       M, gy, nxm, nseg, tmp1);
    const float *zin = tmp1;
    if (ndim == 3) {
        const int64_t n2 = (int64_t)nz * nym * nseg * 64;
        hipLaunchKernelGGL(k_fold_y, dim3(grid_for(n2, 256, 65536)), dim3(256), 0, st, tmp1, nz,
                           ny, nym, nxm, nb, nseg, tmp2);
        zin = tmp2;
    }
    const int64_t n3 = (int64_t)nzm * nym * nseg * 64;
    hipLaunchKernelGGL(k_fold_z, dim3(grid_for(n3, 256, 65536)), dim3(256), 0, st, zin, v, nz,
                       nzm, nym, nxm, nb, nseg, dv);
}

}  // namespace fwi
