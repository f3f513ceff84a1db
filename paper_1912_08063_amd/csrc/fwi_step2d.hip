// fwi_step2d.hip -- the 2-D step kernels (see fwi_kernels.hip for the design).
#include "fwi_device.h"

namespace fwi {

// --------------------------------------------------------------- 2-D step
// One wavefront per block: 64 columns marching down a chunk of rows with a
// (2M+1)-row register queue; the current row with its halo is staged in a
// double-buffered LDS row, and row z+1 is loaded while row z is computed.
template <int M, bool ADJ>
__global__ __launch_bounds__(64) void k_step2d(const Job *__restrict__ jobs,
                                               const int *__restrict__ prefix, int njobs,
                                               int step, int ttiles, int remap, LevelMap lm)
{
    constexpr int TX = kTileX, LX = TX + 2 * M, Q = 2 * M + 1;
    constexpr Weights<M> W{};
    constexpr int KD = kDiffRadii < M ? kDiffRadii : M;   // radii in difference form
    __shared__ float sp[2 * LX];
    __shared__ float sf[ADJ ? 2 * LX : 1];
    __shared__ float sinj[ADJ ? TX : 1];   // adjoint source of the current row

    const int lane = threadIdx.x;
    int b = blockIdx.x;
    if (b >= ttiles) {
        if constexpr (ADJ) return;
        const int gb = b - ttiles;
        const int j = find_job(prefix + njobs + 1, njobs, gb);
        const Job *J = jobs + j;
        gather_block(J, lm, (gb - prefix[njobs + 1 + j]) * blockDim.x + lane, step_level(J, step, false));
        return;
    }
    if (remap) b = xcd_remap(b, ttiles);
    const int j = find_job(prefix, njobs, b);
    const Job *__restrict__ J = jobs + j;
    const int n = step_level(J, step, ADJ);
    if (ADJ ? (n < J->adj_lo || n >= J->adj_hi) : (n < J->fwd_lo || n >= J->fwd_hi)) return;

    const int nz = J->nz, nx = J->nx, pitch = J->pitch, nb = J->nb;
    const int64_t fstride = J->fstride;
    const Job::Tiling &T = J->tile[ADJ ? 1 : 0];
    const int local = b - prefix[j];
    const int tx = local % T.ntx;
    const int tz = local / T.ntx;
    const int z0 = tz * T.zc, z1 = min(z0 + T.zc, nz);
    // adjoint: the psi update adds the adjoint source at this tile's receiver
    // cells (a list sorted by row; at most one cell per column)
    int rp = 0, re = 0;
    if constexpr (ADJ) {
        rp = J->rt_start[tx * nz + z0];
        re = J->rt_start[tx * nz + z1];
    }

    const gfloat *cur, *prv;
    gfloat *out;
    const gfloat *fwd = nullptr;
    gfloat *grad = nullptr;
    bool accum = false;
    if constexpr (ADJ) {
        cur = gptr(J->adj) + (int64_t)((n + 1) & 1) * fstride;
        prv = gptr(J->adj) + (int64_t)(n & 1) * fstride;
        out = gptr(J->adj) + (int64_t)(n & 1) * fstride;
        accum = J->accumulate && n <= J->nt - 1;
        fwd = gptr(level_ptr(J, lm, n));
        grad = gptr(J->grad);
    } else {
        cur = gptr(level_ptr(J, lm, n));
        prv = gptr(level_ptr(J, lm, n - 1));
        out = gptr(level_ptr(J, lm, n + 1));
    }
    const gfloat *kap = gptr(J->kappa);
    const float eta_dt = J->eta_dt;

    const int col = tx * TX + lane;
    const int x = col - M;
    const bool act = x >= 0 && x < nx;
    const int dxs = sponge_depth(x, nx, nb);
    // halo lanes: lane < 2M loads column tx*TX - M + (lane < M ? lane : lane + TX)
    const int hl = lane < M ? lane : lane + TX;
    const int hcol = tx * TX - M + hl;
    const bool hact = lane < 2 * M && hcol >= 0 && hcol < pitch;
    const int hcl = min(max(hcol, 0), pitch - 1);   // a column inside the row
    const bool src_here = !ADJ && J->src_x == x && J->src_z >= z0 && J->src_z < z1;
    const float srcv = src_here ? J->src_scale * J->wavelet[n] : 0.f;
    const int64_t p64 = pitch;

    // Register queue of U = Q + 1 rows: chunk row j (row z0 + j, j = -M ..)
    // in slot (j + M) % U; the front row is loaded straight into the free
    // slot and kappa', the previous level (and g) alternate between two
    // slots, so no freshly loaded register is copied and the wave keeps the
    // next row's loads in flight while it computes (as in the 3-D kernel).
    // Lanes outside the grid load and store zeros in the row's frame and
    // padding, which hold zeros, so stores need no mask.
    constexpr int U = Q + 1;
    float q[U];
    float f[ADJ ? U : 1];
#pragma unroll
    for (int s = 0; s < Q; ++s) {   // rows z0 - M .. z0 + M
        q[s] = act ? cur[(int64_t)(z0 + s) * p64 + col] : 0.f;
        if constexpr (ADJ) f[s] = act ? fwd[(int64_t)(z0 + s) * p64 + col] : 0.f;
    }
    float kv[2], pv[2], gv[2];
    kv[0] = act ? kap[(int64_t)(z0 + M) * p64 + col] : 0.f;
    pv[0] = act ? prv[(int64_t)(z0 + M) * p64 + col] : 0.f;
    gv[0] = 0.f;
    if constexpr (ADJ) gv[0] = act && accum ? grad[(int64_t)(z0 + M) * p64 + col] : 0.f;
    {
        float *L = sp + (z0 & 1) * LX;
        L[M + lane] = q[M];
        if (lane < 2 * M) L[hl] = hact ? cur[(int64_t)(z0 + M) * p64 + hcol] : 0.f;
        if constexpr (ADJ) {
            float *LF = sf + (z0 & 1) * LX;
            LF[M + lane] = f[M];
            if (lane < 2 * M) LF[hl] = hact ? fwd[(int64_t)(z0 + M) * p64 + hcol] : 0.f;
        }
    }
    lds_barrier();

    // row z = z0 + ii; k = ii % U selects the slots
    auto step_row = [&](auto K, const int z, const bool more) __attribute__((always_inline)) {
            constexpr int k = decltype(K)::value;
            const int c = k & 1, cn = c ^ 1;   // pointwise slots of rows z, z+1
            const int fs = (k + U - 1) % U;    // free queue slot: row z+M+1
            // halos of row z+1 (staged at the end of this row) first.  The
            // loads are not predicated (a skipped load would make the wait
            // counts after it inexact): lanes outside the grid read the zero
            // frame and padding of their row, halo lanes a clamped column.
            float nh = 0.f, nfh = 0.f;
            if (more) {
                const int64_t rf = (int64_t)(z + 1 + 2 * M) * p64, rc = (int64_t)(z + 1 + M) * p64;
                const float h = cur[rc + hcl];
                nh = hact ? h : 0.f;
                if constexpr (ADJ) {
                    const float hf = fwd[rc + hcl];
                    nfh = hact ? hf : 0.f;
                }
                q[fs] = cur[rf + col];
                kv[cn] = kap[rc + col];
                pv[cn] = prv[rc + col];
                if constexpr (ADJ) {
                    f[fs] = fwd[rf + col];
                    const float g = grad[rc + col];
                    gv[cn] = accum ? g : 0.f;
                }
            }
            const float *L = sp + (z & 1) * LX;
            const int lx = M + lane;
            const float pc = q[(k + M) % U];
            float acc = 0.f;
#pragma unroll
            for (int m = M; m > KD; --m) {
                const float t = (L[lx + m] + L[lx - m]) + (q[(k + M + m) % U] + q[(k + M - m) % U]);
                acc = fmaf(W.c[m], t, acc);
            }
            if constexpr (KD < M) acc = fmaf(W.t2[KD], pc, acc);
#pragma unroll
            for (int m = KD; m >= 1; --m) {
                const float d = ((L[lx + m] - pc) + (L[lx - m] - pc)) +
                                ((q[(k + M + m) % U] - pc) + (q[(k + M - m) % U] - pc));
                acc = fmaf(W.c[m], d, acc);
            }
            float val = fmaf(kv[c], acc, 2.f * pc);
            if (src_here && z == J->src_z) val += srcv;
            const int dz = sponge_depth(z, nz, nb);
            const int64_t rz = (int64_t)(z + M) * p64 + col;
            float o = leapfrog(val, pv[c], dxs * dxs + dz * dz, eta_dt);
            if constexpr (ADJ) {
                // receivers on row z: lane i takes the list's i-th, and the sum
                // reaches the lane of its column through LDS
                if (rp < re && (J->rt_key[rp] >> 6) == z) {
                    const int idx = rp + lane;
                    const int key = idx < re ? J->rt_key[idx] : -1;
                    const int r = key >= 0 && (key >> 6) == z ? J->rt_rec[idx] : -1;
                    sinj[lane] = 0.f;
                    lds_barrier();
                    if (r >= 0) sinj[key & 63] = adj_source(J, n, r);
                    lds_barrier();
                    if (act) o += kv[c] * sinj[lane];
                    rp += __popcll(__ballot(r >= 0));
                    lds_barrier();
                }
            }
            out[rz] = o;   // zero outside the grid
            if constexpr (ADJ) {
                if (accum) {
                    const float *LF = sf + (z & 1) * LX;
                    const float fc = f[(k + M) % U];
                    float lf = 0.f;
#pragma unroll
                    for (int m = M; m > KD; --m) {
                        const float t = (LF[lx + m] + LF[lx - m]) + (f[(k + M + m) % U] + f[(k + M - m) % U]);
                        lf = fmaf(W.c[m], t, lf);
                    }
                    if constexpr (KD < M) lf = fmaf(W.t2[KD], fc, lf);
#pragma unroll
                    for (int m = KD; m >= 1; --m) {
                        const float d = ((LF[lx + m] - fc) + (LF[lx - m] - fc)) +
                                        ((f[(k + M + m) % U] - fc) + (f[(k + M - m) % U] - fc));
                        lf = fmaf(W.c[m], d, lf);
                    }
                    grad[rz] = fmaf(pc, lf, gv[c]);   // zero outside the grid
                }
            }
            if (more) {
                float *Ln = sp + ((z + 1) & 1) * LX;
                Ln[M + lane] = q[(k + M + 1) % U];
                if (lane < 2 * M) Ln[hl] = nh;
                if constexpr (ADJ) {
                    float *LFn = sf + ((z + 1) & 1) * LX;
                    LFn[M + lane] = f[(k + M + 1) % U];
                    if (lane < 2 * M) LFn[hl] = nfh;
                }
            }
            lds_barrier();
    };
    int zb = z0;
    for (; zb + U < z1; zb += U)
        static_for<0, U>([&](auto K) __attribute__((always_inline)) {
            step_row(K, zb + decltype(K)::value, true);
        });
    static_for<0, U>([&](auto K) __attribute__((always_inline)) {
        const int z = zb + decltype(K)::value;
        if (z < z1) step_row(K, z, z + 1 < z1);
    });
}

// 2-D step for grids too small to fill the GPU: one block per tile row of 64
// columns and one cell per lane, every neighbour loaded straight from memory
// (the fields are cache-resident at these sizes).  Nothing is marched, so a
// launch costs one round of load latency instead of the 2M + 1 row warm-up
// and serial row loop of k_step2d.  The arithmetic is k_step2d's, term by term
// in the same order, so both kernels give bitwise the same fields.  Tiles are
// one row tall (Tiling.zc == 1); the adjoint takes this row's receiver cells
// from the tile's list, as k_step2d does row by row.
template <int M, bool ADJ>
__global__ __launch_bounds__(64) void k_step2d_direct(const Job *__restrict__ jobs,
                                                      const int *__restrict__ prefix, int njobs,
                                                      int step, int ttiles, int remap,
                                                      LevelMap lm)
{
    constexpr int TX = kTileX;
    constexpr Weights<M> W{};
    constexpr int KD = kDiffRadii < M ? kDiffRadii : M;   // radii in difference form
    __shared__ float sinj[ADJ ? TX : 1];   // adjoint source of this row

    const int lane = threadIdx.x;
    int b = blockIdx.x;
    if (b >= ttiles) {
        if constexpr (ADJ) return;
        const int gb = b - ttiles;
        const int j = find_job(prefix + njobs + 1, njobs, gb);
        const Job *J = jobs + j;
        gather_block(J, lm, (gb - prefix[njobs + 1 + j]) * blockDim.x + lane, step_level(J, step, false));
        return;
    }
    if (remap) b = xcd_remap(b, ttiles);
    const int j = find_job(prefix, njobs, b);
    const Job *__restrict__ J = jobs + j;
    const int n = step_level(J, step, ADJ);
    if (ADJ ? (n < J->adj_lo || n >= J->adj_hi) : (n < J->fwd_lo || n >= J->fwd_hi)) return;

    const int nz = J->nz, nx = J->nx, pitch = J->pitch, nb = J->nb;
    const int64_t fstride = J->fstride;
    const Job::Tiling &T = J->tile[ADJ ? 1 : 0];
    const int local = b - prefix[j];
    const int tx = local % T.ntx;
    const int z = local / T.ntx;   // one row per tile
    if (z >= nz) return;

    const gfloat *cur, *prv;
    gfloat *out;
    const gfloat *fwd = nullptr;
    gfloat *grad = nullptr;
    bool accum = false;
    if constexpr (ADJ) {
        cur = gptr(J->adj) + (int64_t)((n + 1) & 1) * fstride;
        prv = gptr(J->adj) + (int64_t)(n & 1) * fstride;
        out = gptr(J->adj) + (int64_t)(n & 1) * fstride;
        accum = J->accumulate && n <= J->nt - 1;
        fwd = gptr(level_ptr(J, lm, n));
        grad = gptr(J->grad);
    } else {
        cur = gptr(level_ptr(J, lm, n));
        prv = gptr(level_ptr(J, lm, n - 1));
        out = gptr(level_ptr(J, lm, n + 1));
    }
    const gfloat *kap = gptr(J->kappa);
    const float eta_dt = J->eta_dt;

    const int col = tx * TX + lane;
    const int x = col - M;
    const bool act = x >= 0 && x < nx;
    // every neighbour of an active cell lies inside the frame (zeros beyond the
    // padded grid), where k_step2d reads the same values from LDS and its queue
    const int64_t p64 = pitch, rz = (int64_t)(z + M) * p64 + col;
    float o = 0.f, pc = 0.f, kv = 0.f, gv = 0.f, lf = 0.f;
    if (act) {
        pc = cur[rz];
        kv = kap[rz];
        const float pv = prv[rz];
        float acc = 0.f;
#pragma unroll
        for (int m = M; m > KD; --m) {
            const float t = (cur[rz + m] + cur[rz - m]) + (cur[rz + m * p64] + cur[rz - m * p64]);
            acc = fmaf(W.c[m], t, acc);
        }
        if constexpr (KD < M) acc = fmaf(W.t2[KD], pc, acc);
#pragma unroll
        for (int m = KD; m >= 1; --m) {
            const float d = ((cur[rz + m] - pc) + (cur[rz - m] - pc)) +
                            ((cur[rz + m * p64] - pc) + (cur[rz - m * p64] - pc));
            acc = fmaf(W.c[m], d, acc);
        }
        float val = fmaf(kv, acc, 2.f * pc);
        // the source term rounded as in k_step2d: its product first, then the
        // sum (never fused into one fma)
        if (!ADJ && J->src_x == x && J->src_z == z) {
#pragma clang fp contract(off)
            const float srcv = J->src_scale * J->wavelet[n];
            val = val + srcv;
        }
        const int dxs = sponge_depth(x, nx, nb), dz = sponge_depth(z, nz, nb);
        o = leapfrog(val, pv, dxs * dxs + dz * dz, eta_dt);
        if constexpr (ADJ) {
            if (accum) {
                gv = grad[rz];
                const float fc = fwd[rz];
#pragma unroll
                for (int m = M; m > KD; --m) {
                    const float t = (fwd[rz + m] + fwd[rz - m]) + (fwd[rz + m * p64] + fwd[rz - m * p64]);
                    lf = fmaf(W.c[m], t, lf);
                }
                if constexpr (KD < M) lf = fmaf(W.t2[KD], fc, lf);
#pragma unroll
                for (int m = KD; m >= 1; --m) {
                    const float d = ((fwd[rz + m] - fc) + (fwd[rz - m] - fc)) +
                                    ((fwd[rz + m * p64] - fc) + (fwd[rz - m * p64] - fc));
                    lf = fmaf(W.c[m], d, lf);
                }
            }
        }
    }
    if constexpr (ADJ) {
        // receivers on this row: lane i takes the list's i-th, and the sum
        // reaches the lane of its column through LDS (block-uniform branch)
        const int rp = J->rt_start[tx * nz + z], re = J->rt_start[tx * nz + z + 1];
        if (rp < re) {
            const int idx = rp + lane;
            const int key = idx < re ? J->rt_key[idx] : -1;
            const int r = key >= 0 ? J->rt_rec[idx] : -1;
            sinj[lane] = 0.f;
            __syncthreads();
            if (r >= 0) sinj[key & 63] = adj_source(J, n, r);
            __syncthreads();
            o += kv * sinj[lane];
        }
    }
    if (act) {
        out[rz] = o;
        if constexpr (ADJ) {
            if (accum) grad[rz] = fmaf(pc, lf, gv);
        }
    }
}
// Several time steps of a 2-D grid in one launch (temporal blocking).  A block
// loads a region of W x H memory cells -- the propagated field's two newest
// levels and kappa' -- and advances it kk steps on the chip, each step on a
// region M cells narrower (the apron of A cells around a tile is computed
// redundantly by the neighbouring blocks), and stores the tile's levels.  Per
// thread: a patch of 4 columns x PZ rows, whose kappa', previous level (and
// gradient) stay in registers; the current level is in LDS, double-buffered,
// so each neighbour is read as a 16-byte vector and a step costs one barrier.
//
// What a launch moves per step and cell falls from 16 B (28 B in the adjoint)
// to (8 + 4 + 8) / kk B of the fields, plus 4 B per level that is stored, so a
// large batch of shots is bound by the arithmetic (24 vector instructions per
// cell and step) instead of HBM, and a single small shot pays the launch and
// the load latency once per kk steps.
//
// Forward: levels n+1 .. n+kk of the tile go to their ring slots (store_all,
// a level store that keeps every level) or only the two newest ones do; traces
// of levels n+1 .. n+kk are written by the block whose tile holds the receiver.
// Adjoint (level k = k0 .. k0-kk+1): psi^{k+1}, psi^{k+2} are read from one
// pair of adjoint fields and the two newest levels written to the other; the
// imaging condition reads p^k (staged through LDS, prefetched one level ahead)
// and keeps g in registers over the launch; the adjoint source is added to
// every receiver cell of the region.  Inputs and outputs are distinct fields:
// no block reads what another writes.
//
// Tiles: column tile i covers memory columns from i * (W - 2A), and the first
// and last tiles have no apron beyond the grid (the frame is zero there).
// Every cell's arithmetic is k_step2d_direct's, term by term, so fields,
// traces and gradients are bitwise those of single steps.
typedef float vf4 __attribute__((ext_vector_type(4)));
typedef unsigned vu4 __attribute__((ext_vector_type(4)));
typedef float vf2 __attribute__((ext_vector_type(2)));
typedef unsigned vu2 __attribute__((ext_vector_type(2)));
struct TbTile {   // output columns (rows) of tile t, relative to its region
    int origin, lo, hi;
};
__device__ __forceinline__ TbTile tb_tile(int t, int nt, int W, int A, int first, int cells)
{
    // first, cells: memory columns (rows) before the grid and up to its end
    TbTile r;
    r.origin = t * (W - 2 * A);
    r.lo = t == 0 ? first : A;
    r.hi = t == nt - 1 ? min(W, cells - r.origin) : W - A;
    return r;
}

// Flags of a multi-step launch: bits 0-1 the pair of fields to read, plus one.
// The launch's integers are separate scalar arguments, few enough to be
// preloaded into registers.
constexpr int kTbRemap = 4, kTbRecord = 8, kTbStoreAll = 16;

// Division of b by d with m = tb_magic(d) from the host (0: divide).
__device__ __forceinline__ int tb_div(int b, int d, uint32_t m)
{
    return m ? (int)__umulhi((uint32_t)b, m) : b / d;
}

template <int M, int W, int H, int PZ, bool ADJ>
__global__ __launch_bounds__((W / 4) * (H / PZ)) void k_step2d_tb(
    const Job *__restrict__ jobs, int njobs, int tiles_per_job, uint32_t magic_job,
    uint32_t magic_tx, int ntx, int ntz, int step, int steps_apron, int flags)
{
    constexpr int NT = (W / 4) * (H / PZ), NR = W * H;
    constexpr int XP = (M + 3) / 4 * 4;                // columns read beside a patch
    constexpr int GUARD = XP + (M % PZ ? (M + PZ) * W : 0);   // never used, only read
    constexpr int NCT = (W + 60 + kTileX - 1) / kTileX;   // receiver-list columns of a region
    constexpr Weights<M> WT{};
    constexpr int KD = kDiffRadii < M ? kDiffRadii : M;
    constexpr int NB = NR + 2 * GUARD;
    __shared__ __align__(16) float sbuf[2 * NB];
    __shared__ __align__(16) float spf[ADJ ? 2 * NB : 4];

    const int tid = threadIdx.x;
    int b = blockIdx.x;
    if (flags & kTbRemap) b = xcd_remap(b, gridDim.x);
    // (every job has the same grid and level)
    const int kk = steps_apron & 0xffff, A = steps_apron >> 16, pair = (flags & 3) - 1;
    const int j = njobs > 1 ? tb_div(b, tiles_per_job, magic_job) : 0;
    const int local = b - j * tiles_per_job, n = step;
    const Job *__restrict__ J = jobs + j;
    const int tz = ntx > 1 ? tb_div(local, ntx, magic_tx) : local, tx = local - tz * ntx;
    const int nz = J->nz, nx = J->nx, pitch = J->pitch, nb = J->nb, nrec = J->nrec;
    const int64_t fstride = J->fstride;
    float *const ring = J->ring, *const adj = J->adj, *const grad = J->grad;
    const float *const kappa = J->kappa;
    const int R = J->R, nt = J->nt;
    // (output columns and rows in whole patches)
    const TbTile X = tb_tile(tx, ntx, W, A, M / 4 * 4, nx + M);
    const TbTile Z = tb_tile(tz, ntz, H, A, M / PZ * PZ, nz + M);

    // this thread's patch: region column lx .. lx+3, rows lz .. lz+PZ-1; memory
    // offsets are from the region's first row, and an offset past the field
    // (rows beyond it, columns beyond the pitch) reads zero and drops stores
    const int lx = 4 * (tid % (W / 4)), lz = PZ * (tid / (W / 4));
    const int c0 = X.origin + lx, r0 = Z.origin + lz;   // memory column, row
    const int64_t row0 = (int64_t)Z.origin * pitch;
    const int rbytes = 4 * min(nz + 2 * M - Z.origin, H) * pitch;
    const uint32_t pb = 4u * (uint32_t)pitch;
    const uint32_t off = c0 < pitch ? 4u * (uint32_t)(lz * pitch + c0) : kDropOffset;
    // output cells: whole patches (one that crosses the grid's end stores zeros
    // into the frame or the row's padding)
    const bool outp = lx >= X.lo && lx < X.hi && lz >= Z.lo && lz < Z.hi;
    const uint32_t soff = outp ? off : kDropOffset;
    auto region = [&](const float *f) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(f + row0), 0, rbytes,
                                                 kRsrcWord3);
    };
    auto load_patch = [&](const float *f, vf4 (&p)[PZ]) __attribute__((always_inline)) {
        const rsrc_t r = region(f);
#pragma unroll
        for (int i = 0; i < PZ; ++i)
            p[i] = __builtin_bit_cast(
                vf4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(off + i * pb), 0, 0));
    };
    auto store_row = [&](const rsrc_t r, int i, vf4 v) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(vu4, v), r,
                                               (int)(soff + i * pb), 0, 0);
    };
    auto store_patch = [&](float *f, const vf4 (&p)[PZ]) __attribute__((always_inline)) {
        const rsrc_t r = region(f);
#pragma unroll
        for (int i = 0; i < PZ; ++i) store_row(r, i, p[i]);
    };
    // forward level L: in the ring, or (pair q >= 0) in the q-th pair of fields
    auto fwd_level = [&](int L, int q) {
        return ring + (int64_t)(q < 0 ? mod_pos(L, R) : 2 * q + (L & 1)) * fstride;
    };
    const float *cur, *prv;
    if constexpr (ADJ) {
        const float *p = adj + (int64_t)(2 * pair) * fstride;
        cur = p + (int64_t)((n + 1) & 1) * fstride;
        prv = p + (int64_t)(n & 1) * fstride;
    } else {
        cur = fwd_level(n, pair);
        prv = fwd_level(n - 1, pair);
    }
    vf4 cv[PZ], pv[PZ], kv[PZ], gv[ADJ ? PZ : 1], fv[ADJ ? PZ : 1] = {};
    load_patch(cur, cv);
    // imaging: patches of the output tile and the forward level around it
    bool img = false, fin = false;
    if constexpr (ADJ) {
        const bool accum = J->accumulate != 0;
        img = accum && outp;
        fin = accum && lx + 4 > X.lo - XP && lx < X.hi + XP && lz + PZ > Z.lo - M && lz < Z.hi + M;
        if (fin && n <= nt - 1) load_patch(fwd_level(n, -1), fv);
    }
    load_patch(prv, pv);
    load_patch(kappa, kv);
    if constexpr (ADJ) {
        if (img) load_patch(grad, gv);
    }

    // receivers of the region: rows z of column tile t are entries
    // rt_start[t nz + z] ..
    const int ez0 = max((ADJ ? 0 : Z.lo) + Z.origin - M, J->rec_z0);
    const int ez1 = min((ADJ ? H : Z.hi) + Z.origin - M, J->rec_z1);
    const bool rec_on = (ADJ || ((flags & kTbRecord) && J->record)) && ez0 < ez1;
    const int tc0 = X.origin / kTileX;
    const GMEM int32_t *rt_start = (const GMEM int32_t *)J->rt_start;
    const GMEM int32_t *rt_key = (const GMEM int32_t *)J->rt_key;
    const GMEM int32_t *rt_rec = (const GMEM int32_t *)J->rt_rec;
    int ebound = 0;   // lane 2t, 2t+1 of each wave: bounds of column tile t
    if (rec_on) {
        const int t = (tid & 63) >> 1;
        if (t < NCT && (tc0 + t) * kTileX < nx + M)
            ebound = rt_start[(tc0 + t) * nz + (tid & 1 ? ez1 : ez0)];
    }
    // wave-uniform: the wave holds sponge or frame cells
    const float eta_dt = J->eta_dt;
    auto inside = [&](int x, int z) { return x >= 0 && x < nx && z >= 0 && z < nz; };
    const bool wedge = __any(min(c0 - M, r0 - M) < nb || c0 + 3 - M >= nx - nb ||
                             r0 + PZ - 1 - M >= nz - nb);
    const bool wframe = __any(min(c0, r0) < M || c0 + 3 - M >= nx || r0 + PZ - 1 - M >= nz);
    // source (forward): its cell within this patch
    const int sx = J->src_x + M - X.origin - lx, sz = J->src_z + M - Z.origin - lz;
    const bool src_here = !ADJ && J->src_x >= 0 && sx >= 0 && sx < 4 && sz >= 0 && sz < PZ;
    const bool wsrc = __any(src_here);
    const gfloat *wavelet = gptr(J->wavelet);
    const float src_scale = J->src_scale;

    float *buf = sbuf + GUARD;
    float *pf = spf + GUARD;
    auto lds_store = [&](float *L, const vf4 (&p)[PZ]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PZ; ++i)
            *reinterpret_cast<vf4 *>(L + (lz + i) * W + lx) = p[i];
    };
    // Sponge factors of the patch (leapfrog's, in waves that hold sponge or
    // frame: out = sa * (val - sb * prev), sa = sb = 1 inside the model, where
    // that is val - prev bit for bit; 0 outside the grid).  Out-of-grid cells
    // are zero at every level: patches that hold some fill both buffers (rows of
    // the frame are not recomputed).
    vf4 sa[PZ], sb[PZ];
    if (wedge) {
#pragma unroll
        for (int i = 0; i < PZ; ++i) {
            const int z = r0 + i - M, dz = sponge_depth(z, nz, nb);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int x = c0 + c - M, dx = sponge_depth(x, nx, nb);
                const int d2 = dx * dx + dz * dz;
                // (d2 = 0: rcp(1) = 1)
                sa[i][c] = __builtin_amdgcn_rcpf(fmaf(eta_dt, (float)d2, 1.f));
                sb[i][c] = fmaf(-eta_dt, (float)d2, 1.f);
                if (!inside(x, z)) {
                    cv[i][c] = pv[i][c] = kv[i][c] = 0.f;
                    sa[i][c] = 0.f;
                }
            }
        }
        if (wframe) lds_store(buf + NB, cv);
    }
    lds_store(buf, cv);
    if constexpr (ADJ) {
        if (fin) lds_store(pf, fv);
    }
    lds_barrier();

    // Thread e holds the e-th receiver entry of the region; entries past NT are
    // walked again when they are needed.  Their loads stay in flight over the
    // first step.
    int elo[NCT] = {}, eend[NCT] = {}, etot = 0;
    if (rec_on) {
#pragma unroll
        for (int t = 0; t < NCT; ++t) {
            elo[t] = __builtin_amdgcn_readlane(ebound, 2 * t);
            etot += __builtin_amdgcn_readlane(ebound, 2 * t + 1) - elo[t];
            eend[t] = etot;
        }
    }
    // entry e: its region cell (-1: outside the region or tile) and receiver
    auto entry = [&](int e, int &cell, int &r) __attribute__((always_inline)) {
        int t = 0, idx = elo[0] + e;
#pragma unroll
        for (int q = 1; q < NCT; ++q)
            if (e >= eend[q - 1]) { t = q; idx = elo[q] + (e - eend[q - 1]); }
        const int key = rt_key[idx];
        r = rt_rec[idx];
        const int x = (tc0 + t) * kTileX + (key & 63) - X.origin, z = (key >> 6) + M - Z.origin;
        const bool in = ADJ ? x >= 0 && x < W : x >= X.lo && x < X.hi;
        cell = in ? z * W + x : -1;
    };
    const gfloat *kap = gptr(kappa) + row0 + X.origin;
    // adjoint source of a receiver cell at level k (as adj_source)
    const gfloat *res = gptr(J->res);
    const GMEM int32_t *rec_next = (const GMEM int32_t *)J->rec_next;
    auto source = [&](int k, int r, int next) __attribute__((always_inline)) {
        const gfloat *q = res + (int64_t)(k - 1) * nrec;
        float s = q[r];
        for (int o = next; o >= 0; o = rec_next[o]) s += q[o];
        return s;
    };
    int ecell = -1, er = 0, enext = -1;
    float ekap = 0.f, esrc = 0.f;
    if (tid < etot) {
        entry(tid, ecell, er);
        if constexpr (ADJ) {
            enext = rec_next[er];
            if (ecell >= 0) {
                ekap = kap[(ecell / W) * pitch + ecell % W];
                esrc = source(n, er, enext);
            }
        }
    }

    // The stencil sum of the patch's row i, column c: w holds the patch's
    // columns (rows lz-M .. lz+PZ-1+M), xr the row's columns lx-XP .. lx+3+XP.
    auto star = [&](const vf4 (&w)[PZ + 2 * M], const float (&xr)[4 + 2 * XP], int i, int c)
        __attribute__((always_inline)) {
        const float pc = w[i + M][c];
        float acc = 0.f;
#pragma unroll
        for (int m = M; m > KD; --m) {
            const float t = (xr[XP + c + m] + xr[XP + c - m]) + (w[i + M + m][c] + w[i + M - m][c]);
            acc = fmaf(WT.c[m], t, acc);
        }
        if constexpr (KD < M) acc = fmaf(WT.t2[KD], pc, acc);
#pragma unroll
        for (int m = KD; m >= 1; --m) {
            const float d = ((xr[XP + c + m] - pc) + (xr[XP + c - m] - pc)) +
                            ((w[i + M + m][c] - pc) + (w[i + M - m][c] - pc));
            acc = fmaf(WT.c[m], d, acc);
        }
        return acc;
    };
    auto window = [&](const float *L, vf4 (&w)[PZ + 2 * M]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < PZ + 2 * M; ++r)
            w[r] = *reinterpret_cast<const vf4 *>(L + (lz + r - M) * W + lx);
    };
    auto row_of = [&](const float *L, const vf4 (&w)[PZ + 2 * M], int i, float (&xr)[4 + 2 * XP])
        __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < XP; q += 4) {
            const vf4 a = *reinterpret_cast<const vf4 *>(L + (lz + i) * W + lx - XP + q);
            const vf4 d = *reinterpret_cast<const vf4 *>(L + (lz + i) * W + lx + 4 + q);
#pragma unroll
            for (int c = 0; c < 4; ++c) { xr[q + c] = a[c]; xr[XP + 4 + q + c] = d[c]; }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) xr[XP + c] = w[i + M][c];
    };

    for (int st = 0; st < kk; ++st) {
        const int L = ADJ ? n - st : n + st;   // the level this step updates from (to, adjoint)
        const float *Lc = buf + (st & 1) * NB;
        float *Ln = buf + ((st & 1) ^ 1) * NB;
        // rows this step still computes
        const int lo = tz == 0 ? M : (st + 1) * M;
        const int hi = tz == ntz - 1 ? nz + M - Z.origin : H - (st + 1) * M;
        vf4 nf[ADJ ? PZ : 1];
        bool nextf = false;
        if constexpr (ADJ) {
            nextf = fin && st + 1 < kk;
            if (nextf) load_patch(fwd_level(L - 1, -1), nf);
        }
        if (lz + PZ > lo && lz < hi) {
            vf4 w[PZ + 2 * M];
            window(Lc, w);
            rsrc_t ro;
            if constexpr (!ADJ) ro = region(fwd_level(L + 1, -1));
#pragma unroll
            for (int i = 0; i < PZ; ++i) {
                float xr[4 + 2 * XP];
                row_of(Lc, w, i, xr);
                vf4 o;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    o[c] = fmaf(kv[i][c], star(w, xr, i, c), 2.f * w[i + M][c]);
                if (wsrc) {
#pragma clang fp contract(off)
                    const float srcv = src_here && sz == i ? src_scale * wavelet[L] : 0.f;
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (src_here && sz == i && sx == c) o[c] = o[c] + srcv;
                }
                if (wedge) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        o[c] = sa[i][c] * fmaf(-sb[i][c], pv[i][c], o[c]);
                        if (wframe) o[c] = sa[i][c] != 0.f ? o[c] : 0.f;
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) o[c] = o[c] - pv[i][c];
                }
                pv[i] = w[i + M];
                *reinterpret_cast<vf4 *>(Ln + (lz + i) * W + lx) = o;
                if constexpr (!ADJ) {
                    if (flags & kTbStoreAll) store_row(ro, i, o);
                }
            }
        }
        if constexpr (ADJ) {
            if (img && L <= nt - 1) {
                const float *Lf = pf + (st & 1) * NB;
                vf4 w[PZ + 2 * M];
                window(Lf, w);
#pragma unroll
                for (int i = 0; i < PZ; ++i) {
                    float xr[4 + 2 * XP];
                    row_of(Lf, w, i, xr);
                    // pv: the patch's psi^{L+1}, which this step read
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        gv[i][c] = fmaf(pv[i][c], star(w, xr, i, c), gv[i][c]);
                    if (wframe) {   // frame cells read past the region
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (!inside(c0 + c - M, r0 + i - M)) gv[i][c] = 0.f;
                    }
                }
            }
            if (nextf) lds_store(pf + ((st & 1) ^ 1) * NB, nf);
        }
        lds_barrier();
        if constexpr (ADJ) {
            // adjoint source of level L at the region's receiver cells
            if (etot > 0) {
                if (ecell >= 0) {
                    Ln[ecell] = fmaf(ekap, esrc, Ln[ecell]);
                    if (st + 1 < kk) esrc = source(L - 1, er, enext);
                }
                for (int e = tid + NT; e < etot; e += NT) {
                    int cell, r;
                    entry(e, cell, r);
                    if (cell >= 0)
                        Ln[cell] = fmaf(kap[(cell / W) * pitch + cell % W],
                                        source(L, r, rec_next[r]), Ln[cell]);
                }
                lds_barrier();
            }
        } else if (etot > 0) {
            gfloat *tr = gptr(J->traces) + (int64_t)L * nrec;   // level L + 1
            // (the first receiver of a cell only: k_trace_duplicates copies its
            // trace to the others at the end of the sweep)
            if (ecell >= 0) tr[er] = Ln[ecell];
            for (int e = tid + NT; e < etot; e += NT) {
                int cell, r;
                entry(e, cell, r);
                if (cell >= 0) tr[r] = Ln[cell];
            }
        }
    }

    // the tile's newest two levels (its newest is in LDS, with the adjoint source)
    const float *Le = buf + (kk & 1) * NB;
    if constexpr (ADJ) {
        float *p = adj + (int64_t)(2 * (pair ^ 1)) * fstride;
        const int kl = n - kk + 1;   // the last level computed
#pragma unroll
        for (int i = 0; i < PZ; ++i)
            cv[i] = *reinterpret_cast<const vf4 *>(Le + (lz + i) * W + lx);
        store_patch(p + (int64_t)(kl & 1) * fstride, cv);
        store_patch(p + (int64_t)((kl + 1) & 1) * fstride, pv);
        if (img) store_patch(grad, gv);
    } else if (!(flags & kTbStoreAll)) {
#pragma unroll
        for (int i = 0; i < PZ; ++i)
            cv[i] = *reinterpret_cast<const vf4 *>(Le + (lz + i) * W + lx);
        const int q = pair < 0 ? -1 : pair ^ 1;
        store_patch(fwd_level(n + kk, q), cv);
        if (q >= 0 || kk > 1) store_patch(fwd_level(n + kk - 1, q), pv);
    }
}

// Two forward steps of a large 2-D launch in one pass over the fields: a wave
// marches 128 columns (two per lane) down a chunk of rows and computes level
// n+1 at row r and level n+2 at row r - M - 1 in the same iteration.  Both
// levels' rows, kappa' (used twice, M + 1 rows apart) and the previous level
// are in register queues indexed by the unrolled phase, loaded two rows ahead;
// the x neighbours of the two centre rows go through one LDS row per level,
// double-buffered.  One wave per block: no barrier.
//
// The launch reads two levels and kappa' and writes two levels, 10 B per cell
// and step instead of 16.  What is computed twice is 8 of 64 lane columns and M
// rows at either end of a chunk; k_step2d_tb, whose blocks recompute an apron
// on four sides, spends twice the instructions per cell on large launches.  32
// shots of 1064 x 360: 48 us per launch, 24 us per step against 33 us with one
// step per launch and 36 us with k_step2d_tb (25 vector instructions per cell
// and step; 5.2 TB/s of fields that the Infinity Cache holds, which bounds it:
// 30 % less arithmetic left the time unchanged).  The same scheme for the
// adjoint (fused with its imaging condition, 197 registers: 67 us per step; as
// two passes, 65 us) was no faster than one step per launch (64 us), so adjoint
// launches take k_step2d_tb.  The cell arithmetic is k_step2d_direct's, term by
// term.
//
// Receivers are sampled one launch later, by extra blocks that read the two
// input levels.
template <int M>
struct Pipe2d {
    static constexpr int W = 128, A = 2 * M;
    static constexpr int D = 2, U = 2 * M + 2 + D;      // rows loaded ahead, queue length
    static constexpr int XH = (M + 1) / 2 * 2;          // columns read beside a pair
    static constexpr int LW = W + 2 * XH;               // LDS row
};

__device__ __forceinline__ void wave_fence()
{
    // orders the wave's own LDS accesses for the compiler (the hardware keeps
    // them in order); no wait is needed
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Stencil sums of a lane's two columns: q(d) is the row d rows below the
// centre, L the lane's place in the LDS copy of the centre row.
template <int M, class Q>
__device__ __forceinline__ vf2 pipe_star(const float *L, Q q)
{
    constexpr int XH = Pipe2d<M>::XH;
    constexpr Weights<M> WT{};
    constexpr int KD = kDiffRadii < M ? kDiffRadii : M;
    float xr[2 + 2 * XH];
#pragma unroll
    for (int c = 0; c < XH; c += 2) {
        const vf2 a = *reinterpret_cast<const vf2 *>(L - XH + c);
        const vf2 d = *reinterpret_cast<const vf2 *>(L + 2 + c);
        xr[c] = a.x; xr[c + 1] = a.y;
        xr[XH + 2 + c] = d.x; xr[XH + 3 + c] = d.y;
    }
    const vf2 pc = q(Int<0>{});
    xr[XH] = pc.x; xr[XH + 1] = pc.y;
    vf2 acc = {0.f, 0.f};
    static_for<0, M - KD>([&](auto I) __attribute__((always_inline)) {
        constexpr int m = M - decltype(I)::value;
        const vf2 up = q(Int<m>{}), dn = q(Int<-m>{});
        const float ta = (xr[XH + m] + xr[XH - m]) + (up.x + dn.x);
        const float tb = (xr[XH + 1 + m] + xr[XH + 1 - m]) + (up.y + dn.y);
        acc.x = fmaf(WT.c[m], ta, acc.x);
        acc.y = fmaf(WT.c[m], tb, acc.y);
    });
    if constexpr (KD < M) {
        acc.x = fmaf(WT.t2[KD], pc.x, acc.x);
        acc.y = fmaf(WT.t2[KD], pc.y, acc.y);
    }
    static_for<0, KD>([&](auto I) __attribute__((always_inline)) {
        constexpr int m = KD - decltype(I)::value;
        const vf2 up = q(Int<m>{}), dn = q(Int<-m>{});
        const float da = ((xr[XH + m] - pc.x) + (xr[XH - m] - pc.x)) +
                         ((up.x - pc.x) + (dn.x - pc.x));
        const float db = ((xr[XH + 1 + m] - pc.y) + (xr[XH + 1 - m] - pc.y)) +
                         ((up.y - pc.y) + (dn.y - pc.y));
        acc.x = fmaf(WT.c[m], da, acc.x);
        acc.y = fmaf(WT.c[m], db, acc.y);
    });
    return acc;
}

// Traces of level n (ring slot s0) and n-1 (s1) at receiver r.
__device__ __forceinline__ void gather_pair(const Job *__restrict__ J, int r, int n, int s0, int s1)
{
    if (!J->record || r >= J->nrec) return;
    const int64_t off = J->rec_off[r];
    float *tr = J->traces + r;
    if (n >= 1) tr[(int64_t)(n - 1) * J->nrec] = J->ring[(int64_t)s0 * J->fstride + off];
    if (n >= 2) tr[(int64_t)(n - 2) * J->nrec] = J->ring[(int64_t)s1 * J->fstride + off];
}

template <int M>
__global__ __launch_bounds__(64) void k_step2d_pipe(
    const Job *__restrict__ jobs, int njobs, int tiles_per_job, uint32_t magic_job,
    uint32_t magic_tx, int ntx, int zc, int n, int s0, int s1, int s2, int s3, int flags)
{
    using P = Pipe2d<M>;
    constexpr int U = P::U, D = P::D, XH = P::XH, LW = P::LW;
    __shared__ __align__(16) float sl[4 * LW];

    const int lane = threadIdx.x;
    const int ttiles = tiles_per_job * njobs;
    int b = blockIdx.x;
    if (b >= ttiles) {   // traces of the input levels n (slot s0) and n-1 (slot s1)
        const int gb = b - ttiles, ng = (int)(gridDim.x - ttiles) / njobs;
        gather_pair(jobs + gb / ng, gb % ng * 64 + lane, n, s0, s1);
        return;
    }
    if (flags & kTbRemap) b = xcd_remap(b, ttiles);
    const int j = njobs > 1 ? tb_div(b, tiles_per_job, magic_job) : 0;
    const int local = b - j * tiles_per_job;
    const int tz = ntx > 1 ? tb_div(local, ntx, magic_tx) : local, tx = local - tz * ntx;
    const Job *__restrict__ J = jobs + j;
    const int nz = J->nz, nx = J->nx, pitch = J->pitch, nb = J->nb;
    const int64_t fstride = J->fstride;
    const float eta_dt = J->eta_dt;
    const TbTile X = tb_tile(tx, ntx, P::W, P::A, M / 2 * 2, nx + M);
    const int z0 = tz * zc, z1 = min(z0 + zc, nz), npl = z1 - z0;

    // fields: level n (slot s0), n-1 (s1), n+1 (s2), n+2 (s3) of the ring
    float *const ring = J->ring;
    const float *cur = ring + (int64_t)s0 * fstride, *prv = ring + (int64_t)s1 * fstride;
    float *o1 = ring + (int64_t)s2 * fstride, *o2 = ring + (int64_t)s3 * fstride;
    const float *kap = J->kappa;

    // this lane's two columns
    const int col = X.origin + 2 * lane, x0 = col - M;
    const uint32_t voff = col < pitch ? 4u * (uint32_t)col : kDropOffset;
    const uint32_t soff = 2 * lane >= X.lo && 2 * lane < X.hi ? voff : kDropOffset;
    const bool xin0 = x0 >= 0 && x0 < nx, xin1 = x0 + 1 >= 0 && x0 + 1 < nx;
    const int dxa = sponge_depth(x0, nx, nb), dxb = sponge_depth(x0 + 1, nx, nb);
    const bool xedge = X.origin - M < nb || X.origin + P::W - 1 - M >= nx - nb;
    // Fields are addressed by one buffer resource each and a 32-bit byte offset
    // (fields are below kPipeFieldBytes): rows and columns outside a field read
    // zero and stores there are dropped.
    const int pb = 4 * pitch, fbytes = pb * (nz + 2 * M);
    auto field = [&](const float *f) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(f), 0, fbytes, kRsrcWord3);
    };
    const rsrc_t rcur = field(cur), rprv = field(prv), rkap = field(kap), ro1 = field(o1),
                 ro2 = field(o2);
    auto ld2 = [&](const rsrc_t f, int rowoff) __attribute__((always_inline)) {
        return __builtin_bit_cast(
            vf2, __builtin_amdgcn_raw_buffer_load_b64(f, (int)(voff + (uint32_t)rowoff), 0, 0));
    };
    auto st2 = [&](const rsrc_t f, int rowoff, vf2 v) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(vu2, v), f,
                                              (int)(soff + (uint32_t)rowoff), 0, 0);
    };
    auto rowof = [&](int z) { return (z + M) * pb; };   // byte offset of row z

    const int src_x = J->src_x, src_z = J->src_z;
    const gfloat *wavelet = gptr(J->wavelet);
    const float src_scale = J->src_scale;
    const int sc = src_x - x0;   // 0 or 1: this lane's column holds the source
    // LDS rows: level n, level n+1, two of each
    float *const l0 = sl + XH + 2 * lane, *const l1 = l0 + 2 * LW;
    // the update of a row: kappa', sum, centre and previous level; level L's
    // source; zero outside the grid
    // (CLEAN: the row holds neither sponge, frame nor source)
    auto update = [&](auto CLEAN, vf2 kv, vf2 lap, vf2 pc, vf2 pv, int z, int L)
        __attribute__((always_inline)) {
        vf2 o;
        o.x = fmaf(kv.x, lap.x, 2.f * pc.x);
        o.y = fmaf(kv.y, lap.y, 2.f * pc.y);
        if constexpr (decltype(CLEAN)::value) {
            o.x = o.x - pv.x;
            o.y = o.y - pv.y;
            return o;
        }
        if (z == src_z) {
#pragma clang fp contract(off)
            const float s = src_scale * wavelet[L];
            if (sc == 0) o.x = o.x + s;
            if (sc == 1) o.y = o.y + s;
        }
        if (xedge || z < nb || z >= nz - nb) {
            const int dz = sponge_depth(z, nz, nb);
            const float ea = (float)(dxa * dxa + dz * dz), eb = (float)(dxb * dxb + dz * dz);
            // (d = 0: 1 * (val - 1 * prev), bit for bit val - prev)
            o.x = __builtin_amdgcn_rcpf(fmaf(eta_dt, ea, 1.f)) *
                  fmaf(-fmaf(-eta_dt, ea, 1.f), pv.x, o.x);
            o.y = __builtin_amdgcn_rcpf(fmaf(eta_dt, eb, 1.f)) *
                  fmaf(-fmaf(-eta_dt, eb, 1.f), pv.y, o.y);
            const bool zin = z >= 0 && z < nz;
            o.x = xin0 && zin ? o.x : 0.f;
            o.y = xin1 && zin ? o.y : 0.f;
        } else {
            o.x = o.x - pv.x;
            o.y = o.y - pv.y;
        }
        return o;
    };

    // Iteration t: level n+1 at row r1 = z0 - M + t, level n+2 at r2 = r1-M-1.
    // Queue slots (mod U): level n row z0 - 2M + i in slot i, so r1 is i = t + M
    // and r2 is i = t - 1; level n+1, kappa' and the previous level by row
    // z0 - M + i, so r1 is i = t and r2 is i = t - M - 1.
    vf2 q0[U], q1[U], kq[U], pq[U];
    auto at = [](int i) constexpr { return ((i % U) + U) % U; };
#pragma unroll
    for (int i = 0; i < 2 * M + D; ++i) q0[at(i)] = ld2(rcur, rowof(z0 - 2 * M + i));
#pragma unroll
    for (int i = 0; i < D; ++i) {
        kq[at(i)] = ld2(rkap, rowof(z0 - M + i));
        pq[at(i)] = ld2(rprv, rowof(z0 - M + i));
    }
    *reinterpret_cast<vf2 *>(l0) = q0[at(M)];
    wave_fence();

    auto iterate = [&](auto CLEAN, auto K, const int t, const bool do2)
        __attribute__((always_inline)) {
        constexpr int k = decltype(K)::value;   // t mod U
        const int r1 = z0 - M + t, r2 = r1 - M - 1;
        // loads D rows ahead
        const int off1 = rowof(r1);
        q0[at(k + 2 * M + D)] = ld2(rcur, off1 + (M + D) * pb);
        kq[at(k + D)] = ld2(rkap, off1 + D * pb);
        pq[at(k + D)] = ld2(rprv, off1 + D * pb);
        constexpr int pc = k & 1, pn = pc ^ 1;   // U is even
        vf2 n1 = {0.f, 0.f};
        {
            const vf2 lap = pipe_star<M>(l0 + pc * LW, [&](auto D) __attribute__((always_inline)) {
                return q0[at(k + M + decltype(D)::value)];
            });
            n1 = update(CLEAN, kq[at(k)], lap, q0[at(k + M)], pq[at(k)], r1, n);
            st2(ro1, r1 >= z0 && r1 < z1 ? off1 : kPipeFieldBytes, n1);
        }
        q1[at(k)] = n1;
        if (do2) {
            const vf2 lap = pipe_star<M>(l1 + pc * LW, [&](auto D) __attribute__((always_inline)) {
                return q1[at(k - M - 1 + decltype(D)::value)];
            });
            const vf2 c1 = q1[at(k - M - 1)], c0 = q0[at(k - 1)];
            const vf2 n2 = update(CLEAN, kq[at(k - M - 1)], lap, c1, c0, r2, n + 1);
            st2(ro2, r2 < z1 ? off1 - (M + 1) * pb : kPipeFieldBytes, n2);
        }
        // centre rows of the next iteration
        *reinterpret_cast<vf2 *>(l0 + pn * LW) = q0[at(k + M + 1)];
        *reinterpret_cast<vf2 *>(l1 + pn * LW) = q1[at(k - M)];
        wave_fence();
    };
    // 2M + 1 iterations fill level n+1's queue
    static_for<0, 2 * M + 1>([&](auto K) __attribute__((always_inline)) {
        iterate(Int<0>{}, K, decltype(K)::value, false);
    });
    // Whole groups of U iterations (past the chunk's end the stores are
    // dropped; chunks are multiples of U rows): without a branch where every row
    // of both levels is clean.  No iteration is skipped, so no queue slot lives
    // longer than its row is needed.
    constexpr int T0 = 2 * M + 1;
    for (int tb = T0; tb < T0 + npl; tb += U) {
        const int za = z0 + tb - 2 * M - 1, zb = z0 + tb + U - 1 - M;   // rows of the group
        const bool clean = !xedge && za >= nb && zb < nz - nb &&
                           (src_z < za || src_z > zb);
        if (clean)
            static_for<0, U>([&](auto I) __attribute__((always_inline)) {
                constexpr int i = decltype(I)::value;
                iterate(Int<1>{}, Int<(T0 + i) % U>{}, tb + i, true);
            });
        else
            static_for<0, U>([&](auto I) __attribute__((always_inline)) {
                constexpr int i = decltype(I)::value;
                iterate(Int<0>{}, Int<(T0 + i) % U>{}, tb + i, true);
            });
    }
}

// Traces of receivers that share a cell with an earlier one, copied from the first
// one of the cell after a sweep of multi-step launches, which sample that one only.
// Walking the others at every step was a chain of dependent loads: 1000 receivers on
// one cell made 100 steps of 168 x 168 cells take 7475 us instead of 295.
__global__ __launch_bounds__(256) void k_trace_duplicates(const Job *__restrict__ jobs,
                                                          int64_t total, int nrec, int nt)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * 256) {
        const Job *J = jobs + i / nrec;
        const int r = (int)(i % nrec), h = J->rec_head[r];
        if (h == r) continue;
        for (int n = blockIdx.y; n < nt; n += gridDim.y) {
            float *tr = J->traces + (int64_t)n * nrec;
            tr[r] = tr[h];
        }
    }
}

__global__ __launch_bounds__(64) void k_gather2(const Job *__restrict__ jobs, int n, int s0, int s1)
{
    gather_pair(jobs + blockIdx.y, blockIdx.x * 64 + threadIdx.x, n, s0, s1);
}

// ---------------------------------------------------------------- launchers
template <int M>
static void launch_2d(int nw, bool adj, const Job *jobs, const int *prefix, int njobs, int step,
                      int ttiles, int grid, int remap, const LevelMap &lm, hipStream_t st)
{
    if (nw == 1) {   // one-row tiles, one cell per lane
        if (adj)
            hipLaunchKernelGGL((k_step2d_direct<M, true>), dim3(grid), dim3(64), 0, st, jobs,
                               prefix, njobs, step, ttiles, remap, lm);
        else
            hipLaunchKernelGGL((k_step2d_direct<M, false>), dim3(grid), dim3(64), 0, st, jobs,
                               prefix, njobs, step, ttiles, remap, lm);
    } else {
        if (adj)
            hipLaunchKernelGGL((k_step2d<M, true>), dim3(grid), dim3(64), 0, st, jobs, prefix,
                               njobs, step, ttiles, remap, lm);
        else
            hipLaunchKernelGGL((k_step2d<M, false>), dim3(grid), dim3(64), 0, st, jobs, prefix,
                               njobs, step, ttiles, remap, lm);
    }
}

void launch_step2d(int M, int nw, bool adj, const Job *jobs, const int *prefix, int njobs,
                   int step, int ttiles, int grid, int remap, const LevelMap &lm, hipStream_t st)
{
    switch (M) {
    case 1: launch_2d<1>(nw, adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    case 2: launch_2d<2>(nw, adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    case 4: launch_2d<4>(nw, adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    case 8: launch_2d<8>(nw, adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    default: break;
    }
}

// Shapes of multi-step 2-D launches: region W x H cells, PZ rows per thread
// (which shape a launch takes: tb_config in the runtime).
#define FWI_TB_SHAPES(X)                                                                        \
    X(0, 48, 40, 1) X(1, 64, 48, 1) X(2, 64, 64, 2) X(3, 128, 64, 2) X(4, 128, 64, 4)

int tb2d_width(int shape)
{
    switch (shape) {
#define FWI_TB(id, W, H, PZ) case id: return W;
        FWI_TB_SHAPES(FWI_TB)
#undef FWI_TB
    }
    return 64;
}
int tb2d_height(int shape)
{
    switch (shape) {
#define FWI_TB(id, W, H, PZ) case id: return H;
        FWI_TB_SHAPES(FWI_TB)
#undef FWI_TB
    }
    return 64;
}

template <int M, bool ADJ>
static void launch_tb(int shape, dim3 g, const Job *jobs, int njobs, const TbLaunch &a,
                      hipStream_t st)
{
    const int flags = (a.pair + 1) | (a.remap ? kTbRemap : 0) | (a.record ? kTbRecord : 0) |
                      (a.store_all ? kTbStoreAll : 0);
    switch (shape) {
#define FWI_TB(id, W, H, PZ)                                                                    \
    case id:                                                                                    \
        if constexpr (tb_has_shape(M, id))                                                      \
            hipLaunchKernelGGL((k_step2d_tb<M, W, H, PZ, ADJ>), g, dim3((W / 4) * (H / PZ)), 0, \
                               st, jobs, njobs, a.tiles_per_job, a.magic_job, a.magic_tx,       \
                               a.ntx, a.ntz, a.step, a.kk | a.A << 16, flags);                  \
        break;
        FWI_TB_SHAPES(FWI_TB)
#undef FWI_TB
    }
}

void launch_step2d_tb(int M, int shape, bool adj, const Job *jobs, int njobs, const TbLaunch &a,
                      hipStream_t st)
{
    const dim3 g(a.tiles_per_job * njobs);
    if (g.x == 0) return;
    switch (M) {
#define FWI_TBM(m)                                                             \
    case m:                                                                    \
        if (adj) launch_tb<m, true>(shape, g, jobs, njobs, a, st);             \
        else launch_tb<m, false>(shape, g, jobs, njobs, a, st);                \
        break;
        FWI_TBM(1)
        FWI_TBM(2)
        FWI_TBM(4)
        FWI_TBM(8)
#undef FWI_TBM
    }
}

// Two-step marching 2-D launches: region width; chunks are multiples of `group`
// rows.
int pipe2d_width() { return Pipe2d<4>::W; }
int pipe2d_group(int M) { return M == 2 ? Pipe2d<2>::U : Pipe2d<4>::U; }

template <int M>
static void launch_pipe(const Job *jobs, int njobs, const PipeLaunch &a, hipStream_t st)
{
    hipLaunchKernelGGL((k_step2d_pipe<M>), dim3((a.tiles_per_job + a.gblocks) * njobs), dim3(64), 0,
                       st, jobs, njobs, a.tiles_per_job, a.magic_job, a.magic_tx, a.ntx, a.zc, a.n,
                       a.slot[0], a.slot[1], a.slot[2], a.slot[3], a.remap ? kTbRemap : 0);
}

void launch_step2d_pipe(int M, const Job *jobs, int njobs, const PipeLaunch &a, hipStream_t st)
{
    if (M == 2) launch_pipe<2>(jobs, njobs, a, st);
    else if (M == 4) launch_pipe<4>(jobs, njobs, a, st);
}

void launch_trace_duplicates(const Job *jobs, int njobs, int nrec, int nt, hipStream_t st)
{
    const int64_t total = (int64_t)njobs * nrec, blocks = (total + 255) / 256;
    if (total > 0)
        hipLaunchKernelGGL(k_trace_duplicates,
                           dim3((int)(blocks < 4096 ? blocks : 4096), nt < 64 ? nt : 64),
                           dim3(256), 0, st, jobs, total, nrec, nt);
}

void launch_gather2(const Job *jobs, int njobs, int nrec, int n, int s0, int s1, hipStream_t st)
{
    if (nrec > 0)
        hipLaunchKernelGGL(k_gather2, dim3((nrec + 63) / 64, njobs), dim3(64), 0, st, jobs, n, s0,
                           s1);
}

}  // namespace fwi
