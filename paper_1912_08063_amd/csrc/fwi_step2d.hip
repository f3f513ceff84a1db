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
        rp = J->rt_start[local];
        re = J->rt_start[local + 1];
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
        const int rp = J->rt_start[local], re = J->rt_start[local + 1];
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
// Several forward steps of a small 2-D grid in one launch (temporal blocking
// for launch-bound grids).  A block loads a region of p^n, p^{n-1} and kappa'
// into LDS that extends the output tile by A = K M cells on every side, then
// advances it kk <= K steps in LDS, each step on a region M cells narrower
// (the apron cells are computed redundantly by neighbouring blocks), and
// stores levels n+kk and n+kk-1 of its output tile.  Cells outside the padded
// grid hold zero and are never updated, as the frame in memory.  Each cell's
// arithmetic is k_step2d_direct's, term by term, so the fields and traces are
// bitwise those of kk single steps.  The launch reads ring slots n, n-1 and
// writes slots n+kk, n+kk-1, which must differ (ring length >= K + 2): no
// block reads what another writes.  Traces of levels n .. n+kk are written by
// the block whose output tile holds the receiver (level n too: a preceding
// single step does not sample the level it produces).
template <int M, int K>
struct Multi2d {
    static constexpr int A = K * M;                     // apron
    static constexpr int RW = 64;                        // region width (one wave per row)
    static constexpr int OX = RW - 2 * A, OZ = 16;       // output tile
    static constexpr int RH = OZ + 2 * A, NR = RW * RH;  // region
    static_assert(OX >= 16, "apron too wide for the region");
};

template <int M, int K>
__global__ __launch_bounds__(1024) void k_step2d_multi(const Job *__restrict__ jobs,
                                                       int tiles_per_job, int ntxm, int step,
                                                       int kk, int record)
{
    using G = Multi2d<M, K>;
    constexpr int A = G::A, RW = G::RW, OX = G::OX, OZ = G::OZ, RH = G::RH, NR = G::NR;
    constexpr int NT = 1024, CPT = (NR + NT - 1) / NT;   // region cells per thread
    constexpr int RPT = 2;                               // receivers resolved per thread
    constexpr Weights<M> W{};
    constexpr int KD = kDiffRadii < M ? kDiffRadii : M;
    __shared__ float s0[NR], s1[NR], sk[NR];

    const int tid = threadIdx.x;
    const int j = blockIdx.x / tiles_per_job, t = blockIdx.x % tiles_per_job;
    const Job *__restrict__ J = jobs + j;
    const int n = step_level(J, step, false);
    const int nz = J->nz, nx = J->nx, pitch = J->pitch, nb = J->nb, nrec = J->nrec;
    const int x0 = (t % ntxm) * OX - A, z0 = (t / ntxm) * OZ - A;   // region origin
    const gfloat *cur = gptr(level_ptr(J, LevelMap{}, n));
    const gfloat *prv = gptr(level_ptr(J, LevelMap{}, n - 1));
    const gfloat *kap = gptr(J->kappa);
    gfloat *o1 = gptr(level_ptr(J, LevelMap{}, n + kk));
    gfloat *o0 = gptr(level_ptr(J, LevelMap{}, n + kk - 1));
    const float eta_dt = J->eta_dt;
    const int64_t p64 = pitch;

    // this thread's region cells: LDS index, grid coordinates, inside the grid
    int ci[CPT], cx[CPT], cz[CPT];
    bool cin[CPT];
#pragma unroll
    for (int q = 0; q < CPT; ++q) {
        ci[q] = tid + q * NT;
        cx[q] = x0 + ci[q] % RW;
        cz[q] = z0 + ci[q] / RW;
        cin[q] = ci[q] < NR && cx[q] >= 0 && cx[q] < nx && cz[q] >= 0 && cz[q] < nz;
    }
#pragma unroll
    for (int q = 0; q < CPT; ++q) {
        if (ci[q] >= NR) continue;
        const int64_t off = (int64_t)(cz[q] + M) * p64 + (cx[q] + M);
        s0[ci[q]] = cin[q] ? cur[off] : 0.f;
        s1[ci[q]] = cin[q] ? prv[off] : 0.f;
        sk[ci[q]] = cin[q] ? kap[off] : 0.f;
    }
    // receivers in this block's output tile: their LDS index (-1: elsewhere).
    // Grids on this path are small, so field offsets fit 32 bits.
    const bool rec_on = record && J->record;
    auto local_of = [&](int r) {
        const int off = (int)J->rec_off[r];
        const int rx = off % pitch - M - x0, rz = off / pitch - M - z0;
        return rx >= A && rx < A + OX && rz >= A && rz < A + OZ ? rz * RW + rx : -1;
    };
    int rl[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = tid + q * NT;
        rl[q] = rec_on && r < nrec ? local_of(r) : -1;
    }
    // traces of level L (1 .. nt) from the LDS field f
    auto sample = [&](const float *f, int L) {
        if (!rec_on || L < 1 || L > J->nt) return;
        float *tr = J->traces + (int64_t)(L - 1) * nrec;
#pragma unroll
        for (int q = 0; q < RPT; ++q)
            if (rl[q] >= 0) tr[tid + q * NT] = f[rl[q]];
        for (int r = tid + RPT * NT; r < nrec; r += NT) {
            const int li = local_of(r);
            if (li >= 0) tr[r] = f[li];
        }
    };
    __syncthreads();
    sample(s0, n);

    float *cu = s0, *pr = s1;   // levels L and L-1; the step writes L+1 over L-1
    for (int st = 0; st < kk; ++st) {
        const int L = n + st, lo = (st + 1) * M;
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            const int i = ci[q], rx = i % RW, rz = i / RW;
            if (!cin[q] || rx < lo || rx >= RW - lo || rz < lo || rz >= RH - lo) continue;
            const int x = cx[q], z = cz[q];
            const float pc = cu[i];
            const float kv = sk[i];
            const float pv = pr[i];
            float acc = 0.f;
#pragma unroll
            for (int m = M; m > KD; --m) {
                const float tt = (cu[i + m] + cu[i - m]) + (cu[i + m * RW] + cu[i - m * RW]);
                acc = fmaf(W.c[m], tt, acc);
            }
            if constexpr (KD < M) acc = fmaf(W.t2[KD], pc, acc);
#pragma unroll
            for (int m = KD; m >= 1; --m) {
                const float d = ((cu[i + m] - pc) + (cu[i - m] - pc)) +
                                ((cu[i + m * RW] - pc) + (cu[i - m * RW] - pc));
                acc = fmaf(W.c[m], d, acc);
            }
            float val = fmaf(kv, acc, 2.f * pc);
            if (J->src_x == x && J->src_z == z) {
#pragma clang fp contract(off)
                const float srcv = J->src_scale * J->wavelet[L];
                val = val + srcv;
            }
            const int dxs = sponge_depth(x, nx, nb), dz = sponge_depth(z, nz, nb);
            pr[i] = leapfrog(val, pv, dxs * dxs + dz * dz, eta_dt);
        }
        __syncthreads();
        float *tmp = cu;
        cu = pr;
        pr = tmp;
        sample(cu, L + 1);
    }

#pragma unroll
    for (int q = 0; q < CPT; ++q) {
        const int i = ci[q], rx = i % RW, rz = i / RW;
        if (!cin[q] || rx < A || rx >= A + OX || rz < A || rz >= A + OZ) continue;
        const int64_t off = (int64_t)(cz[q] + M) * p64 + (cx[q] + M);
        o1[off] = cu[i];
        o0[off] = pr[i];
    }
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

// Multi-step 2-D forward launches: the largest step count per launch, the
// output tile, and the launch itself (M <= 4).
int multi2d_steps() { return 4; }
void multi2d_tile(int M, int *ox, int *oz)
{
    switch (M) {
    case 1: *ox = Multi2d<1, 4>::OX; break;
    case 2: *ox = Multi2d<2, 4>::OX; break;
    default: *ox = Multi2d<4, 4>::OX; break;
    }
    *oz = Multi2d<4, 4>::OZ;
}
void launch_step2d_multi(int M, const Job *jobs, int njobs, int tiles_per_job, int ntxm,
                         int step, int kk, bool record, hipStream_t st)
{
    // 1024 threads: three cells of the 64 x 48 region per thread and step, so
    // a step is a short latency chain (256 threads: 5.3 us per step)
    const dim3 g(njobs * tiles_per_job), b(1024);
    const int rec = record ? 1 : 0;
    switch (M) {
    case 1: hipLaunchKernelGGL((k_step2d_multi<1, 4>), g, b, 0, st, jobs, tiles_per_job, ntxm, step, kk, rec); break;
    case 2: hipLaunchKernelGGL((k_step2d_multi<2, 4>), g, b, 0, st, jobs, tiles_per_job, ntxm, step, kk, rec); break;
    case 4: hipLaunchKernelGGL((k_step2d_multi<4, 4>), g, b, 0, st, jobs, tiles_per_job, ntxm, step, kk, rec); break;
    default: break;
    }
}

}  // namespace fwi
