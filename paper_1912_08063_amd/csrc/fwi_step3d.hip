// fwi_step3d.hip -- the 3-D step kernels (see fwi_kernels.hip for the design).
// Compiled once per stencil radius, FWI_STEP3D_M = 1, 2, 4 or 8, so that the
// radii build in parallel.
#include "fwi_device.h"

#include <stdlib.h>

namespace fwi {

// --------------------------------------------------------------- 3-D step
// One block: NW wavefronts of RY rows each, a 64 (x) x NW*RY (y) tile,
// marching a chunk of z.  Per plane z: the LDS buffer (z & 1) holds plane z of the propagated field
// with an M-cell halo; registers hold the z-queue (planes z-M .. z+M, in a
// ring indexed by the unrolled phase k, so no register moves), kappa' and
// the previous level.  While plane z is computed, plane z+1 is already being
// loaded (the next queue front, kappa', previous level, halos), and written
// to the other LDS buffer afterwards: one barrier per plane.
//
// Step modes: the forward step; the adjoint step with the imaging condition
// fused in (two stencil fields); and the adjoint as two single-field passes,
// the psi update alone and the imaging condition g += psi^{k+1} * L'p^k
// alone, each with the forward step's memory pattern (see launch_3d).
enum StepMode { kFwd = 0, kAdj = 1, kAdjPsi = 2, kImage = 3 };

// Planes a step kernel loads ahead of the one it computes (queue front,
// kappa', previous level).  Two planes ahead measured no faster on the
// 304^3 forward: 86.7 against 85.1 us per step with 4 x 4 blocks (211
// registers), 85.9 with 4 x 2.  No launch bound caps the registers: one
// wave per SIMD more spills (4 x 4 forward at 3 waves: 98 against 85 us;
// fused adjoint at 4 waves: 190 against 171 us).
template <int M, int MODE>
constexpr int kLookahead = 1;

template <int M, int MODE, int NW, int RY>
__global__ __launch_bounds__(64 * NW) void k_step3d(const Job *__restrict__ jobs,
                                                const int *__restrict__ prefix, int njobs,
                                                int step, int ttiles, int remap, LevelMap lm)
{
    constexpr int TX = kTileX, TY = RY * NW, NT = 64 * NW;
    constexpr int LX = TX + 2 * M, LY = TY + 2 * M, Q = 2 * M + 1, LS = LY * LX;
    constexpr int NYH = (2 * M * TX + NT - 1) / NT;   // y-halo cells per thread
    constexpr int NXH = (TY * 2 * M + NT - 1) / NT;   // x-halo cells per thread
    constexpr bool ADJ = MODE != kFwd;     // adjoint time order and tiling
    constexpr bool FUSED = MODE == kAdj;   // second stencil field (p^k) and g
    constexpr bool IMG = MODE == kImage;
    // single-field modes up to 8th order: halos travel with the queue front
    // (loaded at plane z+M, the same iteration in which the neighbouring tiles
    // load those rows as their own front, so the second read is an L2 hit)
    // and wait in a register ring.  At 16th order the ring would hold 5 x 17
    // values per thread; without it the step runs at 4 instead of 2 waves per
    // SIMD and 46 % faster (122 vs 178 us on a 304^3 grid), while at 8th order
    // the ring wins (89 vs 94 us).
    constexpr bool HQ = !FUSED && M <= 4;
    constexpr Weights<M> W{};
    constexpr int KD = kDiffRadii < M ? kDiffRadii : M;   // radii in difference form
    __shared__ float sp[2 * LS];
    __shared__ float sf[FUSED ? 2 * LS : 1];

    const int tid = threadIdx.x;
    int b = blockIdx.x;
    if (b >= ttiles) {   // receiver-sampling blocks (forward launches only)
        if constexpr (ADJ) return;
        const int gb = b - ttiles;
        const int j = find_job(prefix + njobs + 1, njobs, gb);
        const Job *J = jobs + j;
        gather_block(J, lm, (gb - prefix[njobs + 1 + j]) * blockDim.x + tid, step_level(J, step, false));
        return;
    }
    if (remap) b = xcd_remap(b, ttiles);
    const int j = find_job(prefix, njobs, b);
    const Job *__restrict__ J = jobs + j;
    const int n = step_level(J, step, ADJ);
    if (ADJ ? (n < J->adj_lo || n >= J->adj_hi) : (n < J->fwd_lo || n >= J->fwd_hi)) return;

    const int nz = J->nz, ny = J->ny, nx = J->nx, pitch = J->pitch, nb = J->nb;
    const int64_t plane = J->plane, fstride = J->fstride;
    const Job::Tiling &T = J->tile[ADJ ? 1 : 0];
    int local = b - prefix[j];
    int tx, ty, tz;
    if (T.flags & kTileZFast) {
        tz = local % T.nzc;
        local /= T.nzc;
        tx = local % T.ntx;
        ty = local / T.ntx;
    } else {
        tx = local % T.ntx;
        local /= T.ntx;
        ty = local % T.nty;
        tz = local / T.nty;
    }
    const int z0 = tz * T.zc, z1 = min(z0 + T.zc, nz);
    // marching direction: plane i of the chunk (i = 0 .. npl-1) is zs + dir * i
    const int dir = (T.flags & kTileZAlt) && (tz & 1) ? -1 : 1;
    const int zs = dir > 0 ? z0 : z1 - 1, npl = z1 - z0;

    // cur: the stencil field; prv and kap: the two pointwise streams; out.
    // Imaging mode: cur = p^k, prv = psi^{k+1}, kap = out = g.
    const gfloat *cur, *prv, *kap = gptr(J->kappa);
    gfloat *out;
    const gfloat *fwd = nullptr;
    gfloat *grad = nullptr;
    const bool accum = ADJ && J->accumulate && n <= J->nt - 1;
    if constexpr (IMG) {
        if (!accum) return;
        cur = gptr(level_ptr(J, lm, n));
        prv = gptr(J->adj) + (int64_t)((n + 1) & 1) * fstride;
        kap = gptr(J->grad);
        out = gptr(J->grad);
    } else if constexpr (ADJ) {
        cur = gptr(J->adj) + (int64_t)((n + 1) & 1) * fstride;
        prv = gptr(J->adj) + (int64_t)(n & 1) * fstride;
        out = gptr(J->adj) + (int64_t)(n & 1) * fstride;
        if constexpr (FUSED) {
            fwd = gptr(level_ptr(J, lm, n));
            grad = gptr(J->grad);
        }
    } else {
        cur = gptr(level_ptr(J, lm, n));
        prv = gptr(level_ptr(J, lm, n - 1));
        out = gptr(level_ptr(J, lm, n + 1));
    }
    const float eta_dt = J->eta_dt;
    const int pbytes = (int)(plane * (int64_t)sizeof(float));

    // ---- per-thread geometry (loop invariant)
    const int lane = tid & 63, wv = tid >> 6;
    const int col = tx * TX + lane;   // memory column
    const int x = col - M;            // padded-grid x
    const bool ax = x >= 0 && x < nx;
    // Loads are unconditional: a row past the frame is clamped to the last
    // frame row and a column outside the row to its edge.  Both hold zeros
    // (frames and row padding are zero-filled and never written), exactly
    // the values a masked load would give, and no active cell reads them
    // beyond that.  Stores stay masked.
    const int last_row = ny + 2 * M - 1;   // memory rows per plane - 1
    bool act[RY];
    uint32_t roff[RY];   // byte offsets within a plane
    uint32_t soff[RY];   // store offsets: kDropOffset for cells outside the grid
    int dxy2[RY];
    const int dxs = sponge_depth(x, nx, nb);
#pragma unroll
    for (int i = 0; i < RY; ++i) {
        const int yy = ty * TY + wv * RY + i;
        act[i] = ax && yy < ny;
        roff[i] = 4u * (uint32_t)(min(yy + M, last_row) * pitch + col);
        soff[i] = act[i] ? roff[i] : kDropOffset;
        const int d = sponge_depth(yy, ny, nb);
        dxy2[i] = d * d + dxs * dxs;
    }
    uint32_t hyo[NYH], hxo[NXH];
    int hyl[NYH], hxl[NXH];
#pragma unroll
    for (int q = 0; q < NYH; ++q) {   // rows above and below the tile
        const int h = tid + NT * q;
        const int r = (h / TX) % (2 * M), c = h % TX;
        const int ly = r < M ? r : r + TY;
        const int yg = ty * TY - M + ly;
        hyo[q] = 4u * (uint32_t)(min(yg + M, last_row) * pitch + tx * TX + c);
        hyl[q] = h < 2 * M * TX ? ly * LX + M + c : -1;
    }
#pragma unroll
    for (int q = 0; q < NXH; ++q) {   // columns left and right of the tile
        const int h = tid + NT * q;
        const int r = (h / (2 * M)) % TY, c = h % (2 * M);
        const int lc = c < M ? c : c + TX;
        const int cm = min(max(tx * TX - M + lc, 0), pitch - 1);
        const int yg = ty * TY + r;
        hxo[q] = 4u * (uint32_t)(min(yg + M, last_row) * pitch + cm);
        hxl[q] = h < TY * 2 * M ? (M + r) * LX + lc : -1;
    }
    // source (forward): the block that owns it adds it at its plane
    const bool src_blk = !ADJ && J->src_x >= tx * TX - M && J->src_x < tx * TX - M + TX &&
                         J->src_y >= ty * TY && J->src_y < ty * TY + TY && J->src_z >= z0 &&
                         J->src_z < z1;
    float srcv = 0.f;
    int src_row = -1;
    if (src_blk && J->src_x == x) {
        const int r = J->src_y - (ty * TY + wv * RY);
        if (r >= 0 && r < RY) { src_row = r; srcv = J->src_scale * J->wavelet[n]; }
    }

    // ---- register queues.  Chunk plane j (j = -M .. npl-1+M, memory plane
    // zs + dir j + M) lives in queue slot (j + M) % U.  While plane ii is
    // computed from slots ii .. ii+2M (mod U), planes up to ii+M+D-1 are
    // already loaded and the front plane ii+M+D is loaded straight into a
    // free slot (U >= Q + D), so no register is copied after a load and the
    // wave never waits for recent prefetches before it moves on.  kappa', the
    // previous level (and g) of plane ii are in slot ii % (D + 1), loaded D
    // planes ahead.  The plane loop is unrolled by U, a multiple of D + 1,
    // so every slot index is a compile-time constant.  Halos staged from
    // memory at the end of a plane (no halo ring) are loaded one plane ahead,
    // first, so that the wait for them leaves the rest in flight.
    constexpr int D = kLookahead<M, MODE>;
    constexpr int P = D + 1;
    constexpr int U = (Q + D + P - 1) / P * P;
    float q[RY][U];
    float f[FUSED ? RY : 1][FUSED ? U : 1];
    float hy[HQ ? NYH : 1][HQ ? U : 1], hx[HQ ? NXH : 1][HQ ? U : 1];
    if constexpr (HQ) {
        // halos of chunk planes 1 .. M+D-1 (slots M+1 .. 2M+D-1)
#pragma unroll
        for (int s = M + 1; s < Q + D - 1; ++s) {
            if (s - M >= npl) continue;
            const rsrc_t ph = plane_rsrc(cur, zs + dir * (s - M) + M, plane, pbytes);
#pragma unroll
            for (int h = 0; h < NYH; ++h) hy[h][s] = ldb(ph, hyo[h]);
#pragma unroll
            for (int h = 0; h < NXH; ++h) hx[h][s] = ldb(ph, hxo[h]);
        }
    }
    // chunk planes -M .. M+D-1 (plane j is first read by the stencil of
    // plane j - M, so planes past the chunk's last plane + M are skipped)
#pragma unroll
    for (int s = 0; s < Q + D - 1; ++s) {
        if (s >= Q && s - 2 * M >= npl) continue;
        const int zm = zs + dir * (s - M) + M;
        const rsrc_t pc = plane_rsrc(cur, zm, plane, pbytes);
        const rsrc_t pf = plane_rsrc(fwd, zm, plane, pbytes);
#pragma unroll
        for (int i = 0; i < RY; ++i) {
            q[i][s] = ldb(pc, roff[i]);
            if constexpr (FUSED) f[i][s] = ldb(pf, roff[i]);
        }
    }
    float kv[P][RY], pv[P][RY], gv[FUSED ? P : 1][FUSED ? RY : 1];
    // pointwise streams of planes 1 .. D-1
#pragma unroll
    for (int a = 1; a < D; ++a) {
        if (a >= npl) continue;
        const rsrc_t pk = plane_rsrc(kap, zs + dir * a + M, plane, pbytes);
        const rsrc_t pp = plane_rsrc(prv, zs + dir * a + M, plane, pbytes);
#pragma unroll
        for (int i = 0; i < RY; ++i) {
            kv[a][i] = ldb_stream(pk, roff[i]);
            pv[a][i] = ldb_stream(pp, roff[i]);
            if constexpr (FUSED)
                gv[a][i] = accum ? ldb_stream(plane_rsrc(grad, zs + dir * a + M, plane, pbytes), roff[i])
                                 : 0.f;
        }
    }
    {
        const rsrc_t pk = plane_rsrc(kap, zs + M, plane, pbytes);
        const rsrc_t pp = plane_rsrc(prv, zs + M, plane, pbytes);
#pragma unroll
        for (int i = 0; i < RY; ++i) {
            kv[0][i] = ldb(pk, roff[i]);
            pv[0][i] = ldb(pp, roff[i]);
            if constexpr (FUSED)
                gv[0][i] = accum ? ldb(plane_rsrc(grad, zs + M, plane, pbytes), roff[i]) : 0.f;
        }
        const rsrc_t pc = plane_rsrc(cur, zs + M, plane, pbytes);
        const rsrc_t pf = plane_rsrc(fwd, zs + M, plane, pbytes);
        float *L = sp;           // LDS buffer i & 1 holds chunk plane i
        float *LF = FUSED ? sf : nullptr;
#pragma unroll
        for (int i = 0; i < RY; ++i) {
            L[(M + wv * RY + i) * LX + M + lane] = q[i][M];
            if constexpr (FUSED) LF[(M + wv * RY + i) * LX + M + lane] = f[i][M];
        }
#pragma unroll
        for (int h = 0; h < NYH; ++h)
            if (hyl[h] >= 0) {
                L[hyl[h]] = ldb(pc, hyo[h]);
                if constexpr (FUSED) LF[hyl[h]] = ldb(pf, hyo[h]);
            }
#pragma unroll
        for (int h = 0; h < NXH; ++h)
            if (hxl[h] >= 0) {
                L[hxl[h]] = ldb(pc, hxo[h]);
                if constexpr (FUSED) LF[hxl[h]] = ldb(pf, hxo[h]);
            }
    }
    lds_barrier();

    // Plane ii of the chunk; k = ii % U selects the slots.  The main loop
    // runs whole groups of U planes that all have a next plane (more), with
    // no branch around a load or store, so the compiler's wait counts stay
    // exact and only LDS waits remain at the barrier; the last group runs
    // with those checks.
    auto step_plane = [&](auto K, const int ii, const bool more, const bool ahead)
        __attribute__((always_inline)) {
            constexpr int k = decltype(K)::value;
            const int z = zs + dir * ii;   // grid plane computed now
            const int c = k % P, cn = (k + D) % P;   // pointwise slots of planes ii, ii+D
            const int fs = (k + Q - 1 + D) % U;      // free queue slot: chunk plane ii+M+D
            // ---- prefetch: halos of plane z+dir staged at the end of this
            // plane (without a halo ring), then the queue front z+dir(1+M)
            // and the pointwise streams of plane z+dir; memory plane = grid
            // plane + M
            float nhy[HQ ? 1 : NYH], nhx[HQ ? 1 : NXH];
            float nfy[FUSED ? NYH : 1], nfx[FUSED ? NXH : 1];
            const int zf = z + dir * (D + M) + M, zn = z + dir + M, za = z + dir * D + M;
            if (more) {
                if constexpr (!HQ) {
                    const rsrc_t ph = plane_rsrc(cur, zn, plane, pbytes);
#pragma unroll
                    for (int h = 0; h < NYH; ++h) nhy[h] = ldb(ph, hyo[h]);
#pragma unroll
                    for (int h = 0; h < NXH; ++h) nhx[h] = ldb(ph, hxo[h]);
                }
                if constexpr (FUSED) {
                    const rsrc_t fh = plane_rsrc(fwd, zn, plane, pbytes);
#pragma unroll
                    for (int h = 0; h < NYH; ++h) nfy[h] = ldb(fh, hyo[h]);
#pragma unroll
                    for (int h = 0; h < NXH; ++h) nfx[h] = ldb(fh, hxo[h]);
                }
            }
            if (ahead) {
                const rsrc_t pq = plane_rsrc(cur, zf, plane, pbytes);
                const rsrc_t pk = plane_rsrc(kap, za, plane, pbytes);
                const rsrc_t pp = plane_rsrc(prv, za, plane, pbytes);
#pragma unroll
                for (int i = 0; i < RY; ++i) {
                    q[i][fs] = ldb(pq, roff[i]);
                    kv[cn][i] = ldb_stream(pk, roff[i]);
                    pv[cn][i] = ldb_stream(pp, roff[i]);
                }
                if constexpr (HQ) {
#pragma unroll
                    for (int h = 0; h < NYH; ++h) hy[h][fs] = ldb(pq, hyo[h]);
#pragma unroll
                    for (int h = 0; h < NXH; ++h) hx[h][fs] = ldb(pq, hxo[h]);
                }
                if constexpr (FUSED) {
                    const rsrc_t fq = plane_rsrc(fwd, zf, plane, pbytes);
                    const rsrc_t pg = plane_rsrc(grad, za, plane, pbytes);
#pragma unroll
                    for (int i = 0; i < RY; ++i) {
                        f[i][fs] = ldb(fq, roff[i]);
                        gv[cn][i] = accum ? ldb_stream(pg, roff[i]) : 0.f;
                    }
                }
            }
            // ---- plane z (queue slot (k + M + m) % U holds plane z + dir m)
            const float *L = sp + (ii & 1) * LS;
            const float *LF = FUSED ? sf + (ii & 1) * LS : nullptr;
            const rsrc_t po = plane_rsrc(out, z + M, plane, pbytes);
            const rsrc_t pg = plane_rsrc(grad, z + M, plane, pbytes);
            const int dz = sponge_depth(z, nz, nb);
            float res[RY];
#pragma unroll
            for (int i = 0; i < RY; ++i) {
                const int ly = M + wv * RY + i, lx = M + lane;
                const float pc = q[i][(k + M) % U];
                float acc = 0.f;
#pragma unroll
                for (int m = M; m > KD; --m) {
                    const float t = (L[ly * LX + lx + m] + L[ly * LX + lx - m]) +
                                    (L[(ly + m) * LX + lx] + L[(ly - m) * LX + lx]) +
                                    (q[i][(k + M + m) % U] + q[i][(k + M - m) % U]);
                    acc = fmaf(W.c[m], t, acc);
                }
                if constexpr (KD < M) acc = fmaf(W.t3[KD], pc, acc);
#pragma unroll
                for (int m = KD; m >= 1; --m) {
                    const float d = ((L[ly * LX + lx + m] - pc) + (L[ly * LX + lx - m] - pc)) +
                                    ((L[(ly + m) * LX + lx] - pc) + (L[(ly - m) * LX + lx] - pc)) +
                                    ((q[i][(k + M + m) % U] - pc) + (q[i][(k + M - m) % U] - pc));
                    acc = fmaf(W.c[m], d, acc);
                }
                // imaging: g + psi^{k+1} * L'p^k (kv holds g, pv psi^{k+1}),
                // the same operation as the fused kernel's
                res[i] = IMG ? fmaf(pv[c][i], acc, kv[c][i]) : fmaf(kv[c][i], acc, 2.f * pc);
            }
            if (src_blk && z == J->src_z) {
#pragma unroll
                for (int i = 0; i < RY; ++i) res[i] += i == src_row ? srcv : 0.f;
            }
#pragma unroll
            for (int i = 0; i < RY; ++i) {
                if constexpr (IMG)
                    stb_stream(po, soff[i], res[i]);
                else
                    stb_stream(po, soff[i], leapfrog(res[i], pv[c][i], dxy2[i] + dz * dz, eta_dt));
            }
            if constexpr (FUSED) {
                if (accum) {
#pragma unroll
                    for (int i = 0; i < RY; ++i) {
                        const int ly = M + wv * RY + i, lx = M + lane;
                        const float fc = f[i][(k + M) % U];
                        float lf = 0.f;
#pragma unroll
                        for (int m = M; m > KD; --m) {
                            const float t = (LF[ly * LX + lx + m] + LF[ly * LX + lx - m]) +
                                            (LF[(ly + m) * LX + lx] + LF[(ly - m) * LX + lx]) +
                                            (f[i][(k + M + m) % U] + f[i][(k + M - m) % U]);
                            lf = fmaf(W.c[m], t, lf);
                        }
                        if constexpr (KD < M) lf = fmaf(W.t3[KD], fc, lf);
#pragma unroll
                        for (int m = KD; m >= 1; --m) {
                            const float d =
                                ((LF[ly * LX + lx + m] - fc) + (LF[ly * LX + lx - m] - fc)) +
                                ((LF[(ly + m) * LX + lx] - fc) + (LF[(ly - m) * LX + lx] - fc)) +
                                ((f[i][(k + M + m) % U] - fc) + (f[i][(k + M - m) % U] - fc));
                            lf = fmaf(W.c[m], d, lf);
                        }
                        stb_stream(pg, soff[i], fmaf(q[i][(k + M) % U], lf, gv[c][i]));
                    }
                }
            }
            // ---- stage plane z+dir in the other LDS buffer
            if (more) {
                float *Ln = sp + ((ii + 1) & 1) * LS;
                float *LFn = FUSED ? sf + ((ii + 1) & 1) * LS : nullptr;
#pragma unroll
                for (int i = 0; i < RY; ++i) {
                    Ln[(M + wv * RY + i) * LX + M + lane] = q[i][(k + M + 1) % U];
                    if constexpr (FUSED)
                        LFn[(M + wv * RY + i) * LX + M + lane] = f[i][(k + M + 1) % U];
                }
#pragma unroll
                for (int h = 0; h < NYH; ++h)
                    if (hyl[h] >= 0) {
                        if constexpr (HQ) Ln[hyl[h]] = hy[h][(k + M + 1) % U];
                        else Ln[hyl[h]] = nhy[h];
                        if constexpr (FUSED) LFn[hyl[h]] = nfy[h];
                    }
#pragma unroll
                for (int h = 0; h < NXH; ++h)
                    if (hxl[h] >= 0) {
                        if constexpr (HQ) Ln[hxl[h]] = hx[h][(k + M + 1) % U];
                        else Ln[hxl[h]] = nhx[h];
                        if constexpr (FUSED) LFn[hxl[h]] = nfx[h];
                    }
            }
            lds_barrier();
    };
    int ib = 0;
    for (; ib + U - 1 + D < npl; ib += U)
        static_for<0, U>([&](auto K) __attribute__((always_inline)) {
            step_plane(K, ib + decltype(K)::value, true, true);
        });
    static_for<0, U>([&](auto K) __attribute__((always_inline)) {
        const int ii = ib + decltype(K)::value;
        if (ii < npl) step_plane(K, ii, ii + 1 < npl, ii + D < npl);
    });
}
// The 16th-order adjoint runs as two single-field passes (imaging condition,
// then the psi update): the fused kernel carries two 17-plane queues in
// more registers than fit 2 waves per SIMD, each pass one queue.  Both
// compute bitwise the same values.  At 8th order the fused kernel is as
// fast as the two passes and stays; FWI_SPLIT_ADJ=1 selects the two passes
// there too.
template <int M>
static bool split_adjoint()
{
    if constexpr (M >= 8) {
        return true;
    } else if constexpr (M == 4) {
        const char *e = getenv("FWI_SPLIT_ADJ");
        return e && atoi(e) != 0;
    } else {
        return false;
    }
}

template <int M, int NW, int RY>
static void launch_3d(bool adj, const Job *jobs, const int *prefix, int njobs, int step,
                      int ttiles, int grid, int remap, const LevelMap &lm, hipStream_t st)
{
    const dim3 g(grid), b(64 * NW);
    if (!adj) {
        hipLaunchKernelGGL((k_step3d<M, kFwd, NW, RY>), g, b, 0, st, jobs, prefix, njobs, step,
                           ttiles, remap, lm);
        return;
    }
    if constexpr (M >= 4) {
        if (split_adjoint<M>()) {
            // the imaging pass reads psi^{k+1} and p^k, which the psi pass leaves intact
            hipLaunchKernelGGL((k_step3d<M, kImage, NW, RY>), g, b, 0, st, jobs, prefix, njobs,
                               step, ttiles, remap, lm);
            hipLaunchKernelGGL((k_step3d<M, kAdjPsi, NW, RY>), g, b, 0, st, jobs, prefix, njobs,
                               step, ttiles, remap, lm);
            return;
        }
    }
    if constexpr (M < 8)
        hipLaunchKernelGGL((k_step3d<M, kAdj, NW, RY>), g, b, 0, st, jobs, prefix, njobs, step,
                           ttiles, remap, lm);
}

template <int M, int NW, int RY>
static hipError_t occupancy_3d(int *n, bool adj)
{
    const int t = 64 * NW;
    if (!adj) return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, k_step3d<M, kFwd, NW, RY>, t, 0);
    if constexpr (M >= 4) {
        if (split_adjoint<M>()) {
            int a = 0, c = 0;
            hipError_t e =
                hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, k_step3d<M, kAdjPsi, NW, RY>, t, 0);
            if (e == hipSuccess)
                e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&c, k_step3d<M, kImage, NW, RY>, t, 0);
            *n = a < c ? a : c;
            return e;
        }
    }
    if constexpr (M < 8)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, k_step3d<M, kAdj, NW, RY>, t, 0);
    return hipErrorInvalidValue;
}

#define FWI_CAT_(a, b) a##b
#define FWI_CAT(a, b) FWI_CAT_(a, b)

void FWI_CAT(launch_step3d_m, FWI_STEP3D_M)(int nw, bool adj, const Job *jobs, const int *prefix,
                                            int njobs, int step, int ttiles, int grid, int remap,
                                            const LevelMap &lm, hipStream_t st)
{
    constexpr int M = FWI_STEP3D_M;
    switch (nw) {   // wavefronts per block x rows per thread
    case 8: launch_3d<M, 8, 4>(adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    case 42: launch_3d<M, 4, 2>(adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    case 82: launch_3d<M, 8, 2>(adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    default: launch_3d<M, 4, 4>(adj, jobs, prefix, njobs, step, ttiles, grid, remap, lm, st); break;
    }
}

hipError_t FWI_CAT(occupancy_step3d_m, FWI_STEP3D_M)(int nw, bool adj, int *n)
{
    constexpr int M = FWI_STEP3D_M;
    if (nw == 8) return occupancy_3d<M, 8, 4>(n, adj);
    if (nw == 42) return occupancy_3d<M, 4, 2>(n, adj);
    if (nw == 82) return occupancy_3d<M, 8, 2>(n, adj);
    return occupancy_3d<M, 4, 4>(n, adj);
}

}  // namespace fwi
