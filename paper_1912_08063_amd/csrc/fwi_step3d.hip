// fwi_step3d.hip -- the 3-D step kernels (see fwi_kernels.hip for the design).
// Compiled once per stencil radius, FWI_STEP3D_M = 1, 2, 4 or 8, so that the
// radii build in parallel.
#include "fwi_device.h"

#include <stdlib.h>

namespace fwi {

// --------------------------------------------------------------- 3-D step
// Step modes: the forward step; the adjoint step with the imaging condition
// fused in (two stencil fields); and the adjoint as two single-field passes,
// the psi update alone and the imaging condition g += psi^{k+1} * L'p^k
// alone, each with the forward step's memory pattern (see launch_3d).
enum StepMode { kFwd = 0, kAdj = 1, kAdjPsi = 2, kImage = 3 };

typedef float vf4 __attribute__((ext_vector_type(4)));
typedef unsigned vu4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ vf4 ldb4(rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(vf4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ __forceinline__ vf4 ldb4_stream(rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(vf4,
                              __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, kStreamPolicy));
}
__device__ __forceinline__ void stb4_stream(rsrc_t r, uint32_t off, vf4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(vu4, v), r, (int)off, 0,
                                           kStreamPolicy);
}

// Stencil sums of a thread's four columns: L is its place in the staged plane
// (rows LX apart), z(d) its column's plane d planes ahead.
template <int M, int LX, class Z>
__device__ __forceinline__ vf4 star3d(const float *L, Z z)
{
    constexpr Weights<M> W{};
    constexpr int XH = (M + 3) / 4 * 4, KD = kDiffRadii < M ? kDiffRadii : M;
    const vf4 pc = z(Int<0>{});
    float xr[4 + 2 * XH];
#pragma unroll
    for (int c = 0; c < XH; c += 4) {
        const vf4 a = *reinterpret_cast<const vf4 *>(L - XH + c);
        const vf4 d = *reinterpret_cast<const vf4 *>(L + 4 + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) { xr[c + e] = a[e]; xr[XH + 4 + c + e] = d[e]; }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) xr[XH + c] = pc[c];
    vf4 acc = {0.f, 0.f, 0.f, 0.f};
    static_for<0, M>([&](auto I) __attribute__((always_inline)) {
        constexpr int m = M - decltype(I)::value;
        const vf4 yp = *reinterpret_cast<const vf4 *>(L + m * LX);
        const vf4 ym = *reinterpret_cast<const vf4 *>(L - m * LX);
        const vf4 zp = z(Int<m>{}), zm = z(Int<-m>{});
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float xp = xr[XH + c + m], xm = xr[XH + c - m], p = pc[c];
            if constexpr (m == KD && KD < M) acc[c] = fmaf(W.t3[KD], p, acc[c]);
            const float t = m > KD ? (xp + xm) + (yp[c] + ym[c]) + (zp[c] + zm[c])
                                   : ((xp - p) + (xm - p)) + ((yp[c] - p) + (ym[c] - p)) +
                                         ((zp[c] - p) + (zm[c] - p));
            acc[c] = fmaf(W.c[m], t, acc[c]);
        }
    });
    return acc;
}

// 3-D step by z-marching: a block of 16 x 16 threads owns a 64 (x) x 16 (y)
// column of the grid over a chunk of z planes, a thread four columns of one row.
// Its z-queue is a register queue of 2M + 2 planes indexed by the unrolled phase
// (plane j of the chunk in slot (j + M) mod U), so no register is copied after a
// load; the current plane with its M-cell halo is in LDS (double-buffered), and
// the next plane's loads (queue front, halo, kappa', previous level) are in
// flight while a plane is computed; one LDS-only barrier per plane.
//
// All memory and LDS accesses are 16 bytes per lane: a thread's four cells take
// 10 LDS reads (M = 4; one column of four rows per thread, the earlier form,
// took 44 of 4 bytes, and 188 registers with its halo queue), at 111 registers:
// 4 waves per SIMD.  304^3 padded grid, us per step: 8th order forward 82.5 ->
// 74.5 (6.0 TB/s at 16 B per cell), 16th order 97.3 -> 86.8, 8th-order fused
// adjoint with its source 188 -> 175, 560 x 560 x 304 forward 319 -> 294.  A
// halo queue loaded with the queue front (146 registers, 3 waves per SIMD): 77.6;
// capped at 128 registers (spills): 84; the queue front non-temporal: 84.
//
// The adjoint adds its source itself: the bounds of each plane's receivers are
// read where the chunk holds any.
template <int M, int MODE>
__global__ __launch_bounds__(256) void k_step3d(const Job *__restrict__ jobs,
                                                     const int *__restrict__ prefix, int njobs,
                                                     int step, int ttiles, int remap, LevelMap lm)
{
    constexpr int TX = kTileX, TY = kTile3dRows, NT = 256;
    constexpr int XH = (M + 3) / 4 * 4, LX = TX + 2 * XH, LY = TY + 2 * M, LS = LX * LY;
    constexpr int HY = 2 * M * (TX / 4), HX = TY * (XH / 2);   // halo quads: rows, columns
    constexpr int NH = (HY + HX + NT - 1) / NT;
    constexpr int Q = 2 * M + 1, U = Q + 1;
    constexpr bool ADJ = MODE != kFwd, FUSED = MODE == kAdj, IMG = MODE == kImage;
    constexpr bool INJ = MODE == kAdj || MODE == kAdjPsi;
    __shared__ __align__(16) float sp[2 * LS];
    __shared__ __align__(16) float sf[FUSED ? 2 * LS : 4];
    __shared__ __align__(16) float sinj[INJ ? TX * TY : 4];

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
    const int j = njobs > 1 ? find_job(prefix, njobs, b) : 0;
    const Job *__restrict__ J = jobs + j;
    const int n = step_level(J, step, ADJ);
    if (ADJ ? (n < J->adj_lo || n >= J->adj_hi) : (n < J->fwd_lo || n >= J->fwd_hi)) return;
    const int nz = J->nz, ny = J->ny, nx = J->nx, pitch = J->pitch, nb = J->nb;
    const int64_t plane = J->plane, fstride = J->fstride;
    const Job::Tiling &T = J->tile[ADJ ? 1 : 0];
    int local = b - (njobs > 1 ? prefix[j] : 0);
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

    // ---- per-thread geometry (loop invariant).  Loads are unconditional: rows
    // past the frame are clamped to it (zeros); stores of rows outside the grid
    // are dropped, and columns outside it hold and store zeros.
    const int lx = 4 * (tid & 15), ry = tid >> 4;
    const int col = tx * TX + lx, yy = ty * TY + ry;
    const int last_row = ny + 2 * M - 1;
    const uint32_t roff = 4u * (uint32_t)(min(yy + M, last_row) * pitch + col);
    const uint32_t soff = yy < ny ? roff : kDropOffset;
    const int lo = (M + ry) * LX + XH + lx;   // this thread's place in an LDS plane
    uint32_t ho[NH];
    int hl[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const int e = tid + NT * h;
        ho[h] = kDropOffset;
        hl[h] = -1;
        if (e < HY) {   // rows above and below the tile
            const int r = e / (TX / 4), c = e % (TX / 4) * 4, ly = r < M ? r : r + TY;
            ho[h] = 4u * (uint32_t)(min(ty * TY + ly, last_row) * pitch + tx * TX + c);
            hl[h] = ly * LX + XH + c;
        } else if (e < HY + HX) {   // columns left and right of it
            const int g = e - HY, r = g / (XH / 2), c = g % (XH / 2) * 4, lc = c < XH ? c : c + TX;
            ho[h] = 4u * (uint32_t)(min(ty * TY + r + M, last_row) * pitch +
                                    min(max(tx * TX - XH + lc, 0), pitch - 4));
            hl[h] = (M + r) * LX + lc;
        }
    }
    // sponge: squared depth in the plane, and its factors there (leapfrog's with
    // dz = 0; 1 and 1 in the model, where they give val - prev bit for bit)
    int dxy2[4];
    vf4 sa, sb;
    const int dy = sponge_depth(yy, ny, nb);
    bool edge = false;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int dx = sponge_depth(col + c - M, nx, nb);
        dxy2[c] = dx * dx + dy * dy;
        edge = edge || dxy2[c] != 0;
        sa[c] = __builtin_amdgcn_rcpf(fmaf(eta_dt, (float)dxy2[c], 1.f));
        sb[c] = fmaf(-eta_dt, (float)dxy2[c], 1.f);
    }
    const bool wedge = __any(edge);
    // source (forward): the block that owns it adds it at its plane
    const bool src_blk = !ADJ && J->src_x >= tx * TX - M && J->src_x < tx * TX - M + TX &&
                         J->src_y >= ty * TY && J->src_y < ty * TY + TY && J->src_z >= z0 &&
                         J->src_z < z1;
    const int src_z = src_blk ? J->src_z : -1;
    float srcv = 0.f;
    int sc = -1;
    if (src_blk && J->src_y == yy) {
        sc = J->src_x + M - col;   // 0..3: this thread's column
        srcv = J->src_scale * J->wavelet[n];
    }
    // adjoint source: the receivers of the tile in each plane
    const GMEM int32_t *bounds = nullptr;
    if constexpr (INJ)
        if (J->rec_z0 < z1 && J->rec_z1 > z0)
            bounds = (const GMEM int32_t *)J->rt_start + (int64_t)(tx * T.nty + ty) * nz;

    auto pl = [&](const gfloat *f, int zmem) __attribute__((always_inline)) {
        return plane_rsrc(f, zmem, plane, pbytes);
    };
    vf4 q[U], f[FUSED ? U : 1];
    vf4 kv[2], pv[2], gv[FUSED ? 2 : 1];
    // chunk planes -M .. M
#pragma unroll
    for (int s = 0; s < Q; ++s) {
        q[s] = ldb4(pl(cur, zs + dir * (s - M) + M), roff);
        if constexpr (FUSED) f[s] = ldb4(pl(fwd, zs + dir * (s - M) + M), roff);
    }
    kv[0] = ldb4(pl(kap, zs + M), roff);
    pv[0] = ldb4(pl(prv, zs + M), roff);
    if constexpr (FUSED) {
        gv[0] = vf4{0.f, 0.f, 0.f, 0.f};
        if (accum) gv[0] = ldb4(pl(grad, zs + M), roff);
    }
    *reinterpret_cast<vf4 *>(sp + lo) = q[M];
    if constexpr (FUSED) *reinterpret_cast<vf4 *>(sf + lo) = f[M];
#pragma unroll
    for (int h = 0; h < NH; ++h)
        if (hl[h] >= 0) {
            *reinterpret_cast<vf4 *>(sp + hl[h]) = ldb4(pl(cur, zs + M), ho[h]);
            if constexpr (FUSED)
                *reinterpret_cast<vf4 *>(sf + hl[h]) = ldb4(pl(fwd, zs + M), ho[h]);
        }
    lds_barrier();

    // Plane ii of the chunk; k = ii % U selects the slots.  more: a plane follows
    // it.
    auto step_plane = [&](auto K, const int ii, const bool more) __attribute__((always_inline)) {
        constexpr int k = decltype(K)::value, c = k & 1, cn = c ^ 1;   // U is even
        constexpr int fs = (k + Q) % U;   // free queue slot: chunk plane ii+M+1
        const int z = zs + dir * ii;
        vf4 nh[NH], nf[FUSED ? NH : 1];
        if (more) {
            const rsrc_t ph = pl(cur, z + dir + M);
#pragma unroll
            for (int h = 0; h < NH; ++h) nh[h] = ldb4(ph, ho[h]);
            if constexpr (FUSED) {
                const rsrc_t fh = pl(fwd, z + dir + M);
#pragma unroll
                for (int h = 0; h < NH; ++h) nf[h] = ldb4(fh, ho[h]);
            }
            q[fs] = ldb4(pl(cur, z + dir * (1 + M) + M), roff);
            kv[cn] = ldb4_stream(pl(kap, z + dir + M), roff);
            pv[cn] = ldb4_stream(pl(prv, z + dir + M), roff);
            if constexpr (FUSED) {
                f[fs] = ldb4(pl(fwd, z + dir * (1 + M) + M), roff);
                gv[cn] = ldb4_stream(pl(grad, z + dir + M), roff);
            }
        }
        const float *L = sp + (ii & 1) * LS + lo;
        const rsrc_t po = pl(out, z + M);
        const vf4 acc = star3d<M, LX>(L, [&](auto D) __attribute__((always_inline)) {
            return q[(k + M + decltype(D)::value + U) % U];
        });
        vf4 o;
        if constexpr (IMG) {
            // g + psi^{k+1} * L'p^k (kv holds g, pv psi^{k+1})
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(pv[c][e], acc[e], kv[c][e]);
        } else {
            const vf4 pc = q[(k + M) % U];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(kv[c][e], acc[e], 2.f * pc[e]);
            if (!ADJ && z == src_z) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] += e == sc ? srcv : 0.f;
            }
            const int dz = sponge_depth(z, nz, nb);
            if (dz != 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = leapfrog(o[e], pv[c][e], dxy2[e] + dz * dz, eta_dt);
            } else if (wedge) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = sa[e] * fmaf(-sb[e], pv[c][e], o[e]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = o[e] - pv[c][e];
            }
            if constexpr (INJ) {
                if (bounds) {
                    const int e0 = bounds[z], e1 = bounds[z + 1];
                    if (e0 < e1) {
                        *reinterpret_cast<vf4 *>(sinj + ry * TX + lx) = vf4{0.f, 0.f, 0.f, 0.f};
                        lds_barrier();
                        for (int e = e0 + tid; e < e1; e += NT) {
                            const int key = J->rt_key[e];
                            sinj[((key >> 6) & (TY - 1)) * TX + (key & 63)] =
                                adj_source(J, n, J->rt_rec[e]);
                        }
                        lds_barrier();
                        const vf4 s = *reinterpret_cast<const vf4 *>(sinj + ry * TX + lx);
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = fmaf(kv[c][e], s[e], o[e]);
                    }
                }
            }
        }
        stb4_stream(po, soff, o);
        if constexpr (FUSED) {
            if (accum) {
                const vf4 lf = star3d<M, LX>(sf + (ii & 1) * LS + lo,
                                             [&](auto D) __attribute__((always_inline)) {
                                                 return f[(k + M + decltype(D)::value + U) % U];
                                             });
                const vf4 pc = q[(k + M) % U];
                vf4 g;
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] = fmaf(pc[e], lf[e], gv[c][e]);
                stb4_stream(pl(grad, z + M), soff, g);
            }
        }
        // ---- stage the next plane in the other LDS buffer
        if (more) {
            float *Ln = sp + ((ii + 1) & 1) * LS, *LFn = sf + (FUSED ? ((ii + 1) & 1) * LS : 0);
            *reinterpret_cast<vf4 *>(Ln + lo) = q[(k + M + 1) % U];
            if constexpr (FUSED) *reinterpret_cast<vf4 *>(LFn + lo) = f[(k + M + 1) % U];
#pragma unroll
            for (int h = 0; h < NH; ++h)
                if (hl[h] >= 0) {
                    *reinterpret_cast<vf4 *>(Ln + hl[h]) = nh[h];
                    if constexpr (FUSED) *reinterpret_cast<vf4 *>(LFn + hl[h]) = nf[h];
                }
        }
        lds_barrier();
    };
    int ib = 0;
    for (; ib + U < npl; ib += U)
        static_for<0, U>([&](auto K) __attribute__((always_inline)) {
            step_plane(K, ib + decltype(K)::value, true);
        });
    static_for<0, U>([&](auto K) __attribute__((always_inline)) {
        const int ii = ib + decltype(K)::value;
        if (ii < npl) step_plane(K, ii, ii + 1 < npl);
    });
}

// 3-D step without marching, for grids that cannot fill the GPU with long
// z-chunks: a block owns 64 x TY x ZB cells, a thread four columns of one row in
// ZB planes.  All its loads are issued at once -- its columns' ZB + 2M planes,
// kappa', the previous level (and p^k, g) and the halo of the ZB planes, which
// are staged in LDS for the x and y neighbours -- so a launch costs one round of
// load latency and one barrier instead of 2M warm-up planes and a serial plane
// loop, with 16-byte loads.  z is the fastest tile index: the planes that
// neighbouring blocks share are read at the same time on one XCD.  Two planes a
// block: a launch is bound by its latency, and more, smaller blocks hide it better
// than fewer reads of the shared planes (112^3 padded cells, 8th order, us per
// step: 1 plane 9.5, 2 planes 8.4, 3 8.9, 4 9.0, 6 11.2).  The
// arithmetic is k_step3d's, term by term.  The adjoint is fused and adds the
// adjoint source itself, from the receivers of each 64 x TY x 1 slice.
template <int M, bool ADJ>
__global__ __launch_bounds__(kTile3dThreads) void k_step3d_tile(
    const Job *__restrict__ jobs, const int *__restrict__ prefix, int njobs, int step, int ttiles,
    int remap, LevelMap lm)
{
    constexpr int TX = kTileX, TY = kTile3dRows, ZB = kTile3dPlanes, NT = kTile3dThreads;
    constexpr int XH = (M + 3) / 4 * 4, LX = TX + 2 * XH, LY = TY + 2 * M, LP = LX * LY;
    constexpr int NQ = ZB + 2 * M;                       // planes of a column
    constexpr int HY = 2 * M * (TX / 4), HX = TY * (2 * XH / 4);   // halo quads per plane
    constexpr int NYH = (HY * ZB + NT - 1) / NT, NXH = (HX * ZB + NT - 1) / NT;
    static_assert(NT == TX / 4 * TY, "one thread per quad of a plane");
    __shared__ __align__(16) float sp[ZB * LP];
    __shared__ __align__(16) float sf[ADJ ? ZB * LP : 4];

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
    const int j = njobs > 1 ? find_job(prefix, njobs, b) : 0;
    const Job *__restrict__ J = jobs + j;
    const int n = step_level(J, step, ADJ);
    if (ADJ ? (n < J->adj_lo || n >= J->adj_hi) : (n < J->fwd_lo || n >= J->fwd_hi)) return;
    const int nz = J->nz, ny = J->ny, nx = J->nx, pitch = J->pitch, nb = J->nb;
    const int64_t plane = J->plane, fstride = J->fstride;
    const Job::Tiling &T = J->tile[ADJ ? 1 : 0];
    int local = b - (njobs > 1 ? prefix[j] : 0);
    const int nzc = T.nzc, ntx = T.ntx, tz = local % nzc;
    local /= nzc;
    const int ty = local / ntx, tx = local - ty * ntx;
    const int z0 = tz * ZB;

    const gfloat *cur, *prv, *fwd = nullptr;
    gfloat *out;
    bool accum = false;
    if constexpr (ADJ) {
        cur = gptr(J->adj) + (int64_t)((n + 1) & 1) * fstride;
        prv = gptr(J->adj) + (int64_t)(n & 1) * fstride;
        out = gptr(J->adj) + (int64_t)(n & 1) * fstride;
        accum = J->accumulate && n <= J->nt - 1;
        fwd = gptr(level_ptr(J, lm, n));
    } else {
        cur = gptr(level_ptr(J, lm, n));
        prv = gptr(level_ptr(J, lm, n - 1));
        out = gptr(level_ptr(J, lm, n + 1));
    }
    const gfloat *kap = gptr(J->kappa);
    gfloat *grad = gptr(J->grad);
    const float eta_dt = J->eta_dt;
    const int pbytes = (int)(plane * (int64_t)sizeof(float));

    const int qx = tid & 15, ry = tid >> 4, lx = 4 * qx;
    const int col = tx * TX + lx, yy = ty * TY + ry;
    const int last_row = ny + 2 * M - 1, last_plane = nz + 2 * M - 1;
    // rows past the frame and planes past it are clamped to it (zeros)
    const uint32_t roff = 4u * (uint32_t)(min(yy + M, last_row) * pitch + col);
    const uint32_t soff = yy < ny ? roff : kDropOffset;
    auto pl = [&](const gfloat *f, int zmem) __attribute__((always_inline)) {
        return plane_rsrc(f, min(zmem, last_plane), plane, pbytes);
    };
    vf4 q[NQ], kv[ZB], pv[ZB], f[ADJ ? NQ : 1], gv[ADJ ? ZB : 1];
    // the staged planes first, then the halos, then the rest
#pragma unroll
    for (int i = 0; i < ZB; ++i) q[M + i] = ldb4(pl(cur, z0 + M + i), roff);
    vf4 hy[NYH], hx[NXH], fy[ADJ ? NYH : 1], fx[ADJ ? NXH : 1];
    int hyl[NYH], hxl[NXH];
    // a halo quad's plane differs between the lanes of a wave, so its address is
    // one 64-bit pointer per lane
    auto ldh = [&](const gfloat *fld, int i, int row, int c) __attribute__((always_inline)) {
        const int zm = min(z0 + M + i, last_plane);
        typedef GMEM vf4 gvf4;
        return *reinterpret_cast<const gvf4 *>(fld + (int64_t)zm * plane +
                                               (min(row, last_row) * pitch + c));
    };
#pragma unroll
    for (int h = 0; h < NYH; ++h) {   // rows above and below the tile
        const int e = tid + NT * h, i = e / HY, r = e % HY / (TX / 4), c = e % (TX / 4) * 4;
        const int ly = r < M ? r : r + TY;
        hyl[h] = i < ZB ? i * LP + ly * LX + XH + c : -1;
        if (i < ZB) {
            hy[h] = ldh(cur, i, ty * TY + ly, tx * TX + c);
            if constexpr (ADJ) fy[h] = ldh(fwd, i, ty * TY + ly, tx * TX + c);
        }
    }
#pragma unroll
    for (int h = 0; h < NXH; ++h) {   // columns left and right of it
        const int e = tid + NT * h, i = e / HX, r = e % HX / (2 * XH / 4), c = e % (2 * XH / 4) * 4;
        const int lc = c < XH ? c : c + TX;   // LDS column
        const int cm = min(max(tx * TX - XH + lc, 0), pitch - 4);
        hxl[h] = i < ZB ? i * LP + (M + r) * LX + lc : -1;
        if (i < ZB) {
            hx[h] = ldh(cur, i, ty * TY + r + M, cm);
            if constexpr (ADJ) fx[h] = ldh(fwd, i, ty * TY + r + M, cm);
        }
    }
    if constexpr (ADJ) {
#pragma unroll
        for (int i = 0; i < ZB; ++i) f[M + i] = ldb4(pl(fwd, z0 + M + i), roff);
    }
#pragma unroll
    for (int i = 0; i < M; ++i) {
        q[i] = ldb4(pl(cur, z0 + i), roff);
        q[M + ZB + i] = ldb4(pl(cur, z0 + M + ZB + i), roff);
    }
#pragma unroll
    for (int i = 0; i < ZB; ++i) {
        kv[i] = ldb4(pl(kap, z0 + M + i), roff);
        pv[i] = ldb4(pl(prv, z0 + M + i), roff);
    }
    if constexpr (ADJ) {
#pragma unroll
        for (int i = 0; i < M; ++i) {
            f[i] = ldb4(pl(fwd, z0 + i), roff);
            f[M + ZB + i] = ldb4(pl(fwd, z0 + M + ZB + i), roff);
        }
#pragma unroll
        for (int i = 0; i < ZB; ++i) gv[i] = ldb4(pl(grad, z0 + M + i), roff);
    }
    // source (forward)
    const bool src_blk = !ADJ && J->src_x >= tx * TX - M && J->src_x < tx * TX - M + TX &&
                         J->src_y >= ty * TY && J->src_y < ty * TY + TY && J->src_z >= z0 &&
                         J->src_z < z0 + ZB;
    float srcv = 0.f;
    int sc = -1;
    if (src_blk && J->src_y == yy) {
        sc = J->src_x + M - col;   // 0..3: this thread's column
        srcv = J->src_scale * J->wavelet[n];
    }
    int dx2[4];
    const int dy = sponge_depth(yy, ny, nb);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int dx = sponge_depth(col + c - M, nx, nb);
        dx2[c] = dx * dx + dy * dy;
    }
    // receivers of the block's slices (adjoint)
    int e0 = 0, e1 = 0;
    if constexpr (ADJ) {
        if (J->rec_z0 < z0 + ZB && J->rec_z1 > z0) {
            const int bin = (tx * T.nty + ty) * nz;
            e0 = J->rt_start[bin + z0];
            e1 = J->rt_start[bin + min(z0 + ZB, nz)];
        }
    }

    const int lo = (M + ry) * LX + XH + lx;   // this thread's place in an LDS plane
#pragma unroll
    for (int i = 0; i < ZB; ++i) {
        *reinterpret_cast<vf4 *>(sp + i * LP + lo) = q[M + i];
        if constexpr (ADJ) *reinterpret_cast<vf4 *>(sf + i * LP + lo) = f[M + i];
    }
#pragma unroll
    for (int h = 0; h < NYH; ++h)
        if (hyl[h] >= 0) {
            *reinterpret_cast<vf4 *>(sp + hyl[h]) = hy[h];
            if constexpr (ADJ) *reinterpret_cast<vf4 *>(sf + hyl[h]) = fy[h];
        }
#pragma unroll
    for (int h = 0; h < NXH; ++h)
        if (hxl[h] >= 0) {
            *reinterpret_cast<vf4 *>(sp + hxl[h]) = hx[h];
            if constexpr (ADJ) *reinterpret_cast<vf4 *>(sf + hxl[h]) = fx[h];
        }
    lds_barrier();

    auto st4 = [&](gfloat *fld, int i, vf4 v) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_buffer_store_b128(
            __builtin_bit_cast(vu4, v), plane_rsrc(fld, z0 + M + i, plane, pbytes),
            (int)(z0 + i < nz ? soff : kDropOffset), 0, 0);
    };
    vf4 o[ZB];
    static_for<0, ZB>([&](auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        const vf4 acc = star3d<M, LX>(sp + i * LP + lo, [&](auto D) __attribute__((always_inline)) {
            return q[M + i + decltype(D)::value];
        });
        const int dz = sponge_depth(z0 + i, nz, nb);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float r = fmaf(kv[i][c], acc[c], 2.f * q[M + i][c]);
            if (src_blk && z0 + i == J->src_z) r += c == sc ? srcv : 0.f;
            o[i][c] = leapfrog(r, pv[i][c], dx2[c] + dz * dz, eta_dt);
        }
        if constexpr (!ADJ) st4(out, i, o[i]);
    });
    if constexpr (ADJ) {
        if (accum) {
            static_for<0, ZB>([&](auto I) __attribute__((always_inline)) {
                constexpr int i = decltype(I)::value;
                const vf4 lf = star3d<M, LX>(sf + i * LP + lo, [&](auto D) __attribute__((always_inline)) {
                    return f[M + i + decltype(D)::value];
                });
                vf4 g;
#pragma unroll
                for (int c = 0; c < 4; ++c) g[c] = fmaf(q[M + i][c], lf[c], gv[i][c]);
                st4(grad, i, g);
            });
        }
        if (e0 < e1) {   // adjoint source, through the psi tile's LDS
            lds_barrier();
#pragma unroll
            for (int i = 0; i < ZB; ++i)
                *reinterpret_cast<vf4 *>(sp + i * LP + lo) = vf4{0.f, 0.f, 0.f, 0.f};
            lds_barrier();
            for (int e = e0 + tid; e < e1; e += NT) {
                const int key = J->rt_key[e];
                sp[((key >> kKeyBits3d) - z0) * LP + (M + ((key >> 6) & (TY - 1))) * LX + XH +
                   (key & 63)] = adj_source(J, n, J->rt_rec[e]);
            }
            lds_barrier();
#pragma unroll
            for (int i = 0; i < ZB; ++i) {
                const vf4 s = *reinterpret_cast<const vf4 *>(sp + i * LP + lo);
#pragma unroll
                for (int c = 0; c < 4; ++c) o[i][c] = fmaf(kv[i][c], s[c], o[i][c]);
            }
        }
#pragma unroll
        for (int i = 0; i < ZB; ++i) st4(out, i, o[i]);
    }
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

#define FWI_CAT_(a, b) a##b
#define FWI_CAT(a, b) FWI_CAT_(a, b)

void FWI_CAT(launch_step3d_m, FWI_STEP3D_M)(int nw, bool adj, const Job *jobs, const int *prefix,
                                            int njobs, int step, int ttiles, int grid, int remap,
                                            const LevelMap &lm, hipStream_t st)
{
    constexpr int M = FWI_STEP3D_M;
    const dim3 g(grid), b(kTile3dThreads);
    if (nw == kTile3dCode) {
        if (!adj)
            hipLaunchKernelGGL((k_step3d_tile<M, false>), g, b, 0, st, jobs, prefix, njobs, step,
                               ttiles, remap, lm);
        else if constexpr (M <= 4)
            hipLaunchKernelGGL((k_step3d_tile<M, true>), g, b, 0, st, jobs, prefix, njobs, step,
                               ttiles, remap, lm);
        return;
    }
    if (!adj) {
        hipLaunchKernelGGL((k_step3d<M, kFwd>), g, b, 0, st, jobs, prefix, njobs, step, ttiles,
                           remap, lm);
        return;
    }
    if constexpr (M >= 4) {
        if (split_adjoint<M>()) {
            // the imaging pass reads psi^{k+1} and p^k, which the psi pass leaves intact
            hipLaunchKernelGGL((k_step3d<M, kImage>), g, b, 0, st, jobs, prefix, njobs, step,
                               ttiles, remap, lm);
            hipLaunchKernelGGL((k_step3d<M, kAdjPsi>), g, b, 0, st, jobs, prefix, njobs, step,
                               ttiles, remap, lm);
            return;
        }
    }
    if constexpr (M < 8)
        hipLaunchKernelGGL((k_step3d<M, kAdj>), g, b, 0, st, jobs, prefix, njobs, step, ttiles,
                           remap, lm);
}

}  // namespace fwi
