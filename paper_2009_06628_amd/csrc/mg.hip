// Matrix-free multigrid-preconditioned conjugate gradients on the uniform
// grid (gfx950).  The elliptic solver is not fixed by the paper (its coupled
// system goes to Krylov solvers with ASM / algebraic-multigrid
// preconditioners, and it names matrix-free multigrid as future work); this
// is a geometric cell-centred multigrid:
//   * operator       (A x)_c = s_c x_c + sum_b cs_b(c)(x_c - x_{c-e_b})
//                                       + cs_b(c+e_b)(x_c - x_{c+e_b}),
//   * smoother       red-black Gauss-Seidel; pre-smoothing (red, black) from
//                    a zero guess, post-smoothing (black, red): the V-cycle is
//                    a symmetric positive definite preconditioner;
//   * transfers      cell-centred bilinear / trilinear prolongation P and
//                    full-weighting restriction R = P^T / 2^d;
//   * coarse levels  re-discretised: s averaged over children, face
//                    coefficients averaged over the fine faces of a coarse
//                    face and divided by 4 (spacing doubles);
//   * coarsest       explicit FP64 inverse (Gauss-Jordan, in one workgroup
//                    up to kLdsInverse cells, else by block steps of the
//                    whole chip) with a rank-one shift tau 1 1^T for the singular
//                    pressure operator.
// Launch structure (a launch costs a few microseconds whatever its size):
//   * 2D levels above kSBCells cells: two tile kernels per level, one for
//     the way down (pre-smoothing, residual, restriction) and one for the
//     way up (prolongation, black sweep, red sweep), on LDS tiles with halos;
//   * 3D levels above kSBCells cells: two kernels per level as well, columns
//     that march along z (k_down3, k_sweep3), on levels of few cells LDS tiles;
//   * all smaller levels: ONE single-workgroup kernel that holds their
//     coefficients in registers and x in LDS.
// Reductions are deterministic and fence-free: per-block partials from a
// fixed grid-stride partition, summed in a fixed order either by a
// one-workgroup finalize kernel or redundantly by every block of the kernel
// that consumes them.  PCG scalars live on the device; every iteration
// kernel returns at once when the device "done" flag is set, so the host
// launches iterations in chunks and checks the flag once per chunk.
#include <type_traits>
#include <utility>

#include "mgdev.h"
#include "solvers.h"
#include "tile2d.h"

namespace chns {

static int sb_cells() { return kSBCells; }

// Grid-stride loop over cells, XCD-contiguous
#define GRID_LOOP(N) \
    for (int c = xcd_block() * (int)blockDim.x + (int)threadIdx.x; c < (int)(N); c += (int)(gridDim.x * blockDim.x))

// Two consecutive values along x (the pair starts at an even index).
template <typename T>
struct Pair2 {
    T v[2];
};

// ---------------------------------------------------------------------------
// 2D tile kernels of the grid levels (bodies in tile2d.h); tiles along x
// ---------------------------------------------------------------------------
template <typename T, typename TB>
__global__ void __launch_bounds__(kTileThreads) k_down_tile2(Level<T> L, Geo gc, const TB *__restrict__ b,
                                                             T *__restrict__ xs, T *__restrict__ bc, int ntx,
                                                             int ntiles, const int *__restrict__ done) {
    const int tile = xcd_block();
    if (tile >= ntiles) return;
    const int ty = tile / ntx, tx = tile - ty * ntx;
    down_tile2<T, kTileThreads>(L, gc, RhsStored<TB>{b}, xs, bc, tx, ty, *done);
}

template <typename T, typename TB>
__global__ void __launch_bounds__(kTileThreads) k_up_tile2(Level<T> L, Geo gc, const T *__restrict__ xc,
                                                           const TB *__restrict__ b, const T *__restrict__ xs,
                                                           T *__restrict__ x, int ntx, int ntiles,
                                                           const int *__restrict__ done) {
    const int tile = xcd_block();
    if (tile >= ntiles) return;
    const int ty = tile / ntx, tx = tile - ty * ntx;
    up_tile2<T, kTileThreads>(L, gc, xc, RhsStored<TB>{b}, xs, x, tx, ty, *done);
}

// Level 0 of the preconditioner of CG iteration k, fused with the update
// that precedes it: alpha = rz / p.q (every block sums the apply's partials
// in the same order), x += alpha p on the tile's cells, the partial of r.r
// per tile for r - alpha q, and the way down from r - alpha q.  r itself is
// not stored here (neighbouring tiles still read the old r in their halos):
// the next operator apply stores it.
template <typename T, typename TR>
__global__ void __launch_bounds__(kTileThreads) k_down_tile2_cg(Level<T> L, Geo gc, const TR *__restrict__ r,
                                                                const TR *__restrict__ q, const TR *__restrict__ p,
                                                                TR *__restrict__ x, T *__restrict__ xs,
                                                                T *__restrict__ bc, int ntx, int ntiles, Scal *sc,
                                                                const double *__restrict__ part_pq, int npq,
                                                                double *__restrict__ part_rr) {
    const int tile = xcd_block();
    if (tile >= ntiles) return;
    if (sc->done) return;
    __shared__ double bcast;
    double pq = 0.0, u0 = 0.0, u1 = 0.0;
    for (int i = (int)threadIdx.x; i < npq; i += kTileThreads) pq += part_pq[i];
    tile_sum3<kTileThreads>(pq, u0, u1);
    if (threadIdx.x == 0) bcast = pq;
    __syncthreads();
    pq = bcast;
    const double alpha = pq != 0.0 ? sc->rz / pq : 0.0;
    if (tile == 0 && threadIdx.x == 0) {
        sc->pq = pq;
        sc->alpha = alpha;
    }
    const int ty = tile / ntx, tx = tile - ty * ntx;
    down_tile2<T, kTileThreads>(L, gc, RhsPending<TR, T>{r, q, alpha}, xs, bc, tx, ty, 0);
    const int nx = (int)L.g.n[0], ny = (int)L.g.n[1];
    double rr = 0.0;
    u0 = u1 = 0.0;
    for (int j = (int)threadIdx.x; j < kTFX * kTFY; j += kTileThreads) {
        const int ly = j / kTFX, lx = j - ly * kTFX;
        const int gx = tx * kTFX + lx, gy = ty * kTFY + ly;
        if (gx < nx && gy < ny) {
            const int g = gx + nx * gy;
            x[g] = (TR)((double)x[g] + alpha * (double)p[g]);
            const double rc = cg_residual((double)r[g], (double)q[g], alpha);
            rr += rc * rc;
        }
    }
    tile_sum3<kTileThreads>(rr, u0, u1);
    if (threadIdx.x == 0) part_rr[tile] = rr;
}

// Level 0 of the way up inside CG: right-hand side as stored (b) or pending
// (r - alpha q, bpend); dmode 0: no partials, 1: partials of r.z, sum z,
// sum r per tile with r as stored, 2: with r pending.
template <typename T, typename TR>
__global__ void __launch_bounds__(kTileThreads) k_up_tile2_cg(Level<T> L, Geo gc, const T *__restrict__ xc,
                                                              const T *__restrict__ b, const TR *__restrict__ r,
                                                              const TR *__restrict__ q, const T *__restrict__ xs,
                                                              T *__restrict__ x, int ntx, int ntiles,
                                                              const Scal *__restrict__ sc, int bpend, int dmode,
                                                              double *__restrict__ p0, double *__restrict__ p1,
                                                              double *__restrict__ p2,
                                                              const int *__restrict__ done) {
    const int tile = xcd_block();
    if (tile >= ntiles) return;
    const int ty = tile / ntx, tx = tile - ty * ntx;
    const double alpha = (bpend || dmode == 2) ? sc->alpha : 0.0;
    const int skip = *done;
    if (dmode == 0) {
        up_tile2<T, kTileThreads>(L, gc, xc, RhsPending<TR, T>{r, q, alpha}, xs, x, tx, ty, skip);
        return;
    }
    const RzDots<TR> d{r, q, alpha, dmode == 2, p0, p1, p2, tile};
    if (bpend)
        up_tile2<T, kTileThreads>(L, gc, xc, RhsPending<TR, T>{r, q, alpha}, xs, x, tx, ty, skip, d);
    else
        up_tile2<T, kTileThreads>(L, gc, xc, RhsStored<T>{b}, xs, x, tx, ty, skip, d);
}

// Level 0 of a solve with one reduction point per iteration (tile2d.h).
template <typename T, typename TR>
__global__ void __launch_bounds__(kTileThreads) k_cg_down_tile2(Level<T> L, Geo gc, CgVec2<TR> v,
                                                                const T *__restrict__ z, T *__restrict__ xs,
                                                                T *__restrict__ bc, int ntx, int ntiles, int k,
                                                                int singular, Scal *sc, CgPart pt,
                                                                double *__restrict__ part_rr) {
    const int tile = xcd_block();
    if (tile >= ntiles) return;
    const int ty = tile / ntx, tx = tile - ty * ntx;
    cg_down_tile2<T, TR>(L, gc, v, z, xs, bc, tx, ty, tile, k, singular, sc, pt, ntiles, part_rr);
}

template <typename T, typename TR>
__global__ void __launch_bounds__(kTileThreads) k_cg_up_tile2(Level<T> L, Geo gc, const T *__restrict__ xc,
                                                              const TR *__restrict__ r, const T *__restrict__ xs,
                                                              T *__restrict__ z, TR *__restrict__ w, Level<TR> A,
                                                              int ntx, int ntiles, int singular, CgPart pt,
                                                              const int *__restrict__ done) {
    const int tile = xcd_block();
    if (tile >= ntiles) return;
    const int ty = tile / ntx, tx = tile - ty * ntx;
    cg_up_tile2<T, TR>(L, gc, xc, r, xs, z, w, A, tx, ty, tile, singular, pt, *done);
}

// ---------------------------------------------------------------------------
// single-workgroup kernels for the small levels
// ---------------------------------------------------------------------------
template <typename T, typename TB, int DIM>
__global__ void __launch_bounds__(kSBThreads) k_vcycle_block(Slot<T> S, int l0, const TB *__restrict__ b0,
                                                             T *__restrict__ x0, const int *__restrict__ done) {
    if (*done) return;
    vcycle_block_dev<T, TB, DIM>(S, l0, b0, x0);
}

// End of a CG iteration: r.r, the iteration count and the stop flags (thread
// 0; v: the scalars as they were, or *sc itself, so read before sc is written)
__device__ inline void pcg_fin_rr_dev(Scal *sc, const Scal &v, double rr) {
    if (threadIdx.x != 0) return;
    const int iter = v.iter + 1, max_iter = v.max_iter;
    const double lim = v.rtol2 * v.bb;
    sc->rr = rr;
    sc->iter = iter;
    if (!isfinite(rr)) {
        sc->nonfinite = 1;
        sc->done = 1;
    } else if (rr <= lim) {
        sc->done = 1;
    } else if (iter >= max_iter) {
        sc->unconverged = 1;
        sc->done = 1;
    }
}

// Levels [l0, nlev) in one workgroup (vcycle_small_dev).  fin (when given): the
// CG update of this iteration left nfin partials of r.r there and its end
// (pcg_fin_rr_dev) is taken here, in the one workgroup every cycle passes
// through, instead of in a launch of its own; the cycle that follows the
// last update is completed for nothing.
template <typename T, int DIM>
__global__ void __launch_bounds__(kVsThreads) k_vcycle_lds(VsArgs<T, DIM> A, const int *__restrict__ done, Scal *fsc,
                                                           const double *__restrict__ fin, int nfin) {
    const int dn = *done;
    extern __shared__ uint4 lds_words[];
    __shared__ double ws[kVsThreads / kWave];
    double rr = 0.0;
    for (int i = (int)threadIdx.x; i < nfin; i += kVsThreads) rr += fin[i];
    Scal sv{};   // read with the other loads; the sums of the waves meet after the cycle's barriers
    if (nfin && threadIdx.x == 0) sv = *fsc;
    vcycle_small_dev<T, DIM>(A, (T *)lds_words, dn, [&] {
        if (!nfin) return;
        rr = wave_sum(rr);
        if ((threadIdx.x & (kWave - 1)) == 0) ws[threadIdx.x / kWave] = rr;
    });
    if (dn || !nfin || threadIdx.x != 0) return;
    rr = 0.0;
    for (int q = 0; q < kVsThreads / kWave; ++q) rr += ws[q];
    pcg_fin_rr_dev(fsc, sv, rr);
}

template <typename T, int DIM>
__global__ void __launch_bounds__(kSBThreads) k_setup_block(Slot<T> S, int l0, double *mat) {
    __shared__ SetupLdsLev<T, DIM> sh;
    setup_lds_dev<T, DIM>(S, l0, sh, mat);
}

// One block step of the Gauss-Jordan inversion of the n x n SPD matrix src (no
// pivoting between blocks), for a coarsest level of more than kLdsInverse
// cells: pivots k0 .. k0 + kGjB - 1, from src to dst, a kGjT x kGjT tile per
// workgroup.  With P the inverse of the pivot block (formed in every
// workgroup; past n the identity) and W = P src[K, :], and P itself in the
// columns K: rows K become W, the others src - src[:, K] W, with 0 for src in
// the columns K.  The inversion in one workgroup makes a pass over the matrix
// per pivot from one CU; here a launch of the whole chip takes kGjB pivots.
// Whole steps: drops on 40 x 72 x 72 (405 coarsest cells, four set-ups) 25.7 ms
// before, 3.2 here; 64 x 56 x 64 (448 cells) 33.4 / 2.8 ms; about 6 us per
// launch, so bound by latency.
constexpr int kGjB = 16, kGjT = 32;
__global__ void __launch_bounds__(kBlock) k_gj_step(int n, int k0, const double *__restrict__ src,
                                                    double *__restrict__ dst) {
    __shared__ double P[kGjB][kGjB + 1], Kr[kGjB][kGjT + 1], Kc[kGjT][kGjB + 1], W[kGjB][kGjT + 1];
    static_assert(kBlock == kGjB * kGjB, "one pivot entry per thread");
    const int tid = (int)threadIdx.x, i0 = (int)blockIdx.y * kGjT, j0 = (int)blockIdx.x * kGjT;
    auto at = [&](int i, int j) { return i < n && j < n ? src[i * n + j] : 0.0; };
    const int pi = tid / kGjB, pj = tid % kGjB;
    P[pi][pj] = k0 + pi < n && k0 + pj < n ? src[(k0 + pi) * n + k0 + pj] : (pi == pj ? 1.0 : 0.0);
    for (int e = tid; e < kGjB * kGjT; e += kBlock) {
        Kr[e / kGjT][e % kGjT] = at(k0 + e / kGjT, j0 + e % kGjT);
        Kc[e / kGjB][e % kGjB] = at(i0 + e / kGjB, k0 + e % kGjB);
    }
    double old[kGjT * kGjT / kBlock];
#pragma unroll
    for (int r = 0; r < kGjT * kGjT / kBlock; ++r) {
        const int e = tid + r * kBlock;
        old[r] = at(i0 + e / kGjT, j0 + e % kGjT);
    }
    __syncthreads();
    double v = P[pi][pj];
    for (int p = 0; p < kGjB; ++p) {
        const double piv = 1.0 / P[p][p], row = P[p][pj], c = P[pi][p];
        __syncthreads();
        if (pi == p)
            v = pj == p ? piv : row * piv;
        else
            v = pj == p ? -c * piv : v - c * (row * piv);
        P[pi][pj] = v;
        __syncthreads();
    }
    for (int e = tid; e < kGjB * kGjT; e += kBlock) {
        const int m = e / kGjT, j = e % kGjT, kj = j0 + j - k0;
        double w = 0.0;
        for (int q = 0; q < kGjB; ++q) w = fma(P[m][q], Kr[q][j], w);
        W[m][j] = kj >= 0 && kj < kGjB ? P[m][kj] : w;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kGjT * kGjT / kBlock; ++r) {
        const int e = tid + r * kBlock, i = e / kGjT, j = e % kGjT, gi = i0 + i, gj = j0 + j;
        const int ki = gi - k0, kj = gj - k0;
        double x = kj >= 0 && kj < kGjB ? 0.0 : old[r];
        for (int q = 0; q < kGjB; ++q) x = fma(-Kc[i][q], W[q][j], x);
        if (ki >= 0 && ki < kGjB) x = W[ki][j];
        if (gi < n && gj < n) dst[gi * n + gj] = x;
    }
}

template <typename T, int DIM>
__global__ void __launch_bounds__(kBlock) k_invd(Level<T> L) {
    GRID_LOOP(L.g.N) invd_cell<T, DIM>(L, c);
}

template <typename T, int DIM>
__global__ void __launch_bounds__(kBlock) k_coarsen(Level<T> F, Level<T> C) {
    GRID_LOOP(C.g.N) coarsen_cell<T, DIM>(F, C, c);
}

// ---------------------------------------------------------------------------
// PCG kernels
// ---------------------------------------------------------------------------

// fixed-order sum of partials, returned to every thread of the block
__device__ inline double sum_parts_all(const double *__restrict__ part, int nparts, double *lds) {
    double v = 0.0;
    for (int k = threadIdx.x; k < nparts; k += blockDim.x) v += part[k];
    return block_sum_all(v, lds);
}

// Start of CG iteration k, evaluated by every block of the kernel that
// consumes it (the sums are the same in every block): rz = r.(z - zmean)
// from the partials of k_pcg_rz, zmean = mean(z) for a singular operator
// (else 0), beta = rz / rz_previous (0 for k = 0).  For a singular
// (pure Neumann / periodic) operator the preconditioned vector is projected
// onto the range: the V-cycle amplifies the constant mode, and without the
// projection rounding noise in that mode destroys the conjugacy of the
// search directions.  Block 0 stores rz in sc->rzs[k & 1] while the blocks
// read the previous value from the other entry, and publishes rz, zmean,
// beta; a non-finite rz ends the solve.  Returns false when the solve ends.
struct IterStart {
    double rz, zm, beta;
};
__device__ inline bool iter_start(Scal *sc, const double *__restrict__ p0, const double *__restrict__ p1,
                                  const double *__restrict__ p2, int nparts, long long N, int k, int singular,
                                  IterStart &o) {
    // the three sums in one pass: the same per-thread and per-wave order as
    // three separate block sums, one round of barriers
    __shared__ double wsum[3][kBlock / kWave];
    double trz = 0.0, tz = 0.0, tr = 0.0;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x) {
        trz += p0[i];
        if (singular) {
            tz += p1[i];
            tr += p2[i];
        }
    }
    trz = wave_sum(trz);
    tz = wave_sum(tz);
    tr = wave_sum(tr);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) {
        wsum[0][w] = trz;
        wsum[1][w] = tz;
        wsum[2][w] = tr;
    }
    __syncthreads();
    trz = tz = tr = 0.0;
    for (int q = 0; q < (int)(blockDim.x / kWave); ++q) {
        trz += wsum[0][q];
        tz += wsum[1][q];
        tr += wsum[2][q];
    }
    __syncthreads();
    if (!singular) tz = tr = 0.0;
    o.zm = singular ? tz / (double)N : 0.0;
    o.rz = trz - o.zm * tr;
    const double prev = k > 0 ? sc->rzs[(k + 1) & 1] : 0.0;
    o.beta = (k == 0 || prev == 0.0) ? 0.0 : o.rz / prev;
    const bool ok = isfinite(o.rz);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (ok) {
            sc->rzs[k & 1] = o.rz;
            sc->rz = o.rz;
            sc->zmean = o.zm;
            sc->beta = o.beta;
        } else {
            sc->nonfinite = 1;
            sc->done = 1;
        }
    }
    return ok;
}

// p_new = (z - zmean) + beta p_old (beta = 0: p_new = z - zmean);
// q = A p_new (slot operator); partial p.q.  RHO (3D pressure operator): the
// face coefficients formed from the cell densities with the set-up's
// expression instead of read, as in k_pcg_apply3_march below.
template <typename T, typename TZ, int DIM, bool RHO>
__global__ void __launch_bounds__(kBlock) k_pcg_apply_slot(Level<T> L, const TZ *__restrict__ z,
                                                           const T *__restrict__ pold, T *__restrict__ pnew,
                                                           T *__restrict__ q, Scal *sc, double *__restrict__ part,
                                                           const double *__restrict__ rz0,
                                                           const double *__restrict__ rz1,
                                                           const double *__restrict__ rz2, int nrz, int k,
                                                           int singular, T *__restrict__ rpend,
                                                           const double *__restrict__ rho, double rho_ih2) {
    if (sc->done) return;
    __shared__ double lds[kBlock / kWave];
    const double alpha_prev = rpend ? sc->alpha : 0.0;   // read before iter_start
    IterStart it;
    if (!iter_start(sc, rz0, rz1, rz2, nrz, L.g.N, k, singular, it)) return;
    const double beta = it.beta, zm = it.zm;
    auto pv = [&](int e) { return ((double)z[e] - zm) + (beta != 0.0 ? beta * (double)pold[e] : 0.0); };
    double acc = 0.0;
    GRID_LOOP(L.g.N) {
        int ia[3];
        coords_of<DIM>(L.g, c, ia);
        // residual of the previous iteration, stored before q is overwritten
        if (rpend) rpend[c] = (T)cg_residual((double)rpend[c], (double)q[c], alpha_prev);
        const double pc = pv(c);
        // a singular (pressure) operator has s = +0: not read
        double sv = 0.0;
        if (!singular) sv = (double)L.s[c];
        double qc = sv * pc;
#pragma unroll
        for (int b = 0; b < DIM; ++b) {   // branch-free: a missing neighbour is c itself with weight 0
            const int lo = nb_lo(L.g, c, ia[b], b);
            const int hi = nb_hi(L.g, c, ia[b], b);
            const int l = lo >= 0 ? lo : c, h = hi >= 0 ? hi : c;
            const double vl = pv(l), vh = pv(h);
            const double wl = RHO ? 1.0 / (0.5 * (rho[c] + rho[l])) * rho_ih2 : (double)L.cs[b][c];
            const double wh = RHO ? 1.0 / (0.5 * (rho[h] + rho[c])) * rho_ih2 : (double)L.cs[b][h];
            qc += (lo >= 0 ? wl : 0.0) * (pc - vl);
            qc += (hi >= 0 ? wh : 0.0) * (pc - vh);
        }
        pnew[c] = (T)pc;
        q[c] = (T)qc;
        acc += pc * qc;
    }
    const double s = block_sum(acc, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// The same apply on a 3D grid (no pending residual), marching along z:
// logical block b owns the kMX x kMY x zc cells of column tile b mod ncol and
// z chunk b / ncol, one cell per thread and plane.  p = (z - zmean) + beta p_old of
// the column and a one-cell halo is formed once per plane into a ring of
// three LDS planes, where the grid-stride form above evaluates it at all
// seven stencil points of every cell (128^3: 4 TB/s).  q, p_new and the
// per-cell arithmetic are those of k_pcg_apply_slot (a missing neighbour
// enters as the cell itself with weight 0); one p.q partial per block.
constexpr int kMX = 32, kMY = kBlock / kMX, kMW = kMX + 2, kMH = kMY + 2;
#ifndef CHNS_MARCH_PLANES
#define CHNS_MARCH_PLANES 8
#endif
constexpr int kMarchPlanes = CHNS_MARCH_PLANES;   // z planes per block (more on grids too large for the partials)
// A block marches its planes one after another, so the apply is as long as
// one block's chain unless the chip holds several blocks per CU: the planes
// per block are halved until there are kMarchApplyBlocks blocks (96^3, FP64:
// 432 blocks of 8 planes 21.4 us, 864 of 4 planes 18.1, 1728 of 2 planes
// 17.5; a target of 2048 halves 128^3 too, 28.2 -> 31.1 us).  Below
// kMarchApplyCells cells one cell per thread (k_pcg_apply_slot) has no chain
// at all: 64^3 17.3 us marching 8 planes, 10.7 with 1024 blocks, 9.3
// grid-stride; 32^3 14.8 / 6.3 / 5.5 us; 96^3 17.5 against 18.8 the other way.
constexpr int kMarchApplyBlocks = 1024;
constexpr long long kMarchApplyCells = 1LL << 19;
// RHO (pressure operator): the face coefficients 1/(rho_f h^2) are formed
// from the cell densities rho (a second ring of planes) with the set-up's
// expression, instead of read as s and cs[3]: 8 bytes per cell instead of 32
// for six divisions per cell.  Used on grids past the Infinity Cache (the
// marching-sweep threshold of the slot): 512^3 apply 2.00 -> 1.50 ms; at
// 128^3, where the coefficients come from the cache, the divisions cost more
// than the bytes save.
template <typename T, typename TZ, bool RHO>
__global__ void __launch_bounds__(kBlock) k_pcg_apply3_march(Level<T> L, const TZ *__restrict__ z,
                                                             const T *__restrict__ pold, T *__restrict__ pnew,
                                                             T *__restrict__ q, Scal *sc, double *__restrict__ part,
                                                             const double *__restrict__ rz0,
                                                             const double *__restrict__ rz1,
                                                             const double *__restrict__ rz2, int nrz, int k,
                                                             int singular, int ncolx, int ncol, int zc,
                                                             const double *__restrict__ rho, double rho_ih2) {
    if (sc->done) return;
    __shared__ double pl[3][kMH * kMW];
    __shared__ double rl[RHO ? 3 : 1][RHO ? kMH * kMW : 1];
    __shared__ double lds[kBlock / kWave];
    IterStart it;
    if (!iter_start(sc, rz0, rz1, rz2, nrz, L.g.N, k, singular, it)) return;
    const double beta = it.beta, zm = it.zm;
    const Geo &g = L.g;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    // XCD-contiguous numbering: the column tiles of a z chunk, whose halos
    // overlap, run on the same XCD and share its L2 (128^3: 32 -> 28 us)
    const int lb = xcd_block();
    const int col = lb % ncol, z0 = (lb / ncol) * zc;
    const int x0 = (col % ncolx) * kMX, y0 = (col / ncolx) * kMY;
    const int z1 = z0 + zc < nz ? z0 + zc : nz;
    // coordinate of a halo position on one axis (wrapped on a periodic axis);
    // false outside a walled one
    auto wrapc = [](int v, int n, int per, int &w) {
        if (v >= 0 && v < n) {
            w = v;
            return true;
        }
        w = v < 0 ? v + n : v - n;
        return per != 0 && w >= 0 && w < n;
    };
    // p of plane zz and its halo into P (0 outside the domain; never used
    // with a nonzero weight there)
    auto form = [&](int zz, int slot) {
        double *P = pl[slot];
        int gz;
        const bool vz = wrapc(zz, nz, g.per[2], gz);
        for (int i = (int)threadIdx.x; i < kMH * kMW; i += kBlock) {
            const int ly = i / kMW, lx = i - ly * kMW;
            int gx, gy;
            const bool vx = wrapc(x0 - 1 + lx, nx, g.per[0], gx);
            const bool vy = wrapc(y0 - 1 + ly, ny, g.per[1], gy);
            const bool v = vx && vy && vz;
            double pv = 0.0, rv = 0.0;
            if (v) {
                const int e = gx + nx * (gy + ny * gz);
                pv = ((double)z[e] - zm) + (beta != 0.0 ? beta * (double)pold[e] : 0.0);
                if (RHO) rv = rho[e];
            }
            P[i] = pv;
            if (RHO) rl[slot][i] = rv;
        }
    };
    const int tx = (int)threadIdx.x % kMX, ty = (int)threadIdx.x / kMX;
    const int gx = x0 + tx, gy = y0 + ty, li = (ty + 1) * kMW + tx + 1;
    const bool own = gx < nx && gy < ny;
    form(z0 - 1, (z0 + 2) % 3);
    form(z0, z0 % 3);
    double acc = 0.0;
    for (int zz = z0; zz < z1; ++zz) {
        form(zz + 1, (zz + 1) % 3);
        __syncthreads();
        const double *Pm = pl[(zz + 2) % 3], *P0 = pl[zz % 3], *Pp = pl[(zz + 1) % 3];
        if (own) {
            const int c = gx + nx * (gy + ny * zz);
            const int ia[3] = {gx, gy, zz};
            const double pc = P0[li];
            const double nbv[3][2] = {{P0[li - 1], P0[li + 1]}, {P0[li - kMW], P0[li + kMW]}, {Pm[li], Pp[li]}};
            double rc = 0.0, nbr[3][2] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
            if (RHO) {
                const double *Rm = rl[(zz + 2) % 3], *R0 = rl[zz % 3], *Rp = rl[(zz + 1) % 3];
                rc = R0[li];
                nbr[0][0] = R0[li - 1];
                nbr[0][1] = R0[li + 1];
                nbr[1][0] = R0[li - kMW];
                nbr[1][1] = R0[li + kMW];
                nbr[2][0] = Rm[li];
                nbr[2][1] = Rp[li];
            }
            // s = +0 on a singular (pressure) operator: not read
            double sv = 0.0;
            if (!RHO && !singular) sv = (double)L.s[c];
            double qc = sv * pc;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const int lo = nb_lo(g, c, ia[b], b);
                const int hi = nb_hi(g, c, ia[b], b);
                const int h = hi >= 0 ? hi : c;
                const double vl = lo >= 0 ? nbv[b][0] : pc, vh = hi >= 0 ? nbv[b][1] : pc;
                double wl, wh;
                if (RHO) {
                    // the set-up's 1.0 / (0.5 * (rho_c + rho_lo)) * ih2 for the faces c and c + e_b
                    wl = lo >= 0 ? 1.0 / (0.5 * (rc + nbr[b][0])) * rho_ih2 : 0.0;
                    wh = hi >= 0 ? 1.0 / (0.5 * (nbr[b][1] + rc)) * rho_ih2 : 0.0;
                } else {
                    wl = (double)L.cs[b][c];
                    wh = (double)L.cs[b][h];
                }
                qc += (lo >= 0 ? wl : 0.0) * (pc - vl);
                qc += (hi >= 0 ? wh : 0.0) * (pc - vh);
            }
            pnew[c] = (T)pc;
            q[c] = (T)qc;
            acc += pc * qc;
        }
        __syncthreads();   // the next plane overwrites this iteration's lower plane
    }
    const double s = block_sum(acc, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// ---------------------------------------------------------------------------
// 3D V-cycle passes on cubic tiles (levels of at most Slot::tile_cells cells
// above the single-workgroup part): ONE launch per level on the way down
// (zero-guess pre-smoothing, residual, restriction) and one on the way up
// (prolongation, black sweep, red sweep), as the columns below have, without
// their march: on these levels a chain of planes takes longer than recomputing
// halos (kTileCycleCells).  A workgroup owns a kTF^3 block of fine cells (kTC^3 coarse
// cells) and recomputes into LDS what its cells' stencils reach in the
// neighbouring tiles:
//   down: b / d of the red cells on a halo of 3, x on a halo of 2, the
//         residual of the red cells on a halo of 1 (the restriction's outer
//         taps; that of a black cell is 0);
//   up:   red x + P e on a halo of 2, the black GS values on a halo of 1,
//         then the red GS values of the owned cells.
// Each value is formed with the arithmetic and order of the per-cell
// bodies (presmooth_cell, apply_at, restrict_cell, prolong_at,
// gs_color_cell), so both forms give the same bits.  The pre-smoothed x of
// the owned cells goes to the level's r array (the residual stays in LDS)
// and the way up reads it there, writing the smoothed x: a workgroup writes
// its cells while its neighbours still read their halo values.  Positions
// past a wall hold 0 and enter only with weight 0, as a missing neighbour
// does in the per-cell bodies (the zero product added to a sum that starts
// at +0 leaves it unchanged).
// ---------------------------------------------------------------------------
constexpr int kTF = 8, kTC = kTF / 2;   // fine / coarse cells per tile edge
// Threads per tile: at most one cell of each region per thread (two of the
// widest halo), so that all loads of a tile kernel are issued together.
constexpr int kT3Threads = 1024;

// Global index and coordinates of position (lx, ly, lz) of a tile whose
// first fine cell is f0, with a halo of H cells, wrapped on periodic axes;
// ok = false past a wall (the index is then that of a cell inside).
template <int H>
__device__ inline int tile_cell(const Geo &g, const int f0[3], int lx, int ly, int lz, int ia[3], bool &ok) {
    const int l[3] = {lx, ly, lz};
    ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int p = f0[a] - H + l[a];
        if (p < 0 || p >= g.n[a]) {
            ok = ok && g.per[a] != 0;
            p %= g.n[a];
            p = p < 0 ? p + g.n[a] : p;
        }
        ia[a] = p;
    }
    return ia[0] + g.n[0] * (ia[1] + g.n[1] * ia[2]);
}

// x-pair k of a region of edge E (E even, halo H): position of the member
// of colour col (colour = parity of the global coordinates; the tile origin
// is even and periodic extents are even, so it is the parity of the
// unwrapped position)
template <int E, int H>
__device__ inline void tile_pair(int k, int col, int &lx, int &ly, int &lz) {
    const int kx = k % (E / 2), r = k / (E / 2);
    ly = r % E;
    lz = r / E;
    lx = 2 * kx + ((H + ly + lz + col) & 1);
}

template <int E>
__device__ inline void tile_split(int q, int &lx, int &ly, int &lz) {
    lx = q % E;
    const int r = q / E;
    ly = r % E;
    lz = r / E;
}

// The loads of one cell's stencil, issued at the start of a tile kernel
// (each kernel then waits on one round of loads, not one per pass):
// neighbour existence (nb_lo / nb_hi), b and 1 / d (for a sweep) and the
// coefficients of the faces towards the neighbours.
template <typename T>
struct TileSt {
    bool lo[3], hi[3];
    T bv, dv, wl[3], wh[3];
};

template <typename T, typename TB, bool RES>
__device__ inline void tile_load(const Level<T> &L, const TB *__restrict__ b, int c, const int ia[3], TileSt<T> &S) {
    using R = T;
    if (!RES) {
        S.bv = (R)b[c];
        S.dv = (R)L.invd[c];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int lo = nb_lo(L.g, c, ia[a], a);
        const int hi = nb_hi(L.g, c, ia[a], a);
        const int h = hi >= 0 ? hi : c;
        S.lo[a] = lo >= 0;
        S.hi[a] = hi >= 0;
        S.wl[a] = (R)L.cs[a][c];
        S.wh[a] = (R)L.cs[a][h];
    }
}

// sum_b cs * v_nb from the neighbours' values at stride offsets of position q
// of an LDS region of edge E (offsum_at's order; a missing neighbour enters
// as 0 with weight 0): the residual of a red cell after the black sweep
template <typename T, int E>
__device__ inline T tile_offsum(const TileSt<T> &S, const T *v, int q) {
    using R = T;
    constexpr int st[3] = {1, E, E * E};
    R acc = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const R vl = S.lo[a] ? (R)v[q - st[a]] : (R)0, vh = S.hi[a] ? (R)v[q + st[a]] : (R)0;
        acc = fmar(S.lo[a] ? S.wl[a] : (R)0, vl, acc);
        acc = fmar(S.hi[a] ? S.wh[a] : (R)0, vh, acc);
    }
    return acc;
}
// GS value (b_c + sum_b cs * v_nb) / d_c
template <typename T, int E>
__device__ inline T tile_gs(const TileSt<T> &S, const T *v, int q) {
    return (T)((S.bv + tile_offsum<T, E>(S, v, q)) * S.dv);
}

// P e at fine cell fi: the eight coarse taps loaded up front, then
// prolong_at's weights and summation order
template <typename T>
struct TilePro {
    T X[2][2][2];
    T w0[3], w1[3];
};

template <typename T>
__device__ inline void pro_load(const Geo &gc, const T *__restrict__ xc, const int fi[3], TilePro<T> &P) {
    using R = T;
    int c0[3], c1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) pro_axis<R>(fi[a], gc.n[a], gc.per[a], c0[a], c1[a], P.w0[a], P.w1[a]);
    const int nx = gc.n[0], nxy = gc.n[0] * gc.n[1];
#pragma unroll
    for (int dz = 0; dz < 2; ++dz) {
        const int kz = (dz ? c1[2] : c0[2]) * nxy;
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
            const int ky = kz + (dy ? c1[1] : c0[1]) * nx;
            P.X[dz][dy][0] = xc[ky + c0[0]];
            P.X[dz][dy][1] = xc[ky + c1[0]];
        }
    }
}

template <typename T>
__device__ inline T pro_value(const TilePro<T> &P) {
    using R = T;
    R v = 0.0;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz) {
        const R wz = dz ? P.w1[2] : P.w0[2];
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
            const R wyz = wz * (dy ? P.w1[1] : P.w0[1]);
            v = pro_row(v, wyz, P.w0[0], (R)P.X[dz][dy][0], P.w1[0], (R)P.X[dz][dy][1]);
        }
    }
    return v;
}

template <typename T, typename TB>
__global__ void __launch_bounds__(kT3Threads) k_down3_tile(Level<T> L, Geo gc, const TB *__restrict__ b,
                                                           T *__restrict__ bc, int ntx, int nty, int ntiles,
                                                           const int *__restrict__ done) {
    using R = T;
    const int tile = xcd_block();
    if (tile >= ntiles || *done) return;
    constexpr int E3 = kTF + 6, E2 = kTF + 4, E1 = kTF + 2;
    constexpr int N3 = E3 * E3 * E3 / 2, N2 = E2 * E2 * E2 / 2, N1 = E1 * E1 * E1 / 2;
    constexpr int K3 = (N3 + kT3Threads - 1) / kT3Threads;
    static_assert(N2 <= kT3Threads && N1 <= kT3Threads, "one x pair and one red residual per thread");
    __shared__ T sd[E3 * E3 * E3];   // red b / d, halo 3
    __shared__ T sx[E2 * E2 * E2];   // pre-smoothed x, halo 2
    __shared__ T sr[E1 * E1 * E1];   // residual of the red cells, halo 1
    const Geo &g = L.g;
    const int tz = tile / (ntx * nty), trem = tile - tz * ntx * nty, ty = trem / ntx, tx = trem - ty * ntx;
    const int f0[3] = {tx * kTF, ty * kTF, tz * kTF};
    const int tid = (int)threadIdx.x;
    // loads: red b and 1 / d (halo 3), the black member of an x-pair (halo 2),
    // a red residual (halo 1)
    R rb[K3], rd[K3];
    int rq[K3];
    bool rok[K3];
#pragma unroll
    for (int j = 0; j < K3; ++j) {
        const int k = tid + j * kT3Threads;
        int lx, ly, lz, ia[3];
        tile_pair<E3, 3>(k < N3 ? k : N3 - 1, 0, lx, ly, lz);
        const int c = tile_cell<3>(g, f0, lx, ly, lz, ia, rok[j]);
        rq[j] = lx + E3 * (ly + E3 * lz);
        rb[j] = (R)b[c];
        rd[j] = (R)L.invd[c];
    }
    int x2, y2, z2, ia2[3];
    bool ok2;
    tile_pair<E2, 2>(tid < N2 ? tid : 0, 1, x2, y2, z2);
    TileSt<T> S2;
    tile_load<T, TB, false>(L, b, tile_cell<2>(g, f0, x2, y2, z2, ia2, ok2), ia2, S2);
    int x1, y1, z1, ia1[3];
    bool ok1;
    tile_pair<E1, 1>(tid < N1 ? tid : 0, 0, x1, y1, z1);
    TileSt<T> S1;
    tile_load<T, TB, true>(L, b, tile_cell<1>(g, f0, x1, y1, z1, ia1, ok1), ia1, S1);
#pragma unroll
    for (int j = 0; j < K3; ++j)
        if (tid + j * kT3Threads < N3) sd[rq[j]] = rok[j] ? (T)(rb[j] * rd[j]) : (T)0;
    __syncthreads();
    // x: black GS from the red neighbours' b / d, red b / d
    if (tid < N2) {
        const int q = x2 + E2 * (y2 + E2 * z2);
        const int q3 = (x2 + 1) + E3 * ((y2 + 1) + E3 * (z2 + 1));
        const T v = tile_gs<T, E3>(S2, sd, q3);
        sx[q] = ok2 ? v : (T)0;
        const int d = 1 - 2 * (x2 & 1);   // the red member of the x-pair
        sx[q + d] = sd[q3 + d];
    }
    __syncthreads();
    // red residuals
    if (tid < N1) {
        const T v = tile_offsum<T, E2>(S1, sx, (x1 + 1) + E2 * ((y1 + 1) + E2 * (z1 + 1)));
        sr[x1 + E1 * (y1 + E1 * z1)] = ok1 ? v : (T)0;
    }
    // the owned cells' pre-smoothed x (read back on the way up)
    if (tid < kTF * kTF * kTF) {
        int lx, ly, lz;
        tile_split<kTF>(tid, lx, ly, lz);
        const int gx = f0[0] + lx, gy = f0[1] + ly, gz = f0[2] + lz;
        if (gx < g.n[0] && gy < g.n[1] && gz < g.n[2])
            L.r[gx + g.n[0] * (gy + g.n[1] * gz)] = sx[(lx + 2) + E2 * ((ly + 2) + E2 * (lz + 2))];
    }
    __syncthreads();
    // restriction (restrict_cell's weights and order, the red taps) of the tile's coarse cells
    if (tid < kTC * kTC * kTC) {
        int cx, cy, cz;
        tile_split<kTC>(tid, cx, cy, cz);
        const int I[3] = {tx * kTC + cx, ty * kTC + cy, tz * kTC + cz};
        if (I[0] < gc.n[0] && I[1] < gc.n[1] && I[2] < gc.n[2]) {
            int f[4];
            R wx[4], wy[4], wz[4];
            res_axis<R>(I[0], gc.n[0], g.n[0], gc.per[0], f, wx);
            res_axis<R>(I[1], gc.n[1], g.n[1], gc.per[1], f, wy);
            res_axis<R>(I[2], gc.n[2], g.n[2], gc.per[2], f, wz);
            R acc = 0.0;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const R wza = wz[a];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const T *row = &sr[2 * cx + E1 * ((2 * cy + q) + E1 * (2 * cz + a))];
                    R s = 0.0;
#pragma unroll
                    for (int e = (1 + q + a) & 1; e < 4; e += 2) s = fmar(wx[e], (R)row[e], s);   // (tap 2 I - 1 + e, ..)
                    acc = fmar(wy[q] * wza, s, acc);
                }
            }
            bc[(I[2] * gc.n[1] + I[1]) * gc.n[0] + I[0]] = (T)acc;
        }
    }
}

// !PRO: the symmetric sweep from zero that ends a truncated cycle (red b / d,
// black, red) instead of the way up.
template <typename T, typename TB, bool PRO = true>
__global__ void __launch_bounds__(kT3Threads) k_up3_tile(Level<T> L, Geo gc, const T *__restrict__ xc,
                                                         const TB *__restrict__ b, const T *__restrict__ xpre,
                                                         T *__restrict__ x, int ntx, int nty, int ntiles,
                                                         const int *__restrict__ done) {
    using R = T;
    const int tile = xcd_block();
    if (tile >= ntiles || *done) return;
    constexpr int E2 = kTF + 4, E1 = kTF + 2;
    constexpr int N2 = E2 * E2 * E2 / 2, N1 = E1 * E1 * E1 / 2, N0 = kTF * kTF * kTF / 2;
    static_assert(N2 <= kT3Threads, "one red cell of the halo-2 region per thread");
    __shared__ T se[E2 * E2 * E2];   // red x + P e, halo 2
    __shared__ T sb[E1 * E1 * E1];   // black GS values, halo 1
    const Geo &g = L.g;
    const int tz = tile / (ntx * nty), trem = tile - tz * ntx * nty, ty = trem / ntx, tx = trem - ty * ntx;
    const int f0[3] = {tx * kTF, ty * kTF, tz * kTF};
    const int tid = (int)threadIdx.x;
    // loads: a red cell's x and coarse taps (halo 2), a black cell (halo 1),
    // an owned x-pair
    int x2, y2, z2, ia2[3];
    bool ok2;
    tile_pair<E2, 2>(tid < N2 ? tid : 0, 0, x2, y2, z2);
    const int c2 = tile_cell<2>(g, f0, x2, y2, z2, ia2, ok2);
    R rx, rd = (R)0;
    TilePro<T> P;
    if (PRO) {
        rx = (R)xpre[c2];
        pro_load<T>(gc, xc, ia2, P);
    } else {
        rx = (R)b[c2];
        rd = (R)L.invd[c2];
    }
    int x1, y1, z1, ia1[3];
    bool ok1;
    tile_pair<E1, 1>(tid < N1 ? tid : 0, 1, x1, y1, z1);
    TileSt<T> S1;
    tile_load<T, TB, false>(L, b, tile_cell<1>(g, f0, x1, y1, z1, ia1, ok1), ia1, S1);
    int x0, y0, z0;
    tile_pair<kTF, 0>(tid < N0 ? tid : 0, 0, x0, y0, z0);
    int ia0[3] = {f0[0] + x0, f0[1] + y0, f0[2] + z0};
    // whole pairs (even extents): the red member inside <=> the pair inside
    const bool own0 = tid < N0 && ia0[0] < g.n[0] && ia0[1] < g.n[1] && ia0[2] < g.n[2];
    if (!own0) ia0[0] = ia0[1] = ia0[2] = 0;
    const int c0 = ia0[0] + g.n[0] * (ia0[1] + g.n[1] * ia0[2]);
    TileSt<T> S0;
    tile_load<T, TB, false>(L, b, c0, ia0, S0);
    if (tid < N2) {
        const T v = (T)(PRO ? rx + pro_value<T>(P) : rx * rd);
        se[x2 + E2 * (y2 + E2 * z2)] = ok2 ? v : (T)0;
    }
    __syncthreads();
    if (tid < N1) {
        const T v = tile_gs<T, E2>(S1, se, (x1 + 1) + E2 * ((y1 + 1) + E2 * (z1 + 1)));
        sb[x1 + E1 * (y1 + E1 * z1)] = ok1 ? v : (T)0;
    }
    __syncthreads();
    if (own0) {
        const int q1 = (x0 + 1) + E1 * ((y0 + 1) + E1 * (z0 + 1));
        const int d = 1 - 2 * (x0 & 1);   // the black member of the x-pair
        x[c0] = tile_gs<T, E1>(S0, sb, q1);
        x[c0 + d] = sb[q1 + d];
    }
}

// ---------------------------------------------------------------------------
// 3D post-smoothing in one pass over the level: red values, black sweep, red
// sweep (and the r.z partials of CG) on columns that march along z.
//   PRO   red start = x + P e (the way up: x the pre-smoothed one, e the
//         coarse correction)
//   !PRO  red start = b / d (the symmetric sweep from zero that ends a
//         truncated cycle)
// A block owns kUX x kUY cells of every plane of its z chunk.  Its waves split
// by role: the first form the red start values with a halo of two cells, the
// others, two planes behind, the black values with a halo of one and then the
// red values of the plane below and store that plane.  Values pass through
// rings of planes in LDS, stored by x-pair (one red and one black cell; the red
// one is at x = 2 m + parity), so one barrier per plane is enough, and every
// role loads operands two planes before it works on them.  The lanes of a wave
// of the second role have rows of one parity, so which cell of a pair is red
// is known at compile time and one load per pair serves the black and the red
// value (a load of every second cell touches as many cache lines); the black
// cells above and below a red one are in the lane's own pair.
// The stored x may not be the one read (neighbouring blocks still read their
// halos): the way down leaves the pre-smoothed x in the level's r array.
// Per-cell arithmetic and order are those of prolong_at / presmooth_cell and
// gs_color_cell (a neighbour past a wall enters as 0 with weight 0).
// x, b, 1 / d and three coefficients are read once and x is written once, 56 B
// per cell in FP64, where three passes (prolongation, black, red) moved 129.
// Measured against these, with r.z, alone on the chip (a pressure solve): 128^3
// FP64 46.6 us -> 24.9, FP32 29.6 -> 20; 96^3 FP64 26.5 -> 16.4, FP32 19.1 -> 14.5;
// 80^3 FP64 19.4 -> 15.2; 512^3 4.0 ms -> 1.95.
// 128^3 FP64 moves 117 MB, 24.6 us at the rate of a large copy; 512^3 moves
// 1.6 times its bytes (halos that have left the L2) at 5.7 TB/s; smaller levels
// are bound by the rounds of steps.  With the black and the red values in roles
// of their own, each loading its half of every pair: 128^3 FP64 32.2, 96^3 22.1.
// ---------------------------------------------------------------------------
constexpr int kUX = 32, kUY = 16, kUM = kUX / 2 + 2;   // owned cells; pairs per row with one more on each side
constexpr int kCUs = 256;

// LDS of one plane is written before and read after: the barrier alone, without
// waiting for the loads in flight
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Cell (x, y, z) wrapped on periodic axes; false past a wall (indices inside).
__device__ inline bool wrap_axis(int v, int n, int per, int &w) {
    w = v < 0 ? v + n : (v >= n ? v - n : v);
    const bool ok = (v >= 0 && v < n) || per != 0;
    w = w < 0 ? 0 : (w >= n ? n - 1 : w);   // past a wall, or past the tile's part of the grid
    return ok;
}

// Element at byte offset off of a plane (a scalar base and one vector register)
template <typename T>
__device__ inline T plane_at(const T *plane, unsigned off) {
    return *(const T *)((const char *)plane + off);
}

template <typename T>
__device__ inline Pair2<T> pair_at(const T *plane, unsigned off) {
    return *(const Pair2<T> *)((const char *)plane + off);
}

// A lane of the role that works on pairs of ROWS rows (halo H in y, one pair in
// x) of the tile at (x0, y0): waves 0 .. wHalf - 1 hold the even rows, the next
// wHalf the odd ones.
template <int ROWS, int H>
struct PairLane {
    static constexpr int half = ROWS / 2 * kUM, wHalf = (half + kWave - 1) / kWave, waves = 2 * wHalf;
    int rp, ly, m;        // row parity, row, pair in the row
    bool on, own, ok;     // has a pair; of the owned cells; inside the grid
    unsigned c, n, h;     // cell indices in a plane: the pair, the cell above it in x, the pair above in y
    template <typename G>
    __device__ inline PairLane(const G &g, int wave, int lane, int x0, int y0) {
        rp = wave / wHalf;
        const int u = (wave - rp * wHalf) * kWave + lane;
        on = u < half;
        const int row = on ? u / kUM : 0;
        m = (on ? u : 0) - row * kUM;
        ly = 2 * row + rp;
        const int ex = x0 - 2 + 2 * m, ey = y0 - H + ly;
        int gx, gy;
        ok = wrap_axis(ex, g.n[0], g.per[0], gx) & wrap_axis(ey, g.n[1], g.per[1], gy);
        gx &= ~1;
        own = on && m >= 1 && m <= kUX / 2 && ly >= H && ly < ROWS - H && ex < g.n[0] && ey < g.n[1];
        c = (unsigned)(gx + g.n[0] * gy);
        // (nothing above at a wall: the coefficient multiplies 0 and may be any)
        const int hx = nb_hi(g, (int)c + 1, gx + 1, 0), hy = nb_hi(g, (int)c, gy, 1);
        n = hx >= 0 ? (unsigned)hx : c + 1;
        h = hy >= 0 ? (unsigned)hy : c;
    }
};

// One role of the pass: body(s, K, o) for the steps from FIRST on, in whole
// groups of four until `last` is past, a barrier after every one of `total`
// steps; load(s, P, o) fetches a step's operands two steps ahead of its body,
// into one of two sets of registers.  The group has no branch in it: with a
// test around a load or a body the compiler cannot know which loads are in
// flight and waits for all of them in every step, which makes a step as long
// as the way to memory.  (The up to three steps past `last` work on clamped
// planes and write only ring planes that are no longer read.)  K = s mod 4
// and P = s mod 2 are constants, so that ring planes are immediate offsets
// and a lane's two alternating cells cost no arithmetic.
template <int FIRST, typename O, typename LOAD, typename BODY>
__device__ __forceinline__ void sweep_role(int last, int total, LOAD load, BODY body) {
    O o0, o1;
    load(FIRST, std::integral_constant<int, FIRST & 1>(), o0);
    load(FIRST + 1, std::integral_constant<int, (FIRST + 1) & 1>(), o1);
    for (int s = 0; s < FIRST; ++s) lds_barrier();
    auto step = [&](int s, auto J, O &o) {
        constexpr int k = (FIRST + decltype(J)::value) & 3;
        body(s, std::integral_constant<int, k>(), o);
        __builtin_amdgcn_sched_barrier(0);   // (loads moved up into the body need a third set of registers)
        load(s + 2, std::integral_constant<int, (k & 1)>(), o);
        lds_barrier();
    };
    int s = FIRST;
    for (; s <= last; s += 4) {
        step(s, std::integral_constant<int, 0>(), o0);
        step(s + 1, std::integral_constant<int, 1>(), o1);
        step(s + 2, std::integral_constant<int, 2>(), o0);
        step(s + 3, std::integral_constant<int, 3>(), o1);
    }
    for (; s < total; ++s) lds_barrier();
}

// Pairs per plane of the red start / black values, coarse cells per plane that
// the red start reads, waves of the first role, threads.
struct SweepShape {
    static constexpr int rows = kUY + 2, E = (kUY + 4) * kUM, B = rows * kUM;
    static constexpr int CX = kUX / 2 + 4, CY = kUY / 2 + 4, C = CX * CY;
    using Lane = PairLane<rows, 1>;
    static constexpr int wB = (E + kWave - 1) / kWave, nB = Lane::waves;
    static constexpr int threads = (wB + nB) * kWave;
};

// r.z, sum z, sum r of a thread's pair, and the block's partials of them (u:
// thread of the second role)
template <typename TR, typename T>
__device__ inline void sweep_dots(const Pair2<TR> &r, const Pair2<T> &z, double &arz, double &az, double &ar) {
#pragma clang fp contract(off)   // z as stored: not fused with the product it comes from
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        arz = fmar((double)r.v[e], (double)z.v[e], arz);
        az += (double)z.v[e];
        ar += (double)r.v[e];
    }
}
__device__ inline void sweep_partials(double arz, double az, double ar, int u, double (*ws)[SweepShape::nB],
                                      double *p0, double *p1, double *p2) {
    arz = wave_sum(arz);
    az = wave_sum(az);
    ar = wave_sum(ar);
    if ((u & (kWave - 1)) == 0) {
        ws[0][u / kWave] = arz;
        ws[1][u / kWave] = az;
        ws[2][u / kWave] = ar;
    }
    lds_barrier();
    if (u == 0) {
        arz = az = ar = 0.0;
        for (int k = 0; k < SweepShape::nB; ++k) {
            arz += ws[0][k];
            az += ws[1][k];
            ar += ws[2][k];
        }
        *p0 = arz;
        *p1 = az;
        *p2 = ar;
    }
}

template <typename T, typename TB, bool PRO, bool DOTS, typename TR>
__global__ void __launch_bounds__(SweepShape::threads) k_sweep3(Level<T> L, const TB *__restrict__ b,
                                                      const T *__restrict__ xpre, Geo gc,
                                                      const T *__restrict__ xc, T *__restrict__ x, int ntx, int ncol,
                                                      int zc, int ntiles, const int *__restrict__ done,
                                                      const TR *__restrict__ r, double *__restrict__ p0,
                                                      double *__restrict__ p1, double *__restrict__ p2) {
    using Sh = SweepShape;
    const int tile = xcd_block();
    if (tile >= ntiles || *done) return;
    static_assert(sizeof(T) == sizeof(TB), "offsets in bytes of both");
    __shared__ T E[4][Sh::E], B[2][Sh::B], C[4][PRO ? Sh::C : 1];
    __shared__ double ws[3][Sh::nB];
    static_assert(Sh::C <= Sh::wB * kWave, "one coarse cell per lane of the first role");
    const Geo &g = L.g;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int col = tile % ncol, z0 = (tile / ncol) * zc, z1 = z0 + zc < nz ? z0 + zc : nz;
    const int x0 = (col % ntx) * kUX, y0 = (col / ntx) * kUY;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const long long nxy = (long long)nx * ny;
    const int n = z1 - z0, total = n + 8;   // every role ends its group of four within these steps
    if (wave < Sh::wB) {
        // red start of plane z0 - 2 + s, into E[s & 3]
        const int u = (int)threadIdx.x;
        const bool on = u < Sh::E;
        const int ly = on ? u / kUM : 0, m = (on ? u : 0) - ly * kUM;
        int gy;
        const bool oky = wrap_axis(y0 - 2 + ly, ny, g.per[1], gy);
        bool ok[2];
        unsigned off[2];
        int t00[2], t01[2], t10[2], t11[2];   // coarse taps (y, x) in a plane of C
        T w0x[2], w1x[2], w0y = 0, w1y = 0;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int par = (y0 + ly + z0 + p) & 1;   // of plane z0 - 2 + s, s = p mod 2
            int gx;
            ok[p] = wrap_axis(x0 - 2 + 2 * m + par, nx, g.per[0], gx) && oky;
            off[p] = (unsigned)(gx + nx * gy) * sizeof(T);
            if (PRO) {   // weights of prolong_at; a tap past a wall has weight 0
                int c0, c1;
                pro_axis<T>(gx, gc.n[0], gc.per[0], c0, c1, w0x[p], w1x[p]);
                pro_axis<T>(gy, gc.n[1], gc.per[1], c0, c1, w0y, w1y);
                const int a0 = m + 1, a1 = a0 + (par ? 1 : -1);
                const int b0 = (ly >> 1) + 1, b1 = b0 + ((ly & 1) ? 1 : -1);   // (y0 is even)
                t00[p] = a0 + Sh::CX * b0;
                t01[p] = a1 + Sh::CX * b0;
                t10[p] = a0 + Sh::CX * b1;
                t11[p] = a1 + Sh::CX * b1;
            }
        }
        // coarse cell u of the planes around (z0 is even): plane Zc of the
        // coarse level is at C[Zc & 3]; fine planes 2 Z and 2 Z + 1 read
        // Z - 1, Z and Z + 1, and plane Z + 2 is stored in the first of their steps
        const int Zf = z0 / 2 - 1;
        T cnext = (T)0;
        const T *cu = xc;
        const bool con = PRO && u < Sh::C;
        auto cplane = [&](int Z) {
            int w;
            (void)wrap_axis(Z, gc.n[2], gc.per[2], w);
            return cu[(long long)w * gc.n[0] * gc.n[1]];
        };
        if (PRO) {
            const int ry = u / Sh::CX, rx = u - ry * Sh::CX;
            int cx, cy;
            (void)wrap_axis(x0 / 2 - 2 + rx, gc.n[0], gc.per[0], cx);
            (void)wrap_axis(y0 / 2 - 2 + ry, gc.n[1], gc.per[1], cy);
            cu = xc + (cx + gc.n[0] * cy);
            const T c0 = cplane(Zf - 1), c1 = cplane(Zf), c2 = cplane(Zf + 1);
            cnext = cplane(Zf + 2);
            if (con) {
                C[(Zf - 1) & 3][u] = c0;
                C[Zf & 3][u] = c1;
                C[(Zf + 1) & 3][u] = c2;
            }
            lds_barrier();
        }
        struct Ops {
            T a, b;
        };
        sweep_role<0, Ops>(
            n + 3, total,
            [&](int s, auto P, Ops &o) {
                constexpr int p = decltype(P)::value;
                int gz;
                (void)wrap_axis(z0 - 2 + s, nz, g.per[2], gz);
                const long long z = (long long)gz * nx * ny;
                if (PRO) {
                    o.a = plane_at(xpre + z, off[p]);
                } else {
                    o.a = (T)plane_at(b + z, off[p]);
                    o.b = plane_at(L.invd + z, off[p]);
                }
            },
            [&](int s, auto K, const Ops &o) {
                constexpr int k = decltype(K)::value, p = k & 1;
                int gz;
                const bool okz = wrap_axis(z0 - 2 + s, nz, g.per[2], gz);
                T v;
                if (PRO) {   // prolong_at's weights and order
                    const int Z = Zf + (s >> 1);
                    int c0, c1;
                    T w0, w1;
                    pro_axis<T>(gz, gc.n[2], gc.per[2], c0, c1, w0, w1);
                    const T *e0 = C[Z & 3], *e1 = C[(p ? Z + 1 : Z - 1) & 3];
                    v = pro_row((T)0, w0 * w0y, w0x[p], e0[t00[p]], w1x[p], e0[t01[p]]);
                    v = pro_row(v, w0 * w1y, w0x[p], e0[t10[p]], w1x[p], e0[t11[p]]);
                    v = pro_row(v, w1 * w0y, w0x[p], e1[t00[p]], w1x[p], e1[t01[p]]);
                    v = pro_row(v, w1 * w1y, w0x[p], e1[t10[p]], w1x[p], e1[t11[p]]);
                    v = o.a + v;
                    if (p == 0) {
                        if (con) C[(Z + 2) & 3][u] = cnext;
                        cnext = cplane(Z + 3);
                    }
                } else {
                    v = o.a * o.b;
                }
                if (on) E[k][u] = okz && ok[p] ? v : (T)0;
            });
        if (DOTS) lds_barrier();
        return;
    }
    // black values of plane z0 - 4 + s into B[s & 1] (the red start around it is
    // in E[s - 3 .. s - 1]); red values of the plane below, whose black values
    // are in B[s - 1], and its store
    const typename Sh::Lane P(g, wave - Sh::wB, (int)threadIdx.x & (kWave - 1), x0, y0);
    const int q = (P.ly + 1) * kUM + P.m, qb = P.ly * kUM + P.m;
    // (the outermost pairs' and rows' outer neighbours are not used)
    const int ql = P.m > 0 ? q - 1 : q, qh = P.m < kUM - 1 ? q + 1 : q;
    const int xl = P.m > 0 ? qb - 1 : qb, xh = P.m < kUM - 1 ? qb + 1 : qb;
    const int yl = P.ly > 0 ? qb - kUM : qb, yh = P.ly < Sh::rows - 1 ? qb + kUM : qb;
    const unsigned off = P.c * (unsigned)sizeof(T), offn = P.n * (unsigned)sizeof(T), offh = P.h * (unsigned)sizeof(T);
    constexpr bool same = std::is_same<T, TR>::value;   // r is b
    double arz = 0.0, az = 0.0, ar = 0.0;
    if (PRO) lds_barrier();
    struct Ops {
        Pair2<T> b, d, c0, c1, h1, c2;   // c2: of the plane above
        T n;
        Pair2<TR> r;                     // of the plane below
    };
    auto run = [&](auto RP) {
        constexpr int rpar = decltype(RP)::value;
        asm volatile("; rows of parity %0" ::"n"(rpar));   // keeps the two parities' loads apart
        // of the plane below: b, the red cell's 1 / d and coefficients but the
        // upper one, the black value; the black value below that
        Pair2<T> kb;
        T kd = 0.0, kw[5], v1 = 0.0, v2 = 0.0;
        kb.v[0] = kb.v[1] = (T)0;
#pragma unroll
        for (int i = 0; i < 5; ++i) kw[i] = (T)0;
        int gf;
        (void)wrap_axis(z0 - 1, nz, g.per[2], gf);
        Pair2<T> c2 = pair_at(L.cs[2] + gf * nxy, off);
        sweep_role<3, Ops>(
            n + 4, total,
            [&](int s, auto, Ops &o) {
                int gz, gh;
                (void)wrap_axis(z0 - 4 + s, nz, g.per[2], gz);
                (void)wrap_axis(z0 - 3 + s, nz, g.per[2], gh);
                const long long z = gz * nxy;
                o.b = pair_at((const T *)(const void *)b + z, off);
                o.d = pair_at(L.invd + z, off);
                o.c0 = pair_at(L.cs[0] + z, off);
                o.n = plane_at(L.cs[0] + z, offn);
                o.c1 = pair_at(L.cs[1] + z, off);
                o.h1 = pair_at(L.cs[1] + z, offh);
                o.c2 = pair_at(L.cs[2] + gh * nxy, off);
                if (DOTS && !same) {
                    const int zr = z0 - 5 + s < z0 ? z0 : (z0 - 5 + s < nz ? z0 - 5 + s : nz - 1);
                    o.r = pair_at(r + zr * nxy, P.c * (unsigned)sizeof(TR));
                }
            },
            [&](int s, auto K, const Ops &o) {
                constexpr int k = decltype(K)::value, blk = (rpar + k) & 1, red = 1 - blk;
                const int p = z0 - 4 + s;
                int gz;
                const bool okz = wrap_axis(p, nz, g.per[2], gz);
                T val;
                {
                    const T *e0 = E[(k + 2) & 3], *em = E[(k + 1) & 3], *ep = E[(k + 3) & 3];
                    const T v[6] = {blk ? e0[q] : e0[ql], blk ? e0[qh] : e0[q], e0[q - kUM], e0[q + kUM], em[q], ep[q]};
                    const T w[6] = {o.c0.v[blk], blk ? o.n : o.c0.v[1], o.c1.v[blk], o.h1.v[blk], c2.v[blk], o.c2.v[blk]};
                    T acc = 0.0;
#pragma unroll
                    for (int i = 0; i < 6; ++i) acc = fmar(w[i], v[i], acc);
                    val = (o.b.v[blk] + acc) * o.d.v[blk];
                    val = okz && P.ok ? val : (T)0;
                    if (P.on) B[k & 1][qb] = val;
                }
                {
                    // (the plane below has its red and black cells the other way round)
                    const T *a = B[(k + 1) & 1];
                    const T v[6] = {blk ? v1 : a[xl], blk ? a[xh] : v1, a[yl], a[yh], v2, val};
                    T acc = 0.0;
#pragma unroll
                    for (int i = 0; i < 5; ++i) acc = fmar(kw[i], v[i], acc);
                    acc = fmar(c2.v[blk], v[5], acc);
                    Pair2<T> t;
                    t.v[blk] = (kb.v[blk] + acc) * kd;
                    t.v[red] = v1;
                    if (P.own && p > z0 && p <= z1) {
                        *(Pair2<T> *)((char *)(x + (p - 1) * nxy) + off) = t;
                        if (DOTS) {
                            if constexpr (same)
                                sweep_dots(kb, t, arz, az, ar);
                            else
                                sweep_dots(o.r, t, arz, az, ar);
                        }
                    }
                }
                kb = o.b;
                kd = o.d.v[red];
                kw[0] = o.c0.v[red];
                kw[1] = red ? o.n : o.c0.v[1];
                kw[2] = o.c1.v[red];
                kw[3] = o.h1.v[red];
                kw[4] = c2.v[red];
                c2 = o.c2;
                v2 = v1;
                v1 = val;
            });
    };
    if (P.rp)
        run(std::integral_constant<int, 1>());
    else
        run(std::integral_constant<int, 0>());
    if (DOTS) sweep_partials(arz, az, ar, (int)threadIdx.x - Sh::wB * kWave, ws, p0 + tile, p1 + tile, p2 + tile);
}

// The same partials in the same order as a pass of its own, for a level 0
// that runs the tile passes: one block per block of the sweep, one thread per
// pair of cells of its column, marching along z.  Both forms of the cycle then
// give the same bits.  Its few blocks cost nothing against k_pcg_rz (their
// partials are what the next kernel sums): whole pressure solves with it and with
// k_pcg_rz, FP64, 16^3 638 and 662 us, 32^3 923 and 948, 48^3 1047 and 1075.
template <typename T, typename TZ>
__global__ void __launch_bounds__(SweepShape::nB * kWave) k_pcg_rz3(Geo g, const T *__restrict__ r,
                                                                    const TZ *__restrict__ z,
                                                                    const Scal *__restrict__ sc,
                                                                    double *__restrict__ p0, double *__restrict__ p1,
                                                                    double *__restrict__ p2, int ntx, int ncol, int zc,
                                                                    int ntiles) {
    const int tile = xcd_block();
    if (tile >= ntiles || sc->done) return;
    __shared__ double ws[3][SweepShape::nB];
    const int nxy = g.n[0] * g.n[1];
    const int col = tile % ncol, z0 = (tile / ncol) * zc, z1 = z0 + zc < g.n[2] ? z0 + zc : g.n[2];
    const SweepShape::Lane P(g, __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), (int)threadIdx.x & (kWave - 1),
                             (col % ntx) * kUX, (col / ntx) * kUY);
    double arz = 0.0, az = 0.0, ar = 0.0;
    if (P.own) {
#pragma unroll 4
        for (int kz = z0; kz < z1; ++kz) {
            const Pair2<T> rc = *(const Pair2<T> *)(r + P.c + (long long)kz * nxy);
            const Pair2<TZ> zv = *(const Pair2<TZ> *)(z + P.c + (long long)kz * nxy);
            sweep_dots(rc, zv, arz, az, ar);
        }
    }
    sweep_partials(arz, az, ar, (int)threadIdx.x, ws, p0 + tile, p1 + tile, p2 + tile);
}

// ---------------------------------------------------------------------------
// 3D way down of a level in one pass: zero-guess pre-smoothing (red x = b / d,
// black from those), the residual, its restriction.  After the black sweep the
// residual of a black cell is 0 and that of a red cell is the sum of its
// black neighbours' x over the face coefficients (d x = b cancels), so only
// red residuals are formed, s is not read, and the restriction takes the 32
// red of its 64 taps.
// Columns of kUX x kUY cells march along z as in k_sweep3, with three roles:
// red values b / d (halo of 3 cells), black values and, two planes behind, the
// red residuals (halos of 2 and 1), and two waves with a coarse cell per lane,
// which add a plane of residuals per step to the two coarse planes it
// contributes to.  The lanes of a wave of the second role have rows of one parity,
// so which cell of a pair is red is known at compile time and both cells'
// coefficients come from one load per pair (a load of every second cell
// touches as many cache lines).
// b, 1 / d and three coefficients are read and x written once: 48 B per cell in
// FP64 where pre-smoothing, residual and restriction moved 121.  Measured
// against these three: 128^3 FP64 43.7 us -> 21.3, FP32 29.8 -> 14.9; 96^3 FP64
// 34.3 -> 14.2; 512^3 3.37 ms -> 1.82.  What bounds it is, at 512^3, memory (the
// least bytes take 1.35 ms; halo lines that have left the L2 make it fetch 1.7
// times them), and below the cache lines a CU can look up (halos of 3, 2 and
// 1 cells) and the steps by which the roles trail.  b and 1 / d go to the second
// role through LDS: with loads of its own, 128^3 24.7, 96^3 15.7, 512^3 2.06.
// 8 rows per column instead of 16: 96^3 level and 128^3 10 % slower, 512^3 solve
// 377 ms against 350.
// ---------------------------------------------------------------------------
struct DownShape {
    static constexpr int DM = kUX / 2 + 4, D = (kUY + 6) * DM;   // pairs of the red values: per row, per plane
    static constexpr int rows = kUY + 4, X = rows * kUM;         // black values and residuals
    using Lane = PairLane<rows, 2>;
    static constexpr int wX = (D + kWave - 1) / kWave, wC = wX + Lane::waves;
    static constexpr int wN = kUX / 2 * kUY / 2 / kWave;   // a coarse cell per lane
    static constexpr int threads = (wC + wN) * kWave;
};

template <typename T, typename TB>
__global__ void __launch_bounds__(DownShape::threads) k_down3(Level<T> L, const TB *__restrict__ b, Geo gc,
                                                              T *__restrict__ xp, T *__restrict__ bc, int ntx,
                                                              int ncol, int zc, int ntiles,
                                                              const int *__restrict__ done) {
    using Sh = DownShape;
    const int tile = xcd_block();
    if (tile >= ntiles || *done) return;
    static_assert(sizeof(T) == sizeof(TB), "offsets in bytes of both");
    __shared__ T D[4][Sh::D], X[2][Sh::X], R[2][Sh::X];
    __shared__ Pair2<T> F[4][2][Sh::D];   // b, 1 / d of the pairs of D
    const Geo &g = L.g;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const long long nxy = (long long)nx * ny;
    const int col = tile % ncol, z0 = (tile / ncol) * zc, z1 = z0 + zc < nz ? z0 + zc : nz, n = z1 - z0;
    const int x0 = (col % ntx) * kUX, y0 = (col / ntx) * kUY;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = (int)threadIdx.x & (kWave - 1);
    const int total = n + 11;   // every role ends its group of four within these steps
    if (wave < Sh::wX) {
        // red b / d of plane z0 - 3 + s, into D[s & 3]; b and 1 / d of both
        // cells for the second role, which would fetch the lines again two
        // planes later
        const int u = (int)threadIdx.x;
        const bool on = u < Sh::D;
        const int ly = on ? u / Sh::DM : 0, m = (on ? u : 0) - ly * Sh::DM;
        int gx, gy;
        const bool ok = wrap_axis(x0 - 4 + 2 * m, nx, g.per[0], gx) & wrap_axis(y0 - 3 + ly, ny, g.per[1], gy);
        gx &= ~1;
        const unsigned off = (unsigned)(gx + nx * gy) * sizeof(T);
        struct Ops {
            Pair2<T> a, d;
        };
        sweep_role<0, Ops>(
            n + 5, total,
            [&](int s, auto, Ops &o) {
                int gz;
                (void)wrap_axis(z0 - 3 + s, nz, g.per[2], gz);
                const long long z = gz * nxy;
                o.a = pair_at((const T *)(const void *)b + z, off);
                o.d = pair_at(L.invd + z, off);
            },
            [&](int s, auto K, const Ops &o) {
                int gz;
                const bool okz = wrap_axis(z0 - 3 + s, nz, g.per[2], gz);
                constexpr int k = decltype(K)::value;
                const bool hi = (ly + k) & 1;   // the red cell of the pair (y0 - 3 + ly + z0 - 3 + s even: the lower one)
                const T v = (hi ? o.a.v[1] : o.a.v[0]) * (hi ? o.d.v[1] : o.d.v[0]);
                if (on) {
                    D[k][u] = okz && ok ? v : (T)0;
                    F[k][0][u] = o.a;
                    F[k][1][u] = o.d;
                }
            });
        return;
    }
    if (wave < Sh::wC) {
        // black values of plane z0 - 5 + s into X[s & 1] (the red ones around
        // it are in D[s - 3 .. s - 1]); red residuals of the plane below into
        // R[s & 1] (its black values are in X[s - 1]; the black cells above and
        // below a red one are in this lane's pair)
        const typename Sh::Lane P(g, wave - Sh::wX, lane, x0, y0);
        const bool on = P.on, ok = P.ok, own = P.own;
        const int ly = P.ly, m = P.m;
        const unsigned off = P.c * (unsigned)sizeof(T), offn = P.n * (unsigned)sizeof(T), offh = P.h * (unsigned)sizeof(T);
        const int q = (ly + 1) * Sh::DM + m + 1, qx = ly * kUM + m;
        // (the outermost pairs' and rows' outer neighbours are not used)
        const int xl = m > 0 ? qx - 1 : qx, xh = m < kUM - 1 ? qx + 1 : qx;
        const int yl = ly > 0 ? qx - kUM : qx, yh = ly < Sh::rows - 1 ? qx + kUM : qx;
        struct Ops {
            T n;
            Pair2<T> c0, c1, h1, c2;   // c2: of the plane above
        };
        auto run = [&](auto RP) {
            constexpr int rpar = decltype(RP)::value;
        asm volatile("; rows of parity %0" ::"n"(rpar));   // keeps the two parities' loads apart
            // of the plane below: the red cell's coefficients but the upper one,
            // the black value; the black value below that
            T keep[5], v1 = 0.0, v2 = 0.0;
#pragma unroll
            for (int i = 0; i < 5; ++i) keep[i] = (T)0;
            int gf;
            (void)wrap_axis(z0 - 2, nz, g.per[2], gf);
            Pair2<T> c2 = pair_at(L.cs[2] + gf * nxy, off);
            sweep_role<3, Ops>(
                n + 6, total,
                [&](int s, auto, Ops &o) {
                    int gz, gh;
                    (void)wrap_axis(z0 - 5 + s, nz, g.per[2], gz);
                    (void)wrap_axis(z0 - 4 + s, nz, g.per[2], gh);
                    const long long z = gz * nxy;
                    o.c0 = pair_at(L.cs[0] + z, off);
                    o.n = plane_at(L.cs[0] + z, offn);
                    o.c1 = pair_at(L.cs[1] + z, off);
                    o.h1 = pair_at(L.cs[1] + z, offh);
                    o.c2 = pair_at(L.cs[2] + gh * nxy, off);
                },
                [&](int s, auto K, const Ops &o) {
                    constexpr int k = decltype(K)::value, blk = (rpar + k) & 1, red = 1 - blk;   // the pair's black and red cell
                    const int p = z0 - 5 + s;
                    int gz;
                    const bool okz = wrap_axis(p, nz, g.per[2], gz);
                    T val;
                    {
                        const T *d0 = D[(k + 2) & 3], *dm = D[(k + 1) & 3], *dp = D[(k + 3) & 3];
                        const T dq = d0[q];
                        const T v[6] = {blk ? dq : d0[q - 1], blk ? d0[q + 1] : dq, d0[q - Sh::DM], d0[q + Sh::DM], dm[q], dp[q]};
                        const T wt[6] = {o.c0.v[blk], blk ? o.n : o.c0.v[1], o.c1.v[blk], o.h1.v[blk], c2.v[blk], o.c2.v[blk]};
                        T acc = 0.0;
#pragma unroll
                        for (int i = 0; i < 6; ++i) acc = fmar(wt[i], v[i], acc);
                        val = (F[(k + 2) & 3][0][q].v[blk] + acc) * F[(k + 2) & 3][1][q].v[blk];
                        val = okz && ok ? val : (T)0;
                        if (on) X[k & 1][qx] = val;
                        if (own && p >= z0 && p < z1) {
                            Pair2<T> t;
                            t.v[blk] = val;
                            t.v[red] = dq;
                            *(Pair2<T> *)((char *)(xp + p * nxy) + off) = t;
                        }
                    }
                    {
                        // (the plane below has its red and black cells the other way round)
                        const T *a = X[(k + 1) & 1];
                        const T v[6] = {blk ? v1 : a[xl], blk ? a[xh] : v1, a[yl], a[yh], v2, val};
                        T acc = 0.0;
#pragma unroll
                        for (int i = 0; i < 5; ++i) acc = fmar(keep[i], v[i], acc);
                        acc = fmar(c2.v[blk], v[5], acc);
                        if (on) R[k & 1][qx] = acc;
                    }
                    keep[0] = o.c0.v[red];
                    keep[1] = red ? o.n : o.c0.v[1];
                    keep[2] = o.c1.v[red];
                    keep[3] = o.h1.v[red];
                    keep[4] = c2.v[red];
                    c2 = o.c2;
                    v2 = v1;
                    v1 = val;
                });
        };
        if (P.rp)
            run(std::integral_constant<int, 1>());
        else
            run(std::integral_constant<int, 0>());
        return;
    }
    // coarse cell (I, J) of this lane: plane z0 - 7 + s of the residual (in
    // R[s - 1]) is tap 2 of coarse plane Z and tap 0 of Z + 1 (an odd plane), or
    // tap 3, the last, of Z and tap 1 of Z + 1
    const int u = (int)threadIdx.x - Sh::wC * kWave, i = u % (kUX / 2), j = u / (kUX / 2), I = x0 / 2 + i, J = y0 / 2 + j;
    const bool own = I < gc.n[0] && J < gc.n[1];
    int f[4];
    T wx[4], wy[4], wo[4], wn[4];
    res_axis<T>(own ? I : 0, gc.n[0], nx, gc.per[0], f, wx);
    res_axis<T>(own ? J : 0, gc.n[1], ny, gc.per[1], f, wy);
    res_axis<T>(z0 / 2, gc.n[2], nz, gc.per[2], f, wn);
#pragma unroll
    for (int a = 0; a < 4; ++a) wo[a] = (T)0;
    T ao = 0.0, an = 0.0;   // sums of Z and Z + 1
    struct None {};
    sweep_role<6, None>(
        n + 7, total, [](int, auto, None &) {},
        [&](int s, auto K, const None &) {
            constexpr int k = decltype(K)::value, odd = (k + 1) & 1;
            const T *r = R[(k + 1) & 1];
            T sum[4];
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                // row 2 J - 1 + y: its red cells are at even or (par) odd x (z0 and y0 are even)
                const int par = (y + 1 + odd) & 1;
                const T *rr = r + (2 * j + y + 1) * kUM + i + (par ? 0 : 1);
                sum[y] = fmar(wx[par ? 2 : 3], rr[1], fmar(wx[par ? 0 : 1], rr[0], (T)0));
            }
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                ao = fmar(wy[y] * wo[odd ? 2 : 3], sum[y], ao);
                an = fmar(wy[y] * wn[odd ? 0 : 1], sum[y], an);
            }
            if (!odd) {
                const int Z = (z0 - 7 + s) / 2 - 1;
                if (own && s >= 9 && s <= n + 7) bc[(Z * gc.n[1] + J) * gc.n[0] + I] = ao;
                ao = an;
                an = (T)0;
#pragma unroll
                for (int a = 0; a < 4; ++a) wo[a] = wn[a];
                const int Zn = Z + 2 < gc.n[2] ? Z + 2 : gc.n[2] - 1;
                res_axis<T>(Zn, gc.n[2], nz, gc.per[2], f, wn);
            }
        });
}

// Columns, planes per block (a multiple of 4) and blocks of these passes.  A CU
// holds one block (12 or 15 waves of up to 128 registers), so a pass takes
// ceil(blocks / CUs) rounds of a chunk's planes and the steps by which its
// roles trail: the planes that make this least.  Whole FP64 pressure solves with
// 4, 8, 16, 32 and 64 planes on every level: 64^3 1.45, 1.59, 1.77, 2.15, 2.96 ms;
// 96^3 2.43, 2.23, 2.41, 2.82, 3.67; 128^3 5.24, 4.66, 4.56, 5.53, 7.80 (the rule,
// level by level, 4.14); 192^3 20.0, 17.3, 16.4, 16.1, 17.3 (14.3); 256^3 57.7, 48.6,
// 43.0, 40.0, 43.5 (34.9).  max_blocks: more planes where the blocks outnumber
// the partials of r.z.
constexpr int kSweepTrail = 8, kDownTrail = 11;
static int march3_grid(const Geo &g, int trail, int max_blocks, int &ntx, int &ncol, int &zc, int &ntiles) {
    ntx = (g.n[0] + kUX - 1) / kUX;
    ncol = ntx * ((g.n[1] + kUY - 1) / kUY);
    auto blocks = [&](int z) { return ncol * ((g.n[2] + z - 1) / z); };
    auto steps = [&](int z) { return (long long)((blocks(z) + kCUs - 1) / kCUs) * (z + trail); };
    zc = 4;
    for (int z = 8; z / 2 < g.n[2]; z *= 2)
        if (steps(z) < steps(zc) || (max_blocks && blocks(zc) > max_blocks)) zc = z;
    ntiles = blocks(zc);
    return ntiles > 8 ? (ntiles + 7) & ~7 : ntiles;
}
static int sweep3_grid(const Geo &g, int &ntx, int &ncol, int &zc, int &ntiles) {
    return march3_grid(g, kSweepTrail, kRedBlocks, ntx, ncol, zc, ntiles);
}

// Whether level l of a 3D slot runs the tile passes: above the
// single-workgroup part, below march_cells and at most tile_cells cells,
// with even extents (every level that has a coarser one).
template <typename T>
static bool tile3_level(const Slot<T> &S, int l) {
    const Geo &g = S.lev[l].g;
    return l + 1 < S.nlev && g.N <= S.tile_cells && g.N < S.march_cells && (g.n[0] & 1) == 0 &&
           (g.n[1] & 1) == 0 && (g.n[2] & 1) == 0;
}

static inline int tile3_grid(const Geo &gc, int &ntx, int &nty, int &ntiles) {
    ntx = (gc.n[0] + kTC - 1) / kTC;
    nty = (gc.n[1] + kTC - 1) / kTC;
    ntiles = ntx * nty * ((gc.n[2] + kTC - 1) / kTC);
    return ntiles > 8 ? (ntiles + 7) & ~7 : ntiles;
}

// CH operator, first half: p_new = z + beta p_old, t = L p_new.
template <typename T, typename TZ, int DIM>
__global__ void __launch_bounds__(kBlock) k_pcg_ch_lap(Geo g, double ih2, const TZ *__restrict__ z,
                                                       const T *__restrict__ pold, T *__restrict__ pnew,
                                                       T *__restrict__ t, Scal *sc, const double *__restrict__ rz0,
                                                       int nrz, int k, T *__restrict__ rpend,
                                                       const T *__restrict__ q) {
    if (sc->done) return;
    const double alpha_prev = rpend ? sc->alpha : 0.0;
    IterStart it;
    if (!iter_start(sc, rz0, rz0, rz0, nrz, g.N, k, 0, it)) return;
    const double beta = it.beta;
    auto pv = [&](int e) { return (double)z[e] + (beta != 0.0 ? beta * (double)pold[e] : 0.0); };
    GRID_LOOP(g.N) {
        int ia[3];
        coords_of<DIM>(g, c, ia);
        // residual of the previous iteration (q is rewritten by the second half)
        if (rpend) rpend[c] = (T)cg_residual((double)rpend[c], (double)q[c], alpha_prev);
        pnew[c] = (T)pv(c);
        t[c] = (T)lap_at<DIM>(g, c, ia, ih2, pv);
    }
}

// CH operator, second half: q = p - a t + b L t; partial p.q.
template <typename T, int DIM>
__global__ void __launch_bounds__(kBlock) k_pcg_ch_apply(Geo g, double ih2, double ca, double cb,
                                                         const T *__restrict__ p, const T *__restrict__ t,
                                                         T *__restrict__ q, const Scal *__restrict__ sc,
                                                         double *__restrict__ part) {
    if (sc->done) return;
    __shared__ double lds[kBlock / kWave];
    auto tv = [&](int e) { return (double)t[e]; };
    double acc = 0.0;
    GRID_LOOP(g.N) {
        int ia[3];
        coords_of<DIM>(g, c, ia);
        const double pc = (double)p[c];
        const double qc = pc - ca * (double)t[c] + cb * lap_at<DIM>(g, c, ia, ih2, tv);
        q[c] = (T)qc;
        acc += pc * qc;
    }
    const double s = block_sum(acc, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// alpha = rz / sum(part_pq) (every block, same order); x += alpha p;
// r -= alpha q; partial r.r.  TP != T: also rp = r rounded to TP (the
// right-hand side of the preconditioner in its own precision).
template <typename T, typename TP = T>
__global__ void __launch_bounds__(kBlock) k_pcg_update(int N, const T *__restrict__ p, const T *__restrict__ q,
                                                       T *__restrict__ x, T *__restrict__ r, Scal *sc,
                                                       const double *__restrict__ part_pq, int nparts,
                                                       double *__restrict__ part_rr, TP *__restrict__ rp = nullptr) {
    if (sc->done) return;
    __shared__ double lds[kBlock / kWave];
    const double pq = sum_parts_all(part_pq, nparts, lds);
    const double alpha = pq != 0.0 ? sc->rz / pq : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->pq = pq;
        sc->alpha = alpha;
    }
    double acc = 0.0;
    GRID_LOOP(N) {
        x[c] = (T)((double)x[c] + alpha * (double)p[c]);
        const double rc = cg_residual((double)r[c], (double)q[c], alpha);
        r[c] = (T)rc;
        if constexpr (!std::is_same<T, TP>::value) rp[c] = (TP)(T)rc;
        acc += rc * rc;
    }
    const double s = block_sum(acc, lds);
    if (threadIdx.x == 0) part_rr[blockIdx.x] = s;
}

// rp = r rounded to the preconditioner's precision
template <typename T, typename TP>
__global__ void __launch_bounds__(kBlock) k_round_vec(int N, const T *__restrict__ r, TP *__restrict__ rp) {
    GRID_LOOP(N) rp[c] = (TP)r[c];
}

// one workgroup: rr = sum(part_rr); iteration count; convergence flag
__global__ void __launch_bounds__(kBlock) k_pcg_fin_rr(Scal *sc, const double *__restrict__ part_rr, int nparts) {
    if (sc->done) return;
    __shared__ double lds[kBlock / kWave];
    pcg_fin_rr_dev(sc, *sc, sum_parts_all(part_rr, nparts, lds));
}

// partials of r.z, sum z, sum r
template <typename T, typename TZ>
__global__ void __launch_bounds__(kBlock) k_pcg_rz(int N, const T *__restrict__ r, const TZ *__restrict__ z,
                                                   const Scal *__restrict__ sc, double *__restrict__ p0,
                                                   double *__restrict__ p1, double *__restrict__ p2, int singular) {
    if (sc->done) return;
    __shared__ double lds[kBlock / kWave];
    double arz = 0.0, az = 0.0, ar = 0.0;
    GRID_LOOP(N) {
        const double rc = (double)r[c], zc = (double)z[c];
        arz += rc * zc;
        az += zc;
        ar += rc;
    }
    const double s0 = block_sum(arz, lds);
    const double s1 = singular ? block_sum(az, lds) : 0.0;
    const double s2 = singular ? block_sum(ar, lds) : 0.0;
    if (threadIdx.x == 0) {
        p0[blockIdx.x] = s0;
        p1[blockIdx.x] = s1;
        p2[blockIdx.x] = s2;
    }
}

// r = b - A x (slot operator); partials of b.b and r.r; rp (when given):
// r rounded to the preconditioner's precision.  conv: also the level-0
// arrays of the preconditioner's hierarchy B that the set-up would write
// (a cycle that ends on the grid needs nothing else): 1 / diag, and for a
// lower precision the rounded s and cs[b], with the arithmetic and order of
// k_invd / k_conv_coef (bit for bit).
template <typename T, int DIM, typename TP = T>
__global__ void __launch_bounds__(kBlock) k_pcg_init_slot(Level<T> L, const T *__restrict__ b,
                                                          const T *__restrict__ x, T *__restrict__ r,
                                                          double *__restrict__ p0, double *__restrict__ p1,
                                                          TP *__restrict__ rp, Level<TP> B, int conv) {
    constexpr bool kSame = std::is_same<T, TP>::value;
    __shared__ double lds[kBlock / kWave];
    double bb = 0.0, rr = 0.0;
    GRID_LOOP(L.g.N) {
        int ia[3];
        coords_of<DIM>(L.g, c, ia);
        const double bc = (double)b[c];
        const double rc = bc - apply_at<T, DIM>(L, x, c, ia);
        r[c] = (T)rc;
        if (rp) rp[c] = (TP)(T)rc;   // the preconditioner's copy (k_round_vec's value)
        bb += bc * bc;
        rr += rc * rc;
        if (conv) {
            const TP sv = (TP)L.s[c];
            if (!kSame) B.s[c] = sv;
            TP d = sv;
#pragma unroll
            for (int q = 0; q < DIM; ++q) {
                const TP w = (TP)L.cs[q][c];
                if (!kSame) B.cs[q][c] = w;
                if (nb_lo(L.g, c, ia[q], q) >= 0) d += w;
                const int hi = nb_hi(L.g, c, ia[q], q);
                if (hi >= 0) d += (TP)L.cs[q][hi];
            }
            B.invd[c] = (TP)1 / d;
        }
    }
    const double s0 = block_sum(bb, lds);
    const double s1 = block_sum(rr, lds);
    if (threadIdx.x == 0) {
        p0[blockIdx.x] = s0;
        p1[blockIdx.x] = s1;
    }
}

// zero initial guess: x = 0, r = b; partials of b.b (twice)
template <typename T>
__global__ void __launch_bounds__(kBlock) k_pcg_init_zero(int N, const T *__restrict__ b, T *__restrict__ x,
                                                          T *__restrict__ r, double *__restrict__ p0,
                                                          double *__restrict__ p1) {
    __shared__ double lds[kBlock / kWave];
    double bb = 0.0;
    GRID_LOOP(N) {
        const T bc = b[c];
        x[c] = (T)0;
        r[c] = bc;
        bb += (double)bc * (double)bc;
    }
    const double s0 = block_sum(bb, lds);
    if (threadIdx.x == 0) {
        p0[blockIdx.x] = s0;
        p1[blockIdx.x] = s0;
    }
}

template <typename T, int DIM>
__global__ void __launch_bounds__(kBlock) k_ch_lap_plain(Geo g, double ih2, const T *__restrict__ x,
                                                         T *__restrict__ t) {
    auto xv = [&](int e) { return (double)x[e]; };
    GRID_LOOP(g.N) {
        int ia[3];
        coords_of<DIM>(g, c, ia);
        t[c] = (T)lap_at<DIM>(g, c, ia, ih2, xv);
    }
}

// CH: r = b - (x - a t + b L t) with t = L x; partials b.b, r.r
template <typename T, int DIM>
__global__ void __launch_bounds__(kBlock) k_pcg_init_ch(Geo g, double ih2, double ca, double cb,
                                                        const T *__restrict__ b, const T *__restrict__ x,
                                                        const T *__restrict__ t, T *__restrict__ r,
                                                        double *__restrict__ p0, double *__restrict__ p1) {
    __shared__ double lds[kBlock / kWave];
    auto tv = [&](int e) { return (double)t[e]; };
    double bb = 0.0, rr = 0.0;
    GRID_LOOP(g.N) {
        int ia[3];
        coords_of<DIM>(g, c, ia);
        const double Mx = (double)x[c] - ca * (double)t[c] + cb * lap_at<DIM>(g, c, ia, ih2, tv);
        const double bc = (double)b[c];
        const double rc = bc - Mx;
        r[c] = (T)rc;
        bb += bc * bc;
        rr += rc * rc;
    }
    const double s0 = block_sum(bb, lds);
    const double s1 = block_sum(rr, lds);
    if (threadIdx.x == 0) {
        p0[blockIdx.x] = s0;
        p1[blockIdx.x] = s1;
    }
}

// one workgroup: initialise the scalars from the b.b and r0.r0 partials
__global__ void __launch_bounds__(kBlock) k_pcg_fin_init(Scal *sc, const double *__restrict__ p0,
                                                         const double *__restrict__ p1, int nparts, double rtol,
                                                         int max_iter) {
    __shared__ double lds[kBlock / kWave];
    const double tb = sum_parts_all(p0, nparts, lds);
    const double tr = sum_parts_all(p1, nparts, lds);
    if (threadIdx.x == 0) {
        sc->bb = tb > tr ? tb : tr;
        sc->rr = tr;
        sc->rtol2 = rtol * rtol;
        sc->iter = 0;
        sc->max_iter = max_iter;
        sc->unconverged = 0;
        sc->nonfinite = 0;
        sc->beta = 0.0;
        sc->rz = 0.0;
        sc->zmean = 0.0;
        sc->alpha = 0.0;
        sc->done = 0;
        if (!isfinite(tr) || !isfinite(tb)) {
            sc->nonfinite = 1;
            sc->done = 1;
        } else if (tr <= sc->rtol2 * sc->bb) {
            sc->done = 1;
        }
    }
}

// mean removal: partial sums, then every block sums them and subtracts
template <typename T>
__global__ void __launch_bounds__(kBlock) k_sum(int N, const T *__restrict__ x, double *__restrict__ part) {
    __shared__ double lds[kBlock / kWave];
    double acc = 0.0;
    GRID_LOOP(N) acc += (double)x[c];
    const double s = block_sum(acc, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// x -= mean(x); copy (when given) receives the same values
template <typename T>
__global__ void __launch_bounds__(kBlock) k_sub_mean(int N, T *__restrict__ x, const double *__restrict__ part,
                                                     int nparts, T *__restrict__ copy) {
    __shared__ double lds[kBlock / kWave];
    const double m = sum_parts_all(part, nparts, lds) / (double)N;
    GRID_LOOP(N) {
        const T v = (T)((double)x[c] - m);
        x[c] = v;
        if (copy) copy[c] = v;
    }
}

template <typename T, int DIM>
__global__ void __launch_bounds__(kBlock) k_slot_apply(Level<T> L, const T *__restrict__ x, T *__restrict__ y) {
    GRID_LOOP(L.g.N) {
        int ia[3];
        coords_of<DIM>(L.g, c, ia);
        y[c] = (T)apply_at<T, DIM>(L, x, c, ia);
    }
}

// ---------------------------------------------------------------------------
// host drivers
// ---------------------------------------------------------------------------
#define LAUNCH(cls, bytes, kern, n, st, ...) TLAUNCH(cls, bytes, kern, dim3(grid_for(n)), dim3(kBlock), st, __VA_ARGS__)
#define LAUNCH1(cls, bytes, kern, threads, st, ...) TLAUNCH(cls, bytes, kern, dim3(1), dim3(threads), st, __VA_ARGS__)
// kernels that produce per-block partials use at most kRedBlocks blocks
#define LAUNCHR(cls, bytes, kern, n, st, ...) TLAUNCH(cls, bytes, kern, dim3(grid_red(n)), dim3(kBlock), st, __VA_ARGS__)

// First level handled by the single-workgroup kernel.
template <typename T>
static int single_block_level(const Slot<T> &S) {
    int l = 0;
    const int lim = sb_cells();
    while (l < S.nlev - 1 && S.lev[l].g.N > lim) ++l;
    return l;
}

// Level at which the V-cycle of S ends (-1: it runs down to the coarsest).
template <typename T>
static int trunc_level(const Slot<T> &S, int dim) {
    return dim == 3 && S.ltrunc >= 0 && S.ltrunc < S.lsb ? S.ltrunc : -1;
}

template <typename T, int DIM>
static void mg_setup_d(Slot<T> &S, hipStream_t st, bool invd0) {
    constexpr double W = sizeof(T);
    S.lsb = single_block_level(S);
    const int lsb = S.lsb;
    const int lt = trunc_level(S, DIM);
    if (lsb > 0 && invd0)
        LAUNCH(K_MG_SETUP, W * (2 + DIM) * S.lev[0].g.N, (k_invd<T, DIM>), S.lev[0].g.N, st, S.lev[0]);
    for (int l = 1; l < (lt >= 0 ? lt + 1 : lsb); ++l) {
        LAUNCH(K_MG_SETUP, W * (1 + DIM) * (S.lev[l - 1].g.N + S.lev[l].g.N), (k_coarsen<T, DIM>), S.lev[l].g.N, st,
               S.lev[l - 1], S.lev[l]);
        LAUNCH(K_MG_SETUP, W * (2 + DIM) * S.lev[l].g.N, (k_invd<T, DIM>), S.lev[l].g.N, st, S.lev[l]);
    }
    if (lt >= 0) return;   // the cycle ends at level lt: no small levels, no coarsest inverse
    double bytes = 0.0;
    for (int l = lsb; l < S.nlev; ++l) bytes += W * (2 + 2 * DIM) * S.lev[l].g.N;
    bytes += 8.0 * S.ncoarse * S.ncoarse;
    const int n = S.ncoarse, nb = (n + kGjB - 1) / kGjB;
    if (n <= kLdsInverse) {
        LAUNCH1(K_MG_SETUP, bytes, (k_setup_block<T, DIM>), kSBThreads, st, S, lsb, (double *)nullptr);
        return;
    }
    // the block steps go back and forth between aug and Ainv and end in Ainv
    double *a = (nb & 1) ? S.aug : S.Ainv, *b = (nb & 1) ? S.Ainv : S.aug;
    LAUNCH1(K_MG_SETUP, bytes, (k_setup_block<T, DIM>), kSBThreads, st, S, lsb, a);
    const dim3 tiles((n + kGjT - 1) / kGjT, (n + kGjT - 1) / kGjT);
    for (int k = 0; k < nb; ++k) {
        TLAUNCH(K_MG_SETUP, 16.0 * n * n, (k_gj_step), tiles, dim3(kBlock), st, n, k * kGjB, (const double *)a, b);
        std::swap(a, b);
    }
}

template <typename T>
void mg_setup(Slot<T> &S, int dim, hipStream_t st, bool invd0) {
    if (dim == 2)
        mg_setup_d<T, 2>(S, st, invd0);
    else
        mg_setup_d<T, 3>(S, st, invd0);
}

// 2D tile grid of a level: tiles along x, rounded up to whole XCD groups
// Level-0 role of a 2D V-cycle inside CG (tile kernels only): down_upd:
// the way down also performs the CG update of the iteration
// (k_down_tile2_cg, then k_pcg_fin_rr); bpend: the right-hand side is the
// pending residual r - alpha q; dmode: partials of r.z, sum z, sum r on the
// way up (0 none, 1 r as stored, 2 r pending).
template <typename TR>
struct L0Cg {
    int down_upd, bpend, dmode;
    const TR *r, *q, *p;
    TR *x;
    Scal *sc;
    const double *part_pq;
    int npq;
    double *part_rr;
    double *rz0, *rz1, *rz2;
};

static void tile_grid2(const Geo &g, int &ntx, int &ntiles, int &grid) {
    ntx = ((int)g.n[0] + kTFX - 1) / kTFX;
    ntiles = ntx * (((int)g.n[1] + kTFY - 1) / kTFY);
    grid = ntiles > 8 ? (ntiles + 7) & ~7 : ntiles;
}

// The r.z partials of CG (k_pcg_rz) taken by the last pass of a 3D
// preconditioner, k_sweep3 on level 0: *nparts is the number of partials
// where that pass took them, one per block.
template <typename TR>
struct RzFuse {
    const TR *r;
    double *p0, *p1, *p2;
    int *nparts;
};

// The post-smoothing of a 3D level in one pass (k_sweep3): from the
// pre-smoothed xpre and the coarse correction xc (PRO), or the symmetric sweep
// from zero; x != xpre; with the r.z partials when rz is given.
template <bool PRO, typename T, typename TB, typename TR>
static void sweep3(const Level<T> &L, const TB *b, const T *xpre, const Geo &gc, const T *xc, T *x, const int *done,
                   hipStream_t st, const RzFuse<TR> *rz) {
    int ntx, ncol, zc, ntiles;
    const int grid = sweep3_grid(L.g, ntx, ncol, zc, ntiles);
    const double N = (double)L.g.N;
    // b, 1 / d, cs, (x and e) in; x out
    const double bytes = sizeof(T) * (5 + (PRO ? 1 : 0)) * N + sizeof(TB) * N + (PRO ? sizeof(T) * (double)gc.N : 0.0);
    if (rz && ntiles <= kRedBlocks) {
        const double r_bytes = std::is_same<T, TR>::value ? 0.0 : sizeof(TR) * N;   // (of one type: r is b)
        TLAUNCH(K_SMOOTH, bytes + r_bytes, (k_sweep3<T, TB, PRO, true, TR>), dim3(grid),
                dim3(SweepShape::threads), st, L, b, xpre, gc, xc, x, ntx, ncol, zc, ntiles, done, rz->r, rz->p0,
                rz->p1, rz->p2);
        *rz->nparts = ntiles;
    } else {
        TLAUNCH(K_SMOOTH, bytes, (k_sweep3<T, TB, PRO, false, TR>), dim3(grid), dim3(SweepShape::threads), st, L, b,
                xpre, gc, xc, x, ntx, ncol, zc, ntiles, done, (const TR *)nullptr, (double *)nullptr,
                (double *)nullptr, (double *)nullptr);
    }
}

template <typename T, typename TB, int DIM, typename TR = T>
static void vcycle_down(Slot<T> &S, int l, const TB *b, T *x, const int *done, hipStream_t st,
                        const L0Cg<TR> *cg = nullptr) {
    constexpr double W = sizeof(T);
    Level<T> &lv = S.lev[l];
    const int N = (int)lv.g.N, Nc = (int)S.lev[l + 1].g.N;
    if (DIM == 2) {
        int ntx, ntiles, grid;
        tile_grid2(lv.g, ntx, ntiles, grid);
        if (cg && cg->down_upd) {
            constexpr double WR = sizeof(TR);
            // r, q, p, x in, x out; invd, cs in; x, bc out
            const double bytes = 5.0 * WR * N + W * (2 + DIM) * N + W * Nc;
            TLAUNCH(K_MG_DOWN, bytes, (k_down_tile2_cg<T, TR>), dim3(grid), dim3(kTileThreads), st, lv,
                    S.lev[l + 1].g, cg->r, cg->q, cg->p, cg->x, lv.r, S.lev[l + 1].b, ntx, ntiles, cg->sc,
                    cg->part_pq, cg->npq, cg->part_rr);
            LAUNCH1(K_PCG_UPDATE, 8.0 * ntiles, (k_pcg_fin_rr), kBlock, st, cg->sc, (const double *)cg->part_rr,
                    ntiles);
            return;
        }
        const double bytes = (sizeof(TB) + W * (2 + DIM)) * N + W * Nc;   // b, invd, cs in; x, bc out
        TLAUNCH(K_MG_DOWN, bytes, (k_down_tile2<T, TB>), dim3(grid), dim3(kTileThreads), st, lv, S.lev[l + 1].g, b,
                lv.r, S.lev[l + 1].b, ntx, ntiles, done);
        return;
    }
    if (DIM == 3 && tile3_level(S, l)) {
        // b, invd, cs in; pre-smoothed x (to r) and the coarse b out
        int ntx, nty, ntiles;
        const int grid = tile3_grid(S.lev[l + 1].g, ntx, nty, ntiles);
        TLAUNCH(K_MG_DOWN, (sizeof(TB) + W * (2 + DIM)) * N + W * Nc, (k_down3_tile<T, TB>), dim3(grid),
                dim3(kT3Threads), st, lv, S.lev[l + 1].g, b, S.lev[l + 1].b, ntx, nty, ntiles, done);
        return;
    }
    if constexpr (DIM == 3) {
        // b, invd, cs in; pre-smoothed x (to r: the way up reads it there while it writes x) and the coarse b out
        int ntx, ncol, zc, ntiles;
        const int grid = march3_grid(lv.g, kDownTrail, 0, ntx, ncol, zc, ntiles);
        TLAUNCH(K_MG_DOWN, (sizeof(TB) + W * (2 + DIM)) * N + W * Nc, (k_down3<T, TB>), dim3(grid),
                dim3(DownShape::threads), st, lv, b, S.lev[l + 1].g, lv.r, S.lev[l + 1].b, ntx, ncol, zc, ntiles, done);
    }
}

template <typename T, typename TB, int DIM, typename TR = T>
static void vcycle_up(Slot<T> &S, int l, const TB *b, T *x, const int *done, hipStream_t st,
                      const L0Cg<TR> *cg = nullptr, const RzFuse<TR> *rz = nullptr) {
    constexpr double W = sizeof(T);
    Level<T> &lv = S.lev[l];
    const int N = (int)lv.g.N, Nc = (int)S.lev[l + 1].g.N;
    if (DIM == 2) {
        int ntx, ntiles, grid;
        tile_grid2(lv.g, ntx, ntiles, grid);
        if constexpr (std::is_same<TB, T>::value) {
            if (cg && (cg->bpend || cg->dmode)) {
                constexpr double WR = sizeof(TR);
                // right-hand side (r, q when pending), invd, cs, x, xc in; x out; r (and q) for the dots
                const double rhs = cg->bpend ? 2.0 * WR : (double)sizeof(TB);
                const double dots = cg->dmode == 0 ? 0.0 : (cg->bpend ? 0.0 : (cg->dmode == 2 ? 2.0 : 1.0) * WR);
                const double bytes = (rhs + dots + W * (3 + DIM)) * N + W * Nc;
                TLAUNCH(K_MG_UP, bytes, (k_up_tile2_cg<T, TR>), dim3(grid), dim3(kTileThreads), st, lv,
                        S.lev[l + 1].g, (const T *)S.lev[l + 1].x, (const T *)b, cg->r, cg->q, (const T *)lv.r, x,
                        ntx, ntiles, (const Scal *)cg->sc, cg->bpend, cg->dmode, cg->rz0, cg->rz1, cg->rz2, done);
                return;
            }
        }
        const double bytes = (sizeof(TB) + W * (3 + DIM)) * N + W * Nc;   // b, invd, cs, x, xc in; x out
        TLAUNCH(K_MG_UP, bytes, (k_up_tile2<T, TB>), dim3(grid), dim3(kTileThreads), st, lv, S.lev[l + 1].g,
                (const T *)S.lev[l + 1].x, b, (const T *)lv.r, x, ntx, ntiles, done);
        return;
    }
    if (DIM == 3 && tile3_level(S, l)) {
        // pre-smoothed x (from r), b, invd, cs, coarse x in; x out
        int ntx, nty, ntiles;
        const int grid = tile3_grid(S.lev[l + 1].g, ntx, nty, ntiles);
        TLAUNCH(K_MG_UP, (sizeof(TB) + W * (3 + DIM)) * N + W * Nc, (k_up3_tile<T, TB>), dim3(grid),
                dim3(kT3Threads), st, lv, S.lev[l + 1].g, (const T *)S.lev[l + 1].x, b, (const T *)lv.r, x, ntx, nty,
                ntiles, done);
        return;
    }
    if constexpr (DIM == 3)
        sweep3<true, T, TB, TR>(lv, b, (const T *)lv.r, S.lev[l + 1].g, (const T *)S.lev[l + 1].x, x, done, st, rz);
}

// The levels [S.lsb, nlev) in one workgroup; b0 / x0: right-hand side and
// result of level 0 where the whole grid is among them.  fin: partials of
// r.r that end the CG iteration of sc (0: none).
template <typename T, typename TB, int DIM>
static void vcycle_small(Slot<T> &S, const TB *b0, T *x0, const int *done, hipStream_t st, Scal *sc = nullptr,
                         const double *fin = nullptr, int nfin = 0) {
    constexpr double W = sizeof(T);
    const int lsb = S.lsb;
    if (const size_t lds = vs_lds_bytes(S, lsb, DIM)) {
        // s, cs, 1 / diag of the swept levels, b and x of the first, the coarsest inverse
        double bytes = 2.0 * W * S.lev[lsb].g.N + 8.0 * S.ncoarse * S.ncoarse + 8.0 * nfin;
        for (int l = lsb; l < S.nlev - 1; ++l) bytes += W * (2 + DIM) * S.lev[l].g.N;
        TLAUNCHS(K_COARSE_SOLVE, bytes, (k_vcycle_lds<T, DIM>), dim3(1), dim3(kVsThreads), lds, st,
                 (vs_args<T, DIM>(S, lsb)), done, sc, fin, nfin);
        return;
    }
    if (nfin) LAUNCH1(K_PCG_UPDATE, 8.0 * nfin, (k_pcg_fin_rr), kBlock, st, sc, fin, nfin);
    double bytes = 8.0 * S.ncoarse * S.ncoarse;
    for (int l = lsb; l < S.nlev; ++l) bytes += W * 12.0 * S.lev[l].g.N;
    if (lsb == 0)
        LAUNCH1(K_COARSE_SOLVE, bytes, (k_vcycle_block<T, TB, DIM>), kSBThreads, st, S, 0, b0, x0, done);
    else
        LAUNCH1(K_COARSE_SOLVE, bytes, (k_vcycle_block<T, T, DIM>), kSBThreads, st, S, lsb, (const T *)S.lev[lsb].b,
                S.lev[lsb].x, done);
}

// One V-cycle of slot S: x0 ~ A^{-1} b0 (b0 may be stored in another
// precision than the hierarchy).
template <typename T, typename TB, int DIM, typename TR = T>
static void vcycle_d(Slot<T> &S, const TB *b0, T *x0, const int *done, hipStream_t st,
                     const L0Cg<TR> *cg = nullptr, const RzFuse<TR> *rz = nullptr) {
    constexpr double W = sizeof(T);
    const int lsb = S.lsb;
    if (const int lt = trunc_level(S, DIM); lt >= 0) {
        // truncated cycle (3D): down to level lt, which is solved by one
        // symmetric red-black Gauss-Seidel sweep from zero (red, black as the
        // zero-guess pre-smoothing, then red again: the backward sweep's black
        // half would repeat the forward one), then back up; at lt = 0 the
        // preconditioner is that sweep alone
        auto sgs = [&](Level<T> &L, const auto *b, T *x, const RzFuse<TR> *rzl) {
            sweep3<false>(L, b, (const T *)nullptr, L.g, (const T *)nullptr, x, done, st, rzl);
        };
        if (lt == 0) {
            sgs(S.lev[0], b0, x0, rz);
            return;
        }
        vcycle_down<T, TB, DIM, TR>(S, 0, b0, x0, done, st, cg);
        for (int l = 1; l < lt; ++l) vcycle_down<T, T, DIM>(S, l, S.lev[l].b, S.lev[l].x, done, st);
        if (DIM == 3 && tile3_level(S, lt)) {
            // (32^3 FP64 5.9 us against 8.6 in k_sweep3, whose 16 blocks march)
            Level<T> &L = S.lev[lt];
            int ntx, nty, ntiles;
            const int grid = tile3_grid(S.lev[lt + 1].g, ntx, nty, ntiles);
            // b, invd, cs in; x out
            TLAUNCH(K_SMOOTH, W * (3 + DIM) * L.g.N, (k_up3_tile<T, T, false>), dim3(grid), dim3(kT3Threads), st, L,
                    S.lev[lt + 1].g, (const T *)nullptr, (const T *)L.b, (const T *)nullptr, L.x, ntx, nty, ntiles, done);
        } else {
            sgs(S.lev[lt], (const T *)S.lev[lt].b, S.lev[lt].x, nullptr);
        }
        for (int l = lt - 1; l >= 1; --l) vcycle_up<T, T, DIM>(S, l, S.lev[l].b, S.lev[l].x, done, st);
        vcycle_up<T, TB, DIM, TR>(S, 0, b0, x0, done, st, cg, rz);
        return;
    }
    if (lsb > 0) {
        vcycle_down<T, TB, DIM, TR>(S, 0, b0, x0, done, st, cg);
        for (int l = 1; l < lsb; ++l) vcycle_down<T, T, DIM>(S, l, S.lev[l].b, S.lev[l].x, done, st);
    }
    vcycle_small<T, TB, DIM>(S, b0, x0, done, st);
    if (lsb > 0) {
        for (int l = lsb - 1; l >= 1; --l) vcycle_up<T, T, DIM>(S, l, S.lev[l].b, S.lev[l].x, done, st);
        vcycle_up<T, TB, DIM, TR>(S, 0, b0, x0, done, st, cg, rz);
    }
}

template <typename T>
void mg_vcycle(Slot<T> &S, int dim, const T *b0, T *x0, const int *done, hipStream_t st) {
    if (dim == 2)
        vcycle_d<T, T, 2>(S, b0, x0, done, st);
    else
        vcycle_d<T, T, 3>(S, b0, x0, done, st);
}

// Preconditioner z = B r with the hierarchy SP (precision TP); r in T.
// rz: the r.z partials of CG (vector precision TR) may ride on the last pass.
template <typename T, typename TP, int DIM, typename TR = T>
static void precond_d(Slot<TP> &SP, OpKind kind, const T *r, TP *z, TP *w, const int *done, hipStream_t st,
                      const RzFuse<TR> *rz = nullptr) {
    if (kind == OP_CH) {
        // M ~ (I - c L)^2 with c = sqrt(b): two V-cycles of the slot operator
        vcycle_d<TP, T, DIM>(SP, r, w, done, st);
        vcycle_d<TP, TP, DIM>(SP, w, z, done, st);
    } else {
        vcycle_d<TP, T, DIM, TR>(SP, r, z, done, st, nullptr, rz);
    }
}

// The same inside CG with the level-0 roles of cg (2D tile levels); for the
// CH operator the first V-cycle takes the update and the pending
// right-hand side, the second the dot products.
template <typename TP, int DIM, typename TR>
static void precond_cg_d(Slot<TP> &SP, OpKind kind, const TP *r, TP *z, TP *w, const int *done, hipStream_t st,
                         const L0Cg<TR> &cg) {
    if (kind == OP_CH) {
        L0Cg<TR> c1 = cg, c2 = cg;
        c1.dmode = 0;
        c2.down_upd = 0;
        c2.bpend = 0;
        vcycle_d<TP, TP, DIM, TR>(SP, r, w, done, st, &c1);
        vcycle_d<TP, TP, DIM, TR>(SP, w, z, done, st, &c2);
    } else {
        vcycle_d<TP, TP, DIM, TR>(SP, r, z, done, st, &cg);
    }
}

// Tiles up to which a 2D solve takes the form with one reduction point per
// iteration.  Every tile of its way down sums four partials per tile, which
// grows with the square of the tiles, and both tile passes stage a wider halo;
// what it saves, two launches and a pass over p and q, grows with the tiles.
// Against launches of their own for apply, update and sums, walled drops, FP64 /
// FP32 hierarchy, pressure solve and whole step: 1152 tiles (768^2) 4 / 3 % and
// 2 / 1 % faster, 1280 (1024 x 640) 4 / 4 and 3 / 2 %, 1408 (1024 x 704) 0 / 1 and
// -1 / 0 %, 1536 (1024 x 768) -1 / 0 and 0 / 0 %, 1792 (1024 x 896) 0 / 0 and
// -2 / -1 %, 2048 (1024^2) -4 / -3 and -5 / -4 % (step 3059 against 3231 us).
constexpr int kCgTiles = 1408;
bool one_reduction_grid(const Geo &g, int dim) {
    int ntx, ntiles, grid;
    if (dim != 2 || g.N <= kSBCells) return false;
    tile_grid2(g, ntx, ntiles, grid);
    return ntiles <= kCgTiles;
}

// The preconditioner of iteration k of such a solve, and the update before
// it (k < 0: the first one, from the initial residual b0; no update): level 0
// through cg_down_tile2 / cg_up_tile2, the levels below as in vcycle_d.
template <typename TP, typename TR>
static void cg_cycle2(Slot<TP> &SP, const Level<TR> &A, const TP *b0, TP *z, const PcgVecs2<TR, TP> &v, TR *x, int k,
                      const Red &red, hipStream_t st) {
    constexpr double W = sizeof(TP), WR = sizeof(TR);
    Level<TP> &lv = SP.lev[0];
    const Geo &gc = SP.lev[1].g;
    const double N = (double)lv.g.N, Nc = (double)gc.N;
    const int *done = &red.scal->done;
    const CgPart pt{red.rz0, red.rz1, red.rz2, red.part0};
    TR *const R[2] = {v.r, v.p1}, *const Sv[2] = {v.q, v.t};
    int ntx, ntiles, grid;
    tile_grid2(lv.g, ntx, ntiles, grid);
    if (k < 0) {
        vcycle_down<TP, TP, 2>(SP, 0, b0, z, done, st);
    } else {
        const CgVec2<TR> cv{R[k & 1], Sv[k & 1], v.az, R[(k + 1) & 1], Sv[(k + 1) & 1], v.p0, x};
        // r, s, w, p, x, z in; r, s, p, x out; invd, cs in; x, bc out
        TLAUNCH(K_MG_DOWN, (9.0 * WR + W) * N + W * 4 * N + W * Nc, (k_cg_down_tile2<TP, TR>), dim3(grid),
                dim3(kTileThreads), st, lv, gc, cv, (const TP *)z, lv.r, SP.lev[1].b, ntx, ntiles, k, SP.singular,
                red.scal, pt, red.part1);
    }
    for (int l = 1; l < SP.lsb; ++l) vcycle_down<TP, TP, 2>(SP, l, SP.lev[l].b, SP.lev[l].x, done, st);
    vcycle_small<TP, TP, 2>(SP, b0, z, done, st, red.scal, (const double *)red.part1, k < 0 ? 0 : ntiles);
    for (int l = SP.lsb - 1; l >= 1; --l) vcycle_up<TP, TP, 2>(SP, l, SP.lev[l].b, SP.lev[l].x, done, st);
    // r, x, invd, cs, xc in; z, w out; the CG's own cs where they differ, and its s
    const double own = (W < WR ? 2.0 : 0.0) + (SP.singular ? 0.0 : 1.0);
    TLAUNCH(K_MG_UP, (2.0 + own) * WR * N + W * 5 * N + W * Nc, (k_cg_up_tile2<TP, TR>), dim3(grid),
            dim3(kTileThreads), st, lv, gc, (const TP *)SP.lev[1].x, (const TR *)R[(k + 1) & 1],
            (const TP *)lv.r, z, v.az, A, ntx, ntiles, SP.singular, pt, done);
}

// PCG in precision T (operator SA level 0, vectors, updates) preconditioned
// by V-cycles of the hierarchy SP in precision TP.
template <typename T, typename TP, int DIM>
static hipError_t pcg_d(Slot<T> &SA, Slot<TP> &SP, OpKind kind, ChOp ch, const T *b, T *x, double rtol, int max_iter,
                        int predict, Red &red, const PcgVecs2<T, TP> &v, hipStream_t st, SolveOut *out,
                        int zero_guess, int conv0 = 0) {
    constexpr double W = sizeof(T);
    constexpr double WP = sizeof(TP);
    const Level<T> &L0 = SA.lev[0];
    const Geo g = L0.g;
    const int N = (int)g.N;
    const int nb = grid_red(N);
    const int singular = SP.singular;
    Scal *sc = red.scal;
    const int *done = &sc->done;
    if (zero_guess) {
        LAUNCHR(K_PCG_INIT, W * 3 * N, (k_pcg_init_zero<T>), N, st, N, b, x, v.r, red.part0, red.part1);
    } else if (kind == OP_SLOT) {
        constexpr bool split = !std::is_same<T, TP>::value;
        // conv0: the level-0 set-up of SP's cycle rides on this pass
        const double conv_bytes = conv0 ? (split ? WP * (2 + DIM) : WP) * N : 0.0;
        LAUNCHR(K_PCG_INIT, W * (4 + DIM) * N + (split ? WP * N : 0.0) + conv_bytes, (k_pcg_init_slot<T, DIM, TP>), N,
                st, L0, b, (const T *)x, v.r, red.part0, red.part1, split ? (TP *)v.rp : (TP *)nullptr, SP.lev[0],
                conv0);
    } else {
        LAUNCH(K_PCG_INIT, W * 2 * N, (k_ch_lap_plain<T, DIM>), N, st, g, ch.ih2, (const T *)x, v.t);
        LAUNCHR(K_PCG_INIT, W * 4 * N, (k_pcg_init_ch<T, DIM>), N, st, g, ch.ih2, ch.a, ch.b, b, (const T *)x,
               (const T *)v.t, v.r, red.part0, red.part1);
    }
    LAUNCH1(K_PCG_INIT, 16.0 * nb, (k_pcg_fin_init), kBlock, st, sc, (const double *)red.part0,
            (const double *)red.part1, nb, rtol, max_iter);
    Scal hs;
    // With a lower-precision hierarchy the V-cycle reads the residual
    // already rounded to its precision (the value its sweeps would round it
    // to), so the level-0 passes read 4 instead of 8 bytes per cell of it.
    constexpr bool split = !std::is_same<T, TP>::value;
    const TP *rpre = split ? (const TP *)v.rp : (const TP *)(const void *)v.r;
    if (split && !(kind == OP_SLOT && !zero_guess))   // (the slot init writes rp itself)
        LAUNCH(K_PCG_INIT, (W + WP) * N, (k_round_vec<T, TP>), N, st, N, (const T *)v.r, v.rp);
    // preconditioner, then the r.z partials (in 3D with the slot operator
    // they ride on the preconditioner's last pass where that can take them)
    int nrz = nb;   // partials of r.z, sum z, sum r
    auto precond_rz = [&]() {
        int taken = 0;
        const RzFuse<T> rzf{(const T *)v.r, red.rz0, red.rz1, red.rz2, &taken};
        precond_d<TP, TP, DIM, T>(SP, kind, rpre, v.z, v.w, done, st, DIM == 3 && kind == OP_SLOT ? &rzf : nullptr);
        nrz = taken ? taken : nb;
        if (taken) return;
        if constexpr (DIM == 3) {
            int ntx, ncol, zc, ntiles;
            const int grid = sweep3_grid(g, ntx, ncol, zc, ntiles);
            if (kind == OP_SLOT && SP.lsb > 0 && ntiles <= kRedBlocks) {   // (level 0 above the small levels: even extents)
                TLAUNCH(K_PCG_DOT, (W + WP) * N, (k_pcg_rz3<T, TP>), dim3(grid), dim3(SweepShape::nB * kWave), st, g,
                        (const T *)v.r, (const TP *)v.z, (const Scal *)sc, red.rz0, red.rz1, red.rz2, ntx, ncol, zc,
                        ntiles);
                nrz = ntiles;
                return;
            }
        }
        LAUNCHR(K_PCG_DOT, (W + WP) * N, (k_pcg_rz<T, TP>), N, st, N, (const T *)v.r, (const TP *)v.z,
                (const Scal *)sc, red.rz0, red.rz1, red.rz2, singular);
    };
    // 2D with tiled level 0 of at most kRedBlocks tiles, the Cahn-Hilliard
    // operator or no vector for A z: the update and the r.z partials ride on
    // the level-0 tile passes (one partial per tile), and the residual store
    // moves to the next operator apply
    int ntiles0 = 0;
    if (DIM == 2 && SP.lsb > 0) {
        int ntx, grid;
        tile_grid2(SP.lev[0].g, ntx, ntiles0, grid);
    }
    // one reduction point per iteration: the operator apply rides on the
    // preconditioner's last pass as well
    const bool one = kind == OP_SLOT && SP.lsb > 0 && v.az && one_reduction_grid(g, DIM);
    const bool fuse = !one && DIM == 2 && SP.lsb > 0 && ntiles0 <= kRedBlocks;
    if (fuse) nrz = ntiles0;
    L0Cg<T> cg{0, 0, 1, (const T *)v.r, (const T *)v.q, nullptr, x, sc, (const double *)red.part0, nb,
               red.part1, red.rz0, red.rz1, red.rz2};
    if (one) {
        if constexpr (DIM == 2) cg_cycle2<TP, T>(SP, L0, rpre, v.z, v, x, -1, red, st);
    } else if (fuse) {
        precond_cg_d<TP, DIM, T>(SP, kind, rpre, v.z, v.w, done, st, cg);
    } else {
        precond_rz();
    }
    // 3D slot operator: the z-marching apply (kMarchPlanes planes per block,
    // fewer where that leaves the chip short of blocks, more when the grid
    // would exceed the partial-sum slots)
    struct {
        int nb = 0, ncolx = 0, ncol = 0, zc = 0;
    } march;
    bool dens = false;   // coefficients from the density (Slot::rho)
    if (DIM == 3 && kind == OP_SLOT) {
        const Geo &g0 = L0.g;
        march.ncolx = (g0.n[0] + kMX - 1) / kMX;
        march.ncol = march.ncolx * ((g0.n[1] + kMY - 1) / kMY);
        dens = march.ncol <= kMaxBlocks && SA.rho && g0.N >= SA.march_cells;
        if (march.ncol <= kMaxBlocks && g0.N >= kMarchApplyCells) {   // else the grid-stride apply
            march.zc = kMarchPlanes;
            while (march.zc > 1 && march.ncol * ((g0.n[2] + march.zc - 1) / march.zc) < kMarchApplyBlocks)
                march.zc /= 2;
            while (march.zc < g0.n[2] && (long long)march.ncol * ((g0.n[2] + march.zc - 1) / march.zc) > kMaxBlocks)
                march.zc *= 2;
            march.nb = march.ncol * ((g0.n[2] + march.zc - 1) / march.zc);
        }
    }
    // of an apply with stored coefficients: p_old, p_new, q, cs and, unless the operator is singular, s
    const double WA = W * (3 + DIM + (singular ? 0 : 1));
    int launched = 0;
    int chunk = predict < 1 ? 1 : predict;
    for (;;) {
        if (chunk > max_iter - launched) chunk = max_iter - launched;
        for (int it = 0; it < chunk; ++it) {
            const int k = launched + it;
            if (one) {
                if constexpr (DIM == 2) cg_cycle2<TP, T>(SP, L0, rpre, v.z, v, x, k, red, st);
                continue;
            }
            T *pnew = (k & 1) ? v.p1 : v.p0;
            T *pold = (k & 1) ? v.p0 : v.p1;
            // the consumer of the r.z partials starts the iteration (beta);
            // fused: it also stores the previous iteration's residual
            T *rpend = fuse && k > 0 ? v.r : nullptr;
            const double WRP = rpend ? 2.0 * W : 0.0;   // r read and written
            if (kind == OP_SLOT && march.nb && dens) {
                // rho, p_old read; p_new, q written; z in its precision
                TLAUNCH(K_PCG_APPLY, 8.0 * N + 3.0 * W * N + WP * N, (k_pcg_apply3_march<T, TP, true>),
                        dim3(march.nb), dim3(kBlock), st, L0, (const TP *)v.z, (const T *)pold, pnew, v.q, sc,
                        red.part0, (const double *)red.rz0, (const double *)red.rz1, (const double *)red.rz2, nrz, k,
                        singular, march.ncolx, march.ncol, march.zc, SA.rho, SA.rho_ih2);
            } else if (kind == OP_SLOT && march.nb) {
                TLAUNCH(K_PCG_APPLY, WA * N + WP * N, (k_pcg_apply3_march<T, TP, false>), dim3(march.nb),
                        dim3(kBlock), st, L0, (const TP *)v.z, (const T *)pold, pnew, v.q, sc, red.part0,
                        (const double *)red.rz0, (const double *)red.rz1, (const double *)red.rz2, nrz, k, singular,
                        march.ncolx, march.ncol, march.zc, (const double *)nullptr, 0.0);
            } else if (kind == OP_SLOT && dens) {
                // a threshold set below kMarchApplyCells: same bits as the stored coefficients give
                if constexpr (DIM == 3)
                    LAUNCHR(K_PCG_APPLY, 8.0 * N + 3.0 * W * N + WP * N, (k_pcg_apply_slot<T, TP, DIM, true>), N, st,
                            L0, (const TP *)v.z, (const T *)pold, pnew, v.q, sc, red.part0, (const double *)red.rz0,
                            (const double *)red.rz1, (const double *)red.rz2, nrz, k, singular, (T *)nullptr, SA.rho,
                            SA.rho_ih2);
            } else if (kind == OP_SLOT) {
                LAUNCHR(K_PCG_APPLY, WA * N + WP * N + WRP * N, (k_pcg_apply_slot<T, TP, DIM, false>), N,
                        st, L0, (const TP *)v.z, (const T *)pold, pnew, v.q, sc, red.part0, (const double *)red.rz0,
                        (const double *)red.rz1, (const double *)red.rz2, nrz, k, singular, rpend,
                        (const double *)nullptr, 0.0);
            } else {
                LAUNCHR(K_PCG_APPLY, W * 3 * N + WP * N + WRP * N, (k_pcg_ch_lap<T, TP, DIM>), N, st, g, ch.ih2,
                        (const TP *)v.z, (const T *)pold, pnew, v.t, sc, (const double *)red.rz0, nrz, k, rpend,
                        (const T *)v.q);
                LAUNCHR(K_PCG_APPLY, W * 3 * N, (k_pcg_ch_apply<T, DIM>), N, st, g, ch.ih2, ch.a, ch.b, (const T *)pnew,
                       (const T *)v.t, v.q, (const Scal *)sc, red.part0);
            }
            if (fuse) {
                L0Cg<T> c = cg;
                c.down_upd = 1;
                c.bpend = 1;
                c.dmode = 2;
                c.p = pnew;
                precond_cg_d<TP, DIM, T>(SP, kind, rpre, v.z, v.w, done, st, c);
                continue;
            }
            // (a last-block finalize inside the update would need a
            // device-scope fence per block, which costs more than this launch)
            LAUNCHR(K_PCG_UPDATE, W * 6 * N + (split ? WP * N : 0.0), (k_pcg_update<T, TP>), N, st, N,
                    (const T *)pnew, (const T *)v.q, x, v.r, sc, (const double *)red.part0,
                    kind == OP_SLOT && march.nb ? march.nb : nb, red.part1, split ? v.rp : (TP *)nullptr);
            LAUNCH1(K_PCG_UPDATE, 8.0 * nb, (k_pcg_fin_rr), kBlock, st, sc, (const double *)red.part1, nb);
            precond_rz();
        }
        launched += chunk;
        hipError_t e = hipMemcpyAsync(&hs, sc, sizeof(Scal), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        if (hs.done || launched >= max_iter) break;
        chunk = 2;
    }
    if (out) {
        out->iters = hs.iter;
        out->rel_res = hs.bb > 0.0 ? sqrt(hs.rr / hs.bb) : 0.0;
        out->unconverged = hs.unconverged || !hs.done;
        out->nonfinite = hs.nonfinite;
    }
    return hipGetLastError();
}

template <typename T>
hipError_t pcg_solve(Slot<T> &S, int dim, OpKind kind, ChOp ch, const T *b, T *x, double rtol, int max_iter,
                     int predict, Red &red, PcgVecs<T> &v, hipStream_t st, SolveOut *out, int zero_guess,
                     int conv0) {
    const PcgVecs2<T, T> v2{v.r, v.p0, v.p1, v.q, v.t, v.z, v.t, nullptr, v.w};
    if (dim == 2)
        return pcg_d<T, T, 2>(S, S, kind, ch, b, x, rtol, max_iter, predict, red, v2, st, out, zero_guess, conv0);
    return pcg_d<T, T, 3>(S, S, kind, ch, b, x, rtol, max_iter, predict, red, v2, st, out, zero_guess, conv0);
}

// ---------------------------------------------------------------------------
// precision form: FP64 CG preconditioned by the FP32 hierarchy.  x, r, p,
// q, the level-0 operator of the CG recurrence, its updates and every dot
// product are FP64; the V-cycle runs on FP32 coefficients, sweeps and
// transfers (FP64 coarsest inverse) and returns z in FP32.  The initial
// residual is the true FP64 residual b - A x of the starting iterate and the
// recurrence residual is that of an FP64 CG, so the solve stops on the FP64
// form's test, ||r||_2 <= rtol max(||b||_2, ||r_0||_2).
// ---------------------------------------------------------------------------
template <int DIM>
// FP32 copy of the level-0 coefficients and their 1 / diag (invd_cell's
// sum, in FP32, of the rounded values: the upper faces' coefficients are
// read from the neighbours' FP64 entries and rounded the same way)
__global__ void __launch_bounds__(kBlock) k_conv_coef(Level<double> A, Level<float> B) {
    GRID_LOOP(A.g.N) {
        int ia[3];
        coords_of<DIM>(A.g, c, ia);
        const float sc = (float)A.s[c];
        B.s[c] = sc;
        float d = sc;
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
            const float w = (float)A.cs[b][c];
            B.cs[b][c] = w;
            if (nb_lo(A.g, c, ia[b], b) >= 0) d += w;
            const int hi = nb_hi(A.g, c, ia[b], b);
            if (hi >= 0) d += (float)A.cs[b][hi];
        }
        B.invd[c] = 1.0f / d;
    }
}

void convert_level0(const Slot<double> &A, Slot<float> &B, int dim, hipStream_t st) {
    const int N = A.lev[0].g.N;
    const double bytes = (8.0 + 4.0) * (1 + dim) * N + 4.0 * N;
    if (dim == 2)
        LAUNCH(K_MG_SETUP, bytes, (k_conv_coef<2>), N, st, A.lev[0], B.lev[0]);
    else
        LAUNCH(K_MG_SETUP, bytes, (k_conv_coef<3>), N, st, A.lev[0], B.lev[0]);
}

template <int DIM>
static hipError_t refine_d(Slot<double> &S64, Slot<float> &S32, OpKind kind, ChOp ch, const double *b, double *x,
                           double rtol, int max_iter, int *predict, Red &red, const PcgVecs2<double, float> &v,
                           hipStream_t st, SolveOut *out, int conv0) {
    SolveOut o;
    hipError_t e =
        pcg_d<double, float, DIM>(S64, S32, kind, ch, b, x, rtol, max_iter, *predict, red, v, st, &o, 0, conv0);
    if (e != hipSuccess) return e;
    if (o.iters > 0) *predict = o.iters;
    if (out) *out = o;
    return hipGetLastError();
}

hipError_t refine_solve(Slot<double> &S64, Slot<float> &S32, int dim, OpKind kind, ChOp ch, const double *b,
                        double *x, double rtol, int max_iter, int *predict, Red &red,
                        const PcgVecs2<double, float> &v, hipStream_t st, SolveOut *out, int conv0) {
    if (dim == 2) return refine_d<2>(S64, S32, kind, ch, b, x, rtol, max_iter, predict, red, v, st, out, conv0);
    return refine_d<3>(S64, S32, kind, ch, b, x, rtol, max_iter, predict, red, v, st, out, conv0);
}

template <typename T>
void remove_mean(const Geo &g, T *x, Red &red, hipStream_t st, T *copy) {
    const int N = (int)g.N;
    const int nb = grid_red(N);
    LAUNCHR(K_MEAN, sizeof(T) * N, (k_sum<T>), N, st, N, (const T *)x, red.part0);
    LAUNCHR(K_MEAN, (copy ? 3.0 : 2.0) * sizeof(T) * N, (k_sub_mean<T>), N, st, N, x, (const double *)red.part0, nb,
            copy);
}

template <typename T>
void slot_apply(Slot<T> &S, int dim, const T *x, T *y, hipStream_t st) {
    if (dim == 2)
        LAUNCH(K_PCG_APPLY, 0, (k_slot_apply<T, 2>), S.lev[0].g.N, st, S.lev[0], x, y);
    else
        LAUNCH(K_PCG_APPLY, 0, (k_slot_apply<T, 3>), S.lev[0].g.N, st, S.lev[0], x, y);
}

template void mg_setup<double>(Slot<double> &, int, hipStream_t, bool);
template void mg_vcycle<double>(Slot<double> &, int, const double *, double *, const int *, hipStream_t);
template hipError_t pcg_solve<double>(Slot<double> &, int, OpKind, ChOp, const double *, double *, double, int, int,
                                      Red &, PcgVecs<double> &, hipStream_t, SolveOut *, int, int);
template void mg_setup<float>(Slot<float> &, int, hipStream_t, bool);
template hipError_t pcg_solve<float>(Slot<float> &, int, OpKind, ChOp, const float *, float *, double, int, int,
                                     Red &, PcgVecs<float> &, hipStream_t, SolveOut *, int, int);
template void remove_mean<double>(const Geo &, double *, Red &, hipStream_t, double *);
template void slot_apply<double>(Slot<double> &, int, const double *, double *, hipStream_t);

}  // namespace chns
