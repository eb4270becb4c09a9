// Device building blocks of the multigrid: per-cell operator, smoother and
// transfer bodies, the workgroup-level V-cycle and hierarchy set-up, and the
// Laplacian of the CH operator.  Shared by the grid-wide kernels (one pass
// per launch), the single-workgroup coarse-level kernels and the batched
// workgroup-per-problem step.
#pragma once
#include <algorithm>

#include "common.h"

namespace chns {

// ---------------------------------------------------------------------------
// per-cell building blocks (shared by the grid-wide and single-block kernels)
// ---------------------------------------------------------------------------
template <int DIM>
__device__ inline void coords_of(const Geo &g, int c, int ia[3]) {
    if (DIM == 2)
        cell_coords2(g, c, ia[0], ia[1], ia[2]);
    else
        cell_coords(g, c, ia[0], ia[1], ia[2]);
}

// Neighbour stencils are branch-free: a missing neighbour (outside a walled
// axis) is replaced by the cell itself with weight 0, so every load of a
// stencil is unconditional and can be issued together (adding 0 leaves the
// sums unchanged).

// a * b + c, rounded once.  The stencil sums of the multigrid spell their
// fused multiply-adds out: left to contraction, a sum that starts with two
// products is fused on one or the other depending on the surrounding code,
// and the grid-wide, marching, tile and LDS forms of a pass must round alike
// (they are compared bit for bit).
__device__ inline float fmar(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fmar(double a, double b, double c) { return __builtin_fma(a, b, c); }

// (A x)_c
template <typename T, int DIM>
__device__ inline T apply_at(const Level<T> &L, const T *__restrict__ x, int c, const int ia[3]) {
    using R = T;
    const Geo &g = L.g;
    const R xc = (R)x[c];
    R acc = (R)L.s[c] * xc;
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
        const int lo = nb_lo(g, c, ia[b], b);
        const int hi = nb_hi(g, c, ia[b], b);
        const int l = lo >= 0 ? lo : c, h = hi >= 0 ? hi : c;
        const R xl = (R)x[l], xh = (R)x[h];
        const R wl = (R)L.cs[b][c], wh = (R)L.cs[b][h];
        acc = fmar(lo >= 0 ? wl : (R)0, xc - xl, acc);
        acc = fmar(hi >= 0 ? wh : (R)0, xc - xh, acc);
    }
    return acc;
}

// sum_b cs * x_nb over the neighbours (x given by a functor)
template <typename T, int DIM, typename F>
__device__ inline T offsum_at(const Level<T> &L, int c, const int ia[3], F xv) {
    using R = T;
    const Geo &g = L.g;
    R acc = 0.0;
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
        const int lo = nb_lo(g, c, ia[b], b);
        const int hi = nb_hi(g, c, ia[b], b);
        const int l = lo >= 0 ? lo : c, h = hi >= 0 ? hi : c;
        const R vl = xv(l), vh = xv(h);
        const R wl = (R)L.cs[b][c], wh = (R)L.cs[b][h];
        acc = fmar(lo >= 0 ? wl : (R)0, vl, acc);
        acc = fmar(hi >= 0 ? wh : (R)0, vh, acc);
    }
    return acc;
}

template <typename T, int DIM>
__device__ inline void invd_cell(const Level<T> &L, int c) {
    using R = T;
    int ia[3];
    coords_of<DIM>(L.g, c, ia);
    R d = (R)L.s[c];
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
        if (nb_lo(L.g, c, ia[b], b) >= 0) d += (R)L.cs[b][c];
        const int hi = nb_hi(L.g, c, ia[b], b);
        if (hi >= 0) d += (R)L.cs[b][hi];
    }
    L.invd[c] = (T)((R)1 / d);
}

// zero-guess pre-smoothing: red x = b / d, black from those red values
template <typename T, typename TB, int DIM>
__device__ inline void presmooth_cell(const Level<T> &L, const TB *__restrict__ b, T *__restrict__ x, int c) {
    using R = T;
    int ia[3];
    coords_of<DIM>(L.g, c, ia);
    const int col = (ia[0] + ia[1] + ia[2]) & 1;
    if (col == 0) {
        x[c] = (T)((R)b[c] * (R)L.invd[c]);
    } else {
        auto red = [&](int e) { return (R)b[e] * (R)L.invd[e]; };
        x[c] = (T)(((R)b[c] + offsum_at<T, DIM>(L, c, ia, red)) * (R)L.invd[c]);
    }
}

template <typename T, typename TB, int DIM>
__device__ inline void residual_cell(const Level<T> &L, const TB *__restrict__ b, const T *__restrict__ x,
                                     int c) {
    using R = T;
    int ia[3];
    coords_of<DIM>(L.g, c, ia);
    L.r[c] = (T)((R)b[c] - apply_at<T, DIM>(L, x, c, ia));
}

// One (z, y) row of the prolongation: v + wyz (w0 a + w1 b)
template <typename R>
__device__ inline R pro_row(R v, R wyz, R w0, R a, R w1, R b) {
    return fmar(wyz, fmar(w0, a, w1 * b), v);
}

// cell-centred linear prolongation along one axis: fine f takes 3/4 of its
// parent f/2 and 1/4 of the coarse neighbour on its side; past a wall the
// neighbour is the parent itself (weight 1 in total)
template <typename R>
__device__ inline void pro_axis(int f, int nc, int per, int &c0, int &c1, R &w0, R &w1) {
    const int p = f >> 1;
    const int q = (f & 1) ? p + 1 : p - 1;
    const bool out = q < 0 || q >= nc, wall = out && !per;
    c0 = p;
    c1 = out ? (per ? (q < 0 ? nc - 1 : 0) : p) : q;
    w0 = wall ? (R)1 : (R)0.75;
    w1 = wall ? (R)0 : (R)0.25;
}

template <typename T, int DIM, typename G>
__device__ inline T prolong_at(const G &gf, const G &gc, const T *__restrict__ xc, const int fi[3]) {
    using R = T;
    int c0[3], c1[3];
    R w0[3], w1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (a < DIM) {
            pro_axis<R>(fi[a], gc.n[a], gc.per[a], c0[a], c1[a], w0[a], w1[a]);
        } else {
            c0[a] = c1[a] = 0;
            w0[a] = 1.0;
            w1[a] = 0.0;
        }
    }
    const int nx = gc.n[0], nxy = (int)gc.n[0] * gc.n[1];
    R v = 0.0;
#pragma unroll
    for (int dz = 0; dz < (DIM == 3 ? 2 : 1); ++dz) {
        const int kz = (dz ? c1[2] : c0[2]) * nxy;
        const R wz = dz ? w1[2] : w0[2];
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
            const int ky = kz + (dy ? c1[1] : c0[1]) * nx;
            const R wyz = wz * (dy ? w1[1] : w0[1]);
            v = pro_row(v, wyz, w0[0], (R)xc[ky + c0[0]], w1[0], (R)xc[ky + c1[0]]);
        }
    }
    return v;
}

// full weighting along one axis: the four fine cells 2I-1 .. 2I+2 with
// weights (1,3,3,1)/8; at a wall the missing outer cell's weight moves to the
// adjacent child (4,3,1)/8 -- exactly the transpose of pro_axis / 2.  Always
// four taps (an absent one gets weight 0 and a valid index) so that the
// loads of a fully unrolled stencil issue together.
template <typename R>
__device__ inline void res_axis(int I, int nc, int nf, int per, int f[4], R w[4]) {
    const bool lo = (I > 0) || per, hi = (I < nc - 1) || per;
    f[0] = I > 0 ? 2 * I - 1 : (per ? nf - 1 : 0);
    w[0] = lo ? (R)0.125 : (R)0;
    f[1] = 2 * I;
    w[1] = lo ? (R)0.375 : (R)0.5;
    f[2] = 2 * I + 1;
    w[2] = hi ? (R)0.375 : (R)0.5;
    f[3] = I < nc - 1 ? 2 * I + 2 : (per ? 0 : nf - 1);
    w[3] = hi ? (R)0.125 : (R)0;
}

template <typename T, int DIM>
__device__ inline void restrict_cell(const Geo &gf, const Geo &gc, const T *__restrict__ rf, T *__restrict__ bc,
                                     int c) {
    using R = T;
    int I[3];
    coords_of<DIM>(gc, c, I);
    int fx[4], fy[4], fz[4];
    R wx[4], wy[4], wz[4];
    res_axis<R>(I[0], gc.n[0], gf.n[0], gc.per[0], fx, wx);
    res_axis<R>(I[1], gc.n[1], gf.n[1], gc.per[1], fy, wy);
    if (DIM == 3) res_axis<R>(I[2], gc.n[2], gf.n[2], gc.per[2], fz, wz);
    const int nx = gf.n[0], nxy = (int)gf.n[0] * gf.n[1];
    R v = 0.0;
#pragma unroll
    for (int a = 0; a < (DIM == 3 ? 4 : 1); ++a) {
        const int kz = DIM == 3 ? fz[a] * nxy : 0;
        const R wza = DIM == 3 ? wz[a] : 1.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = kz + fy[q] * nx;
            R s = 0.0;
#pragma unroll
            for (int e = 0; e < 4; ++e) s = fmar(wx[e], (R)rf[row + fx[e]], s);
            v = fmar(wy[q] * wza, s, v);
        }
    }
    bc[c] = (T)v;
}

// fused prolongation + black sweep: writes tmp = {red: x + P e, black:
// GS update from those red values}; x is left untouched
template <typename T, typename TB, int DIM>
__device__ inline void prolong_black_cell(const Level<T> &L, const Geo &gc, const T *__restrict__ xc,
                                          const TB *__restrict__ b, const T *__restrict__ x, T *__restrict__ tmp,
                                          int c) {
    using R = T;
    int ia[3];
    coords_of<DIM>(L.g, c, ia);
    const int col = (ia[0] + ia[1] + ia[2]) & 1;
    if (col == 0) {
        tmp[c] = (T)((R)x[c] + prolong_at<T, DIM>(L.g, gc, xc, ia));
    } else {
        auto red = [&](int e) {
            int ie[3];
            coords_of<DIM>(L.g, e, ie);
            return (R)x[e] + prolong_at<T, DIM>(L.g, gc, xc, ie);
        };
        tmp[c] = (T)(((R)b[c] + offsum_at<T, DIM>(L, c, ia, red)) * (R)L.invd[c]);
    }
}

// red sweep from tmp: x = {red: GS update from black tmp values, black: tmp}
template <typename T, typename TB, int DIM>
__device__ inline void red_from_tmp_cell(const Level<T> &L, const TB *__restrict__ b, const T *__restrict__ tmp,
                                         T *__restrict__ x, int c) {
    using R = T;
    int ia[3];
    coords_of<DIM>(L.g, c, ia);
    const int col = (ia[0] + ia[1] + ia[2]) & 1;
    if (col == 1) {
        x[c] = tmp[c];
    } else {
        auto blk = [&](int e) { return (R)tmp[e]; };
        x[c] = (T)(((R)b[c] + offsum_at<T, DIM>(L, c, ia, blk)) * (R)L.invd[c]);
    }
}

// in-place Gauss-Seidel update of one colour (neighbours have the other colour)
template <typename T, typename TB, int DIM>
__device__ inline void gs_color_cell(const Level<T> &L, const TB *__restrict__ b, T *__restrict__ x, int color, int c) {
    using R = T;
    int ia[3];
    coords_of<DIM>(L.g, c, ia);
    if (((ia[0] + ia[1] + ia[2]) & 1) != color) return;
    auto xv = [&](int e) { return (R)x[e]; };
    x[c] = (T)(((R)b[c] + offsum_at<T, DIM>(L, c, ia, xv)) * (R)L.invd[c]);
}

template <typename T, int DIM>
__device__ inline void coarsen_cell(const Level<T> &F, const Level<T> &C, int c) {
    int I[3];
    coords_of<DIM>(C.g, c, I);
    const Geo &gf = F.g;
    double s = 0.0;
    double cs[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int dz = 0; dz < (DIM == 3 ? 2 : 1); ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
                const int d3[3] = {dx, dy, dz};
                const int f =
                    (2 * I[0] + dx) + (int)gf.n[0] * ((2 * I[1] + dy) + (int)gf.n[1] * (2 * I[2] + dz));
                s += (double)F.s[f];
#pragma unroll
                for (int b = 0; b < DIM; ++b)
                    if (d3[b] == 0) cs[b] += (double)F.cs[b][f];   // fine faces on the coarse lower b-face
            }
    constexpr double nchild = (DIM == 3) ? 8.0 : 4.0;
    C.s[c] = (T)(s / nchild);
    // a face on a wall holds 0: every other pass masks it, and the LDS
    // V-cycle relies on it to index walled axes as periodic ones
#pragma unroll
    for (int b = 0; b < DIM; ++b)
        C.cs[b][c] = (C.g.per[b] || I[b] > 0) ? (T)(cs[b] / (nchild * 0.5) * 0.25) : (T)0;
}


// ---------------------------------------------------------------------------
// single-workgroup kernels for the small levels
// ---------------------------------------------------------------------------
#define BLOCK_LOOP(N) for (int c = (int)threadIdx.x; c < (int)(N); c += (int)blockDim.x)

// Red-black sweeps on each side of the cycle on the levels of at most
// kSmallSweepCells cells, the part run by one workgroup (one sweep on the
// larger levels).  With one sweep there, the coarse levels of a high-
// contrast system (density ratio 1000) leave most of the error: a CPU
// emulation of the bubble's pressure system at 256 x 512 needs 30 CG
// iterations with one sweep, 18 with two and 15 with three on these
// levels, which cost LDS passes but no launches (measured on the device:
// 30 / 19 / 17 iterations, 2.67 / 2.25 / 2.17 ms per bubble step).  The
// pre-sweeps run red then black, the post-sweeps black then red, so the
// cycle stays symmetric.
#ifndef CHNS_SMALL_SWEEPS
#define CHNS_SMALL_SWEEPS 3
#endif
constexpr int kSmallSweeps = CHNS_SMALL_SWEEPS;
constexpr int kSmallSweepCells = 2048;

// x = Ainv b on the coarsest level (FP64 matrix, block-wide)
template <typename T, typename TB>
__device__ inline void coarse_solve_block(int n, const double *__restrict__ Ainv, const TB *__restrict__ b,
                                          T *__restrict__ x) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        double v = 0.0;
        const double *row = Ainv + i * n;
        for (int j = 0; j < n; ++j) v += row[j] * (double)b[j];
        x[i] = (T)v;
    }
}

template <typename T, typename TB, int DIM>
__device__ inline void block_down(const Slot<T> &S, int l, const TB *__restrict__ b, T *__restrict__ x) {
    const Level<T> &lv = S.lev[l];
    BLOCK_LOOP(lv.g.N) presmooth_cell<T, TB, DIM>(lv, b, x, c);
    __syncthreads();
    if (lv.g.N <= kSmallSweepCells)
        for (int sw = 1; sw < kSmallSweeps; ++sw) {
            BLOCK_LOOP(lv.g.N) gs_color_cell<T, TB, DIM>(lv, b, x, 0, c);
            __syncthreads();
            BLOCK_LOOP(lv.g.N) gs_color_cell<T, TB, DIM>(lv, b, x, 1, c);
            __syncthreads();
        }
    BLOCK_LOOP(lv.g.N) residual_cell<T, TB, DIM>(lv, b, x, c);
    __syncthreads();
    BLOCK_LOOP(S.lev[l + 1].g.N) restrict_cell<T, DIM>(lv.g, S.lev[l + 1].g, lv.r, S.lev[l + 1].b, c);
    __syncthreads();
}

template <typename T, typename TB, int DIM>
__device__ inline void block_up(const Slot<T> &S, int l, const TB *__restrict__ b, T *__restrict__ x) {
    const Level<T> &lv = S.lev[l];
    BLOCK_LOOP(lv.g.N) prolong_black_cell<T, TB, DIM>(lv, S.lev[l + 1].g, S.lev[l + 1].x, b, x, lv.r, c);
    __syncthreads();
    BLOCK_LOOP(lv.g.N) red_from_tmp_cell<T, TB, DIM>(lv, b, lv.r, x, c);
    __syncthreads();
    if (lv.g.N <= kSmallSweepCells)
        for (int sw = 1; sw < kSmallSweeps; ++sw) {
            BLOCK_LOOP(lv.g.N) gs_color_cell<T, TB, DIM>(lv, b, x, 1, c);
            __syncthreads();
            BLOCK_LOOP(lv.g.N) gs_color_cell<T, TB, DIM>(lv, b, x, 0, c);
            __syncthreads();
        }
}

// V-cycle over levels [l0, nlev) in one workgroup.  b0 / x0 are the
// right-hand side / result of level l0 (they replace its own arrays; b0 may
// be stored in another precision).  Ends with a workgroup barrier.
template <typename T, typename TB, int DIM>
__device__ inline void vcycle_block_dev(const Slot<T> &S, int l0, const TB *__restrict__ b0, T *__restrict__ x0) {
    const int L = S.nlev;
    if (l0 == L - 1) {
        coarse_solve_block<T, TB>((int)S.lev[L - 1].g.N, S.Ainv, b0, x0);
        __syncthreads();
        return;
    }
    block_down<T, TB, DIM>(S, l0, b0, x0);
    for (int l = l0 + 1; l < L - 1; ++l) block_down<T, T, DIM>(S, l, S.lev[l].b, S.lev[l].x);
    coarse_solve_block<T, T>((int)S.lev[L - 1].g.N, S.Ainv, S.lev[L - 1].b, S.lev[L - 1].x);
    __syncthreads();
    for (int l = L - 2; l > l0; --l) block_up<T, T, DIM>(S, l, S.lev[l].b, S.lev[l].x);
    block_up<T, TB, DIM>(S, l0, b0, x0);
}

// ---------------------------------------------------------------------------
// V-cycle of the small levels in registers and LDS
// ---------------------------------------------------------------------------
// Levels [l0, nlev), l0 >= 1, of at most 4 kVsThreads cells, in one workgroup
// of kVsThreads threads, with the arithmetic of vcycle_block_dev per cell:
//   pre-smoothing  red x = b / d, black GS from those values, then
//                  kSmallSweeps - 1 more red | black sweeps
//   post-smoothing red x += P e, then kSmallSweeps x (black GS | red GS)
//                  (black x is overwritten by its GS update, so only red
//                  cells take the prolonged correction)
// A thread takes pairs of cells 2m, 2m + 1 of a row (x extents are even), one
// red and one black: two pairs of level l0, one of each level below.
//
// One workgroup is alone with its latencies: memory (a launch may land on an
// XCD whose L2 holds none of this), the index arithmetic and coefficient
// loads of every level, and per pass one LDS round trip, a chain of multiply-
// adds and a barrier.  So everything a thread ever needs from memory, for all
// levels, is loaded into its registers in one round at the start (1 / diag,
// the face coefficients and s of its pairs, b of level l0, its entries of
// the coarsest inverse), the index arithmetic (quotients of small integers
// through a float reciprocal) runs while those loads are in flight, and only x,
// the residual and the coarser right-hand sides are in LDS.  x and the
// residual are stored by colour while a level is swept (red of pair k at k,
// black at N / 2 + k): a pass reads consecutive words where the x order reads
// every second one (two-way bank conflicts), and a pair's partner is in a
// register.  512 threads instead of 1024 leave each twice the registers (all
// levels' coefficients stay resident) and half the waves at each barrier.
// Faces on walls hold 0 on these levels (coarsen_cell), so every axis is
// indexed as periodic: the wrapped neighbour of a cell on a wall enters with
// weight 0, where the masked stencils add 0 for the missing neighbour.
// Launch in a pressure solve, FP64 (before: every level staged in LDS in x order,
// 1024 threads): 256 x 512 (levels 2048, 512, 128, 32) 15.7 -> 14.0 us and 64^2
// 11.6 -> 10.2, with the end of the CG iteration taken in; 96^3 (1728, 216, 27)
// 16.7 -> 13.4, 64^3 9.6 -> 8.4; bit for bit the same.  What is left is the 41 dependent passes, 250 to 400 cycles each.
constexpr int kVsThreads = 512;
template <int DIM>
constexpr int kVsLevels = DIM == 2 ? 3 : 2;   // levels swept: N > 64 on each, at most 2048 on the first

template <typename T>
struct VsTwo {
    typedef T type __attribute__((ext_vector_type(2)));
};

// LDS bytes of that V-cycle, or 0 where it does not apply (then
// vcycle_block_dev): lsb == 0, a larger level or more levels.  x and r per
// swept level, b below the first; b and x of the coarsest.
template <typename T>
inline size_t vs_lds_bytes(const Slot<T> &S, int lsb, int dim) {
    if (lsb <= 0 || S.lev[lsb].g.N > 4 * kVsThreads) return 0;
    if (S.nlev - 1 - lsb > (dim == 2 ? kVsLevels<2> : kVsLevels<3>)) return 0;
    size_t n = 2 * (size_t)S.ncoarse;
    for (int l = lsb; l < S.nlev - 1; ++l) n += (l == lsb ? 2 : 3) * (size_t)S.lev[l].g.N;
    return (n * sizeof(T) + 15) & ~(size_t)15;
}

// What the kernel needs to know, at fixed places: indexing the slot's levels
// by l0 in the kernel's arguments costs a scalar load from memory before the
// address of the next is known.  Entries past the coarsest repeat level l0.
struct VsGeo {
    int n[3], per[3];
};
template <typename T, int DIM>
struct VsArgs {
    int ns, n;             // levels swept, cells of the coarsest
    VsGeo g[kVsLevels<DIM> + 1];
    const T *s[kVsLevels<DIM>], *cs[kVsLevels<DIM>][DIM], *invd[kVsLevels<DIM>];
    const T *b;            // level l0
    T *x;
    const double *Ainv;
};
template <typename T, int DIM>
__host__ __device__ inline VsArgs<T, DIM> vs_args(const Slot<T> &S, int l0) {
    VsArgs<T, DIM> A;
    A.ns = S.nlev - 1 - l0;
    A.n = S.ncoarse;
#pragma unroll
    for (int j = 0; j <= kVsLevels<DIM>; ++j) {
        const Level<T> &L = S.lev[j <= A.ns ? l0 + j : l0];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            A.g[j].n[a] = L.g.n[a];
            A.g[j].per[a] = L.g.per[a];
        }
        if (j < kVsLevels<DIM>) {
            A.s[j] = L.s;
            A.invd[j] = L.invd;
#pragma unroll
            for (int a = 0; a < DIM; ++a) A.cs[j][a] = L.cs[a];
        }
    }
    A.b = S.lev[l0].b;
    A.x = S.lev[l0].x;
    A.Ainv = S.Ainv;
    return A;
}
template <int DIM>
__device__ inline int vs_cells(const VsGeo &g) {
    return g.n[0] * g.n[1] * (DIM == 3 ? g.n[2] : 1);
}

// a / b for 0 <= a < 2^20, b >= 1: (a + 1/2) / b is at least 1 / (2 b) away
// from an integer, more than its error of 2^-22 a / b
__device__ inline int small_div(int a, int b) {
    return (int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b));
}

template <typename T, int DIM>
struct VsPair {
    bool on;
    int k, par;            // pair index; the red cell's parity in x: red at 2m + par
    int adj[2];            // the other pair in the row that the red / black cell touches
    int nb[2 * DIM - 2];   // pairs across the y faces (, z faces)
    int xh;                // pair of the upper x neighbour of the odd cell
    int ia[3];             // coordinates of the red cell
    T b[2], v[2];          // right-hand side and x: red, black
    T invd[2], s[2];
    T cw[2][2 * DIM];      // coefficients of the faces: x low, x high, y low, y high (, z low, z high)
};

template <typename T, int DIM>
__device__ inline void vs_index(const VsGeo &g, int k, VsPair<T, DIM> &P) {
    const int nx = g.n[0], ny = g.n[1], nz = DIM == 3 ? g.n[2] : 1, nxh = nx >> 1;
    P.on = k < nxh * ny * nz;
    P.k = P.on ? k : 0;
    const int row = small_div(P.k, nxh), m = P.k - row * nxh;   // row = y + ny z
    const int z = DIM == 3 ? small_div(row, ny) : 0;
    const int y = row - z * ny;
    P.par = (y + z) & 1;
    P.ia[0] = 2 * m + P.par;
    P.ia[1] = y;
    P.ia[2] = z;
    const int ml = P.k + (m > 0 ? -1 : nxh - 1);
    P.xh = P.k + (m < nxh - 1 ? 1 : 1 - nxh);
    P.adj[0] = P.par ? P.xh : ml;
    P.adj[1] = P.par ? ml : P.xh;
    P.nb[0] = P.k + (y > 0 ? -nxh : nxh * (ny - 1));
    P.nb[1] = P.k + (y < ny - 1 ? nxh : -nxh * (ny - 1));
    if (DIM == 3) {
        const int nxyh = nxh * ny;
        P.nb[2 * DIM - 4] = P.k + (z > 0 ? -nxyh : nxyh * (nz - 1));
        P.nb[2 * DIM - 3] = P.k + (z < nz - 1 ? nxyh : -nxyh * (nz - 1));
    }
}

// even / odd cell -> red / black
template <typename T, int DIM, typename V>
__device__ inline void vs_order(const VsPair<T, DIM> &P, V v, T (&o)[2]) {
    o[0] = P.par ? v.y : v.x;
    o[1] = P.par ? v.x : v.y;
}

// The pair's coefficients and b in device memory, as loaded: one aligned load
// per array and pair.  The loads of every level are issued before any of
// them is used (vs_take), without a branch between them: a level per branch
// waited for one memory round trip after another (7600 cycles for
// five, 4900 for all at once).
template <typename T>
struct VsRaw {
    typename VsTwo<T>::type invd, s, b, f0, f1, h1, f2, h2;
    T x2;
};
template <typename T, int DIM>
__device__ inline void vs_load(const VsArgs<T, DIM> &A, int j, const VsPair<T, DIM> &P, VsRaw<T> &r) {
    using GV = const __attribute__((address_space(1))) typename VsTwo<T>::type;
    using G1 = const __attribute__((address_space(1))) T;
    auto two = [](const T *p, int k) { return ((GV *)p)[k]; };
    r.invd = two(A.invd[j], P.k);
    r.s = two(A.s[j], P.k);
    r.f0 = two(A.cs[j][0], P.k);
    r.x2 = ((G1 *)A.cs[j][0])[2 * P.xh];
    r.f1 = two(A.cs[j][1], P.k);
    r.h1 = two(A.cs[j][1], P.nb[1]);
    if (DIM == 3) {
        r.f2 = two(A.cs[j][DIM - 1], P.k);
        r.h2 = two(A.cs[j][DIM - 1], P.nb[2 * DIM - 3]);
    }
    r.b = j == 0 ? two(A.b, P.k) : r.s;   // (below level l0 the restriction provides b)
}
template <typename T, int DIM>
__device__ inline void vs_take(const VsRaw<T> &r, VsPair<T, DIM> &P) {
    vs_order(P, r.invd, P.invd);
    vs_order(P, r.s, P.s);
    vs_order(P, r.b, P.b);
    typename VsTwo<T>::type h0;
    h0.x = r.f0.y;
    h0.y = r.x2;
    T t[2];
    auto put = [&](typename VsTwo<T>::type v, int i) {
        vs_order(P, v, t);
        P.cw[0][i] = t[0];
        P.cw[1][i] = t[1];
    };
    put(r.f0, 0);
    put(h0, 1);
    put(r.f1, 2);
    put(r.h1, 3);
    if (DIM == 3) {
        put(r.f2, 2 * DIM - 2);
        put(r.h2, 2 * DIM - 1);
    }
}

// Values across the faces of cell Q of the pair, in the order of cw: x holds
// the other colour by pair.
template <int Q, typename T, int DIM>
__device__ inline void vs_faces(const VsPair<T, DIM> &P, const T *x, T (&v)[2 * DIM]) {
    const T other = x[P.adj[Q]], mine = P.v[1 - Q];
    // red: its partner is the upper x neighbour for par 0; black: the lower one
    const bool low = Q == 0 ? P.par != 0 : P.par == 0;
    v[0] = low ? mine : other;
    v[1] = low ? other : mine;
#pragma unroll
    for (int i = 0; i < 2 * DIM - 2; ++i) v[2 + i] = x[P.nb[i]];
}

// Gauss-Seidel value of cell Q of the pair
template <int Q, typename T, int DIM>
__device__ inline T vs_gs(const VsPair<T, DIM> &P, const T *x) {
    T v[2 * DIM], acc = 0.0;
    vs_faces<Q>(P, x, v);
#pragma unroll
    for (int i = 0; i < 2 * DIM; ++i) acc = fmar(P.cw[Q][i], v[i], acc);
    return (P.b[Q] + acc) * P.invd[Q];
}

// residual b - A x at cell Q of the pair
template <int Q, typename T, int DIM>
__device__ inline T vs_residual(const VsPair<T, DIM> &P, const T *x) {
    T v[2 * DIM], acc = P.s[Q] * P.v[Q];
    vs_faces<Q>(P, x, v);
#pragma unroll
    for (int i = 0; i < 2 * DIM; ++i) acc = fmar(P.cw[Q][i], P.v[Q] - v[i], acc);
    return P.b[Q] - acc;
}

// restrict_cell at coarse coordinates I from a fine residual stored by colour
// (r: red, then black from half on): the taps are the odd cell of pair I - 1,
// both cells of pair I and the even cell of pair I + 1 of each row.
template <typename T, int DIM>
__device__ inline T vs_restrict(const VsGeo &gf, const VsGeo &gc, const T *r, const int I[3]) {
    int fx[4], fy[4], fz[4];
    T wx[4], wy[4], wz[4];
    res_axis<T>(I[0], gc.n[0], gf.n[0], gc.per[0], fx, wx);
    res_axis<T>(I[1], gc.n[1], gf.n[1], gc.per[1], fy, wy);
    if (DIM == 3) res_axis<T>(I[2], gc.n[2], gf.n[2], gc.per[2], fz, wz);
    const int nxh = gf.n[0] >> 1, half = nxh * gf.n[1] * (DIM == 3 ? gf.n[2] : 1);
    T v = 0.0;
#pragma unroll
    for (int a = 0; a < (DIM == 3 ? 4 : 1); ++a) {
        const int kz = DIM == 3 ? fz[a] * gf.n[1] : 0;
        const T wza = DIM == 3 ? wz[a] : (T)1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = (kz + fy[q]) * nxh;
            const int par = (fy[q] + (DIM == 3 ? fz[a] : 0)) & 1;
            // (a clamped tap at a wall has weight 0: any value of its row does)
            const int odd = row + (par ? 0 : half), even = row + (par ? half : 0);
            T s = 0.0;
#pragma unroll
            for (int e = 0; e < 4; ++e) s = fmar(wx[e], r[((e & 1) ? even : odd) + (fx[e] >> 1)], s);
            v = fmar(wy[q] * wza, s, v);
        }
    }
    return v;
}

// x = Ainv b on the coarsest level: G lanes per row (a power of two, at most
// a wave, G n <= 1024 where n allows), lane q summing columns q, q + G, ...
// in order, then a butterfly over the G lanes.  For n <= 64 a thread's
// entries (two rows, four columns at most) are in a, loaded at the start.
constexpr int kVsRows = 2, kVsCols = 4;
__device__ inline int vs_lanes(int n, int &lg) {
    int G = 1;
    lg = 0;
    while (G < kWave && 2 * G * n <= 1024) {
        G *= 2;
        ++lg;
    }
    return G;
}
__device__ inline void vs_load_inverse(int n, const double *Ainv, double (&a)[kVsRows][kVsCols]) {
    int lg;
    const int G = vs_lanes(n, lg), q = (int)threadIdx.x & (G - 1), i0 = (int)threadIdx.x >> lg;
#pragma unroll
    for (int r = 0; r < kVsRows; ++r)
#pragma unroll
        for (int c = 0; c < kVsCols; ++c) {
            const int i = i0 + r * (kVsThreads >> lg), j = q + c * G;
            a[r][c] = Ainv[i < n && j < n ? i * n + j : 0];
        }
}
// v of the lane that a DPP control pairs with this one
template <int CTRL>
__device__ inline double vs_dpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// Sum of the two 16-lane (32-lane) halves of each group, in both
__device__ inline double vs_sum16(double v) {
    const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
__device__ inline double vs_sum32(double v) {
    const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
// Butterfly sum over groups of G = 16, 32 or 64 lanes, the widest step first
// (the sums of __shfl_xor with offsets G / 2 .. 1 without its LDS round trips:
// coarse solve of 32 cells 2600 -> 1150 cycles).  After the step of
// distance 8 the values repeat every 8 lanes, so a rotation by 4 within 16
// is the exchange at distance 4.
__device__ inline double vs_butterfly(double v, int G) {
    if (G > 32) v = vs_sum32(v);
    if (G > 16) v = vs_sum16(v);
    v += vs_dpp<0x128>(v);   // row_ror:8
    v += vs_dpp<0x124>(v);   // row_ror:4
    v += vs_dpp<0x4E>(v);    // quad_perm 2 3 0 1
    v += vs_dpp<0xB1>(v);    // quad_perm 1 0 3 2
    return v;
}
template <typename T>
__device__ inline void vs_coarse(int n, const double *Ainv, const double (&a)[kVsRows][kVsCols], const T *b, T *x) {
    int lg;
    const int G = vs_lanes(n, lg), q = (int)threadIdx.x & (G - 1), i0 = (int)threadIdx.x >> lg;
    if (n <= kLdsInverse) {
        double bv[kVsCols];
#pragma unroll
        for (int c = 0; c < kVsCols; ++c) bv[c] = (double)b[q + c * G < n ? q + c * G : 0];
        double v[kVsRows] = {0.0, 0.0};
#pragma unroll
        for (int c = 0; c < kVsCols; ++c) {
            if (c * G >= n) break;
            const bool in = q + c * G < n;
#pragma unroll
            for (int r = 0; r < kVsRows; ++r) v[r] = in ? v[r] + a[r][c] * bv[c] : v[r];
        }
#pragma unroll
        for (int r = 0; r < kVsRows; ++r) v[r] = vs_butterfly(v[r], G);
#pragma unroll
        for (int r = 0; r < kVsRows; ++r) {
            const int i = i0 + r * (kVsThreads >> lg);
            if (q == 0 && i < n) x[i] = (T)v[r];
        }
        return;
    }
    for (int i = i0; i < n; i += kVsThreads >> lg) {
        const double *row = Ainv + i * n;
        double v = 0.0;
        for (int j = q; j < n; j += G) v += row[j] * (double)b[j];
        for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
        if (q == 0) x[i] = (T)v;
    }
}

// One side of the cycle on one level (NP pairs per thread; X, R: x and
// residual by colour, half = N / 2).
template <typename T, int DIM, int NP>
__device__ inline void vs_down(VsPair<T, DIM> (&P)[NP], T *X, T *R, int half) {
#pragma unroll
    for (int p = 0; p < NP; ++p)
        if (P[p].on) X[P[p].k] = P[p].v[0] = P[p].b[0] * P[p].invd[0];
    __syncthreads();
    for (int sw = 0;; ++sw) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (P[p].on) X[half + P[p].k] = P[p].v[1] = vs_gs<1>(P[p], X);
        __syncthreads();
        if (sw + 1 >= kSmallSweeps) break;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (P[p].on) X[P[p].k] = P[p].v[0] = vs_gs<0>(P[p], X + half);
        __syncthreads();
    }
#pragma unroll
    for (int p = 0; p < NP; ++p)
        if (P[p].on) {
            R[P[p].k] = vs_residual<0>(P[p], X + half);
            R[half + P[p].k] = vs_residual<1>(P[p], X);
        }
    __syncthreads();
}
// out: x in cell order
template <typename T, int DIM, int NP>
__device__ inline void vs_up(VsPair<T, DIM> (&P)[NP], const VsGeo &gf, const VsGeo &gc, const T *xc, T *X, int half,
                             T *out) {
#pragma unroll
    for (int p = 0; p < NP; ++p)
        if (P[p].on) X[P[p].k] = P[p].v[0] = P[p].v[0] + prolong_at<T, DIM>(gf, gc, xc, P[p].ia);
    __syncthreads();
    for (int sw = 0; sw < kSmallSweeps; ++sw) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (P[p].on) X[half + P[p].k] = P[p].v[1] = vs_gs<1>(P[p], X);
        __syncthreads();
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (P[p].on) {
                P[p].v[0] = vs_gs<0>(P[p], X + half);
                if (sw + 1 < kSmallSweeps) X[P[p].k] = P[p].v[0];
            }
        if (sw + 1 < kSmallSweeps) __syncthreads();
    }
    using V = typename VsTwo<T>::type;
#pragma unroll
    for (int p = 0; p < NP; ++p)
        if (P[p].on) {
            V t;
            t.x = P[p].par ? P[p].v[1] : P[p].v[0];
            t.y = P[p].par ? P[p].v[0] : P[p].v[1];
            *(V *)(out + 2 * P[p].k) = t;
        }
    __syncthreads();
}

// The whole V-cycle: b of level l0 and x of level l0 are the level's arrays.
// skip: stop once the loads have been issued (nothing is written).  fin: see
// the kernel.
template <typename T, int DIM, typename FIN>
__device__ __forceinline__ void vcycle_small_dev(const VsArgs<T, DIM> &A, T *lds, int skip, FIN fin) {
    constexpr int NL = kVsLevels<DIM>;
    const int ns = A.ns, n = A.n, tid = (int)threadIdx.x;
    VsPair<T, DIM> top[2], low[NL - 1][1];
    // loads of every level and of the coarsest inverse (a level the cycle does
    // not have: those of pair 0 of level l0, unused)
    vs_index(A.g[0], tid, top[0]);
    vs_index(A.g[0], tid + kVsThreads, top[1]);
    VsRaw<T> rt[2], rl[NL - 1];
    vs_load(A, 0, top[0], rt[0]);
    vs_load(A, 0, top[1], rt[1]);
#pragma unroll
    for (int j = 1; j < NL; ++j) {
        vs_index(A.g[j], j < ns ? tid : 1 << 19, low[j - 1][0]);
        vs_load(A, j, low[j - 1][0], rl[j - 1]);
    }
    double ai[kVsRows][kVsCols];
    vs_load_inverse(n, A.Ainv, ai);
    if (skip) return;
    fin();
    vs_take(rt[0], top[0]);
    vs_take(rt[1], top[1]);
#pragma unroll
    for (int j = 1; j < NL; ++j) vs_take(rl[j - 1], low[j - 1][0]);
    // LDS: x, r of level l0; b, x, r of the levels below; b, x of the coarsest
    T *X[NL], *R[NL], *B[NL + 1];
    int half[NL];
    {
        T *o = lds;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int N = j < ns ? vs_cells<DIM>(A.g[j]) : 0;
            half[j] = N / 2;
            B[j] = o;
            if (j) o += N;
            X[j] = o;
            R[j] = o + N;
            o += 2 * N;
        }
        B[NL] = o;   // coarsest b; x follows
    }
    T *const bc = B[NL], *const xcs = B[NL] + n;
    auto restrict_to = [&](int j, const T *r) {   // onto level j (of the cycle's levels) from the one above
        const VsGeo &gc = A.g[j];
        if (tid < vs_cells<DIM>(gc)) {
            int I[3];
            const int t = small_div(tid, gc.n[0]);
            I[0] = tid - t * gc.n[0];
            I[2] = DIM == 3 ? small_div(t, gc.n[1]) : 0;
            I[1] = t - I[2] * gc.n[1];
            (j == ns ? bc : B[j])[tid] = vs_restrict<T, DIM>(A.g[j - 1], gc, r, I);
        }
        __syncthreads();
    };
    if (ns == 0) {
        for (int c = tid; c < n; c += kVsThreads) bc[c] = A.b[c];
        __syncthreads();
    } else {
        vs_down<T, DIM, 2>(top, X[0], R[0], half[0]);
        restrict_to(1, R[0]);
    }
#pragma unroll
    for (int j = 1; j < NL; ++j)
        if (j < ns) {
            using V = typename VsTwo<T>::type;
            VsPair<T, DIM>(&P)[1] = low[j - 1];
            if (P[0].on) vs_order(P[0], ((const V *)B[j])[P[0].k], P[0].b);
            vs_down<T, DIM, 1>(P, X[j], R[j], half[j]);
            restrict_to(j + 1, R[j]);
        }
    vs_coarse<T>(n, A.Ainv, ai, bc, xcs);
    __syncthreads();
    if (ns == 0) {
        for (int c = tid; c < n; c += kVsThreads) A.x[c] = xcs[c];
        return;
    }
#pragma unroll
    for (int j = NL - 1; j >= 1; --j)
        if (j < ns)
            vs_up<T, DIM, 1>(low[j - 1], A.g[j], A.g[j + 1], j + 1 == ns ? xcs : R[j + 1 < NL ? j + 1 : 0], X[j], half[j],
                             R[j]);
    vs_up<T, DIM, 2>(top, A.g[0], A.g[1], ns == 1 ? xcs : R[1], X[0], half[0], A.x);
}

// In-place Gauss-Jordan inversion of the n x n SPD matrix held in A (no
// pivoting), block-wide; f is a scratch row of n doubles.
__device__ inline void gauss_jordan_inplace(double *A, int n, double *f, double *piv) {
    for (int k = 0; k < n; ++k) {
        __syncthreads();
        if (threadIdx.x == 0) *piv = 1.0 / A[k * n + k];
        for (int i = threadIdx.x; i < n; i += blockDim.x) f[i] = A[i * n + k];
        __syncthreads();
        const double p = *piv;
        for (int j = threadIdx.x; j < n; j += blockDim.x) A[k * n + j] = (j == k) ? p : A[k * n + j] * p;
        __syncthreads();
        for (int e = threadIdx.x; e < n * n; e += blockDim.x) {
            const int i = e / n, j = e % n;
            if (i == k) continue;
            const double fi = f[i];
            A[e] = (j == k) ? -fi * p : A[e] - fi * A[k * n + j];
        }
    }
    __syncthreads();
}

// Gauss-Jordan inversion as above with the matrix in registers: thread
// (ti, tj) of the first 256 holds the entries (ti + 16 p, tj + 16 q), p, q <
// NB (n <= 16 NB; entries past n are 0 and stay 0), and only the pivot row,
// the pivot column and the pivot's reciprocal go through LDS, in two slots by
// pivot parity: one barrier per pivot.  The chain of a pivot is one LDS read,
// two multiply-adds, a division and one LDS write; with the matrix in LDS
// (read and written once per pivot, 96 KB of LDS traffic for n = 64) a pivot
// took 1.2 us at n = 64.  Block-wide (at least 256 threads); A (n x n, LDS)
// is replaced by its inverse.  Ends with a workgroup barrier.
struct GjLds {
    double row[2][kLdsInverse], col[2][kLdsInverse], rp[2];
};
template <int NB>
__device__ inline void gauss_jordan_regs(double *A, int nn, GjLds &g) {
    const int n = __builtin_amdgcn_readfirstlane(nn);   // pivot tests in scalar registers
    const int tid = (int)threadIdx.x, ti = tid >> 4, tj = tid & 15;
    const bool on = tid < 256;
    double a[NB][NB];
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int i = ti + 16 * p, j = tj + 16 * q;
            a[p][q] = on && i < n && j < n ? A[i * n + j] : 0.0;
        }
    if (tid < kLdsInverse) {
        g.row[0][tid] = tid == 0 ? 1.0 : (tid < n ? A[tid] : 0.0);   // 1 at the pivot: the scaled row holds its reciprocal there
        g.col[0][tid] = tid < n ? A[tid * n] : 0.0;
        if (tid == 0) g.rp[0] = 1.0 / A[0];
    }
    __syncthreads();
    for (int k = 0; k < n; ++k) {
        if (on) {
            const int s = k & 1, kn = k + 1;
            const double p = g.rp[s];
            double c[NB], akj[NB];   // the pivot column, the scaled pivot row
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                c[q] = g.col[s][ti + 16 * q];
                akj[q] = g.row[s][tj + 16 * q];
            }
#pragma unroll
            for (int q = 0; q < NB; ++q) akj[q] = akj[q] * p;
#pragma unroll
            for (int pi = 0; pi < NB; ++pi)
#pragma unroll
                for (int q = 0; q < NB; ++q) a[pi][q] = a[pi][q] - c[pi] * akj[q];
            // column k, then row k, then the next pivot's row and column out
            // (the block index of a pivot is the same in every thread)
            const int kt = k & 15, kq = k >> 4, nt = kn & 15, nq = kn >> 4;
#pragma unroll
            for (int x = 0; x < NB; ++x)
                if (x == kq) {
                    if (tj == kt)
#pragma unroll
                        for (int pi = 0; pi < NB; ++pi) a[pi][x] = -c[pi] * p;
                    if (ti == kt)
#pragma unroll
                        for (int q = 0; q < NB; ++q) a[x][q] = akj[q];
                }
#pragma unroll
            for (int x = 0; x < NB; ++x)
                if (x == nq) {
                    if (ti == nt)
#pragma unroll
                        for (int q = 0; q < NB; ++q) g.row[s ^ 1][tj + 16 * q] = q == x && tj == nt ? 1.0 : a[x][q];
                    if (tj == nt) {
#pragma unroll
                        for (int pi = 0; pi < NB; ++pi) g.col[s ^ 1][ti + 16 * pi] = a[pi][x];
                        if (ti == nt) g.rp[s ^ 1] = 1.0 / a[x][x];
                    }
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int i = ti + 16 * p, j = tj + 16 * q;
            if (on && i < n && j < n) A[i * n + j] = a[p][q];
        }
    __syncthreads();
}

// LDS of the set-up: the coarsest matrix (in LDS when it has at most
// kLdsInverse cells), a scratch row, reduction slots and the pivot.
struct SetupLds {
    double A[kLdsInverse * kLdsInverse];
    double f[kMaxCoarse];
    double red[kSBThreads / kWave];
    double piv;
};

// The dense operator of the coarsest level C into M (n x n), shifted by the
// mean of its trace / n for a singular slot.  Block-wide; ends with a barrier.
template <typename T, int DIM>
__device__ inline void coarse_matrix_block(const Level<T> &C, int singular, double *M, double *red) {
    const int n = (int)C.g.N;
    for (int e = threadIdx.x; e < n * n; e += blockDim.x) M[e] = 0.0;
    __syncthreads();
    double dsum = 0.0;
    for (int c = threadIdx.x; c < n; c += blockDim.x) {
        int ia[3];
        coords_of<DIM>(C.g, c, ia);
        double d = (double)C.s[c];
        for (int b = 0; b < DIM; ++b) {
            const int lo = nb_lo(C.g, c, ia[b], b);
            const int hi = nb_hi(C.g, c, ia[b], b);
            if (lo >= 0) {
                const double w = (double)C.cs[b][c];
                d += w;
                M[c * n + lo] -= w;
            }
            if (hi >= 0) {
                const double w = (double)C.cs[b][hi];
                d += w;
                M[c * n + hi] -= w;
            }
        }
        M[c * n + c] += d;
        dsum += d;
    }
    const double tot = block_sum_all(dsum, red);
    if (singular) {
        const double tau = (tot / n) / n;
        for (int e = threadIdx.x; e < n * n; e += blockDim.x) M[e] += tau;
    }
    __syncthreads();
}

// Set-up of the small levels in one workgroup: coarsen from level
// max(l0,1) - 1 downwards, inverse diagonals, then the coarsest inverse
// (in LDS when it has at most kLdsInverse cells, else in S.aug).  Ends with
// a workgroup barrier.  mat (when given): the coarsest matrix is left there and
// not inverted.
template <typename T, int DIM>
__device__ inline void setup_block_dev(const Slot<T> &S, int l0, SetupLds &sh, double *mat = nullptr) {
    const int L = S.nlev;
    if (l0 == 0) {
        BLOCK_LOOP(S.lev[0].g.N) invd_cell<T, DIM>(S.lev[0], c);
        __syncthreads();
    }
    for (int l = (l0 > 1 ? l0 : 1); l < L; ++l) {
        BLOCK_LOOP(S.lev[l].g.N) coarsen_cell<T, DIM>(S.lev[l - 1], S.lev[l], c);
        __syncthreads();
        BLOCK_LOOP(S.lev[l].g.N) invd_cell<T, DIM>(S.lev[l], c);
        __syncthreads();
    }
    // dense coarsest operator
    const int n = (int)S.lev[L - 1].g.N;
    double *M = mat ? mat : (n <= kLdsInverse ? sh.A : S.aug);
    coarse_matrix_block<T, DIM>(S.lev[L - 1], S.singular, M, sh.red);
    if (mat) return;
    gauss_jordan_inplace(M, n, sh.f, &sh.piv);
    for (int e = threadIdx.x; e < n * n; e += blockDim.x) S.Ainv[e] = M[e];
    __syncthreads();
}

// The same set-up (the same arithmetic per entry) for a slot whose coarsest
// level has at most kLdsInverse cells, in at least 256 threads: the levels it
// writes are also kept in LDS, where the next level's coarsening, the inverse
// diagonals and the coarsest matrix read them (the global-memory form waits
// for a round trip in each of these passes), and the coarsest matrix is
// inverted in registers.  Falls back to setup_block_dev where that does not
// apply (a larger coarsest level, or no level below the grid).
// Whole set-up kernel, FP64, with the levels in memory and the matrix in LDS
// before: 64^2 (n = 64) 91 -> 44 us, 256 x 512 (n = 32) 29 -> 23 us, 96^3
// (n = 27) 32 -> 25 us, all bit for bit the same; 512 batched problems, FP32,
// 134 -> 56 us.
constexpr int kSetupLdsCells = kSBThreads * 2 * 4 / 3 + 32;   // all levels from 2 kSBThreads cells down (2D; fewer in 3D)
template <typename T, int DIM>
struct SetupLdsLev {
    SetupLds base;
    GjLds gj;
    T lev[(1 + DIM) * kSetupLdsCells];
};
template <typename T, int DIM>
__device__ inline void setup_lds_dev(const Slot<T> &S, int l0, SetupLdsLev<T, DIM> &sh, double *mat = nullptr) {
    const int L = S.nlev, n = (int)S.lev[L - 1].g.N;
    if (n > kLdsInverse || L < 2 || S.lev[l0 > 1 ? l0 : 1].g.N > 2 * kSBThreads) {
        setup_block_dev<T, DIM>(S, l0, sh.base, mat);
        return;
    }
    if (l0 == 0) BLOCK_LOOP(S.lev[0].g.N) invd_cell<T, DIM>(S.lev[0], c);
    const int l1 = l0 > 1 ? l0 : 1;
    int off = 0;
    auto image = [&](int l, int o) {   // level l with s, cs in LDS
        Level<T> C = S.lev[l];
        const int N = (int)C.g.N;
        C.s = sh.lev + o;
#pragma unroll
        for (int b = 0; b < DIM; ++b) C.cs[b] = sh.lev + o + (1 + b) * N;
        return C;
    };
    auto publish = [&](const Level<T> &C, int l) {   // 1 / diag, and s, cs to the level's own arrays
        BLOCK_LOOP(C.g.N) {
            invd_cell<T, DIM>(C, c);
            S.lev[l].s[c] = C.s[c];
#pragma unroll
            for (int b = 0; b < DIM; ++b) S.lev[l].cs[b][c] = C.cs[b][c];
        }
    };
    Level<T> C = image(l1, 0);
    BLOCK_LOOP(C.g.N) coarsen_cell<T, DIM>(S.lev[l1 - 1], C, c);
    __syncthreads();
    publish(C, l1);
    for (int l = l1 + 1; l < L; ++l) {
        const Level<T> F = image(l - 1, off);
        off += (1 + DIM) * (int)F.g.N;
        C = image(l, off);
        BLOCK_LOOP(C.g.N) coarsen_cell<T, DIM>(F, C, c);
        __syncthreads();
        publish(C, l);
    }
    double *M = sh.base.A;
    coarse_matrix_block<T, DIM>(image(L - 1, off), S.singular, M, sh.base.red);
    if (n <= 16)
        gauss_jordan_regs<1>(M, n, sh.gj);
    else if (n <= 32)
        gauss_jordan_regs<2>(M, n, sh.gj);
    else if (n <= 48)
        gauss_jordan_regs<3>(M, n, sh.gj);
    else
        gauss_jordan_regs<4>(M, n, sh.gj);
    for (int e = threadIdx.x; e < n * n; e += blockDim.x) S.Ainv[e] = M[e];
    __syncthreads();
}


// Lap(x) at c for the CH operator (walled axes Neumann), x given by a functor
// (branch-free like apply_at)
template <int DIM, typename F>
__device__ inline double lap_at(const Geo &g, int c, const int ia[3], double ih2, F val) {
    const double xc = val(c);
    double acc = 0.0;
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
        const int lo = nb_lo(g, c, ia[b], b);
        const int hi = nb_hi(g, c, ia[b], b);
        const double vl = val(lo >= 0 ? lo : c), vh = val(hi >= 0 ? hi : c);
        acc += lo >= 0 ? vl - xc : 0.0;
        acc += hi >= 0 ? vh - xc : 0.0;
    }
    return acc * ih2;
}

}  // namespace chns
