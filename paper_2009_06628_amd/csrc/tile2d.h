// Device bodies of the 2D multigrid tile passes (gfx950).
#pragma once
#include "mgdev.h"

namespace chns {

// ---------------------------------------------------------------------------
// 2D tile passes of the grid levels: one for the way down, one for the way
// up (shared by the single-grid kernels and the tiled batched form)
// ---------------------------------------------------------------------------
// A workgroup owns kTFX x kTFY fine cells (kTFX/2 x kTFY/2 coarse cells) and
// stages the level on the tile plus a halo in LDS.  Cells outside a walled
// axis are zero with zero coupling, which is what the branch-free per-cell
// stencils add for a missing neighbour; periodic axes wrap.  Halo values are
// recomputed by every tile that needs them, with the arithmetic of the
// per-cell passes in the same order, so the results are those of the
// separate passes.  Levels here have even extents (only the coarsest may
// not), so colours do not change across a periodic seam.
#ifndef CHNS_TILE2_X
#define CHNS_TILE2_X 32
#endif
#ifndef CHNS_TILE2_Y
#define CHNS_TILE2_Y 16
#endif
#ifndef CHNS_TILE2_THREADS
#define CHNS_TILE2_THREADS 512
#endif
#ifndef CHNS_TILE2_BATCH_THREADS
#define CHNS_TILE2_BATCH_THREADS 256
#endif
constexpr int kTFX = CHNS_TILE2_X, kTFY = CHNS_TILE2_Y;   // fine cells per tile (even)
// Threads per tile: a single grid has few tiles per CU, so more threads per
// tile shorten each phase; the batched form has many tiles per CU and
// prefers more workgroups of fewer threads (measured).
constexpr int kTileThreads = CHNS_TILE2_THREADS;              // single-grid kernels
constexpr int kTileThreadsBatch = CHNS_TILE2_BATCH_THREADS;   // batched form
static_assert(kTFX % 2 == 0 && kTFY % 2 == 0, "tile extents must be even");

// Local x of the m-th cell of colour col in local row ly of a region that
// starts at local x 1 and has an even width, for a tile whose local (0, 0)
// has global parity par: the colour of a cell is the parity of its global
// x + y.
__device__ inline int tile_color_x(int m, int ly, int par, int col) {
    return 1 + 2 * m + ((ly + par + col + 1) & 1);
}

// Local index -> global coordinate along one axis: wrapped on a periodic
// axis; v tells whether the cell exists.
__device__ inline int tile_coord(int g, int n, int per, bool &v) {
    v = per || (g >= 0 && g < n);
    return per ? ((g % n) + n) % n : g;
}

// Right-hand side of a tile pass, staged in the hierarchy's precision T.
// As stored:
template <typename TB>
struct RhsStored {
    const TB *b;
    template <typename T>
    __device__ T at(int g) const {
        return (T)b[g];
    }
};
// The residual r - alpha q of a CG iteration whose store is still pending
// (the next operator apply stores it): the value the update stores in the
// CG precision TR, as read by the hierarchy through its right-hand side
// type TB.
__device__ inline double cg_residual(double r, double q, double alpha) { return fma(-alpha, q, r); }
template <typename TR, typename TB>
struct RhsPending {
    const TR *r, *q;
    double alpha;
    template <typename T>
    __device__ T at(int g) const {
        return (T)(TB)(TR)cg_residual((double)r[g], (double)q[g], alpha);
    }
};

// Sums of three per-thread values over a workgroup of NT threads, valid in
// thread 0 (fixed order: waves by shuffles, then the waves in order).
template <int NT>
__device__ inline void tile_sum3(double &a, double &b, double &c) {
    __shared__ double ws[3][NT / kWave];
    a = wave_sum(a);
    b = wave_sum(b);
    c = wave_sum(c);
    const int lane = (int)threadIdx.x & (kWave - 1), w = (int)threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) {
        ws[0][w] = a;
        ws[1][w] = b;
        ws[2][w] = c;
    }
    __syncthreads();
    a = b = c = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < NT / kWave; ++k) {
            a += ws[0][k];
            b += ws[1][k];
            c += ws[2][k];
        }
}

// Epilogue of the way up: nothing, or the partials of r.z, sum z and sum r
// over the tile's cells for the CG iteration that consumes z (r as stored,
// or pending as in RhsPending).
struct NoDots {
    __device__ void add(int, double) {}
    template <int NT>
    __device__ void finish() {}
};
template <typename TR>
struct RzDots {
    const TR *r, *q;
    double alpha;
    int pending;
    double *p0, *p1, *p2;
    int slot;
    double arz = 0.0, az = 0.0, ar = 0.0;
    __device__ void add(int g, double z) {
        const double rc =
            pending ? (double)(TR)cg_residual((double)r[g], (double)q[g], alpha) : (double)r[g];
        arz += rc * z;
        az += z;
        ar += rc;
    }
    template <int NT>
    __device__ void finish() {
        tile_sum3<NT>(arz, az, ar);
        if (threadIdx.x == 0) {
            p0[slot] = arz;
            p1[slot] = az;
            p2[slot] = ar;
        }
    }
};

// Way down: zero-guess pre-smoothing (red x = b / d, black GS from those),
// residual, restriction to the coarse right-hand side bc.  After the black
// sweep the residual of a black cell is 0 and that of a red cell is the sum of
// its black neighbours' x over the face coefficients (d x = b cancels): only
// the red ones are formed, s is not read and the restriction takes the red
// half of its taps (with s and every residual: 256 x 512 bubble step 1233 us,
// 1185 without; 768^2 drop step 2.12 -> 2.05 ms).
// FULL (the batched form): b - A x in every cell instead, whose rounding in the
// FP32 hierarchy that form's iterates carry: its refinement rounds end far
// above FP64 rounding, and without the rounding its velocities move by 1e-8.
// Writes the smoothed x of the tile to xs (the level's residual array, which
// no longer holds a residual: the way up reads x from there while it writes
// the level's x) and bc on the tile's coarse cells.
constexpr int kDownH = 3, kDownWX = kTFX + 2 * kDownH, kDownWY = kTFY + 2 * kDownH, kDownNL = kDownWX * kDownWY;
template <typename T, bool FULL>
struct DownTile {
    T sB[kDownNL], sI[kDownNL], sC0[kDownNL], sC1[kDownNL];
    T sX[kDownNL];   // x of the black cells, residual of the red ones (FULL: x)
    T sS[FULL ? kDownNL : 1], sR[FULL ? kDownNL : 1];
};

// The passes of the way down on a staged tile (sB .. sC1 filled, barrier done).
template <typename T, int NT, bool FULL>
__device__ inline void down_passes2(DownTile<T, FULL> &t, const Level<T> &L, const Geo &gc, T *__restrict__ xs,
                                    T *__restrict__ bc, int tx, int ty);

template <typename T, int NT, bool FULL = false, typename BS>
__device__ inline void down_tile2(const Level<T> &L, const Geo &gc, const BS &b, T *__restrict__ xs,
                                  T *__restrict__ bc, int tx, int ty, int skip) {
    constexpr int H = kDownH, WX = kDownWX, NL = kDownNL;
    constexpr int KL = (NL + NT - 1) / NT;   // staged cells per thread
    __shared__ DownTile<T, FULL> tile;
    const int nx = (int)L.g.n[0], ny = (int)L.g.n[1];
    const int px = L.g.per[0], py = L.g.per[1];
    const int gx0 = tx * kTFX - H, gy0 = ty * kTFY - H;
    // Stage: every load of the thread is issued before the first LDS store
    // (indices past the region are clamped to its last cell, which is then
    // stored again with the same values).
    T lb[KL], li[KL], ls[KL], l0[KL], l1[KL];
    bool lv[KL], m0[KL], m1[KL];
#pragma unroll
    for (int k = 0; k < KL; ++k) {
        const int i0 = (int)threadIdx.x + k * NT, i = i0 < NL ? i0 : NL - 1;
        const int ly = i / WX, lx = i - ly * WX;
        bool vx, vy;
        const int gx = tile_coord(gx0 + lx, nx, px, vx), gy = tile_coord(gy0 + ly, ny, py, vy);
        const bool v = vx && vy;
        const int g = v ? gx + nx * gy : 0;
        lb[k] = b.template at<T>(g);
        li[k] = L.invd[g];
        if (FULL) ls[k] = L.s[g];
        l0[k] = L.cs[0][g];
        l1[k] = L.cs[1][g];
        lv[k] = v;
        m0[k] = v && (px || gx > 0);   // a wall face couples nothing
        m1[k] = v && (py || gy > 0);
    }
    if (skip) return;   // tested once the staging loads are in flight
    // masks applied as factors 0 / 1 (the values come from valid addresses and
    // are finite), so that no load turns into a branch of its own
#pragma unroll
    for (int k = 0; k < KL; ++k) {
        const int i0 = (int)threadIdx.x + k * NT, i = i0 < NL ? i0 : NL - 1;
        const T fv = lv[k] ? (T)1 : (T)0;
        tile.sB[i] = lb[k] * fv;
        tile.sI[i] = li[k] * fv;
        if (FULL) tile.sS[i] = ls[k] * fv;
        tile.sC0[i] = l0[k] * (m0[k] ? (T)1 : (T)0);
        tile.sC1[i] = l1[k] * (m1[k] ? (T)1 : (T)0);
    }
    __syncthreads();
    down_passes2<T, NT, FULL>(tile, L, gc, xs, bc, tx, ty);
}

template <typename T, int NT, bool FULL>
__device__ inline void down_passes2(DownTile<T, FULL> &t, const Level<T> &L, const Geo &gc, T *__restrict__ xs,
                                    T *__restrict__ bc, int tx, int ty) {
    using R = T;
    constexpr int H = kDownH, WX = kDownWX, WY = kDownWY;
    T *const sB = t.sB, *const sI = t.sI, *const sC0 = t.sC0, *const sC1 = t.sC1, *const sX = t.sX;
    T *const sR = FULL ? t.sR : t.sX;
    const int nx = (int)L.g.n[0], ny = (int)L.g.n[1];
    const int gx0 = tx * kTFX - H, gy0 = ty * kTFY - H;
    // black x on the tile and 2 halo cells (local [1, WX-1) x [1, WY-1), rows
    // of even width): the k-th black cell in one thread, so no wave runs both
    // colours' branches
    const int par = (gx0 + gy0) & 1;
    constexpr int XP = (WX - 2) / 2;   // cells of one colour per row
    for (int k = (int)threadIdx.x; k < XP * (WY - 2); k += NT) {
        const int row = k / XP, m = k - row * XP, ly = 1 + row;
        const int i = ly * WX + tile_color_x(m, ly, par, 1);
        auto red = [&](int j) { return (R)sB[j] * (R)sI[j]; };
        R acc = 0.0;
        acc += (R)sC0[i] * red(i - 1);
        acc += (R)sC0[i + 1] * red(i + 1);
        acc += (R)sC1[i] * red(i - WX);
        acc += (R)sC1[i + WX] * red(i + WX);
        sX[i] = (T)(((R)sB[i] + acc) * (R)sI[i]);
        if (FULL) {
            const int ir = ly * WX + tile_color_x(m, ly, par, 0);
            sX[ir] = (T)((R)sB[ir] * (R)sI[ir]);
        }
    }
    __syncthreads();
    // red residuals on the tile and 1 halo cell (local [2, WX-2) x [2, WY-2))
    constexpr int RW = WX - 4, RP = RW / 2;
    if (FULL) {
        for (int j = (int)threadIdx.x; j < RW * (WY - 4); j += NT) {
            const int ry = j / RW, i = (ry + 2) * WX + (j - ry * RW) + 2;
            const R xc = (R)sX[i];
            R acc = (R)t.sS[i] * xc;
            acc += (R)sC0[i] * (xc - (R)sX[i - 1]);
            acc += (R)sC0[i + 1] * (xc - (R)sX[i + 1]);
            acc += (R)sC1[i] * (xc - (R)sX[i - WX]);
            acc += (R)sC1[i + WX] * (xc - (R)sX[i + WX]);
            sR[i] = (T)((R)sB[i] - acc);
        }
    } else {
        for (int k = (int)threadIdx.x; k < RP * (WY - 4); k += NT) {
            const int row = k / RP, m = k - row * RP, ly = 2 + row;
            const int i = ly * WX + 2 + 2 * m + ((ly + par) & 1);
            R acc = (R)sC0[i] * (R)sX[i - 1];
            acc += (R)sC0[i + 1] * (R)sX[i + 1];
            acc += (R)sC1[i] * (R)sX[i - WX];
            acc += (R)sC1[i + WX] * (R)sX[i + WX];
            sX[i] = (T)acc;
        }
    }
    __syncthreads();
    // restriction (taps 2I-1 .. 2I+2 per axis; an absent tap has weight 0)
    constexpr int CX = kTFX / 2, CY = kTFY / 2;
    const int ncx = (int)gc.n[0], ncy = (int)gc.n[1];
    for (int j = (int)threadIdx.x; j < CX * CY; j += NT) {
        const int cy = j / CX, cx = j - cy * CX;
        const int I = tx * CX + cx, J = ty * CY + cy;
        if (I >= ncx || J >= ncy) continue;
        int fx[4], fy[4];
        R wx[4], wy[4];
        res_axis<R>(I, ncx, nx, gc.per[0], fx, wx);
        res_axis<R>(J, ncy, ny, gc.per[1], fy, wy);
        R v = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = (2 * cy + H - 1 + q) * WX + 2 * cx + H - 1;
            R s = 0.0;
#pragma unroll
            for (int e = FULL ? 0 : q & 1; e < 4; e += FULL ? 1 : 2) s += wx[e] * (R)sR[row + e];   // (red taps: 2 I - 1 + e of row 2 J - 1 + q)
            v += (wy[q] * (R)1.0) * s;
        }
        bc[I + ncx * J] = (T)v;
    }
    // x of the tile's own cells
    for (int j = (int)threadIdx.x; j < kTFX * kTFY; j += NT) {
        const int ly = j / kTFX, lx = j - ly * kTFX;
        const int gx = tx * kTFX + lx, gy = ty * kTFY + ly;
        const int i = (ly + H) * WX + lx + H;
        if (gx < nx && gy < ny) xs[gx + nx * gy] = FULL || (gx + gy) & 1 ? sX[i] : (T)((R)sB[i] * (R)sI[i]);
    }
}

// Way up: red x += P e, black GS, red GS (the post-smoothing), with e the
// coarse correction xc and the pre-smoothed x read from xs.  Writes x on the
// tile (never read here, so tiles do not race on their halos).
template <typename T, int NT, typename BS, typename DOTS = NoDots>
__device__ inline void up_tile2(const Level<T> &L, const Geo &gc, const T *__restrict__ xc, const BS &b,
                                const T *__restrict__ xs, T *__restrict__ x, int tx, int ty, int skip,
                                DOTS dots = DOTS()) {
    using R = T;
    constexpr int H = 2, WX = kTFX + 2 * H, WY = kTFY + 2 * H, NL = WX * WY;
    constexpr int KL = (NL + NT - 1) / NT;
    __shared__ T sB[NL], sI[NL], sC0[NL], sC1[NL], sX[NL];
    const int nx = (int)L.g.n[0], ny = (int)L.g.n[1];
    const int px = L.g.per[0], py = L.g.per[1];
    const int gx0 = tx * kTFX - H, gy0 = ty * kTFY - H;
    // Stage as on the way down; the prolongation is evaluated for every
    // staged cell (at coordinate 0 for cells that do not exist) and kept for
    // the red cells only.
    T lb[KL], li[KL], l0[KL], l1[KL], lx_[KL];
    bool lv[KL], m0[KL], m1[KL];
#pragma unroll
    for (int k = 0; k < KL; ++k) {
        const int i0 = (int)threadIdx.x + k * NT, i = i0 < NL ? i0 : NL - 1;
        const int ly = i / WX, lx = i - ly * WX;
        bool vx, vy;
        const int gx = tile_coord(gx0 + lx, nx, px, vx), gy = tile_coord(gy0 + ly, ny, py, vy);
        const bool v = vx && vy;
        const int g = v ? gx + nx * gy : 0;
        lb[k] = b.template at<T>(g);
        li[k] = L.invd[g];
        l0[k] = L.cs[0][g];
        l1[k] = L.cs[1][g];
        const int ia[3] = {v ? gx : 0, v ? gy : 0, 0};
        const R pe = prolong_at<T, 2>(L.g, gc, xc, ia);
        const T red = (v && ((gx0 + lx + gy0 + ly) & 1) == 0) ? (T)1 : (T)0;
        lx_[k] = (T)((R)xs[g] + pe) * red;
        lv[k] = v;
        m0[k] = v && (px || gx > 0);
        m1[k] = v && (py || gy > 0);
    }
    if (skip) return;
#pragma unroll
    for (int k = 0; k < KL; ++k) {
        const int i0 = (int)threadIdx.x + k * NT, i = i0 < NL ? i0 : NL - 1;
        const T fv = lv[k] ? (T)1 : (T)0;
        sB[i] = lb[k] * fv;
        sI[i] = li[k] * fv;
        sC0[i] = l0[k] * (m0[k] ? (T)1 : (T)0);
        sC1[i] = l1[k] * (m1[k] ? (T)1 : (T)0);
        sX[i] = lx_[k];
    }
    __syncthreads();
    auto gs = [&](int i) {
        R acc = 0.0;
        acc += (R)sC0[i] * (R)sX[i - 1];
        acc += (R)sC0[i + 1] * (R)sX[i + 1];
        acc += (R)sC1[i] * (R)sX[i - WX];
        acc += (R)sC1[i + WX] * (R)sX[i + WX];
        return (T)(((R)sB[i] + acc) * (R)sI[i]);
    };
    // black on the tile and 1 halo cell (local [1, WX-1) x [1, WY-1); reads
    // red cells only)
    const int par = (gx0 + gy0) & 1;
    constexpr int XP = (WX - 2) / 2;
    for (int k = (int)threadIdx.x; k < XP * (WY - 2); k += NT) {
        const int row = k / XP, m = k - row * XP, ly = 1 + row;
        const int i = ly * WX + tile_color_x(m, ly, par, 1);
        sX[i] = gs(i);
    }
    __syncthreads();
    // red on the tile (reads black cells only); both colours written out
    for (int j = (int)threadIdx.x; j < kTFX * kTFY; j += NT) {
        const int ly = j / kTFX, lx = j - ly * kTFX;
        const int gx = tx * kTFX + lx, gy = ty * kTFY + ly;
        if (gx >= nx || gy >= ny) continue;
        const int i = (ly + H) * WX + lx + H;
        const T v = ((gx + gy) & 1) == 0 ? gs(i) : sX[i];
        x[gx + nx * gy] = v;
        dots.add(gx + nx * gy, (double)v);
    }
    dots.template finish<NT>();
}

// ---------------------------------------------------------------------------
// Level 0 of a 2D solve with one reduction point per CG iteration (Chronopoulos
// and Gear's arrangement of conjugate gradients): the way up also forms
// w = A z, so both inner products r.z and w.z are taken there, and the next
// way down forms beta, alpha, p = z + beta p, s = w + beta s (= A p),
// x += alpha p and r -= alpha s before it smooths.  The iterates are those of
// the usual order in exact arithmetic.  On a singular operator the update also
// takes the mean of r off: the recurrence of s collects rounding, so the sum of r
// drifts from 0, and what cannot be solved for stays in r (768 x 512, density
// ratio 1e4: r stalled at 2e-11 of b; of 360 solves to 1e-13 at ratios of 1e3 to
// 1e5, 512^2 to 1024 x 640, 141 did not end, 43 with two reductions, none now).
// What goes is the launch of the operator apply (5.7 us at 128 x 256, 6.8 us at
// 256 x 512, FP64), which on these grids costs its latency, against a longer way
// down (6.7 -> 7.4 us, 7.0 -> 8.1) and way up (5.9 -> 6.5, 6.2 -> 6.8); the end of
// the iteration moves from a launch of its own (2.7 us) into the single-workgroup
// coarse kernel.  Residuals and solutions agree with the two-reduction form to
// rounding (224 solves of 64^2 to 1024 x 640, ratios 10 to 1e4: the same
// iteration counts up to -6 and +2, true residuals 2 % larger on average).
// ---------------------------------------------------------------------------
// Sums of four per-thread values over a workgroup of NT threads, in every
// thread (fixed order: waves by shuffles, then the waves in order).
template <int NT>
__device__ inline void tile_sum4_all(double v[4], double (*ws)[NT / kWave]) {
    const int lane = (int)threadIdx.x & (kWave - 1), w = (int)threadIdx.x / kWave;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[q] = wave_sum(v[q]);
        if (lane == 0) ws[q][w] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[q] = 0.0;
        for (int k = 0; k < NT / kWave; ++k) v[q] += ws[q][k];
    }
}

// Partials per tile of the way up: r.z, sum z, sum r, w.z.
struct CgPart {
    double *rz, *z, *r, *wz;
};
// Vectors of the way down of iteration k (r, s: old; rn, sn: new, other
// buffers, since neighbouring tiles read the old ones in their halos).
template <typename TR>
struct CgVec2 {
    const TR *r, *s, *w;
    TR *rn, *sn, *p, *x;
};

// One tile of the way down of CG iteration k: scalars, vector updates on the
// tile's cells (one per thread), the partial of r.r, and the passes of
// down_tile2 from the new residual.  The old s is not read for k = 0.
template <typename T, typename TR>
__device__ inline void cg_down_tile2(const Level<T> &L, const Geo &gc, const CgVec2<TR> &v, const T *__restrict__ z,
                                     T *__restrict__ xs, T *__restrict__ bc, int tx, int ty, int tile_id, int k,
                                     int singular, Scal *sc, const CgPart &pt, int nparts,
                                     double *__restrict__ part_rr) {
    constexpr int NT = kTileThreads, H = kDownH, WX = kDownWX, NL = kDownNL;
    constexpr int KL = (NL + NT - 1) / NT;
    static_assert(kTFX * kTFY == NT, "one owned cell per thread");
    __shared__ DownTile<T, false> tile;
    __shared__ double ws[4][NT / kWave], wr[NT / kWave];
    const int tid = (int)threadIdx.x;
    const int nx = (int)L.g.n[0], ny = (int)L.g.n[1];
    const int px = L.g.per[0], py = L.g.per[1];
    const int gx0 = tx * kTFX - H, gy0 = ty * kTFY - H;
    // every load of the thread is issued before anything is waited for
    const int dn = sc->done;
    const double prev_rz = k > 0 ? sc->rzs[(k + 1) & 1] : 0.0, prev_al = k > 0 ? sc->als[(k + 1) & 1] : 0.0;
    TR lr[KL], lw[KL], lo[KL];
    T li[KL], l0[KL], l1[KL];
    bool lv[KL], m0[KL], m1[KL];
#pragma unroll
    for (int q = 0; q < KL; ++q) {
        const int i0 = tid + q * NT, i = i0 < NL ? i0 : NL - 1;
        const int ly = i / WX, lx = i - ly * WX;
        bool vx, vy;
        const int gx = tile_coord(gx0 + lx, nx, px, vx), gy = tile_coord(gy0 + ly, ny, py, vy);
        const bool in = vx && vy;
        const int g = in ? gx + nx * gy : 0;
        lr[q] = v.r[g];
        lw[q] = v.w[g];
        lo[q] = (TR)0;
        if (k > 0) lo[q] = v.s[g];
        li[q] = L.invd[g];
        l0[q] = L.cs[0][g];
        l1[q] = L.cs[1][g];
        lv[q] = in;
        m0[q] = in && (px || gx > 0);
        m1[q] = in && (py || gy > 0);
    }
    const int oy = tid / kTFX, ox = tid - oy * kTFX;
    const int cx = tx * kTFX + ox, cy = ty * kTFY + oy;
    const bool own = cx < nx && cy < ny;
    const int c = own ? cx + nx * cy : 0;
    const double oz = (double)z[c], oxx = (double)v.x[c], orr = (double)v.r[c], ow = (double)v.w[c];
    double op = 0.0, os = 0.0;
    if (k > 0) {
        op = (double)v.p[c];
        os = (double)v.s[c];
    }
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = tid; i < nparts; i += NT) {
        sum[0] += pt.rz[i];
        sum[1] += pt.wz[i];
        if (singular) {
            sum[2] += pt.z[i];
            sum[3] += pt.r[i];
        }
    }
    if (dn) return;
    tile_sum4_all<NT>(sum, ws);
    // a singular operator's z is projected onto its range (mean removed); A z
    // does not see the constant
    const double zm = singular ? sum[2] / (double)L.g.N : 0.0, rm = singular ? sum[3] / (double)L.g.N : 0.0;
    const double rz = sum[0] - zm * sum[3];
    const double beta = (k == 0 || prev_rz == 0.0) ? 0.0 : rz / prev_rz;
    const double back = (k == 0 || prev_al == 0.0) ? 0.0 : beta * rz / prev_al;
    const double pq = sum[1] - back;
    const double alpha = pq != 0.0 ? rz / pq : 0.0;
    const bool ok = isfinite(rz) && isfinite(alpha);
    if (tile_id == 0 && tid == 0) {
        if (ok) {
            sc->rzs[k & 1] = rz;
            sc->als[k & 1] = alpha;
        } else {
            sc->nonfinite = 1;
            sc->done = 1;
        }
    }
    if (!ok) return;
    auto residual = [&](double r, double s) { return (TR)fma(-alpha, s, r - rm); };
#pragma unroll
    for (int q = 0; q < KL; ++q) {
        const int i0 = tid + q * NT, i = i0 < NL ? i0 : NL - 1;
        const T fv = lv[q] ? (T)1 : (T)0;
        const TR sn = (TR)fma(beta, (double)lo[q], (double)lw[q]);
        tile.sB[i] = (T)residual((double)lr[q], (double)sn) * fv;
        tile.sI[i] = li[q] * fv;
        tile.sC0[i] = l0[q] * (m0[q] ? (T)1 : (T)0);
        tile.sC1[i] = l1[q] * (m1[q] ? (T)1 : (T)0);
    }
    double rr = 0.0;
    if (own) {
        const double pn = (oz - zm) + beta * op;
        const TR sn = (TR)fma(beta, os, ow), rn = residual(orr, (double)sn);
        v.p[c] = (TR)pn;
        v.x[c] = (TR)(oxx + alpha * pn);
        v.sn[c] = sn;
        v.rn[c] = rn;
        rr = (double)rn * (double)rn;
    }
    rr = wave_sum(rr);
    if ((tid & (kWave - 1)) == 0) wr[tid / kWave] = rr;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int q = 0; q < NT / kWave; ++q) t += wr[q];
        part_rr[tile_id] = t;
    }
    down_passes2<T, NT, false>(tile, L, gc, xs, bc, tx, ty);
}

// One tile of the way up that ends the preconditioner of a CG iteration:
// red x += P e, black GS, red GS as in up_tile2 but on one halo cell more
// (staged halo 3, black on 2, red on 1), then w = A z and the partials of
// r.z, sum z, sum r and w.z on the tile's cells.  rhs: the CG residual.
// A singular operator has s = +0: not read.
template <typename T, typename TR>
__device__ inline void cg_up_tile2(const Level<T> &L, const Geo &gc, const T *__restrict__ xc,
                                   const TR *__restrict__ r, const T *__restrict__ xs, T *__restrict__ z,
                                   TR *__restrict__ w, const Level<TR> &A, int tx, int ty, int tile_id, int singular,
                                   const CgPart &pt, int skip) {
    using R = T;
    constexpr int NT = kTileThreads, H = 3, WX = kTFX + 2 * H, WY = kTFY + 2 * H, NL = WX * WY;
    constexpr int KL = (NL + NT - 1) / NT;
    static_assert(kTFX * kTFY == NT, "one owned cell per thread");
    __shared__ T sB[NL], sI[NL], sC0[NL], sC1[NL], sX[NL];
    __shared__ double ws[4][NT / kWave];
    const int tid = (int)threadIdx.x;
    const int nx = (int)L.g.n[0], ny = (int)L.g.n[1];
    const int px = L.g.per[0], py = L.g.per[1];
    const int gx0 = tx * kTFX - H, gy0 = ty * kTFY - H;
    T lb[KL], li[KL], l0[KL], l1[KL], lx_[KL];
    bool lv[KL], m0[KL], m1[KL];
#pragma unroll
    for (int q = 0; q < KL; ++q) {
        const int i0 = tid + q * NT, i = i0 < NL ? i0 : NL - 1;
        const int ly = i / WX, lx = i - ly * WX;
        bool vx, vy;
        const int gx = tile_coord(gx0 + lx, nx, px, vx), gy = tile_coord(gy0 + ly, ny, py, vy);
        const bool in = vx && vy;
        const int g = in ? gx + nx * gy : 0;
        lb[q] = (T)r[g];
        li[q] = L.invd[g];
        l0[q] = L.cs[0][g];
        l1[q] = L.cs[1][g];
        const int ia[3] = {in ? gx : 0, in ? gy : 0, 0};
        const R pe = prolong_at<T, 2>(L.g, gc, xc, ia);
        const T red = (in && ((gx0 + lx + gy0 + ly) & 1) == 0) ? (T)1 : (T)0;
        lx_[q] = (T)((R)xs[g] + pe) * red;
        lv[q] = in;
        m0[q] = in && (px || gx > 0);
        m1[q] = in && (py || gy > 0);
    }
    // the owned cell's operator row (in the CG's precision) and residual
    const int oy = tid / kTFX, ox = tid - oy * kTFX;
    const int cx = tx * kTFX + ox, cy = ty * kTFY + oy;
    const bool own = cx < nx && cy < ny;
    const int ca[3] = {own ? cx : 0, own ? cy : 0, 0};
    const int c = ca[0] + nx * ca[1];
    const int xl = nb_lo(A.g, c, ca[0], 0), xh = nb_hi(A.g, c, ca[0], 0);
    const int yl = nb_lo(A.g, c, ca[1], 1), yh = nb_hi(A.g, c, ca[1], 1);
    const double a0 = (double)A.cs[0][c], a1 = (double)A.cs[0][xh >= 0 ? xh : c];
    const double a2 = (double)A.cs[1][c], a3 = (double)A.cs[1][yh >= 0 ? yh : c];
    double as = 0.0;
    if (!singular) as = (double)A.s[c];
    const double rc = (double)r[c];
    if (skip) return;
#pragma unroll
    for (int q = 0; q < KL; ++q) {
        const int i0 = tid + q * NT, i = i0 < NL ? i0 : NL - 1;
        const T fv = lv[q] ? (T)1 : (T)0;
        sB[i] = lb[q] * fv;
        sI[i] = li[q] * fv;
        sC0[i] = l0[q] * (m0[q] ? (T)1 : (T)0);
        sC1[i] = l1[q] * (m1[q] ? (T)1 : (T)0);
        sX[i] = lx_[q];
    }
    __syncthreads();
    auto gs = [&](int i) {
        R acc = 0.0;
        acc += (R)sC0[i] * (R)sX[i - 1];
        acc += (R)sC0[i + 1] * (R)sX[i + 1];
        acc += (R)sC1[i] * (R)sX[i - WX];
        acc += (R)sC1[i + WX] * (R)sX[i + WX];
        return (T)(((R)sB[i] + acc) * (R)sI[i]);
    };
    const int par = (gx0 + gy0) & 1;
    // black on the tile and 2 halo cells (local [1, WX-1) x [1, WY-1))
    constexpr int XB = (WX - 2) / 2;
    for (int q = tid; q < XB * (WY - 2); q += NT) {
        const int row = q / XB, m = q - row * XB, ly = 1 + row;
        const int i = ly * WX + tile_color_x(m, ly, par, 1);
        sX[i] = gs(i);
    }
    __syncthreads();
    // red on the tile and 1 halo cell (local [2, WX-2) x [2, WY-2)): every
    // second cell of the rows, whose x of that colour starts at 2 or 3
    constexpr int XR = (WX - 4) / 2;
    for (int q = tid; q < XR * (WY - 4); q += NT) {
        const int row = q / XR, m = q - row * XR, ly = 2 + row;
        const int i = ly * WX + 2 + 2 * m + ((ly + par) & 1);
        sX[i] = gs(i);
    }
    __syncthreads();
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    if (own) {
        const int i = (oy + H) * WX + ox + H;
        const double zc = (double)sX[i];
        double wv = as * zc;
        wv += (xl >= 0 ? a0 : 0.0) * (zc - (double)sX[i - 1]);
        wv += (xh >= 0 ? a1 : 0.0) * (zc - (double)sX[i + 1]);
        wv += (yl >= 0 ? a2 : 0.0) * (zc - (double)sX[i - WX]);
        wv += (yh >= 0 ? a3 : 0.0) * (zc - (double)sX[i + WX]);
        z[c] = (T)sX[i];
        w[c] = (TR)wv;
        sum[0] = rc * zc;
        sum[1] = zc;
        sum[2] = rc;
        sum[3] = wv * zc;
    }
    tile_sum4_all<NT>(sum, ws);
    if (tid == 0) {
        pt.rz[tile_id] = sum[0];
        pt.z[tile_id] = sum[1];
        pt.r[tile_id] = sum[2];
        pt.wz[tile_id] = sum[3];
    }
}

}  // namespace chns
