"""GPU solver kernels at the sizes where their launch form changes, against
the FP64 CPU oracle's operators.

Bar of a manufactured solve: the right-hand side is the oracle operator
applied to a known field, the solve stops at a relative residual of 1e-13,
and the V-cycle-preconditioned operator has a condition number of a few
units per decade of density contrast, so the field comes back to 1e-9 as in
the pressure parity tests.
"""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import MACGrid, Params
from oracle import chns as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _lib():
    import paper_2009_06628_amd as P
    return P


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def manufactured(n, per, ratio, seed):
    """Density of a drop, a known mean-free field and the oracle's operator on it."""
    g = MACGrid(n, 1.0 / n[0], per)
    X = g.coords()
    r2 = sum((X[a] - 0.5 * g.n[a] * g.h) ** 2 for a in range(g.dim))
    phi = np.tanh((np.sqrt(r2) - 0.25) / (np.sqrt(2.0) * 1.5 * g.h))
    rho = 0.5 * (1 - ratio) * phi + 0.5 * (1 + ratio)
    rng = np.random.default_rng(seed)
    x = np.ones(g.shape)
    for a in range(g.dim):
        x = x * np.cos(2.0 * np.pi * (X[a] / (g.n[a] * g.h)) + 0.4 * a)
    x = x + 0.1 * rng.normal(size=g.shape)
    x -= x.mean()
    rhs = -g.div([g.grad(x, a) / g.avg(rho, a) for a in range(g.dim)])
    return g, rho, x, rhs


def solve_error(n, per, ratio=0.1, precision=0, seed=3, tile_cells=None):
    P = _lib()
    g, rho, x, rhs = manufactured(n, per, ratio, seed)
    h = P.create_grid(n, g.h, ["periodic" if q else "wall" for q in per], precision=precision)
    if tile_cells is not None:   # largest 3D level of the tile passes
        h.set_option(P.CHNS_OPT_TILE_CYCLE_CELLS, tile_cells)
    p = dev(np.zeros(g.shape))
    out = h.solve_pressure(dev(rho), dev(rhs), p, rtol=1e-13, max_iter=300)
    assert out["rc"] == 0, out
    err = float(np.abs(p.cpu().numpy() - x).max() / np.abs(x).max())
    print("solve", n, per, precision, out, "err %.2e" % err, flush=True)
    return err


@pytest.mark.parametrize("n,per", [((80, 80, 80), (True, True, True)),       # grid-stride apply (below 2^19 cells)
                                   ((96, 80, 80), (False, True, False)),      # marching, 2 planes per block
                                   ((48, 32, 384), (True, False, True)),      # marching, long z, partial x tile
                                   ((128, 128, 64), (False, False, False))])  # marching, 4 planes per block
@pytest.mark.parametrize("precision", [0, 1])
def test_cg_apply_forms(n, per, precision):
    assert solve_error(n, per, precision=precision) <= 1e-9


# coarsest levels of 15, 32, 45, 60, 64 cells (the register inverse with 1 to 4
# entries per thread and axis), 121 (the in-place inverse in memory) and grids
# that are their own coarsest level or one above it
@pytest.mark.parametrize("n,per", [((40, 24), (True, False)), ((64, 128), (False, True)), ((36, 20), (True, True)),
                                   ((48, 80), (False, False)), ((64, 64), (True, True)), ((44, 44), (True, False)),
                                   ((8, 8), (True, True)), ((16, 16), (False, False)), ((24, 24, 24), (True, False, True)),
                                   ((32, 32, 64), (True, True, True))])
@pytest.mark.parametrize("precision", [0, 1])
def test_coarse_setup_forms(n, per, precision):
    assert solve_error(n, per, ratio=0.01, precision=precision) <= 1e-9


# 2D solves with one reduction point per CG iteration: a single row of tiles,
# partial tiles, the most tiles of that form (2048) and the first grid past it
@pytest.mark.parametrize("n,per", [((64, 48), (True, True)), ((72, 88), (False, True)), ((80, 176), (True, False)),
                                   ((2048, 16), (False, False)), ((1024, 1024), (True, False)),
                                   ((1088, 1024), (False, True))])
@pytest.mark.parametrize("precision", [0, 1])
def test_one_reduction_forms(n, per, precision):
    assert solve_error(n, per, ratio=0.01, precision=precision) <= 1e-9


# the one-workgroup V-cycle: one, two and three swept levels, no swept level
# (343 and 270 coarsest cells, inverse read from memory), 121 coarsest cells
# below two swept levels, and rows of one pair
@pytest.mark.parametrize("n,per", [((128, 64), (True, False)), ((96, 96), (False, False)), ((88, 88), (True, True)),
                                   ((512, 8), (True, False)), ((14, 14, 14), (True, False, True)),
                                   ((18, 10, 12), (False, True, True)), ((24, 24, 48), (False, True, False)),
                                   ((16, 16, 32), (True, True, True)), ((8, 32, 32), (True, False, True))])
@pytest.mark.parametrize("precision", [0, 1])
def test_small_level_cycle_forms(n, per, precision):
    assert solve_error(n, per, ratio=0.01, precision=precision) <= 1e-9


# way down and post-smoothing of a 3D level in one pass each: ragged tiles in x and y, chunks of 4,
# 8, 16 and (past 1024 blocks of 16 planes) 32 planes, a single column of tiles
# in x, walls on each axis
@pytest.mark.parametrize("n,per", [((36, 20, 40), (True, False, True)), ((40, 24, 96), (False, True, False)),
                                   ((24, 32, 64), (True, True, True)), ((72, 56, 48), (False, False, False)),
                                   ((80, 144, 80), (True, True, False)), ((160, 80, 80), (False, True, True)),
                                   ((512, 256, 64), (True, False, True))])
@pytest.mark.parametrize("precision", [0, 1])
def test_post_sweep_forms(n, per, precision):
    assert solve_error(n, per, ratio=0.01, precision=precision, tile_cells=0) <= 1e-9


# axis transforms of the direct Cahn-Hilliard solve on 32-wide matrix-core
# tiles: a ragged last tile and k below one chunk (40), k of one chunk and a
# part (72), several chunks with a ragged last one (544).  Bar: MG-PCG stops at
# 1e-10 per solve, as in the parity test of the direct solve.
@pytest.mark.parametrize("n,bc", [((40, 72, 72), ("periodic", "wall", "periodic")), ((576, 544), ("wall", "periodic"))])
def test_axis_transform_forms(n, bc):
    P = _lib()
    prob = W.spinodal(n[0], steps=2, bc=(W.PERIODIC,) * len(n))
    prob = dataclasses.replace(prob, n=n, bc=tuple({"periodic": W.PERIODIC, "wall": W.WALL}[b] for b in bc))
    out = []
    for solver in (P.CHNS_CH_DIRECT, P.CHNS_CH_PCG):
        print("CH solver", n, solver, flush=True)
        g = P.grid_for_problem(prob)
        g.set_option(P.CHNS_OPT_CH_SOLVER, solver)
        st = g.new_state(W.initial_state(prob))
        stats = g.step(st, 2)
        out.append((st["phi"].cpu().numpy(), stats["iters_ch"]))
    (a, ia), (b, ib) = out
    assert ia == 1 and ib > 1
    assert float(np.abs(a - b).max() / np.abs(b).max()) < 1e-8


# coarsest levels inverted by block steps of 16 pivots: 66 and 72 cells (a part
# of a block left over; an odd number of blocks), 255, 306, 448 and 486 cells
@pytest.mark.parametrize("n,per", [((88, 48), (True, False)), ((72, 64), (False, False)), ((34, 30), (True, True)),
                                   ((144, 136), (False, True)), ((56, 64, 64), (False, False, True)),
                                   ((36, 36, 24), (True, True, True))])
@pytest.mark.parametrize("precision", [0, 1])
def test_coarse_inverse_block_forms(n, per, precision):
    assert solve_error(n, per, ratio=0.01, precision=precision) <= 1e-9


# the CG apply that forms the pressure coefficients from the density
# (CHNS_OPT_MARCH_SWEEP_CELLS at or below the grid's cells): the timing record
# shows that it ran (density, p_old and z read, p_new and q written), and the
# solution has the bits of the stored coefficients.  Grids below 2^19 cells (one
# cell per thread) and above (marching), ragged tiles, walls.
@pytest.mark.parametrize("n,per", [((32, 16, 24), (True, True, False)), ((36, 20, 40), (False, False, True)),
                                   ((80, 112, 64), (False, True, False)), ((80, 96, 80), (True, False, True))])
@pytest.mark.parametrize("precision", [0, 1])
def test_density_form_of_the_cg_apply(n, per, precision):
    P = _lib()
    g, rho, x, rhs = manufactured(n, per, 0.01, 5)
    sols = []
    for cells in (1 << 24, 1):
        h = P.create_grid(n, g.h, ["periodic" if q else "wall" for q in per], precision=precision)
        h.set_option(P.CHNS_OPT_MARCH_SWEEP_CELLS, cells)
        h.set_timing(True)
        p = dev(np.zeros(g.shape))
        out = h.solve_pressure(dev(rho), dev(rhs), p, rtol=1e-13, max_iter=300)
        apply = [t for t in h.get_timing() if t["name"] == "pcg_apply"][0]
        print("density form", n, precision, cells, out, apply, flush=True)
        assert out["rc"] == 0
        if cells == 1:
            assert apply["bytes"] == apply["launches"] * (32 + (4 if precision else 8)) * x.size
        sols.append(p)
    assert torch.equal(sols[0], sols[1])
    assert float(np.abs(sols[1].cpu().numpy() - x).max() / np.abs(x).max()) <= 1e-9


# bytes of the timing record: each array a launch reads or writes once (w bytes
# per value of the hierarchy, 8 in the CG), over all launches of a class
def timed_solve(n, precision, **option):
    P = _lib()
    g, rho, x, rhs = manufactured(n, (True,) * len(n), 0.1, 6)
    h = P.create_grid(n, g.h, ["periodic"] * len(n), precision=precision)
    for name, value in option.items():
        h.set_option(getattr(P, name), value)
    h.set_timing(True)
    out = h.solve_pressure(dev(rho), dev(rhs), dev(np.zeros(g.shape)), rtol=1e-10)
    assert out["rc"] == 0
    rec = {t["name"]: (t["launches"], t["bytes"]) for t in h.get_timing()}
    print("bytes", n, precision, option, rec, flush=True)
    return rec


@pytest.mark.parametrize("precision", [0, 1])
def test_timing_bytes_2d(precision):
    """128^2: two tiled levels and 32^2 below them."""
    rec = timed_solve((128, 128), precision)
    w, n0, n1, n2 = (4 if precision else 8), 128 ** 2, 64 ** 2, 32 ** 2
    cycles = rec["mg_down"][0] // 2
    assert rec["mg_down"][0] == 2 * cycles == rec["mg_up"][0]
    # b, 1/d, two cs in, x and the coarse b out; with the update: r, s, w, p, x in, r, s, p, x out and z for b
    assert rec["mg_down"][1] == (5 * w * n0 + w * n1) + (cycles - 1) * ((9 * 8 + 5 * w) * n0 + w * n1) \
        + cycles * (5 * w * n1 + w * n2)
    # level 0: r in, w out, x, 1/d, two cs and the coarse x in, z out, the operator's own cs where they are others
    assert rec["mg_up"][1] == cycles * ((2 * 8 + (2 * 8 if precision else 0) + 5 * w) * n0 + w * n1) \
        + cycles * (6 * w * n1 + w * n2)


@pytest.mark.parametrize("precision", [0, 1])
def test_timing_bytes_3d(precision):
    """32^3: two levels marching along z and 8^3 below them."""
    rec = timed_solve((32, 32, 32), precision, CHNS_OPT_TILE_CYCLE_CELLS=0)
    w, n0, n1, n2 = (4 if precision else 8), 32 ** 3, 16 ** 3, 8 ** 3
    cycles = rec["mg_down"][0] // 2
    assert rec["mg_down"][0] == 2 * cycles == rec["smooth"][0]
    # b, 1/d, three cs in, x and the coarse b out
    assert rec["mg_down"][1] == cycles * (6 * w * n0 + w * n1 + 6 * w * n1 + w * n2)
    # x as well in, and r for r.z where it is not b
    assert rec["smooth"][1] == cycles * ((7 * w + (8 if precision else 0)) * n0 + w * n1 + 7 * w * n1 + w * n2)
    # z, p_old, three cs in, p_new, q out (s of a singular operator is not read)
    assert rec["pcg_apply"][1] == rec["pcg_apply"][0] * (6 * 8 + w) * n0


@pytest.mark.parametrize("precision", [0, 1])
def test_timing_bytes_truncated_cycle(precision):
    """Momentum cycles of 32^3 that end on 16^3 with a symmetric sweep (Re = 50,
    the only launches of the class): b, 1/d, three cs in, x out."""
    P = _lib()
    prob = W.drop3d(32, steps=1, Re=50.0)
    h = P.grid_for_problem(prob, precision)
    st = h.new_state(W.initial_state(prob))
    h.set_timing(True)
    h.step(st, 1)
    rec = {t["name"]: (t["launches"], t["bytes"]) for t in h.get_timing()}
    print("bytes truncated", precision, rec, flush=True)
    assert rec["smooth"][1] == rec["smooth"][0] * 6 * (4 if precision else 8) * 16 ** 3


# momentum solves of a 2D grid past 2048 level-0 tiles (2176), where the update,
# the sums and the operator apply, with the diagonal shift of its rows, are
# launches of their own.  The predicted velocity u* must satisfy the oracle's
# momentum rows.  Bar: the solver stops at a relative residual of rtol_mom on the
# recurred residual; applying A costs a relative 1e-16 of its largest terms,
# which add up to about 100 times b here (4 eta / (Re h^2) against rho / dt), a few
# times per iteration, so 1e-12 on top of twice the tolerance.
@pytest.mark.parametrize("precision", [0, 1])
def test_momentum_past_the_one_reduction_form(precision):
    P = _lib()
    n = (1088, 1024)
    tol = W.PRECISION_FORM_TOLERANCES if precision else {}
    prob = W.Problem("walls", n, 1.0 / n[0], (W.WALL, W.WALL), W.static_drop(n[0], **tol).props, 1, "drop",
                     {"centre": (0.5, 0.45), "radius": 0.25, "velocity": "stream", "vseed": 3, "vamp": 0.05})
    assert (n[0] // 32) * (n[1] // 16) > 2048
    ini = W.initial_state(prob)
    h = P.grid_for_problem(prob, precision)
    st, rec = h.new_state(ini), h.new_record()
    h.step_record(st, rec)
    torch.cuda.synchronize()
    # the right-hand side and rows of the oracle's predictor, from the step's own phi and mu
    g, prm = MACGrid(prob.n, prob.h, prob.periodic), Params.from_props(prob.props)
    alpha, beta, gamma, xi = O.coefficients(prm)
    phi, u = ini["phi"], ini["u"]
    phi_new, mu = rec["phi_new"].cpu().numpy(), rec["mu"].cpu().numpy()
    gmu = [g.grad(mu, a) for a in range(2)]
    m = [np.where(g.wall_face_mask(a), 0.0, g.avg(alpha * phi + beta, a) * u[a] - (alpha / prm.Cn) * gmu[a] / prm.Pe)
         for a in range(2)]
    rho_old, rho_new = alpha * O.pullback(phi) + beta, alpha * O.pullback(phi_new) + beta
    eta = gamma * O.pullback(phi_new) + xi
    for a in range(2):
        rhs = 0.5 * (g.avg(rho_new, a) + g.avg(rho_old, a)) / prm.dt * u[a] - O.skew_advection(g, m, u[a], a)
        rhs = rhs - (1.0 / (prm.We * prm.Cn)) * g.avg(phi, a) * gmu[a]
        A, unk = O.momentum_matrix(g, a, g.avg(rho_new, a) / prm.dt, eta, prm.Re)
        us = rec["ustar"][a].cpu().numpy()
        res = float(np.linalg.norm(rhs[unk] - A @ us[unk]) / np.linalg.norm(rhs[unk]))
        print("momentum residual", precision, a, "%.2e" % res, "change", float(np.abs(us - u[a]).max()), flush=True)
        assert res <= 2.0 * prob.props.rtol_mom + 1e-12
        assert not us[~unk].any()


# the most tiles of the one-reduction form (1408) and the first grid of these
# widths past it (1536), where apply, update and sums are launches of their own
@pytest.mark.parametrize("n,per", [((1024, 704), (False, True)), ((704, 1024), (True, False)),
                                   ((1024, 768), (False, False))])
@pytest.mark.parametrize("precision", [0, 1])
def test_one_reduction_limit(n, per, precision):
    assert solve_error(n, per, ratio=0.01, precision=precision) <= 1e-9


# max_iter is the number of CG iterations a solve may take in every form: 2D with
# one reduction point, 2D with launches of their own, 3D, and the allocation-free
# solve (2D with two reduction points).  Stopped early it reports all of them;
# given exactly the iterations it needs it converges.
@pytest.mark.parametrize("n,alloc", [((64, 64), True), ((1024, 768), True), ((32, 32, 32), True), ((64, 64, 64), True),
                                     ((128, 64), False), ((24, 24, 24), False)])
@pytest.mark.parametrize("precision", [0, 1])
def test_max_iter_counts_every_iteration(n, alloc, precision):
    P = _lib()
    g, rho, x, rhs = manufactured(n, (True,) * len(n), 0.1, 7)
    rho, rhs, bc = dev(rho), dev(rhs), ["periodic"] * len(n)
    h = P.create_grid(n, g.h, bc, precision=precision) if alloc else None

    def solve(max_iter):
        p = dev(np.zeros(g.shape))
        if alloc:
            out = h.solve_pressure(rho, rhs, p, rtol=1e-10, max_iter=max_iter)
        else:
            out = P.solve_pressure_noalloc(n, g.h, bc, rho, rhs, p, rtol=1e-10, max_iter=max_iter, precision=precision)
        print("max_iter", n, alloc, precision, max_iter, out, flush=True)
        return out

    need = solve(300)
    assert need["rc"] == P.CHNS_OK and need["iters"] > 6
    for m in (1, 2, 5, need["iters"] - 1):
        out = solve(m)
        assert out["rc"] == P.CHNS_ENOCONV and out["iters"] == m
    out = solve(need["iters"])
    assert out["rc"] == P.CHNS_OK and out["iters"] == need["iters"]


# large density contrast in the 2D one-reduction form, sources at the interface:
# the residual must fall to rtol (the recurrence's rounding collects in its mean,
# which the operator cannot reduce).  With the mean left in, every one of these
# solves stalls between 1e-13 and 1e-10.
@pytest.mark.parametrize("n,per", [((640, 512), (True, True)), ((512, 768), (True, False)), ((1024, 640), (False, True))])
@pytest.mark.parametrize("precision", [0, 1])
def test_large_contrast_converges(n, per, precision):
    P = _lib()
    g = MACGrid(n, 1.0 / n[0], per)
    X = g.coords()
    r2 = sum((X[a] - 0.5 * g.n[a] * g.h) ** 2 for a in range(2))
    phi = np.tanh((np.sqrt(r2) - 0.25 * min(g.n) * g.h) / (np.sqrt(2.0) * 1.5 * g.h))
    rho = 0.5 * (1 - 1e-5) * phi + 0.5 * (1 + 1e-5)
    rhs = 10.0 * np.random.default_rng(2).normal(size=g.shape) * (1.0 - phi * phi)
    rhs += np.cos(2.0 * np.pi * X[0] / (g.n[0] * g.h)) * np.cos(2.0 * np.pi * X[1] / (g.n[1] * g.h))
    rhs -= rhs.mean()
    h = P.create_grid(n, g.h, ["periodic" if q else "wall" for q in per], precision=precision)
    out = h.solve_pressure(dev(rho), dev(rhs), dev(np.zeros(g.shape)), rtol=1e-13, max_iter=200)
    print("contrast", n, per, precision, out, flush=True)
    assert out["rc"] == P.CHNS_OK
