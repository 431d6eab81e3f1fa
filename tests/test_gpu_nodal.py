"""Nodal projection (Sec. 3.2 Step 11) on the GPU against the nodal oracle:
the node operator, the projection in both precisions over shapes and
boundaries, the full-size workload by properties the oracle checks at any
size, and the error paths."""
import numpy as np
import pytest
import torch

import oracle
from oracle import nodal as nd
from paper_1908_03634_amd import mproj, workloads as W
from tests.gpu_util import N, T, context_for, rel, say

pytestmark = pytest.mark.gpu

BCS = [(0, 0, 1), (1, 1, 1), (0, 0, 0), (1, 0, 1)]
SHAPES = [(16, 16, 16), (32, 24, 20), (48, 32, 40), (12, 10, 14), (8, 8, 6), (7, 9, 5)]


def _mapped(p, precision, **kw):
    ctx = context_for(p, precision, **kw)
    ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center, want_coefs=False)
    return ctx


def _sigma(p):
    g = oracle.Grid.of(p)
    b0 = oracle.fill_beta0(g, p.geometry, p.beta0_1d, p.dr, p.center)
    return g, b0, b0 / p.rho


@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("shape", SHAPES)
def test_node_operator_matches_the_oracle(shape, bc):
    nx, ny, nz = shape
    say("nodal apply", shape, bc)
    p = W.planar_problem(nx=nx, ny=ny, nz=nz, contrast=1e3, bc=bc, seed=7000 + nx, velocity="cells")
    g, _, sigma = _sigma(p)
    ctx = _mapped(p, "fp64")
    assert ctx.node_shape == nd.node_shape(g)
    x = np.random.default_rng(nx * ny).standard_normal(nd.node_shape(g))
    y = N(ctx.nodal_apply(T(x)))
    ref = nd.apply(g, sigma, x)
    assert np.abs(y - ref).max() <= 1e-13 * np.abs(ref).max()
    ctx.close()


def _project_case(p, precision, rtol=1e-12):
    g, b0, sigma = _sigma(p)
    ref = nd.project(p, tol=1e-12)
    ctx = _mapped(p, precision, rtol=rtol)
    ux, uy, uz, S = T(p.ux), T(p.uy), T(p.uz), T(p.S)
    phi, info = ctx.nodal_project(ux, uy, uz, S)
    phi = N(phi)
    assert rel(phi, ref["phi"]) < 1e-9
    assert nd.residual_norm(g, sigma, ref["R"], phi) <= 1.01 * rtol
    assert abs(phi.mean()) <= 1e-12 * np.abs(phi).max()
    for a, b in ((ux, ref["ux"]), (uy, ref["uy"]), (uz, ref["uz"])):
        assert np.abs(N(a) - b).max() <= 1e-9 * np.abs(b).max()
    assert info["rhs_mean"] == pytest.approx(ref["mean"], rel=1e-12, abs=1e-18)
    Rn, _ = nd.rhs(g, b0, *(N(u) for u in (ux, uy, uz)), p.S)
    defect = np.sqrt(nd.node_dot(g, Rn, Rn) / nd.node_dot(g, ref["R"], ref["R"]))
    assert info["div_defect"] == pytest.approx(defect, rel=1e-8)
    ctx.close()
    return info


@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("shape", [(16, 16, 16), (48, 32, 40), (12, 10, 14), (7, 9, 5)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_nodal_projection_matches_the_oracle(shape, bc, precision):
    nx, ny, nz = shape
    say("nodal project", shape, bc, precision)
    p = W.planar_problem(nx=nx, ny=ny, nz=nz, contrast=1e4, bc=bc, seed=7100 + nz, velocity="cells")
    _project_case(p, precision)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_nodal_projection_of_a_64_cube(precision):
    say("nodal project 64^3", precision)
    _project_case(W.planar_problem(64, contrast=1e4, seed=7200, velocity="cells"), precision)


@pytest.mark.parametrize("base", ["irregular", "linear"])
def test_nodal_projection_on_a_star(base):
    say("nodal star", base)
    _project_case(W.spherical_problem(32, contrast=1e5, seed=7300, base=base, velocity="cells"), "mixed")


def test_nodal_projection_full_size():
    """256^3 plane-parallel atmosphere, mixed precision, rtol 1e-10: the
    oracle's FP64 operator confirms the residual of the GPU's phi and its
    gradient confirms the velocity update."""
    say("nodal c2 256^3")
    p = W.config_problem("c2", velocity="cells")
    g, b0, sigma = _sigma(p)
    ctx = _mapped(p, "mixed", rtol=1e-10)
    ux, uy, uz, S = T(p.ux), T(p.uy), T(p.uz), T(p.S)
    phi, info = ctx.nodal_project(ux, uy, uz, S)
    phi = N(phi)
    R, m = nd.rhs(g, b0, p.ux, p.uy, p.uz, p.S)
    assert info["rel_resid"] <= 1e-10
    assert nd.residual_norm(g, sigma, R, phi) <= 1.05e-10
    assert info["rhs_mean"] == pytest.approx(m, rel=1e-12)
    gx, gy, gz = nd.gradient(g, phi)
    w = sigma / b0
    for new, old, gr in ((ux, p.ux, gx), (uy, p.uy, gy), (uz, p.uz, gz)):
        assert np.abs((old - N(new)) - w * gr).max() <= 1e-12 * np.abs(old).max()
    say("nodal c2", info["vcycles"], info["outer_iters"], info["ms_solve"])
    ctx.close()


def test_nodal_projection_is_reproducible_and_warm_starts():
    p = W.planar_problem(32, contrast=1e4, seed=7400, velocity="cells")
    ctx = _mapped(p, "mixed", rtol=1e-11)
    outs = []
    for _ in range(2):
        ux, uy, uz, S = T(p.ux), T(p.uy), T(p.uz), T(p.S)
        phi, info = ctx.nodal_project(ux, uy, uz, S)
        outs.append((N(phi), N(ux)))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    ux, uy, uz, S = T(p.ux), T(p.uy), T(p.uz), T(p.S)
    phi0 = T(outs[0][0])
    _, info = ctx.nodal_project(ux, uy, uz, S, phi=phi0, use_initial_guess=True)
    assert info["outer_iters"] == 0 and info["vcycles"] == 0
    ctx.close()


def test_nodal_sigma_follows_a_new_mapping():
    a = W.planar_problem(16, contrast=1e2, seed=7500, velocity="cells")
    b = W.planar_problem(16, contrast=1e5, seed=7501, velocity="cells")
    ctx = _mapped(a, "mixed")
    ctx.nodal_project(T(a.ux), T(a.uy), T(a.uz), T(a.S))
    ctx.map_base_state(b.geometry, T(b.beta0_1d), T(b.rho), b.dr, b.center, want_coefs=False)
    phi, _ = ctx.nodal_project(T(b.ux), T(b.uy), T(b.uz), T(b.S))
    ref = nd.project(b, tol=1e-12)
    assert rel(N(phi), ref["phi"]) < 1e-6
    ctx.close()


def test_zero_and_rounding_level_right_hand_sides():
    p = W.planar_problem(16, contrast=1e3, seed=7600, velocity="cells")
    ctx = _mapped(p, "mixed")
    z = torch.zeros(p.shape, dtype=torch.float64, device="cuda:0")
    phi, info = ctx.nodal_project(z.clone(), z.clone(), z.clone(), z.clone())
    assert info["rhs_norm"] == 0.0 and np.abs(N(phi)).max() == 0.0
    # beta0 S constant: all of it is the removed mean, R is rounding noise
    _, b0, _ = _sigma(p)
    phi, info = ctx.nodal_project(z.clone(), z.clone(), z.clone(), T(0.25 / b0))
    assert info["rhs_mean"] == pytest.approx(0.25, rel=1e-14)
    assert info["rhs_norm"] <= 1e-13 * np.sqrt(p.ncell)
    assert np.abs(N(phi)).max() <= 1e-12
    ctx.close()


def test_nodal_errors():
    p = W.planar_problem(16, contrast=1e3, seed=7700, velocity="cells")
    ctx = context_for(p, "mixed")
    u = T(p.ux)
    with pytest.raises(mproj.MprojError) as e:
        ctx.nodal_project(u, u.clone(), u.clone(), T(p.S))
    assert e.value.code == 7  # no mapping yet
    ctx.close()
    # 25^3 cells cannot coarsen: 26^3 nodes on the coarsest grid is too many
    q = W.planar_problem(25, contrast=1e3, bc=(1, 1, 1), seed=7701, velocity="cells")
    ctx = _mapped(q, "fp64")
    with pytest.raises(mproj.MprojError) as e:
        ctx.nodal_project(T(q.ux), T(q.uy), T(q.uz), T(q.S))
    assert e.value.code == 1
    ctx.close()


@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("shape", [(32, 24, 20), (12, 10, 14), (64, 64, 64), (8, 8, 6)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_column_kernels_equal_the_one_node_kernels(shape, bc, precision):
    """The z-marching right-hand side, smoother and residuals against the
    one-node kernels (blocked=False).  Each node value is the same expression
    in the same order, but the sums of the right-hand side's node mean and of
    the residual norms run over other block trees, so the removed mean (and in
    mixed precision the refinement scale) moves by rounding: the results agree
    to rounding and take the same number of V-cycles."""
    nx, ny, nz = shape
    say("nodal columns", shape, bc, precision)
    p = W.planar_problem(nx=nx, ny=ny, nz=nz, contrast=1e4, bc=bc, seed=7800 + nx, velocity="cells")
    outs = []
    for blocked in (True, False):
        ctx = _mapped(p, precision, rtol=1e-11, blocked=blocked)
        ux, uy, uz = T(p.ux), T(p.uy), T(p.uz)
        phi, info = ctx.nodal_project(ux, uy, uz, T(p.S))
        outs.append((N(phi), N(ux), info["vcycles"]))
        ctx.close()
    assert outs[0][2] == outs[1][2]
    assert rel(outs[0][0], outs[1][0]) < 1e-8 and rel(outs[0][1], outs[1][1]) < 1e-8


@pytest.mark.parametrize("shape,bc", [((32, 32, 32), (0, 0, 1)), ((48, 32, 40), (1, 1, 1)), ((64, 64, 64), (0, 0, 0)),
                                      ((24, 16, 20), (1, 0, 1))])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_nodal_coarse_cycle_equals_per_level_launches(shape, bc, precision):
    """The single-workgroup coarse cycle (every coarse array in LDS) runs the
    same per-node arithmetic as one launch per operation: the same bits."""
    nx, ny, nz = shape
    say("nodal coarse cycle", shape, bc, precision)
    p = W.planar_problem(nx=nx, ny=ny, nz=nz, contrast=1e4, bc=bc, seed=7900 + nx + nz, velocity="cells")
    outs = []
    for cc in (True, False):
        ctx = _mapped(p, precision, rtol=1e-11, coarse_cycle=cc)
        ux = T(p.ux)
        phi, info = ctx.nodal_project(ux, T(p.uy), T(p.uz), T(p.S))
        outs.append((N(phi), N(ux), info["vcycles"]))
        ctx.close()
    assert outs[0][2] == outs[1][2]
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("shape,bc", [((128, 16, 12), (0, 0, 1)), ((128, 8, 18), (0, 0, 0)), ((128, 8, 34), (0, 0, 1)),
                                      ((256, 12, 10), (0, 0, 1)), ((256, 32, 16), (0, 0, 1)),
                                      ((256, 256, 24), (0, 0, 1)), ((64, 16, 12), (0, 0, 1)), ((64, 6, 10), (0, 0, 0)),
                                      ((32, 8, 10), (0, 0, 1)), ((32, 10, 6), (0, 0, 0))])
def test_two_colour_passes_equal_four_colour_passes(shape, bc):
    """On rows of 32, 64, 128 or 256 nodes (periodic x and y) the
    mixed-precision smoother runs the two colours of each row parity in one
    out-of-place pass (first colour one plane ahead of the second; a
    wavefront holds one, two or four rows); with one pass per colour
    (smoother="per_colour") the projection is the same bit for bit, through
    plane chunks of ragged length, row counts that leave part of a wavefront
    empty, and the coarser levels below a 256-node grid."""
    nx, ny, nz = shape
    say("nodal two-colour passes", shape, bc)
    p = W.planar_problem(nx=nx, ny=ny, nz=nz, contrast=1e4, bc=bc, seed=8100 + nx + ny + nz, velocity="cells")
    outs = []
    for sm in ("auto", "per_colour"):
        ctx = _mapped(p, "mixed", rtol=1e-11, smoother=sm)
        ux, uy, uz = T(p.ux), T(p.uy), T(p.uz)
        phi, info = ctx.nodal_project(ux, uy, uz, T(p.S))
        outs.append((N(phi), N(ux), N(uz), info["vcycles"], info["rel_resid"]))
        ctx.close()
    assert outs[0][3] == outs[1][3] and outs[0][4] <= 1e-11
    for a, b in zip(outs[0][:3], outs[1][:3]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("bc", [(0, 0, 1), (1, 1, 1)])
def test_pressure_from_the_nodal_scalar(bc):
    """pi = s phi bit for bit with the oracle's update; the increment form
    a pi + s phi likewise (a a power of two, so both sides round once); the
    gradient of pi / s reproduces the correction the projection applied."""
    say("nodal pi", bc)
    p = W.planar_problem(nx=24, ny=20, nz=28, contrast=1e4, bc=bc, seed=7800, velocity="cells")
    g, b0, sigma = _sigma(p)
    ctx = _mapped(p, "mixed", rtol=1e-12)
    ux, uy, uz = T(p.ux), T(p.uy), T(p.uz)
    phi, _ = ctx.nodal_project(ux, uy, uz, T(p.S))
    s = 1.0 / 2.5e-3
    pi = ctx.nodal_pi(phi, s)
    torch.cuda.synchronize()
    assert np.array_equal(N(pi), nd.update_pi(N(phi), s))
    gx, gy, gz = nd.gradient(g, N(pi))
    w = sigma / b0 / s
    for new, old, gr in ((ux, p.ux, gx), (uy, p.uy, gy), (uz, p.uz, gz)):
        assert np.abs((old - N(new)) - w * gr).max() <= 1e-12 * np.abs(old).max()
    old = np.random.default_rng(11).standard_normal(ctx.node_shape)
    inc = T(old)
    ctx.nodal_pi(phi, s, pi=inc, a=0.5)
    torch.cuda.synchronize()
    assert np.array_equal(N(inc), nd.update_pi(N(phi), s, pi=old, a=0.5))
    with pytest.raises(mproj.MprojError) as e:
        ctx.nodal_pi(phi, s, pi=phi)
    assert e.value.code == 1
    with pytest.raises(mproj.MprojError) as e:
        ctx.nodal_pi(phi, float("nan"), pi=inc)
    assert e.value.code == 5
    ctx.close()


# the bottom kernel's forms end at 256, 512, 1024, 2048, 3072 and 5120 nodes;
# (48, 40, 56) ends its coarse cycle on 336 nodes, one per thread
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,bc", [((5, 5, 6), (1, 1, 1)), ((7, 7, 7), (1, 1, 1)), ((7, 9, 9), (0, 1, 1)),
                                      ((11, 11, 9), (1, 1, 1)), ((13, 13, 13), (1, 1, 1)), ((15, 17, 15), (0, 0, 1)),
                                      ((17, 17, 17), (1, 1, 1)), ((48, 40, 56), (1, 1, 1))])
def test_nodal_bottom_sizes(shape, bc, precision):
    nx, ny, nz = shape
    say("nodal bottom", shape, bc, precision)
    p = W.planar_problem(nx=nx, ny=ny, nz=nz, contrast=1e3, bc=bc, seed=7800 + nx, velocity="cells")
    info = _project_case(p, precision)
    assert info["bottom_iters_total"] > 0


# two levels in the coarse cycle would leave 1035 nodes to the bottom solve that
# has a node per thread of 1024: these levels keep their own launches
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_nodal_bottom_too_large_for_the_coarse_cycle(precision):
    say("nodal coarse cycle, long bottom", precision)
    p = W.planar_problem(nx=8, ny=8, nz=456, contrast=1e2, bc=(1, 1, 1), seed=7890, velocity="cells")
    outs = []
    for cc in (True, False):
        ctx = _mapped(p, precision, rtol=1e-10, coarse_cycle=cc)
        phi, info = ctx.nodal_project(T(p.ux), T(p.uy), T(p.uz), T(p.S))
        assert info["rel_resid"] <= 1e-10
        outs.append(N(phi))
        ctx.close()
    assert np.array_equal(outs[0], outs[1])


# nodes of a colour on the largest level of the coarse cycle: 1025 (one past a
# place per thread), 1377, 2125 (past two), and 595 on odd extents.  h = 1 / nz:
# 12 h^2, formed in another order inside the cycle, rounds alike on these nz
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,bc", [((16, 16, 80), (1, 1, 1)), ((32, 32, 32), (1, 1, 1)), ((16, 16, 168), (1, 1, 1)),
                                      ((24, 20, 32), (1, 0, 1))])
def test_nodal_coarse_cycle_forms(shape, bc, precision):
    nx, ny, nz = shape
    say("nodal coarse cycle forms", shape, bc, precision)
    p = W.planar_problem(nx=nx, ny=ny, nz=nz, contrast=1e3, bc=bc, seed=7950 + nz, velocity="cells")
    outs = []
    for cc in (True, False):
        ctx = _mapped(p, precision, rtol=1e-10, coarse_cycle=cc)
        ux = T(p.ux)
        phi, _ = ctx.nodal_project(ux, T(p.uy), T(p.uz), T(p.S))
        outs.append((N(phi), N(ux)))
        ctx.close()
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


# two-colour passes of any node grid: rows of 2, 3, 65 and 129 pairs (64 to a
# workgroup), one workgroup's planes and a remainder, every boundary
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,bc", [((4, 4, 4), (0, 0, 0)), ((4, 4, 4), (1, 1, 1)), ((128, 8, 20), (1, 0, 1)),
                                      ((256, 4, 8), (1, 1, 0)), ((20, 36, 132), (0, 1, 1)), ((64, 48, 36), (0, 0, 1)),
                                      ((130, 12, 12), (0, 0, 0)), ((32, 8, 10), (0, 0, 1)), ((256, 12, 10), (0, 0, 1)),
                                      ((160, 160, 160), (1, 1, 1))])
def test_two_colour_passes_of_any_grid_equal_four_colour_passes(shape, bc, precision):
    nx, ny, nz = shape
    say("nodal pair, any grid", shape, bc, precision)
    p = W.planar_problem(nx=nx, ny=ny, nz=nz, contrast=1e3, bc=bc, seed=7700 + nx + nz, velocity="cells")
    outs = []
    # an odd and an even number of sweeps per cycle (the iterate's two buffers);
    # "fused" keeps whole rows per wavefront where it can
    for nu2 in (1, 2):
        for sm in ("auto", "fused", "per_colour"):
            ctx = _mapped(p, precision, rtol=1e-9, smoother=sm, nu1=2, nu2=nu2, coarse_cycle=False)
            ux, uz = T(p.ux), T(p.uz)
            phi, info = ctx.nodal_project(ux, T(p.uy), uz, T(p.S))
            outs.append((N(phi), N(ux), N(uz), info["vcycles"]))
            ctx.close()
        b = outs[-1]
        for a in outs[-3:-1]:
            assert a[3] == b[3] and all(np.array_equal(u, v) for u, v in zip(a[:3], b[:3]))


# without pre-smoothing the first pass after the coarse correction is the first to
# write a level's second buffer: what an earlier call left there (not a number)
# must not reach the rows beside a wall in y
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nu2", [1, 2])
@pytest.mark.parametrize("bc", [(1, 1, 1), (0, 1, 0), (0, 1, 1)])
def test_two_colour_passes_beside_walls_after_a_failed_call(bc, nu2, precision):
    say("nodal pair, walls in y", bc, nu2, precision)
    p = W.planar_problem(nx=16, ny=12, nz=20, contrast=1e3, bc=bc, seed=7730, velocity="cells")
    kw = dict(rtol=1e-8, nu1=0, nu2=nu2, coarse_cycle=False)
    ctx = context_for(p, precision, **kw)
    # values of b / sigma that no double holds
    ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho * 1e300), p.dr, p.center, want_coefs=False)
    with pytest.raises(mproj.MprojError):
        ctx.nodal_project(*(T(u * 1e140) for u in (p.ux, p.uy, p.uz)), T(p.S))
    outs = []
    for c in (ctx, context_for(p, precision, smoother="per_colour", **kw)):
        c.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center, want_coefs=False)
        ux = T(p.ux)
        phi, info = c.nodal_project(ux, T(p.uy), T(p.uz), T(p.S))
        assert info["rel_resid"] <= 1e-8
        outs.append((N(phi), N(ux)))
        c.close()
    assert all(np.array_equal(a, b) for a, b in zip(*outs))


# spacings where 12 h h (inside the cycle) and 12 (h h) (one launch per operation)
# round differently.  One refinement step: about 640 operations in a row (4 cycles,
# 4 levels, 4 sweeps of 10) each carry a unit in the last place; the bottom solves
# agree to their tolerance times a condition number below 100
@pytest.mark.parametrize("precision,tol", [("fp64", 640 * 2.0 ** -53 + 1e-11), ("mixed", 640 * 2.0 ** -24)])
@pytest.mark.parametrize("shape,bc", [((24, 20, 28), (1, 0, 1)), ((12, 28, 56), (1, 1, 1)), ((32, 32, 112), (0, 0, 1))])
def test_nodal_coarse_cycle_on_other_spacings(shape, bc, precision, tol):
    nx, ny, nz = shape
    say("nodal coarse cycle, 12 h^2", shape, bc, precision)
    p = W.planar_problem(nx=nx, ny=ny, nz=nz, contrast=1e3, bc=bc, seed=7960 + nz, velocity="cells")
    outs = []
    for cc in (True, False):
        ctx = _mapped(p, precision, rtol=1e-10, max_outer=1, bottom_rtol=1e-13, coarse_cycle=cc)
        phi, info = ctx.nodal_project(T(p.ux), T(p.uy), T(p.uz), T(p.S), allow_not_converged=True)
        outs.append((N(phi), info["vcycles"]))
        ctx.close()
    assert outs[0][1] == outs[1][1]
    assert np.abs(outs[0][0] - outs[1][0]).max() <= tol * np.abs(outs[1][0]).max()
