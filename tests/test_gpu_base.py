"""Irregular radial base state on the GPU (Sec. 3.1): fill by radius index,
quadratic fill, and the lateral Average, against the oracle; projections on
stars mapped each way."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1908_03634_amd import mproj, workloads as W
from tests.gpu_util import N, T, context_for, gpu_project, rel, say

pytestmark = pytest.mark.gpu


def radii_over_h(nx, ny, nz):
    x = np.arange(nx) + 0.5 - nx / 2
    y = np.arange(ny) + 0.5 - ny / 2
    z = np.arange(nz) + 0.5 - nz / 2
    return np.sqrt(z[:, None, None] ** 2 + y[None, :, None] ** 2 + x[None, None, :] ** 2)


@pytest.mark.parametrize("base", ["irregular", "quadratic", "linear"])
@pytest.mark.parametrize("n", [16, 32])
def test_fill_modes_give_the_oracles_face_coefficients(base, n):
    say("fill", base, n)
    p = W.spherical_problem(n, contrast=1e5, seed=6100 + n, base=base)
    g = oracle.Grid.of(p)
    b0 = oracle.fill_beta0(g, p.geometry, p.beta0_1d, p.dr, p.center)
    ref = oracle.face_coefs(g, b0, p.rho)
    ctx = context_for(p, "fp64")
    got = ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center)
    for a, b in zip(got, ref):
        if base == "irregular":
            assert np.array_equal(N(a), b)  # a lookup: the same bits
        else:
            assert np.abs(N(a) - b).max() <= 1e-14 * np.abs(b).max()
    ctx.close()


def test_irregular_table_of_the_wrong_length_is_rejected():
    p = W.spherical_problem(16, base="irregular", seed=6200)
    ctx = context_for(p, "fp64")
    assert ctx.radius_count() == len(p.beta0_1d) == oracle.radius_count(16, 16, 16)
    with pytest.raises(mproj.MprojError) as e:
        ctx.map_base_state(p.geometry, T(p.beta0_1d[:-1]), T(p.rho), p.dr, p.center)
    assert e.value.code == 1
    ctx.close()


@pytest.mark.parametrize("shape", [(8, 8, 8), (12, 10, 6), (64, 64, 64), (96, 64, 32), (256, 256, 256)])
def test_average_matches_the_oracle(shape):
    nx, ny, nz = shape
    say("average", shape)
    phi = W.random_cells(nx, ny, nz, 6300 + nx)
    avg_ref, cnt_ref = oracle.average_irregular(phi)
    ctx = mproj.Context(nx, ny, nz, bc=(1, 1, 1), precision="fp64")
    assert ctx.radius_count() == len(avg_ref)
    avg, cnt = ctx.average(T(phi))
    avg, cnt = N(avg), N(cnt)
    assert np.array_equal(cnt, cnt_ref)
    assert np.abs(avg - avg_ref).max() <= 1e-13 * np.abs(avg_ref).max()
    # reproducible to the bit
    avg2, _ = ctx.average(T(phi), count=False)
    assert np.array_equal(N(avg2), avg)
    ctx.close()


def test_average_of_a_radial_function_and_the_paper_count():
    """256^3: 24,384 + 1 radii (Sec. 4.1); the average of f(r) is f(r_m)."""
    n = 256
    r = radii_over_h(n, n, n)
    f = np.exp(-r / 40.0)
    ctx = mproj.Context(n, n, n, bc=(1, 1, 1), precision="mixed")
    assert ctx.radius_count() - 1 == 24384
    avg, cnt = ctx.average(T(f))
    avg, cnt = N(avg), N(cnt)
    rm = np.sqrt(0.75 + 2 * np.arange(len(avg)))
    on = cnt > 0
    assert cnt.sum() == n**3
    assert np.allclose(avg[on], np.exp(-rm[on] / 40.0), rtol=1e-13, atol=0)
    assert np.all(avg[~on] == 0)
    ctx.close()


def test_average_needs_even_extents():
    lib = mproj.load_library()
    ctx = mproj.Context(9, 8, 8, bc=(1, 1, 1), precision="fp64")
    assert ctx.radius_count() == 0
    with pytest.raises(mproj.MprojError) as e:
        ctx.average(torch.zeros((8, 8, 9), dtype=torch.float64, device="cuda:0"))
    assert e.value.code == 1
    assert lib.mp_average(ctx._h, None, None, None) == 1
    ctx.close()


@pytest.mark.parametrize("base", ["irregular", "quadratic"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_star_projection_with_each_base_state(base, precision):
    say("star projection", base, precision)
    p = W.spherical_problem(64, contrast=1e5, seed=6400, base=base)
    ref = oracle.mac_project(p, tol=1e-12)
    r = gpu_project(p, precision, rtol=1e-12)
    assert rel(N(r["phi"]), ref["phi"]) < 1e-9
    assert r["info"]["div_defect"] <= 2e-12
    g = ref["grid"]
    assert oracle.residual_norm(g, ref["cx"], ref["cy"], ref["cz"], ref["rhs"], N(r["phi"])) <= 1.01e-12
    r["ctx"].close()


def _split_case(p, precision):
    ref = oracle.mac_project(p, tol=1e-12, split=True)
    ctx = context_for(p, precision, rtol=1e-12)
    ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center, want_coefs=False)
    ux, uy, uz, S = T(p.ux), T(p.uy), T(p.uz), T(p.S)
    sbar = torch.zeros(len(ref["sbar"]), dtype=torch.float64, device="cuda:0")
    phi, info = ctx.mac_project(ux, uy, uz, S, split=True, sbar=sbar)
    phi = N(phi)
    g = ref["grid"]
    assert np.abs(N(sbar) - ref["sbar"]).max() <= 1e-13 * np.abs(ref["sbar"]).max()
    assert rel(phi, ref["phi"]) < 1e-9
    assert oracle.residual_norm(g, ref["cx"], ref["cy"], ref["cz"], ref["rhs"], phi) <= 1.01e-12
    # the split source has a zero sum on every plane / radius: nothing to de-mean
    # (a uniform table filled back by interpolation leaves a small mean, removed)
    if p.geometry in (0, 2):
        assert abs(info["rhs_mean"]) <= 1e-13 * info["rhs_norm"] / np.sqrt(p.ncell)
    else:
        assert info["rhs_mean"] == pytest.approx(ref["mean"], rel=1e-9, abs=1e-13 * info["rhs_norm"])
    assert info["div_defect"] <= 2e-12
    vx, vy, vz = oracle.velocity_correct(g, ref["cx"], ref["cy"], ref["cz"], ref["beta0_cc"], phi, p.ux, p.uy, p.uz)
    for a, b in ((ux, vx), (uy, vy), (uz, vz)):
        assert np.abs(N(a) - b).max() <= 1e-12 * np.abs(b).max()
    ctx.close()


@pytest.mark.parametrize("bc", [(0, 0, 1), (1, 1, 1), (0, 0, 0)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_split_projection_planar_matches_oracle(bc, precision):
    say("split planar", bc, precision)
    _split_case(W.planar_problem(nx=48, ny=32, nz=40, contrast=1e4, bc=bc, seed=6500), precision)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_split_projection_irregular_star_matches_oracle(precision):
    say("split star", precision)
    _split_case(W.spherical_problem(64, contrast=1e5, seed=6600, base="irregular"), precision)


def test_split_projection_full_size_planar():
    say("split c2 256^3")
    _split_case(W.config_problem("c2", seed_offset=300), "mixed")


def test_uniform_split_needs_the_star_on_the_middle_node():
    """The radius averages assume the star centre on the middle node of the
    box: a uniform spherical mapping about another point has no split source."""
    p = W.spherical_problem(16, seed=6700)
    ctx = context_for(p, "fp64")
    off = (0.5 + p.h / 3, 0.5, 0.5)
    ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, off, want_coefs=False)
    with pytest.raises(mproj.MprojError) as e:
        ctx.mac_project(T(p.ux), T(p.uy), T(p.uz), T(p.S), split=True)
    assert e.value.code == 7
    ctx.close()


def test_radius_list_allocation_failure_leaves_the_context_usable(monkeypatch):
    """When the radius list cannot be allocated, a split projection after an
    irregular mapping fails with MP_ERR_NOMEM and frees only the list: the
    context's lateral-average buffer stays owned and valid, so the next split
    projection writes into it (not into memory the failure released, which a
    caller's tensor may now occupy), gives the same bits as a fresh context,
    and mp_free releases every buffer once."""
    p = W.spherical_problem(32, contrast=1e5, seed=6800, base="irregular")
    ctx = context_for(p, "fp64", rtol=1e-12)
    ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center, want_coefs=False)
    monkeypatch.setenv("MP_TEST_FAIL_ALLOC", "radius_list")
    with pytest.raises(mproj.MprojError) as e:
        ctx.mac_project(T(p.ux), T(p.uy), T(p.uz), T(p.S), split=True)
    assert e.value.code == 3
    monkeypatch.delenv("MP_TEST_FAIL_ALLOC")
    nm = ctx.radius_count()
    guards = [torch.full((nm,), 7.0, dtype=torch.float64, device="cuda:0") for _ in range(8)]
    ux, uy, uz = T(p.ux), T(p.uy), T(p.uz)
    phi, _ = ctx.mac_project(ux, uy, uz, T(p.S), split=True)
    torch.cuda.synchronize()
    for gd in guards:
        assert bool((gd == 7.0).all())
    fresh = context_for(p, "fp64", rtol=1e-12)
    fresh.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center, want_coefs=False)
    vx, vy, vz = T(p.ux), T(p.uy), T(p.uz)
    phi2, _ = fresh.mac_project(vx, vy, vz, T(p.S), split=True)
    assert np.array_equal(N(phi), N(phi2))
    assert np.array_equal(N(uz), N(vz))
    fresh.close()
    ctx.close()


@pytest.mark.parametrize("shape", [(8, 8, 8), (24, 4, 4), (12, 8, 20), (64, 48, 32), (256, 256, 256)])
def test_uniform_average_matches_the_oracle(shape):
    """Radius averages interpolated onto r_j = (j + 1/2) dr (the three reached
    radii around the nearest; boxes whose corner regions leave radii
    unreached), against the oracle; reproducible to the bit."""
    nx, ny, nz = shape
    say("uniform average", shape)
    h = 1.0 / max(shape)
    dr = h / 5
    n1d = int(np.ceil(np.sqrt(3.0) * max(shape) * h / dr)) + 4
    phi = W.random_cells(nx, ny, nz, 6900 + nx + nz)
    ref = oracle.average_uniform(phi, h, n1d, dr)
    ctx = mproj.Context(nx, ny, nz, h=h, bc=(1, 1, 1), precision="fp64")
    got = N(ctx.average_uniform(T(phi), n1d, dr))
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
    assert np.array_equal(N(ctx.average_uniform(T(phi), n1d, dr)), got)
    # a radial quadratic is reproduced between the first and last reached radius
    r = radii_over_h(nx, ny, nz) * h
    q = N(ctx.average_uniform(T(1.0 + r - 2.0 * r * r), n1d, dr))
    rj = (np.arange(n1d) + 0.5) * dr
    inside = (rj >= h * np.sqrt(0.75)) & (rj <= r.max())
    assert np.allclose(q[inside], 1.0 + rj[inside] - 2.0 * rj[inside] ** 2, rtol=1e-12, atol=0)
    ctx.close()


def test_average_on_non_cubic_boxes_and_bitwise_reproducible():
    """Octant folding on boxes of three different even extents: counts exact,
    averages to rounding, the same bits on every call."""
    for shape in ((6, 10, 14), (128, 64, 32), (2, 2, 2), (2, 4, 2)):
        nx, ny, nz = shape
        phi = W.random_cells(nx, ny, nz, 7000 + nx)
        avg_ref, cnt_ref = oracle.average_irregular(phi)
        ctx = mproj.Context(nx, ny, nz, bc=(1, 1, 1), precision="fp64")
        a1, c1 = ctx.average(T(phi))
        a2, c2 = ctx.average(T(phi))
        assert np.array_equal(N(c1), cnt_ref) and np.array_equal(N(c2), cnt_ref)
        assert np.array_equal(N(a1), N(a2))
        assert np.abs(N(a1) - avg_ref).max() <= 1e-13 * np.abs(avg_ref).max()
        ctx.close()


@pytest.mark.parametrize("base", ["linear", "quadratic"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_split_projection_uniform_star_matches_oracle(base, precision):
    say("split uniform star", base, precision)
    _split_case(W.spherical_problem(64, contrast=1e5, seed=7100, base=base), precision)


def _w0_edges(p):
    """Centres and edges of the base state of a workload problem."""
    if p.geometry == 0:
        return (np.arange(p.nz) + 0.5) * p.h, np.arange(p.nz + 1) * p.h
    if p.geometry == 2:
        return oracle.irregular_radii(len(p.beta0_1d), p.h)
    n1d = len(p.beta0_1d)
    return (np.arange(n1d) + 0.5) * p.dr, np.arange(n1d + 1) * p.dr


@pytest.mark.parametrize("kind", ["planar", "linear", "quadratic", "irregular"])
def test_add_w0_matches_the_oracle(kind):
    """U~ + w0 e_r on every face: planar (interior z faces), uniform and
    irregular spherical edges; walls unchanged."""
    if kind == "planar":
        p = W.planar_problem(nx=40, ny=24, nz=32, contrast=1e4, seed=7200)
    else:
        p = W.spherical_problem(48, contrast=1e5, seed=7201, base=kind)
    rc, re = _w0_edges(p)
    rng = np.random.default_rng(7202)
    w0 = rng.standard_normal(len(re))
    g = oracle.Grid.of(p)
    center = p.center if p.geometry != 0 else None
    ref = oracle.add_w0(g, 0 if p.geometry == 0 else 1, w0, re, center, p.ux, p.uy, p.uz)
    ctx = context_for(p, "fp64")
    ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center, want_coefs=False)
    ux, uy, uz = T(p.ux), T(p.uy), T(p.uz)
    ctx.add_w0(T(w0), ux, uy, uz, re=T(re) if p.geometry != 0 else None)
    for a, b in zip((ux, uy, uz), ref):
        assert np.abs(N(a) - b).max() <= 1e-14 * np.abs(b).max()
    ctx.close()


def test_add_w0_errors():
    p = W.planar_problem(nx=8, ny=8, nz=8, contrast=1e2, bc=(0, 0, 0), seed=7300)
    ctx = context_for(p, "fp64")
    w = torch.zeros(9, dtype=torch.float64, device="cuda:0")
    with pytest.raises(mproj.MprojError) as e:  # no mapping yet
        ctx.add_w0(w, T(p.ux), T(p.uy), T(p.uz))
    assert e.value.code == 7
    ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center, want_coefs=False)
    with pytest.raises(mproj.MprojError) as e:  # periodic z: no walls for the planar w0
        ctx.add_w0(w, T(p.ux), T(p.uy), T(p.uz))
    assert e.value.code == 7
    ctx.close()


@pytest.mark.parametrize("kind", ["planar", "linear", "irregular"])
def test_full_split_velocity_matches_the_oracle_chain(kind):
    """Appendix A on the GPU: the split projection (U~, Sbar), w0 from Sbar on
    the base state (mp_w0), U = U~ + w0 e_r (mp_add_w0), against the oracle's
    chain fed with the GPU's phi; planar: D(beta0 U) = beta0 (S - psi) with
    psi closing the top wall."""
    say("full split velocity", kind)
    if kind == "planar":
        p = W.planar_problem(nx=48, ny=32, nz=40, contrast=1e4, seed=7400)
    else:
        p = W.spherical_problem(64, contrast=1e5, seed=7401, base=kind)
    ref = oracle.mac_project(p, tol=1e-12, split=True)
    g = ref["grid"]
    rc, re = _w0_edges(p)
    sbar_o = ref["sbar"]
    b1 = p.beta0_1d
    psi = np.full(len(b1), float((b1 * sbar_o).sum() / b1.sum())) if kind == "planar" else np.zeros(len(b1))
    ctx = context_for(p, "fp64", rtol=1e-12)
    ctx.map_base_state(p.geometry, T(b1), T(p.rho), p.dr, p.center, want_coefs=False)
    ux, uy, uz, S = T(p.ux), T(p.uy), T(p.uz), T(p.S)
    sbar = torch.zeros(len(sbar_o), dtype=torch.float64, device="cuda:0")
    phi, _ = ctx.mac_project(ux, uy, uz, S, split=True, sbar=sbar)
    geo = 0 if p.geometry == 0 else 1
    w0 = ctx.w0(geo, T(rc), T(re), T(b1), sbar, T(psi))
    ctx.add_w0(w0, ux, uy, uz, re=T(re) if geo else None)
    torch.cuda.synchronize()
    w0_o = oracle.w0(geo, rc, re, b1, N(sbar), psi)
    assert np.abs(N(w0) - w0_o).max() <= 1e-12 * max(np.abs(w0_o).max(), 1e-300)
    vx, vy, vz = oracle.velocity_correct(g, ref["cx"], ref["cy"], ref["cz"], ref["beta0_cc"], N(phi), p.ux, p.uy,
                                         p.uz)
    vx, vy, vz = oracle.add_w0(g, geo, w0_o, re, p.center if geo else None, vx, vy, vz)
    for a, b in ((ux, vx), (uy, vy), (uz, vz)):
        assert np.abs(N(a) - b).max() <= 1e-12 * np.abs(b).max()
    if kind == "planar":
        d = oracle.beta0_divergence(g, ref["beta0_cc"], N(ux), N(uy), N(uz))
        want = ref["beta0_cc"] * (p.S - psi[:, None, None])
        scale = np.abs(oracle.beta0_divergence(g, ref["beta0_cc"], p.ux, p.uy, p.uz)).max()
        assert np.abs(d - want).max() <= 1e-10 * scale
    ctx.close()


# the edge search starts from a guess (edges equal in r or in r^2): edges far from
# both, a single edge, two edges, and edges that cover a part of the radii only
@pytest.mark.parametrize("edges", ["geometric", "cubic", "random", "one", "two", "inner", "outer"])
def test_add_w0_on_uneven_edges(edges):
    say("add_w0", edges)
    p = W.spherical_problem(32, contrast=1e3, seed=7210, base="linear")
    rng = np.random.default_rng(7211)
    top = p.h * 32
    re = {"geometric": top * 1.05 ** np.arange(-300.0, 1.0), "cubic": top * (np.arange(200) / 199.0) ** 3,
          "random": np.sort(rng.uniform(0.0, top, 777)), "one": np.array([0.3 * top]),
          "two": np.array([0.1, 0.4]) * top, "inner": np.linspace(0.0, 0.2, 50) * top,
          "outer": np.linspace(0.3, 0.35, 64) * top}[edges]
    w0 = rng.standard_normal(len(re))
    ref = oracle.add_w0(oracle.Grid.of(p), 1, w0, re, p.center, p.ux, p.uy, p.uz)
    ctx = context_for(p, "fp64")
    ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center, want_coefs=False)
    u = [T(p.ux), T(p.uy), T(p.uz)]
    ctx.add_w0(T(w0), *u, re=T(re))
    # a radius rounds within 2^-52 r, and w0's slope is at most the largest difference
    # over its interval
    slope = np.abs(np.diff(w0) / np.diff(re)).max() if len(re) > 1 else 0.0
    tol = 1e-14 * max(np.abs(b).max() for b in ref) + 2.0 * slope * top * 2.0 ** -52
    for a, b in zip(u, ref):
        assert np.abs(N(a) - b).max() <= tol
    ctx.close()


# edges that the guess meets at each eighth of the table and misses by hundreds of
# places between them, on both sides (the search steps outwards from the guess),
# and the same spacing without that agreement (halving alone)
@pytest.mark.parametrize("shift", [0.0, 0.04])
def test_add_w0_on_edges_that_wander_from_the_guess(shift):
    say("add_w0 wander", shift)
    p = W.spherical_problem(32, contrast=1e3, seed=7220, base="linear")
    top = p.h * 32
    x = np.arange(20001) / 20000.0
    re = top * (x + 0.015 * (np.sin(16.0 * np.pi * (x + shift)) - np.sin(16.0 * np.pi * shift)))
    assert (np.diff(re) > 0.0).all()
    w0 = np.random.default_rng(7221).standard_normal(len(re))
    ref = oracle.add_w0(oracle.Grid.of(p), 1, w0, re, p.center, p.ux, p.uy, p.uz)
    ctx = context_for(p, "fp64")
    ctx.map_base_state(p.geometry, T(p.beta0_1d), T(p.rho), p.dr, p.center, want_coefs=False)
    u = [T(p.ux), T(p.uy), T(p.uz)]
    ctx.add_w0(T(w0), *u, re=T(re))
    slope = np.abs(np.diff(w0) / np.diff(re)).max()
    tol = 1e-14 * max(np.abs(b).max() for b in ref) + 2.0 * slope * top * 2.0 ** -52
    for a, b in zip(u, ref):
        assert np.abs(N(a) - b).max() <= tol
    ctx.close()
