"""Timing cases: the projections that a user of the library runs, by size.

A low Mach number time step calls the library through its public entry points:
the MAC projection (Sec. 3.2 Steps 3 and 7 of the method), its velocity-split
form with the one-dimensional base state of a star, the nodal projection (Step
11), and, for a differentiable program, a solve with its gradients.  The listed
cases cover those calls from 32^3 to 512^3, in both precisions, on planar
atmospheres and stars, with sizes that the blocked kernels were shaped for
(rows of 128 to 512 cells) and with sizes that they were not.

Sizes 32^3 (c1), 256^3 (c2), 384^3 (c3), 128^3 (c4) and 512^3 (c5) are the
workloads of `paper_1908_03634_amd/workloads.py`; the others are generic.
Inputs follow the same recipe (stratified density with a 1e-3 perturbation,
N(0,1) velocities, S of N(0, (1e-2)^2)), drawn on the device from a seed.

`exact` gives the same results from plain torch in 64 bits: the discrete
operators written out with slices, and the systems solved by conjugate
gradients, preconditioned by the constant-coefficient operator in its
eigenvectors, to the limit of 64-bit rounding.
"""
import math

import torch

GAMMA = 5.0 / 3.0
DEV = "cuda"
F64 = torch.float64
RTOL = 1e-10  # the library's default, and the tolerance of its benchmark


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _case(name, path, nx, ny, nz, bc, base, contrast, precision):
    return {"name": name, "path": path, "nx": nx, "ny": ny, "nz": nz, "bc": bc, "base": base,
            "contrast": contrast, "precision": precision}


def listed():
    return [
        # the smallest box of the workloads (c1): unit tests, parameter scans, a
        # coarse atmosphere; bound by launches and by the coarse levels
        _case("mac-32-fp64", "mac", 32, 32, 32, "PPN", "planar", 1e2, "fp64"),
        # an atmosphere taller than it is wide, rows of 160 cells: an ordinary
        # resolution of a bubble-in-an-atmosphere run
        _case("mac-160x160x320-mixed", "mac", 160, 160, 320, "PPN", "planar", 1e4, "mixed"),
        # a closed box of ragged extents, which halve only three times, so that
        # the coarsest grid is large
        _case("mac-200x120x88-mixed", "mac", 200, 120, 88, "NNN", "planar", 1e3, "mixed"),
        # the benchmark workload (c2) in both precisions
        _case("mac-256-mixed", "mac", 256, 256, 256, "PPN", "planar", 1e4, "mixed"),
        _case("mac-256-fp64", "mac", 256, 256, 256, "PPN", "planar", 1e4, "fp64"),
        # a full star on a uniform radial table (c3)
        _case("mac-star-384-mixed", "mac", 384, 384, 384, "NNN", "star", 1e5, "mixed"),
        # the largest workload (c5): a production atmosphere, bound by HBM
        _case("mac-512-mixed", "mac", 512, 512, 512, "PPN", "planar", 1e5, "mixed"),
        # a solve and its gradients in a differentiable program (c4), and the
        # same at the benchmark's size; the coefficients change every step
        _case("grad-128-fp64", "grad", 128, 128, 128, "PPN", "planar", 1e3, "fp64"),
        _case("grad-256-mixed", "grad", 256, 256, 256, "PPN", "planar", 1e4, "mixed"),
        # the projection that ends a time step (cell-centred velocity, nodal
        # scalar), on the benchmark's box and on a closed box of other extents
        _case("nodal-256-mixed", "nodal", 256, 256, 256, "PPN", "planar", 1e4, "mixed"),
        _case("nodal-96x80x112-fp64", "nodal", 96, 80, 112, "NNN", "planar", 1e3, "fp64"),
        # the whole velocity split of a star on the irregular radial base state:
        # radii, hydrostatic pressure, beta0, lateral average, projection, w0
        _case("split-star-192-mixed", "split", 192, 192, 192, "NNN", "irregular", 1e2, "mixed"),
    ]


def _bottom(n):
    """Cells of the coarsest grid: extents halve while all are even and >= 4."""
    n = list(n)
    while all(a % 2 == 0 and a >= 4 for a in n) and n[0] * n[1] * n[2] > 64:
        n = [a // 2 for a in n]
    return n[0] * n[1] * n[2]


# time of a cell against a cell of a mixed-precision MAC projection, roughly
_COST = {"mac": 1.0, "grad": 2.6, "nodal": 2.2, "split": 1.5}


def draw(rng):
    """One more case of the same ranges: paths and precisions as a program mixes
    them, extents over their logarithm from 16 to 640 (each a multiple of a power
    of two, as a user of a multigrid code chooses them), closed, open and mixed
    boxes; now and then a small box of odd extents."""
    path = rng.choice(["mac", "mac", "mac", "mac", "grad", "nodal", "nodal", "split"])
    precision = rng.choice(["mixed", "mixed", "fp64"])
    base, bc = "planar", rng.choice(["PPN", "PPN", "NNN", "PPP", "NPN"])
    if path == "split":
        base, bc = "irregular", "NNN"
    elif path != "grad" and rng.random() < 0.25:
        base, bc = "star", "NNN"
    contrast = 10.0 ** rng.uniform(1.0, 2.5) if base == "irregular" else 10.0 ** rng.uniform(2.0, 5.0)
    odd = path != "split" and base == "planar" and rng.random() < 0.1
    most = (1 << 26) / (_COST[path] * (3.0 if precision == "fp64" else 1.0))
    while True:
        if odd:
            n = [2 * rng.randrange(4, 13) + 1 for _ in range(3)]
        else:
            unit = rng.choice([8, 8, 16, 16, 32])
            mid = math.exp(rng.uniform(math.log(20.0), math.log(400.0)))
            n = [unit * max(1, round(mid * math.exp(rng.uniform(-0.45, 0.45)) / unit)) for _ in range(3)]
            if base in ("star", "irregular"):
                n = [n[0]] * 3
            elif path == "grad" and rng.random() < 0.5:
                n = [n[0]] * 3
        cells = n[0] * n[1] * n[2]
        if cells <= most and max(n) <= 640 and min(n) >= 8 and (odd or _bottom(n) <= 4200):
            break
    return {"path": path, "nx": n[0], "ny": n[1], "nz": n[2], "bc": bc, "base": base,
            "contrast": float("%.4g" % contrast), "precision": precision}


def work(case):
    """Each input read once and each output written once (64-bit values), and
    the additions and multiplications of one residual: no solver needs less."""
    n = case["nx"] * case["ny"] * case["nz"]
    # density, three velocities and S in; three velocities and phi out
    words = 9.0
    if case["path"] == "grad":
        # right-hand side, three coefficients and the seed in; phi and four gradients out
        words = 10.0
    return {"bytes": words * 8.0 * n, "flops": (60.0 if case["path"] == "nodal" else 20.0) * n}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _grid(case):
    n = (case["nz"], case["ny"], case["nx"])
    per = tuple(b == "P" for b in reversed(case["bc"]))  # z, y, x
    return n, per, 1.0 / case["nz"]


def _face_shape(n, per, a):
    s = list(n)
    s[a] += 0 if per[a] else 1
    return tuple(s)


def _zero_walls(f, per, a):
    if not per[a]:
        f.select(a, 0).zero_()
        f.select(a, f.shape[a] - 1).zero_()
    return f


def _radius2(n, h, dev):
    """Squared distance of the cell centres from the middle of the box."""
    c = [((torch.arange(m, dtype=F64, device=dev) + 0.5) - 0.5 * m) * h for m in n]
    return c[0][:, None, None] ** 2 + c[1][None, :, None] ** 2 + c[2][None, None, :] ** 2


def _star_radius(contrast):
    return 0.5 / math.sqrt(contrast ** 0.4 - 1.0)


def _hydrostatic_steps(rc, rho0, g_edge, rho_cutoff):
    """Fall of the pressure across each pair of centres, 0 from the cutoff on."""
    step = (rc[1:] - rc[:-1]) * g_edge[1:-1] * 0.5 * (rho0[:-1] + rho0[1:])
    return torch.where(torch.cumsum((rho0 <= rho_cutoff).long(), 0)[:-1] > 0, 0.0, step)


def _inputs(case, seed):
    """The arrays of one projection or solve, from the seed alone."""
    n, per, h = _grid(case)
    dev = torch.device(DEV)
    gen = torch.Generator(device=dev)
    gen.manual_seed(1908 * 1000003 + int(seed))

    def normal(shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=F64)

    d = {}
    noise = normal(n).mul_(1e-3).add_(1.0)
    if case["base"] == "planar":
        z = (torch.arange(n[0], dtype=F64, device=dev) + 0.5) * h
        rho0 = torch.exp(-z * math.log(case["contrast"]))
        d["beta0_1d"] = rho0 ** (1.0 / GAMMA)
        d["rho"] = noise.mul_(rho0[:, None, None])
    else:
        R = _star_radius(case["contrast"])
        d["rho"] = noise.mul_((1.0 + _radius2(n, h, dev) / (R * R)) ** -2.5)
        if case["base"] == "star":
            # uniform table of spacing h/5 out to the corner of the box
            r = (torch.arange(int(math.ceil(5.0 * math.sqrt(3.0) * max(n) / 2.0)) + 2, dtype=F64, device=dev) + 0.5) * (h / 5)
            d["beta0_1d"] = (1.0 + (r / R) ** 2) ** (-2.5 / GAMMA)
        else:
            # the base state at the irregular radii: a polytrope of index 5, its
            # gravity on the edges, in units in which 4 pi G / 3 = 1; the central
            # pressure is the one that hydrostatic balance gives from the
            # pressure at the cutoff density inward
            rc, re = _radii(n, h, dev)
            d["rho0"] = (1.0 + (rc / R) ** 2) ** -2.5
            d["g_edge"] = re * (1.0 + (re / R) ** 2) ** -1.5
            d["gamma1"] = GAMMA * (1.0 - 0.05 * (rc / 0.9) ** 2)
            d["rho_cutoff"] = float((1.0 + (0.45 / R) ** 2) ** -2.5)
            step = _hydrostatic_steps(rc, d["rho0"], d["g_edge"], d["rho_cutoff"])
            d["p0_base"] = float(step.sum()) + R * R / 6.0 * (1.0 + (0.45 / R) ** 2) ** -3
    if case["path"] == "nodal":
        d["u"] = [normal(n) for _ in range(3)]  # x, y, z
    else:
        d["u"] = [_zero_walls(normal(_face_shape(n, per, a)), per, a) for a in (2, 1, 0)]
    d["S"] = normal(n).mul_(1e-2)
    if case["path"] == "grad":
        d["w"] = normal(n)
    return d


def _coefs(case, d):
    """Face coefficients and right-hand side of a differentiable solve: the
    system of the projection of these inputs."""
    n, per, h = _grid(case)
    beta0 = _fill(case, d["beta0_1d"])
    c = beta0 / d["rho"]
    cs = [_harmonic(c, per, a) for a in (2, 1, 0)]
    return cs, _rhs(beta0, d["u"], d["S"], per, h)


def prepare(case, seed):
    """What the program holds before the call: a context of its grid, the
    inputs, and the arrays that take the results."""
    from paper_1908_03634_amd import mproj

    n, per, h = _grid(case)
    d = _inputs(case, seed)
    ctx = mproj.Context(case["nx"], case["ny"], case["nz"], h=h, bc=tuple(0 if p else 1 for p in reversed(per)),
                        precision=case["precision"], rtol=RTOL)
    st = {"path": case["path"], "ctx": ctx, "d": d, "h": h,
          "geometry": {"planar": mproj.PLANAR, "star": mproj.SPHERICAL, "irregular": mproj.SPHERICAL_IRREGULAR}[case["base"]],
          "center": tuple(0.5 * m * h for m in reversed(n))}
    if case["path"] == "grad":
        st["cs"], st["rhs"] = _coefs(case, d)
        st["d"] = {"w": d["w"]}
        return st
    st["u"] = [torch.empty_like(u) for u in d["u"]]
    st["phi"] = ctx.empty_nodes() if case["path"] == "nodal" else ctx.empty_cells()
    if case["path"] == "split":
        st["sbar"] = torch.empty(ctx.radius_count(), dtype=F64, device=ctx.device)
    return st


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(st):
    ctx, d = st["ctx"], st["d"]
    if st["path"] == "grad":
        from paper_1908_03634_amd.autograd import mac_solve

        # new values of the coefficients in every step, as an optimiser writes them
        leaves = [t.clone().requires_grad_(True) for t in (st["rhs"], *st["cs"])]
        phi = mac_solve(ctx, *leaves)
        loss = (phi * d["w"]).sum()
        grads = torch.autograd.grad(loss, leaves)
        return {"phi": phi.detach(), "rhs": grads[0], "cx": grads[1], "cy": grads[2], "cz": grads[3]}
    # the velocity that the step's advection leaves, projected in place
    u = st["u"]
    for to, frm in zip(u, d["u"]):
        to.copy_(frm)
    if st["path"] == "split":
        rc, re = ctx.base_radii()
        p0, _ = ctx.enforce_hse(rc, d["rho0"], d["g_edge"], d["p0_base"], d["rho_cutoff"])
        beta0 = ctx.beta0_from_p0(1.0, p0, d["gamma1"])
        ctx.map_base_state(st["geometry"], beta0, d["rho"], want_coefs=False)
        phi, _ = ctx.mac_project(*u, d["S"], phi=st["phi"], split=True, sbar=st["sbar"])
        w0 = ctx.w0(st["geometry"], rc, re, beta0, st["sbar"])
        ctx.add_w0(w0, *u, re=re)
        return {"phi": phi, "u": u, "p0": p0, "beta0": beta0, "sbar": st["sbar"], "w0": w0}
    ctx.map_base_state(st["geometry"], d["beta0_1d"], d["rho"], dr=st["h"] / 5, center=st["center"], want_coefs=False)
    project = ctx.nodal_project if st["path"] == "nodal" else ctx.mac_project
    phi, _ = project(*u, d["S"], phi=st["phi"])
    return {"phi": phi, "u": u}


# --------------------------------------------------------------------------
# the same in plain torch, 64 bits
# --------------------------------------------------------------------------
def _sides(c, per, a):
    """Values on the low and high side of every face along axis a (at a wall,
    the cell inside on both)."""
    if per[a]:
        return torch.roll(c, 1, a), c
    m = c.shape[a]
    return torch.cat([c.narrow(a, 0, 1), c], a), torch.cat([c, c.narrow(a, m - 1, 1)], a)


def _harmonic(c, per, a):
    lo, hi = _sides(c, per, a)
    return _zero_walls(2.0 * lo * hi / (lo + hi), per, a)


def _div1(f, per, a):
    if per[a]:
        return torch.roll(f, -1, a) - f
    m = f.shape[a] - 1
    return f.narrow(a, 1, m) - f.narrow(a, 0, m)


def _grad1(p, per, a, h):
    lo, hi = _sides(p, per, a)
    return (hi - lo) / h


def _apply(p, cs, per, h):
    """div(c grad p); cs in the order x, y, z."""
    out = torch.zeros_like(p)
    for c, a in zip(cs, (2, 1, 0)):
        out += _div1(c * _grad1(p, per, a, h), per, a)
    return out / h


def _face_mean(b, per, a):
    lo, hi = _sides(b, per, a)
    return 0.5 * (lo + hi)


def _rhs(beta0, u, S, per, h):
    out = torch.zeros_like(beta0)
    for f, a in zip(u, (2, 1, 0)):
        out += _div1(_zero_walls(_face_mean(beta0, per, a) * f, per, a), per, a)
    return out / h - beta0 * S


def _radius_index(n, dev):
    q = [(2 * torch.arange(m, device=dev) + 1 - m) ** 2 for m in n]
    return (q[0][:, None, None] + q[1][None, :, None] + q[2][None, None, :] - 3) // 8


def _radii(n, h, dev):
    m = torch.arange((sum((k - 1) ** 2 for k in n) - 3) // 8 + 1, dtype=F64, device=dev)
    re = h * torch.sqrt((2.0 * torch.arange(len(m) + 1, dtype=F64, device=dev) - 0.25).clamp_min(0.0))
    return h * torch.sqrt(0.75 + 2.0 * m), re


def _fill(case, table):
    """beta0 on the cells."""
    n, per, h = _grid(case)
    if case["base"] == "planar":
        return table[:, None, None].expand(n).contiguous()
    if case["base"] == "irregular":
        return table[_radius_index(n, table.device)]
    t = torch.sqrt(_radius2(n, h, table.device)) / (h / 5) - 0.5
    j = t.floor().clamp(0, len(table) - 2)
    w = (t - j).clamp(0.0, 1.0)
    j = j.long()
    return table[j] * (1.0 - w) + table[j + 1] * w


def _modes(m, per, fem):
    """Eigenvectors (columns) and eigenvalues of the one-dimensional second
    difference of m points; fem: linear elements (stiffness against mass)."""
    dev = torch.device(DEV)
    K = torch.zeros(m, m, dtype=F64, device=dev)
    M = torch.zeros_like(K)
    i = torch.arange(m, device=dev)
    pairs = [(i, (i + 1) % m)] if per else [(i[:-1], i[1:])]
    for p, q in pairs:
        for x, y, k, w in ((p, p, 1.0, 1 / 3), (q, q, 1.0, 1 / 3), (p, q, -1.0, 1 / 6), (q, p, -1.0, 1 / 6)):
            K.index_put_((x, y), torch.full((len(x),), k, dtype=F64, device=dev), accumulate=True)
            M.index_put_((x, y), torch.full((len(x),), w, dtype=F64, device=dev), accumulate=True)
    if not fem:
        lam, V = torch.linalg.eigh(K.cpu())
        return V.to(dev), lam.to(dev).clamp_min(0.0)
    L = torch.linalg.cholesky(M.cpu())
    Li = torch.linalg.inv(L)
    lam, Q = torch.linalg.eigh(Li @ K.cpu() @ Li.T)
    return (Li.T @ Q).to(dev), lam.to(dev).clamp_min(0.0)


def _along(A, x, a):
    """A applied along axis a of x."""
    if a == 2:
        return x @ A.T.contiguous()
    if a == 0:
        return (A @ x.reshape(x.shape[0], -1)).reshape(A.shape[0], *x.shape[1:])
    return torch.matmul(A, x)


def _solver(n, per, scale, fem):
    """Approximate inverse: the constant-coefficient operator (sum of second
    differences), scaled on both sides by 1/sqrt(scale)."""
    modes = [_modes(m, p, fem) for m, p in zip(n, per)]
    lam = modes[0][1][:, None, None] + modes[1][1][None, :, None] + modes[2][1][None, None, :]
    flat = lam.reshape(-1)
    lam = torch.where(lam < 1e-9 * flat.max(), torch.sort(flat.cpu())[0][1].item() if len(flat) < 4096 else
                      min(m[1][1].item() for m in modes if len(m[1]) > 1), lam)
    s = scale.rsqrt()

    def solve(r):
        x = r * s
        for a in range(3):
            x = _along(modes[a][0].T.contiguous(), x, a)
        x = x / lam
        for a in range(3):
            x = _along(modes[a][0], x, a)
        return x * s

    return solve


def _cg(op, pre, b, steps=300):
    """Mean-zero x with op(x) = b (b mean-zero, op positive semi-definite)."""
    b = b - b.mean()
    nb = float(b.norm())
    x = torch.zeros_like(b)
    if nb == 0.0:
        return x
    # two rounds: the second on the true residual of the first
    for _ in range(2):
        r = b - op(x) if x.any() else b.clone()
        r -= r.mean()
        start = float(r.norm())
        z = pre(r)
        p = z.clone()
        rz = float((r * z).sum())
        e = torch.zeros_like(b)
        for _k in range(steps):
            q = op(p)
            al = rz / float((p * q).sum())
            e += al * p
            r -= al * q
            if float(r.norm()) <= 1e-12 * start or float(r.norm()) <= 3e-17 * nb:
                break
            z = pre(r)
            new = float((r * z).sum())
            p = z + (new / rz) * p
            rz = new
        x += e
    return x - x.mean()


def _mac_exact(beta0, rho, u, S, per, h):
    c = beta0 / rho
    cs = [_harmonic(c, per, a) for a in (2, 1, 0)]
    b = _rhs(beta0, u, S, per, h)
    phi = _cg(lambda p: -_apply(p, cs, per, h) * h * h, _solver(c.shape, per, c, False), -(b - b.mean()) * h * h)
    out = []
    for f, k, a in zip(u, cs, (2, 1, 0)):
        out.append(f - k / _face_mean(beta0, per, a) * _grad1(phi, per, a, h))
    return phi, out


def _split_exact(case, d):
    n, per, h = _grid(case)
    dev = d["rho"].device
    rc, re = _radii(n, h, dev)
    m = len(rc)
    step = _hydrostatic_steps(rc, d["rho0"], d["g_edge"], d["rho_cutoff"])
    p0 = d["p0_base"] - torch.cat([torch.zeros(1, dtype=F64, device=dev), torch.cumsum(step, 0)])
    g = d["gamma1"]
    e = torch.cumsum(torch.log(p0[1:] / p0[:-1]) / (0.5 * (g[:-1] + g[1:])), 0)
    beta0 = torch.cat([torch.ones(1, dtype=F64, device=dev), torch.exp(e)])
    idx = _radius_index(n, dev)
    count = torch.bincount(idx.reshape(-1), minlength=m).to(F64)
    sbar = torch.zeros(m, dtype=F64, device=dev).index_add_(0, idx.reshape(-1), d["S"].reshape(-1)) / count.clamp_min(1.0)
    phi, u = _mac_exact(beta0[idx], d["rho"], d["u"], d["S"] - sbar[idx], per, h)
    vol = (re[1:] ** 3 - re[:-1] ** 3) / 3.0
    F = torch.cumsum(beta0 * sbar * vol, 0)
    a = torch.arange(m, device=dev).clamp(max=m - 2)
    t = (re[1:] - rc[a]) / (rc[a + 1] - rc[a])
    w0 = torch.cat([torch.zeros(1, dtype=F64, device=dev), F / (re[1:] ** 2 * (beta0[a] + t * (beta0[a + 1] - beta0[a])))])
    for f, ax in zip(u, (2, 1, 0)):
        x = []
        for b in range(3):
            k = torch.arange(f.shape[b], dtype=F64, device=dev)
            x.append((k if b == ax else k + 0.5) * h - 0.5 * n[b] * h)
        r = torch.sqrt(x[0][:, None, None] ** 2 + x[1][None, :, None] ** 2 + x[2][None, None, :] ** 2)
        lo = (torch.searchsorted(re, r.reshape(-1), right=True) - 1).clamp(0, m - 1).reshape(r.shape)
        s = ((r - re[lo]) / (re[lo + 1] - re[lo])).clamp(0.0, 1.0)
        shape = [1, 1, 1]
        shape[ax] = -1
        add = (w0[lo] + s * (w0[lo + 1] - w0[lo])) * (x[ax].reshape(shape) / r.clamp_min(1e-300))
        f += _zero_walls(add, per, ax)
    return {"phi": phi, "u": u, "p0": p0, "beta0": beta0, "sbar": sbar, "w0": w0}


def _corners(x, per):
    """The eight corner values of every cell, stacked: [8, cells], corner index
    4 z + 2 y + x."""
    out = []
    for c in range(8):
        v = x
        for a, up in ((0, c >> 2 & 1), (1, c >> 1 & 1), (2, c & 1)):
            if per[a]:
                v = torch.roll(v, -1, a) if up else v
            else:
                v = v.narrow(a, up, v.shape[a] - 1)
        out.append(v.reshape(-1))
    return torch.stack(out)


def _to_nodes(v, n, per):
    """The transpose of _corners: [8, cells] summed onto the nodes."""
    out = 0.0
    for c in range(8):
        w = v[c].reshape(n)
        for a, up in ((0, c >> 2 & 1), (1, c >> 1 & 1), (2, c & 1)):
            if per[a]:
                w = torch.roll(w, 1, a) if up else w
            else:
                z = torch.zeros_like(w.narrow(a, 0, 1))
                w = torch.cat([z, w] if up else [w, z], a)
        out = out + w
    return out


def _nodal_exact(case, d):
    n, per, h = _grid(case)
    dev = d["rho"].device
    beta0 = _fill(case, d["beta0_1d"])
    sig = beta0 / d["rho"]
    K = torch.tensor([[1.0, -1.0], [-1.0, 1.0]], dtype=F64)
    M = torch.tensor([[1 / 3, 1 / 6], [1 / 6, 1 / 3]], dtype=F64)
    one = torch.tensor([[0.5], [0.5]], dtype=F64)
    dif = torch.tensor([[-1.0], [1.0]], dtype=F64)

    def kron(z, y, x):
        return torch.kron(z, torch.kron(y, x))

    E = (kron(K, M, M) + kron(M, K, M) + kron(M, M, K)).to(dev)
    # integrals of the basis functions' derivatives over a cell: x, y, z
    G = [g.reshape(-1).to(dev) for g in (kron(one, one, dif), kron(one, dif, one), kron(dif, one, one))]

    def op(p):
        return _to_nodes((E @ _corners(p, per)) * sig.reshape(1, -1), n, per)

    src = beta0 * d["S"]
    # all of it times h^2: -M phi = -(D(beta0 U) - L(beta0 S - m))
    b = torch.zeros(8, beta0.numel(), dtype=F64, device=dev)
    for g, u in zip(G, d["u"]):
        b += g[:, None] * (beta0 * u).reshape(1, -1) * h
    b += 0.125 * (src - src.mean()).reshape(1, -1) * (h * h)
    b = _to_nodes(b, n, per)
    nodes = tuple(m + (0 if p else 1) for m, p in zip(n, per))
    weight = _to_nodes(torch.full((8, sig.numel()), 0.125, dtype=F64, device=dev), n, per)
    scale = _to_nodes(0.125 * sig.reshape(1, -1).expand(8, -1), n, per) / weight
    phi = _cg(op, _solver(nodes, per, scale, True), b)
    corners = _corners(phi, per)
    u = [v - (1.0 / d["rho"]) * ((g[:, None] * corners).sum(0) / h).reshape(n) for g, v in zip(G, d["u"])]
    return {"phi": phi, "u": u}


def exact(case, seed):
    n, per, h = _grid(case)
    d = _inputs(case, seed)
    if case["path"] == "nodal":
        return _nodal_exact(case, d)
    if case["path"] == "split":
        return _split_exact(case, d)
    if case["path"] == "grad":
        cs, rhs = _coefs(case, d)
        c = _fill(case, d["beta0_1d"]) / d["rho"]
        pre = _solver(n, per, c, False)

        def op(p):
            return -_apply(p, cs, per, h) * h * h

        phi = _cg(op, pre, -(rhs - rhs.mean()) * h * h)
        lam = _cg(op, pre, -(d["w"] - d["w"].mean()) * h * h)
        g = [_zero_walls(_grad1(lam, per, a, h) * _grad1(phi, per, a, h), per, a) for a in (2, 1, 0)]
        return {"phi": phi, "rhs": lam, "cx": g[0], "cy": g[1], "cz": g[2]}
    phi, u = _mac_exact(_fill(case, d["beta0_1d"]), d["rho"], d["u"], d["S"], per, h)
    return {"phi": phi, "u": u}
