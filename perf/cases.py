"""Timed cases of the framework: the work that its users have it do.

Everything goes through ``Context``, ``SKFn``/``EnergyFn`` and the carbon
model, on seeded diamond-carbon cells (vacancies, voids, thermal noise) like
those of the benchmark and the tests.  Kinds:

  forces       every column of a cell, then rho, pi and the forces through rho
               (the step of a geometry or energy evaluation; what bench.py times)
  grad         positions -> H, S -> free energy -> autograd backward, with the
               work flow (store or recompute) chosen by the caller
  exact        every column, then the exact gradient of the truncated method
  md           MD steps: rebuild, solve, forces, velocity Verlet
  populations  every column, then ICOHP and COHP on an energy grid
  green        Green's-function columns of a few orbitals at complex energies
  cocg         the same columns by the second solver

A case: kind, the cell (n1 x n2 x n3 cubes of 8 sites, vacancy and void
fractions, noise, and the number that its defects and noise are drawn from),
the cluster radius (0: whole cell), the Krylov dimension, and what the kind
needs besides.  Every cell has vacancies or voids, whose states in the gap pin
the chemical potential.  The seed of the inputs moves the whole cell and
varies the bond integrals by a few percent, so every matrix element is another
one while the pattern and the clusters keep their sizes.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_1210_1531_amd import Context, model
from paper_1210_1531_amd.autograd import EnergyFn, SKFn

A_DIAMOND = 3.567
BASIS = np.array([[0, 0, 0], [0, 2, 2], [2, 0, 2], [2, 2, 0],
                  [1, 1, 1], [1, 3, 3], [3, 1, 3], [3, 3, 1]]) / 4.0
KT = 0.1


def _case(name, kind, cells, vac, void, sigma, r, nu, **more):
    n1, n2, n3 = cells
    return dict(name=name, kind=kind, n1=n1, n2=n2, n3=n3, vac=vac, void=void, sigma=sigma,
                defects=more.pop("defects", 7), r=r, nu=nu, **more)


def listed():
    return [
        # smallest calls: a molecule-sized whole cell, where launches and the
        # host path count (the tests' and smoke()'s size)
        _case("cell61_forces_nu30", "forces", (2, 2, 2), 0.05, 0.0, 0.05, 0.0, 30),
        _case("cell61_exact_nu12", "exact", (2, 2, 2), 0.05, 0.0, 0.05, 0.0, 12),
        # a few hundred atoms: the usual relaxation cell, columns ~ 8 per CU
        _case("vac487_forces_nu30", "forces", (4, 4, 4), 0.05, 0.0, 0.05, 6.0, 30),
        # the benchmark's cell: forward and force backward
        _case("vac3892_forces_nu30", "forces", (8, 8, 8), 0.05, 0.0, 0.05, 6.0, 30),
        # the largest: a void cell, 117,000 columns, small Krylov dimension
        _case("void29k_forces_nu20", "forces", (16, 16, 16), 0.0, 0.10, 0.10, 6.0, 20),
        # a large Krylov dimension on ragged clusters
        _case("void3600_forces_nu40", "forces", (8, 8, 8), 0.0, 0.10, 0.10, 6.0, 40),
        # differentiation by autograd in the memory-saving work flow, odd box,
        # smaller clusters
        _case("vac1596_grad_recompute", "grad", (7, 6, 5), 0.05, 0.0, 0.05, 5.0, 30,
              workflow="recompute"),
        # exact gradient at the benchmark's cell
        _case("vac3892_exact_nu30", "exact", (8, 8, 8), 0.05, 0.0, 0.05, 6.0, 30),
        # molecular dynamics: one step (two frames) with everything rebuilt
        _case("vac3892_md_step", "md", (8, 8, 8), 0.05, 0.0, 0.05, 6.0, 30, steps=1,
              exact_forces=False),
        # bond analysis: ICOHP and an energy-resolved COHP on 256 energies
        _case("vac1642_populations", "populations", (6, 6, 6), 0.05, 0.0, 0.05, 6.0, 30, ne=256),
        # local density of states of a few sites: 64 columns, 16 energies
        _case("vac3892_green64", "green", (8, 8, 8), 0.05, 0.0, 0.05, 6.0, 30, ncols=64, nz=16),
        # converged Green's columns by the second solver
        _case("vac487_cocg64", "cocg", (4, 4, 4), 0.05, 0.0, 0.05, 6.0, 30, ncols=64, nz=4,
              eta=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["forces", "forces", "forces", "grad", "exact", "md", "populations",
                       "green", "cocg"])
    big = {"forces": 3600, "grad": 1000, "exact": 512, "md": 700, "populations": 300,
           "green": 1000, "cocg": 150}[kind]  # cells of eight sites at most
    if rng.random() < 0.2:  # a whole cell of at most 192 atoms
        cells, r = rng.choice([(2, 2, 2), (3, 2, 2), (2, 3, 3), (2, 2, 5), (4, 2, 2)]), 0.0
    else:  # every box length is more than twice the radius
        r = rng.choice([4.5, 5.0, 5.5, 6.0])
        lo = 3 if r <= 5.0 else 4
        target = _log_int(rng, lo ** 3, big)
        n1 = min(18, _log_int(rng, lo, max(lo, target // (lo * lo))))
        n2 = min(18, _log_int(rng, lo, max(lo, target // (n1 * lo))))
        n3 = min(18, max(lo, target // (n1 * n2)))
        cells = (n1, n2, n3)
    if r > 0.0 and rng.random() < 0.4:
        vac, void, sigma = 0.0, round(rng.uniform(0.05, 0.12), 3), round(rng.uniform(0.04, 0.1), 3)
    else:
        vac, void, sigma = round(rng.uniform(0.04, 0.08), 3), 0.0, round(rng.uniform(0.03, 0.1), 3)
    if kind in ("forces", "populations", "green"):
        nu = rng.choice([12, 16, 20, 24, 30, 30, 36, 40, 48])
        if kind == "forces" and cells[0] * cells[1] * cells[2] > 1500:
            nu = min(nu, 20)
    else:
        nu = rng.choice([12, 17, 20, 25, 30])
    more = {}
    if kind == "grad":
        more = dict(workflow=rng.choice(["store", "recompute"]))
    elif kind == "md":
        more = dict(steps=rng.choice([1, 2]), exact_forces=cells[0] * cells[1] * cells[2] < 150
                    and rng.random() < 0.5)
    elif kind == "populations":
        more = dict(ne=_log_int(rng, 16, 512))
    elif kind == "green":
        more = dict(ncols=_log_int(rng, 1, 256), nz=_log_int(rng, 1, 32))
    elif kind == "cocg":
        more = dict(ncols=_log_int(rng, 1, 96), nz=rng.choice([1, 2, 3, 4, 6, 8]),
                    eta=rng.choice([0.3, 0.5, 1.0]))
    c = _case("", kind, cells, vac, void, sigma, r, nu, defects=rng.randrange(1 << 20), **more)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _structure(case, seed):
    """(positions, box lengths) of the case's cell: voids of radius 3 to 8 A
    until the fraction is reached, then vacancies, then Gaussian noise."""
    rng = np.random.default_rng([case["defects"], 9001])
    n = np.array([case["n1"], case["n2"], case["n3"]])
    grid = np.stack(np.meshgrid(*[np.arange(k) for k in n], indexing="ij"), -1).reshape(-1, 1, 3)
    pos = ((grid + BASIS[None]) * A_DIAMOND).reshape(-1, 3)
    cell = n * A_DIAMOND
    total = len(pos)
    while case["void"] > 0 and total - len(pos) < case["void"] * total:
        d = pos - rng.uniform(size=3) * cell
        d -= cell * np.round(d / cell)
        pos = pos[(d * d).sum(1) > rng.uniform(3.0, min(8.0, 0.35 * cell.min())) ** 2]
    keep = np.ones(len(pos), bool)
    keep[rng.choice(len(pos), int(case["vac"] * len(pos)), replace=False)] = False
    pos = pos[keep]
    pos = pos + rng.normal(0.0, case["sigma"], pos.shape)
    return np.mod(pos + np.random.default_rng([seed, 9004]).uniform(size=3) * cell, cell), cell


def _parameters(seed):
    """The carbon model with each bond integral scaled by 1 + N(0, 0.02)."""
    rng = np.random.default_rng([seed, 9005])
    p = dict(model.CARBON_SP)
    for k in ("v_ss_sigma", "v_sp_sigma", "v_pp_sigma", "v_pp_pi",
              "s_ss_sigma", "s_sp_sigma", "s_pp_sigma", "s_pp_pi"):
        p[k] *= 1.0 + 0.02 * rng.standard_normal()
    return p


def _columns(case, n_atoms):
    rng = np.random.default_rng([case["defects"], 9002])
    n = min(case["ncols"], 4 * n_atoms)
    return np.sort(rng.choice(4 * n_atoms, n, replace=False)).astype(np.int32)


def _energies(case):
    x = np.linspace(-12.0, 12.0, case["nz"]) if case["nz"] > 1 else np.array([2.0])
    return x + 1j * case.get("eta", 0.05)


def _grid(case):
    return np.linspace(-25.0, 25.0, case["ne"])


def prepare(case, seed):
    pos, cell = _structure(case, seed)
    ctx = Context()
    s = dict(case=case, ctx=ctx, model=model.sk_model(**_parameters(seed)), cell=cell, n_electrons=4.0 * len(pos),
             pos=torch.tensor(pos, dtype=torch.float64, device="cuda"))
    if case["kind"] == "md":
        rng = np.random.default_rng([seed, 9003])
        v = rng.normal(0.0, model.thermal_sigma(300.0), pos.shape)
        s["vel"] = torch.tensor(v - v.mean(0), dtype=torch.float64, device="cuda")
        return s
    ctx.sk_build(s["model"], s["pos"], cell)
    ctx.set_system(*ctx.sk_get_csr(), pos=s["pos"], cell=cell, r_cluster=case["r"])
    if case["kind"] in ("green", "cocg"):
        s["cols"] = _columns(case, len(pos))
        s["z"] = _energies(case)
    return s


# --------------------------------------------------------------- one pass
def run(s):
    case, ctx = s["case"], s["ctx"]
    opts = dict(nu=case["nu"], kT=KT, n_electrons=s["n_electrons"])
    kind = case["kind"]
    if kind == "forces":
        mu, e_band, a_free = ctx.solve(**opts)
        rho, pi = ctx.density_matrix()
        return dict(mu=mu, e_band=e_band, a_free=a_free, rho=rho, pi=pi,
                    forces=ctx.forces(s["model"]))
    if kind == "grad":
        pos = s["pos"].clone().requires_grad_(True)
        h, sv = SKFn.apply(pos, ctx)
        a_free = EnergyFn.apply(h, sv, ctx, dict(opts, workflow=case["workflow"]))
        a_free.backward()
        return dict(a_free=a_free.detach(), grad=pos.grad)
    if kind == "exact":
        mu, e_band, a_free = ctx.solve(keep_exact=True, **opts)
        return dict(mu=mu, e_band=e_band, a_free=a_free, forces=ctx.forces_exact(s["model"]))
    if kind == "md":
        x, v, f, thermo = ctx.md_run(s["model"], s["pos"], s["vel"], s["cell"], 0.5,
                                     model.MASS_CARBON, case["steps"], r_cluster=case["r"],
                                     exact_forces=case["exact_forces"], **model.PAIR_REPULSION,
                                     **opts)
        return dict(x=x, v=v, forces=f, thermo=thermo)
    if kind == "populations":
        mu, e_band, a_free = ctx.solve(workflow="store", **opts)
        b, b_sigma, b_pi = ctx.icohp(s["model"])
        return dict(mu=mu, e_band=e_band, a_free=a_free, icohp=b, icohp_sigma=b_sigma,
                    icohp_pi=b_pi, cohp=ctx.cohp(_grid(case), 0.1))
    if kind == "green":
        g, off = ctx.green_columns(s["cols"], s["z"], nu=case["nu"])
        return dict(g=g, off=off)
    g, off, iters = ctx.cocg_columns(s["cols"], s["z"])
    return dict(g=g, off=off, iters=iters)


# ------------------------------------------------------------------- work
def work(case):
    """Bytes of positions, H, S and what the pass returns; FP64 operations of
    the method: 4 per matrix nonzero and Krylov step, Gram-Schmidt and the two
    projections, the small eigenproblem, and the reverse sweep where there is
    one.  Counts per column from the cell's density and cluster radius."""
    sites = 8 * case["n1"] * case["n2"] * case["n3"]
    n = int(sites * (1.0 - case["vac"]) * (1.0 - case["void"]))
    dens = n / (sites / 8 * A_DIAMOND ** 3)
    nc = 4.0 * (n if case["r"] <= 0 else min(n, dens * 4.18879 * case["r"] ** 3))
    row = 4.0 * (1 + 16 * n / sites)  # nonzeros of a matrix row
    nu, m = case["nu"], 4 * n
    nnz = m * row
    column = 4.0 * nu * nc * row + 5.0 * nc * nu * nu + 20.0 * nu ** 3
    kind = case["kind"]
    if kind in ("forces", "grad"):
        twice = 2 if case.get("workflow") == "recompute" else 1
        return dict(bytes=8.0 * (4 * nnz + 6 * n), flops=twice * m * column + 4.0 * nnz * nu)
    if kind == "exact":
        return dict(bytes=8.0 * (2 * nnz + 6 * n), flops=3.0 * m * column)
    if kind == "md":
        per = 3.0 if case["exact_forces"] else 1.0
        return dict(bytes=8.0 * 15 * n, flops=(case["steps"] + 1) * per * m * column)
    if kind == "populations":
        nblk = nnz / 16
        return dict(bytes=8.0 * (2 * nnz + nblk * (3 + case["ne"])),
                    flops=m * column + nblk * 4.0 * nu * (8.0 + 6.0 * case["ne"]))
    cols = min(case["ncols"], m)
    out = 16.0 * cols * case["nz"] * nc
    if kind == "green":
        return dict(bytes=out + 8.0 * 2 * cols / 4 * nc * row,
                    flops=cols * (column + 8.0 * nc * nu * case["nz"]))
    return dict(bytes=out + 8.0 * 2 * cols / 4 * nc * row,
                flops=cols * case["nz"] * 300.0 * nc * (8.0 * row + 40.0))


# -------------------------------------------------- the same in 64 bits
def _min_image(d, cell):
    return d - cell * np.round(d / cell)


def _pairs(pos, cell):
    """Directed pairs (i, j, d = x_j - x_i), i != j, closer than the cutoff."""
    d = _min_image(pos[None] - pos[:, None], cell)
    r2 = (d * d).sum(-1)
    i, j = np.nonzero(r2 < model.CARBON_SP["r_cut"] ** 2)
    i, j = i[i != j], j[i != j]
    return i, j, d[i, j]


def _sk_blocks(d, v, p):
    """Two-center 4 x 4 blocks (npair, 4, 4) for d = x_j - x_i."""
    r = d.norm(dim=1)
    t = ((r - p["r_on"]) / (p["r_cut"] - p["r_on"])).clamp(0.0, 1.0)
    u = (p["r0"] / r) ** 2 * (1.0 - t ** 3 * (10.0 - 15.0 * t + 6.0 * t * t))
    c = d / r[:, None]
    ss, sp, pps, ppp = v
    blk = d.new_zeros((len(d), 4, 4))
    blk[:, 0, 0] = ss
    blk[:, 0, 1:] = sp * c
    blk[:, 1:, 0] = -sp * c
    cc = c[:, :, None] * c[:, None, :]
    blk[:, 1:, 1:] = pps * cc + ppp * (torch.eye(3, dtype=d.dtype) - cc)
    return blk * u[:, None, None]


def _matrices(d, i, j, n, p):
    """Dense H and S (torch, float64) of the cell."""
    out = []
    for pre, on in (("v", [p["es"]] + 3 * [p["ep"]]), ("s", 4 * [1.0])):
        blk = _sk_blocks(d, [p[pre + k] for k in ("_ss_sigma", "_sp_sigma", "_pp_sigma", "_pp_pi")], p)
        full = torch.zeros((n, n, 4, 4), dtype=torch.float64)
        full = full.index_put((torch.arange(n), torch.arange(n)),
                              torch.diag(torch.tensor(on, dtype=torch.float64)).expand(n, 4, 4))
        full = full.index_put((i, j), blk)
        out.append(full.permute(0, 2, 1, 3).reshape(4 * n, 4 * n))
    return out


def _ritz(h, s, cols, nu):
    """Ritz data of the columns `cols` of the dense pencil (h, s), batched:
    eps (b, nu), Y (b, n, nu), d (b, nu), w (b, nu)."""
    n = h.shape[0]
    q = torch.zeros((len(cols), n), dtype=h.dtype)
    q[torch.arange(len(cols)), torch.as_tensor(cols)] = 1.0
    basis = [q]
    for _ in range(1, min(nu, n)):
        x = basis[-1] @ h
        b = torch.stack(basis, 2)
        for _ in range(2):
            x = x - (b @ (b.transpose(1, 2) @ x[:, :, None]))[:, :, 0]
        basis.append(x / x.norm(dim=1, keepdim=True))
    b = torch.stack(basis, 2)
    hp = b.transpose(1, 2) @ (h @ b)
    sp = b.transpose(1, 2) @ (s @ b)
    low = torch.linalg.cholesky(0.5 * (sp + sp.transpose(1, 2)))
    c = torch.linalg.solve_triangular(low, 0.5 * (hp + hp.transpose(1, 2)), upper=False)
    c = torch.linalg.solve_triangular(low, c.transpose(1, 2), upper=False)
    eps, u = torch.linalg.eigh(0.5 * (c + c.transpose(1, 2)))
    y = torch.linalg.solve_triangular(low.transpose(1, 2), u, upper=True)
    ritz_d = y[:, 0, :]  # the first basis vector is the column's orbital
    w = 2.0 * ritz_d * (sp @ y)[:, 0, :]
    return eps, b @ y, ritz_d, w


def _fermi(x):
    return 0.5 * (1.0 - torch.tanh(0.5 * x))


def _mu(eps, w, ne):
    lo, hi = eps.min() - 40 * KT, eps.max() + 40 * KT
    while hi - lo > 1e-12:
        mid = lo + 0.5 * (hi - lo)
        if mid <= lo or mid >= hi:
            break
        if (w * _fermi((eps - mid) / KT)).sum() < ne:
            lo = mid
        else:
            hi = mid
    return lo + 0.5 * (hi - lo)


def _clusters(case, pos, cell):
    n = len(pos)
    if case["r"] <= 0.0 or 2.0 * case["r"] >= cell.min():
        return [(np.arange(n), np.arange(n))]  # one cluster, every atom's columns
    out = []
    for a in range(n):
        d = _min_image(pos - pos[a], cell)
        out.append((np.nonzero((d * d).sum(1) <= case["r"] ** 2)[0], np.array([a])))
    return out


def exact(case, seed):
    pos, cell = _structure(case, seed)
    n, kind = len(pos), case["kind"]
    if n > 260 or kind == "md":
        return None
    i, j, dv = _pairs(pos, cell)
    it, jt = torch.as_tensor(i), torch.as_tensor(j)
    d = torch.tensor(dv, dtype=torch.float64, requires_grad=True)
    p = _parameters(seed)
    h, s = _matrices(d, it, jt, n, p)
    hd, sd = h.detach(), s.detach()
    groups = _clusters(case, pos, cell)

    def orbitals(atoms):
        return torch.as_tensor((4 * atoms[:, None] + np.arange(4)).ravel())

    def sub(m, atoms):
        o = orbitals(atoms)
        return m[o][:, o]

    if kind in ("green", "cocg"):
        z = _energies(case)
        g, off = [], [0]
        for col in _columns(case, n):
            atoms = groups[0][0] if len(groups) == 1 else groups[col // 4][0]
            loc = 4 * int(np.searchsorted(atoms, col // 4)) + int(col) % 4
            hc, sc = sub(hd, atoms), sub(sd, atoms)
            if kind == "green":
                eps, y, dk, _ = _ritz(hc, sc, [loc], case["nu"])
                for zq in z:
                    g.append(((y[0] * dk[0]).numpy() @ (1.0 / (zq - eps[0].numpy()))))
            else:
                rhs = np.zeros(len(hc), complex)
                rhs[loc] = 1.0
                for zq in z:
                    g.append(np.linalg.solve(zq * sc.numpy() - hc.numpy(), rhs))
            off.append(off[-1] + len(hc))
        out = dict(g=np.concatenate(g), off=np.array(off))
        return dict(out, iters=None) if kind == "cocg" else out

    if kind == "exact" and len(groups) > 1:
        return None  # one reverse sweep per cluster takes too long here
    eps, w, parts = [], [], []
    for atoms, mine in groups:
        loc = [4 * int(np.searchsorted(atoms, a)) + o for a in mine for o in range(4)]
        hc, sc = (sub(h, atoms), sub(s, atoms)) if kind == "exact" else (sub(hd, atoms), sub(sd, atoms))
        e, y, dk, wk = _ritz(hc, sc, loc, case["nu"])
        eps.append(e)
        w.append(wk)
        if kind != "exact":
            parts.append((orbitals(atoms), orbitals(mine), y * dk[:, None, :]))
    eps, w = torch.cat(eps), torch.cat(w)
    mu = _mu(eps.detach(), w.detach(), 4.0 * n)
    f = _fermi((eps.detach() - mu) / KT)
    x = (eps.detach() - mu) / KT
    e_band = float((w.detach() * f * eps.detach()).sum())
    ent = torch.special.entr(f) + torch.special.entr(_fermi(-x))
    a_free = e_band - KT * float((w.detach() * ent).sum())
    head = dict(mu=float(mu), e_band=e_band, a_free=a_free)

    def on_atoms(g):  # d = x_j - x_i, so dA/dx_j += g and dA/dx_i -= g
        grad = torch.zeros((n, 3), dtype=torch.float64)
        return grad.index_add(0, jt, g).index_add(0, it, -g)

    if kind == "exact":
        omega = (w * (-KT) * torch.nn.functional.softplus(-(eps - mu) / KT)).sum()
        omega.backward()
        return dict(head, forces=-on_atoms(d.grad).numpy())

    rho, pi = torch.zeros_like(hd), torch.zeros_like(hd)  # row: the column's own orbital
    k = 0
    for rows, mine, yd in parts:
        fk, ek = f[k:k + len(mine)], eps[k:k + len(mine)]
        k += len(mine)
        rho[mine[:, None], rows[None, :]] = 2.0 * (yd @ fk[:, :, None])[:, :, 0]
        pi[mine[:, None], rows[None, :]] = 2.0 * (yd @ (fk * ek)[:, :, None])[:, :, 0]
    (h * rho - s * pi).sum().backward()
    grad = on_atoms(d.grad).numpy()
    if kind == "grad":
        return dict(a_free=np.float64(a_free), grad=grad)
    blocks = [np.sort(np.append(j[i == a], a)) for a in range(n)]
    if kind == "forces":
        at = np.concatenate([(4 * a + o) * 4 * n + (4 * blocks[a][:, None] + np.arange(4)).ravel()
                             for a in range(n) for o in range(4)])
        return dict(head, rho=rho.reshape(-1)[at].numpy(), pi=pi.reshape(-1)[at].numpy(),
                    forces=-grad)
    # populations: blocks in row order
    bi = np.concatenate([np.full(len(b), a) for a, b in enumerate(blocks)])
    bj = np.concatenate(blocks)
    prod = (hd * rho).reshape(n, 4, n, 4).sum((1, 3))
    hp = torch.zeros((n, n, 4, 4), dtype=torch.float64)
    hp[it, jt] = _sk_blocks(d.detach(), [0.0, 0.0, 0.0, p["v_pp_pi"]], p)
    b_pi = (hp.permute(0, 2, 1, 3).reshape(4 * n, 4 * n) * rho).reshape(n, 4, n, 4).sum((1, 3))
    off = torch.as_tensor(bi != bj)
    b = prod[bi, bj]
    b_pi = b_pi[bi, bj] * off
    grid = torch.as_tensor(_grid(case))
    cohp = torch.zeros((len(bi), len(grid)), dtype=torch.float64)
    col, where = 0, {}
    for rows, mine, yd in parts:
        for q, orb in enumerate(mine.tolist()):
            where[orb] = (rows, yd[q], eps[col])
            col += 1
    for t, (a, c) in enumerate(zip(bi, bj)):
        for o in range(4):
            rows, yd, ek = where[4 * a + o]
            at = int(torch.searchsorted(rows, torch.tensor(4 * c)))
            ck = hd[4 * a + o, 4 * c:4 * c + 4] @ yd[at:at + 4]
            cohp[t] += (2.0 / np.pi) * ((0.1 / ((grid[:, None] - ek) ** 2 + 0.01)) @ ck)
    return dict(head, icohp=b.numpy(), icohp_sigma=((b - b_pi) * off).numpy(),
                icohp_pi=b_pi.numpy(), cohp=cohp.numpy())
