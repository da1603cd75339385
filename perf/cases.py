"""The work that programs have this library do, as measurable cases.

A case is a dict of plain values.  ``kind`` names the entry points that it
goes through, the other keys are sizes and options:

  forward   new walker coordinates -> mo_vgl (values, gradients, Laplacians):
            a Monte Carlo step that evaluates local energies
  gradient  forward, then the adjoint with fixed coefficients: forces and
            electron drift terms from a weight per mo_vgl entry
  train     one optimisation step through torch.autograd, in which the MO
            coefficients and nuclei are parameters and so new on every pass
  batch     many molecules of uneven sizes in one call, forward and adjoint
  value     MO values on points (orbital plots)
  density   electron density of a determinant on a box of grid points
  jastrow   three-body Jastrow factor of every walker
  det       determinants and adjugates of many small matrices

Molecules are seeded stand-ins: carbon and hydrogen atoms at about one atom
per 100 cubic bohr, one contracted Cartesian Gaussian basis per element with
1 to 6 primitives per shell and exponents of 0.1 to 1e4, electrons normally
distributed around the nuclei.  The number of primitives and their exponents
belong to the basis set and do not depend on the seed; geometry, orbitals,
walkers and weights do.

Mixed-precision programs hold their results in FP32, FP64 ones in FP64.
"""
import math

import numpy as np
import torch

import paper_2512_16677_amd as qmk

DEV = "cuda:0"
# angular momenta of the shells of a heavy atom and of hydrogen
SHELLS = {
    "small": ((0, 0, 0, 1, 1, 2), (0, 0, 1)),  # 3s2p1d and 2s1p: 15 and 5 AOs
    "large": ((0, 0, 0, 0, 1, 1, 1, 2, 2, 3), (0, 0, 0, 1, 1, 2)),  # 4s3p2d1f and 3s2p1d: 35 and 15 AOs
}
AO_PER_ATOM = {"small": (15, 5), "large": (35, 15)}
BATCH_ALIGN = 64  # elements: molecules start on whole cache lines of a shared buffer


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # The smallest call: one water molecule, 128 walkers (25 AOs, 25 MOs,
        # 10 electrons).  A short Monte Carlo step, where launches count.
        dict(name="water_forward_fp64", kind="forward", mode="fp64", bits=53, basis="small",
             heavy=1, hydrogen=2, mo=25, walkers=128, screen=False),
        # The same molecule in an optimiser: every step has new coefficients.
        dict(name="water_train_fp64", kind="train", mode="fp64", bits=53, basis="small",
             heavy=1, hydrogen=2, mo=25, walkers=128, screen=False),
        # The ordinary call in full precision: 40 C + 40 H, 800 AOs, 400 MOs,
        # 280 electrons.
        dict(name="medium_forward_fp64", kind="forward", mode="fp64", bits=53, basis="small",
             heavy=40, hydrogen=40, mo=400, walkers=500, screen=False),
        # Forces and drift of the same molecule at half the walkers.
        dict(name="medium_gradient_fp64", kind="gradient", mode="fp64", bits=53, basis="small",
             heavy=40, hydrogen=40, mo=400, walkers=250, screen=False),
        # Odd numbers of everything in FP32: 23 C + 32 H, 505 AOs, 251 MOs, 170
        # electrons.
        dict(name="odd_gradient_f32", kind="gradient", mode="mixed_f32", bits=53, basis="small",
             heavy=23, hydrogen=32, mo=251, walkers=301, screen=False),
        # Wavefunction optimisation in the fastest precision mode.
        dict(name="medium_train_bf16x3", kind="train", mode="mixed_bf16x3", bits=53, basis="small",
             heavy=40, hydrogen=40, mo=400, walkers=256, screen=False),
        # The largest molecule: 150 C + 150 H, 7500 AOs, 1050 MOs, 1050
        # electrons, at the precision parameter that the mixed modes are
        # meant for, with the screened product.
        dict(name="large_forward_bf16x3", kind="forward", mode="mixed_bf16x3", bits=24, basis="large",
             heavy=150, hydrogen=150, mo=1050, walkers=60, screen=True),
        # Many molecules of 4 to 60 atoms with 8 to 128 walkers each, forward
        # and adjoint: the fitting set of a transferable wavefunction.
        dict(name="batch_gradient_fp64", kind="batch", mode="fp64", bits=53, basis="small", molecules=24,
             atoms_min=4, atoms_max=60, walkers_min=8, walkers_max=128),
        dict(name="batch_gradient_bf16x3", kind="batch", mode="mixed_bf16x3", bits=53, basis="small",
             molecules=48, atoms_min=4, atoms_max=60, walkers_min=8, walkers_max=128),
        # Electron density of a closed-shell determinant on a plotting grid:
        # 1085 AOs, 211 occupied orbitals.
        dict(name="grid_density_fp64", kind="density", mode="fp64", bits=53, basis="small",
             heavy=56, hydrogen=49, mo=500, occupied=211, nx=91, ny=97, nz=89),
        # Jastrow factor of the ordinary molecule.
        dict(name="medium_jastrow", kind="jastrow", basis="small", heavy=40, hydrogen=40, walkers=500, nord=5),
        # Slater matrices of small molecules: one per walker and spin.
        dict(name="slater_det_16", kind="det", n=16, batch=50000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(["forward", "forward", "gradient", "gradient", "train", "batch", "value", "density",
                       "jastrow", "det"])
    mode = rng.choice(["fp64", "fp64", "mixed_f32", "mixed_bf16x3"])
    if kind == "det":
        n = rng.randint(2, 32)
        return dict(kind=kind, n=n, batch=_log(rng, 64, max(64, 12800000 // (n * n))))
    if kind == "batch":
        lo = rng.randint(3, 20)
        return dict(kind=kind, mode=mode, bits=53, basis="small", molecules=rng.randint(4, 24), atoms_min=lo,
                    atoms_max=lo + rng.randint(0, 40), walkers_min=rng.randint(4, 16),
                    walkers_max=rng.randint(16, 64))
    basis = "small" if rng.random() < 0.8 else "large"
    heavy = _log(rng, 1, 60 if basis == "small" else 40)
    hydrogen = rng.randint(0, 2 * heavy)
    if kind == "jastrow":
        ne = 6 * heavy + hydrogen
        top = max(1, int(6e7 // (ne * ne)))
        return dict(kind=kind, basis=basis, heavy=heavy, hydrogen=hydrogen, walkers=_log(rng, 1, min(top, 2000)),
                    nord=rng.randint(2, 6))
    ao = heavy * AO_PER_ATOM[basis][0] + hydrogen * AO_PER_ATOM[basis][1]
    if kind == "density":
        mo = max(3, ao // 2)
        return dict(kind=kind, mode=mode, bits=53, basis=basis, heavy=heavy, hydrogen=hydrogen, mo=mo,
                    occupied=rng.randint(1, mo), nx=_log(rng, 8, 64), ny=_log(rng, 8, 64), nz=_log(rng, 8, 64))
    mo = max(1, int(ao * rng.uniform(0.3, 0.7)))
    elec = 6 * heavy + hydrogen
    # at most about 1e11 operations per product and 4e8 AO values in all
    top = int(min(1e11 / (10.0 * ao * mo * elec), 4e8 / (5.0 * ao * elec)))
    case = dict(kind=kind, mode=mode, bits=53, basis=basis, heavy=heavy, hydrogen=hydrogen, mo=mo,
                walkers=_log(rng, 1, max(1, min(1000, top))), screen=False)
    if kind in ("forward", "gradient") and ao > 500 and rng.random() < 0.3:
        case["screen"] = True
    return case


# --------------------------------------------------------------------- inputs
def _rngs(seed):
    return [np.random.default_rng(s) for s in np.random.SeedSequence(seed).spawn(4)]


def _basis(recipe, which):
    """Shells (l, exponents, coefficients) of an element: a fixed table."""
    rng = np.random.default_rng(977 + which)
    shells = []
    for l in recipe:
        n = int(rng.integers(1, 7))
        shells.append((l, np.sort(10.0 ** rng.uniform(-1.0, 4.0, n)), rng.uniform(0.1, 1.0, n)))
    return shells


def _geometry(rng, heavy, hydrogen):
    """Uniform atoms at least 1.5 bohr apart, 100 cubic bohr for each."""
    n = heavy + hydrogen
    side = (100.0 * n) ** (1.0 / 3.0)
    pos = np.empty((n, 3))
    k = 0
    while k < n:
        p = rng.uniform(0.0, side, 3)
        if k == 0 or np.min(np.sum((pos[:k] - p) ** 2, axis=1)) > 2.25:
            pos[k] = p
            k += 1
    return pos


class Molecule:
    def __init__(self, rng, basis, heavy, hydrogen):
        self.pos = _geometry(rng, heavy, hydrogen)
        self.charge = np.array([6] * heavy + [1] * hydrogen)
        tables = [_basis(SHELLS[basis][0], 1), _basis(SHELLS[basis][1], 2)]
        nucleus, ang, off, expo, coef = [], [], [0], [], []
        for a in range(heavy + hydrogen):
            for l, g, c in tables[0 if a < heavy else 1]:
                nucleus.append(a)
                ang.append(l)
                expo.append(g)
                coef.append(c)
                off.append(off[-1] + len(g))
        self.nucleus = np.array(nucleus, dtype=np.int64)
        self.ang = np.array(ang, dtype=np.int32)
        self.off = np.array(off, dtype=np.int64)
        self.expo = np.concatenate(expo)
        self.coef = np.concatenate(coef)
        self.ao = int(sum((l + 1) * (l + 2) // 2 for l in ang))
        self.elec = int(self.charge.sum())

    def walkers(self, gen, n, dtype=torch.float64):
        at = torch.from_numpy(np.repeat(self.pos, self.charge, axis=0)).to(DEV)
        return (at + torch.randn((n, self.elec, 3), generator=gen, device=DEV, dtype=torch.float64)).to(dtype)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 11)
    return g


def _orbitals(rng, mo, ao):
    return rng.normal(0.0, 1.0 / math.sqrt(ao), size=(mo, ao))


def _context(case, mol, coef=None):
    ctx = qmk.Context()
    if "mode" in case:
        ctx.set_precision(case["bits"], case["mode"])
    ctx.set_nucleus(mol.pos)
    ctx.set_basis(mol.nucleus, mol.ang, mol.off, mol.expo, mol.coef)
    if coef is not None:
        ctx.set_mo_coef(coef)
    if case.get("screen"):
        ctx.set_screening(True)
    return ctx


def _real(case):
    """Element type of a program's results."""
    return torch.float64 if case.get("mode", "fp64") == "fp64" else torch.float32


def _atoms(case, k):
    """Atoms and walkers of molecule k of a batch: sizes do not depend on the seed."""
    rng = np.random.default_rng(4099 + k)
    atoms = int(rng.integers(case["atoms_min"], case["atoms_max"] + 1))
    walkers = int(rng.integers(case["walkers_min"], case["walkers_max"] + 1))
    return (atoms + 1) // 2, atoms // 2, walkers


def _inputs(case, seed):
    """Everything of a case that is data: plain arrays and tensors."""
    rg, rc, ro, _ = _rngs(seed)
    gen = _gen(seed)
    kind = case["kind"]
    if kind == "det":
        n = case["n"]
        a = torch.randn((case["batch"], n, n), generator=gen, device=DEV, dtype=torch.float64)
        return dict(a=a / math.sqrt(n))
    if kind == "batch":
        mols = []
        for k in range(case["molecules"]):
            heavy, hydrogen, walkers = _atoms(case, k)
            mol = Molecule(rg, case["basis"], heavy, hydrogen)
            mo = mol.ao // 2
            w = torch.randn((walkers, mol.elec, 5, mo), generator=gen, device=DEV, dtype=torch.float64)
            mols.append(dict(mol=mol, C=_orbitals(rc, mo, mol.ao), r=mol.walkers(gen, walkers),
                             w=w.to(_real(case))))
        return dict(mols=mols)
    mol = Molecule(rg, case["basis"], case["heavy"], case["hydrogen"])
    if kind == "jastrow":
        terms = qmk.jastrow_een_terms(case["nord"])
        return dict(mol=mol, r=mol.walkers(gen, case["walkers"]), kappa=0.6,
                    c=rc.normal(0.0, 1.0, size=(terms, len(mol.charge))) / mol.elec ** 2)
    C = _orbitals(rc, case["mo"], mol.ao)
    if kind == "density":
        lo, hi = mol.pos.min(axis=0) - 4.0, mol.pos.max(axis=0) + 4.0
        axes = [torch.linspace(float(lo[i]), float(hi[i]), case[k], device=DEV, dtype=torch.float64)
                for i, k in enumerate(("nx", "ny", "nz"))]
        grid = torch.stack(torch.meshgrid(*axes, indexing="ij"), dim=-1).reshape(case["nx"], -1, 3)
        occ = np.zeros(case["mo"])
        occ[: case["occupied"]] = 2.0
        return dict(mol=mol, C=C, r=grid.contiguous(), occ=occ)
    d = dict(mol=mol, C=C)
    if kind == "train":
        # parameters and walkers in the program's own element type
        t = _real(case)
        d["C"] = torch.from_numpy(C).to(DEV, t)
        d["R"] = torch.from_numpy(mol.pos).to(DEV, t)
        d["r"] = mol.walkers(gen, case["walkers"], t)
    else:
        d["r"] = mol.walkers(gen, case["walkers"])
    if kind in ("gradient", "train"):
        w = torch.randn((case["walkers"], mol.elec, 5, case["mo"]), generator=gen, device=DEV, dtype=torch.float64)
        d["w"] = w if kind == "train" else w.to(_real(case))
    return d


def _flat(shapes, dtype):
    """One buffer for tensors of all molecules, and a view of it for each."""
    sizes = [-(-int(np.prod(s)) // BATCH_ALIGN) * BATCH_ALIGN for s in shapes]
    buf = torch.zeros(sum(sizes), dtype=dtype, device=DEV)
    views, at = [], 0
    for s, n in zip(shapes, sizes):
        views.append(buf[at: at + int(np.prod(s))].view(s))
        at += n
    return buf, views


def prepare(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    s = dict(case=case, d=d)
    if kind == "det":
        s["ctx"] = qmk.Context()
        return s
    if kind == "batch":
        mols = d["mols"]
        ctxs = [_context(case, m["mol"], m["C"]) for m in mols]
        for c, m in zip(ctxs, mols):
            c.set_point(m["r"])
        s["batch"] = qmk.Batch(ctxs)
        s["out"], s["outs"] = _flat([tuple(m["w"].shape) for m in mols], _real(case))
        grads = {}
        for key, shapes in (("d_coef", [m["C"].shape for m in mols]),
                            ("d_elec", [tuple(m["r"].shape) for m in mols]),
                            ("d_nucl", [m["mol"].pos.shape for m in mols])):
            grads[key] = _flat(shapes, torch.float64)
        s["flat"] = {k: v[0] for k, v in grads.items()}
        s["grads"] = [{k: v[1][i] for k, v in grads.items()} for i in range(len(mols))]
        s["ws"] = [m["w"] for m in mols]
        return s
    if kind == "train":
        s["ctx"] = _context(case, d["mol"], None)
        for k in ("C", "R", "r"):
            d[k].requires_grad_(True)
        return s
    s["ctx"] = _context(case, d["mol"], d.get("C"))
    if kind == "density":
        s["rho"] = torch.empty(d["r"].shape[:2], dtype=torch.float64, device=DEV)
    elif kind == "value":
        s["out"] = torch.empty((*d["r"].shape[:2], case["mo"]), dtype=_real(case), device=DEV)
    elif kind in ("forward", "gradient"):
        s["out"] = torch.empty((*d["r"].shape[:2], 5, case["mo"]), dtype=_real(case), device=DEV)
    return s


# ------------------------------------------------------------------- one pass
def run(s):
    case, d = s["case"], s["d"]
    kind = case["kind"]
    if kind == "det":
        return s["ctx"].det_adj(d["a"])
    if kind == "batch":
        s["batch"].run(outs=s["outs"], ws=s["ws"], grads=s["grads"])
        return [s["out"], {k: v.to(_real(case)) for k, v in s["flat"].items()}]
    ctx = s["ctx"]
    if kind == "train":
        mo = qmk.mo_vgl(ctx, d["C"], d["R"], d["r"])
        return torch.autograd.grad(mo, (d["C"], d["R"], d["r"]), grad_outputs=d["w"])
    ctx.set_point(d["r"])
    if kind == "jastrow":
        return ctx.jastrow_een(case["nord"], d["kappa"], d["c"])
    if kind == "density":
        return ctx.get_density(d["occ"], out=s["rho"])
    if kind == "value":
        return ctx.get_mo_value(out=s["out"])
    mo = ctx.get_mo_vgl(out=s["out"])
    if kind == "forward":
        return mo
    g = ctx.adjoint(d["w"])
    return [mo, {k: v.to(_real(case)) for k, v in g.items()}]


# ------------------------------------------------------- what it cannot do without
def _work(P, K, N, esz, comps, products, coef=1):
    """Points in, results out; `products` contractions over AOs and MOs."""
    return {"bytes": 24.0 * P + coef * 8.0 * K * N + esz * comps * P * N,
            "flops": 2.0 * comps * P * K * N * products}


def _add(a, b):
    return {k: a[k] + b[k] for k in a}


def _grad_work(P, K, N, esz):
    # forward, then both products of the adjoint: weights in, gradients out
    w = _work(P, K, N, esz, 5, 3, coef=2)
    w["bytes"] += esz * 5.0 * P * N + 24.0 * P
    return w


def work(case):
    kind = case["kind"]
    if kind == "det":
        n, b = case["n"], float(case["batch"])
        return {"bytes": 8.0 * b * (2 * n * n + 1), "flops": b * (8.0 / 3.0) * n ** 3}
    esz = 8 if case.get("mode", "fp64") == "fp64" else 4
    if kind == "batch":
        w = {"bytes": 0.0, "flops": 0.0}
        per = AO_PER_ATOM[case["basis"]]
        for k in range(case["molecules"]):
            heavy, hydrogen, walkers = _atoms(case, k)
            K = heavy * per[0] + hydrogen * per[1]
            w = _add(w, _grad_work(walkers * (6 * heavy + hydrogen), K, K // 2, esz))
        return w
    heavy, hydrogen = case["heavy"], case["hydrogen"]
    per = AO_PER_ATOM[case["basis"]]
    K, ne = heavy * per[0] + hydrogen * per[1], 6 * heavy + hydrogen
    if kind == "jastrow":
        nn, nw, nord = heavy + hydrogen, case["walkers"], case["nord"]
        return {"bytes": 24.0 * nw * ne + 8.0 * nw,
                "flops": 2.0 * nw * ne * ne * nn * (nord // 2) * (nord - 1)}
    if kind == "density":
        P = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 32.0 * P + 8.0 * K * case["occupied"], "flops": 2.0 * P * K * case["occupied"]}
    # (screened cases count the dense product: how much of it is zeros depends
    # on the geometry)
    P, N = case["walkers"] * ne, case["mo"]
    if kind in ("gradient", "train"):
        return _grad_work(P, K, N, esz)
    return _work(P, K, N, esz, 1 if kind == "value" else 5, 1)


# ------------------------------------------------------- the same in 64 bits
def _dfact(n):
    return 1.0 if n <= 0 else n * _dfact(n - 2)


def _moment(n, alpha):
    """Integral of t^(2n) exp(-alpha t^2)."""
    return math.gamma(n + 0.5) / alpha ** (n + 0.5)


def _axis(l, alpha):
    return _moment(l, alpha) * _moment(0, alpha) ** 2


def _shell_tables(mol, bits):
    """Shells of each angular momentum: nucleus, exponents and folded
    coefficients padded to six primitives (coefficient 0), first AO."""
    groups = {}
    norms = {}
    ao = 0
    for s in range(len(mol.ang)):
        l = int(mol.ang[s])
        lo, hi = int(mol.off[s]), int(mol.off[s + 1])
        g, a = mol.expo[lo:hi], mol.coef[lo:hi]
        key = (l, g.tobytes(), a.tobytes())
        if key not in norms:
            fa = np.array([c / math.sqrt(_axis(l, 2.0 * x)) for x, c in zip(g, a)])
            ovl = sum(p * q * _axis(l, x + y) for x, p in zip(g, fa) for y, q in zip(g, fa))
            norms[key] = fa / math.sqrt(ovl)
        pad = 6 - (hi - lo)
        groups.setdefault(l, []).append((int(mol.nucleus[s]), np.pad(g, (0, pad), constant_values=1.0),
                                         np.pad(norms[key], (0, pad)), ao))
        ao += (l + 1) * (l + 2) // 2
    out = []
    for l, rows in sorted(groups.items()):
        out.append((l, torch.tensor([r[0] for r in rows], device=DEV),
                    torch.from_numpy(np.array([r[1] for r in rows])).to(DEV),
                    torch.from_numpy(np.array([r[2] for r in rows])).to(DEV),
                    np.array([r[3] for r in rows])))
    order = np.concatenate([(first[None, :] + i).reshape(-1) for l, _, _, _, first in out
                            for i in range((l + 1) * (l + 2) // 2)])
    at = torch.from_numpy(np.argsort(order)).to(DEV)
    return out, at, (bits - 1) * math.log(2.0)


def _ao(tables, r, R, comps=5):
    """AO values (comps = 1), with gradients and Laplacians (5): [comps, points, ao]."""
    groups, at, T = tables
    cols = [[] for _ in range(comps)]
    for l, nuc, g, c, _ in groups:
        d = r[:, None, :] - R[nuc][None, :, :]
        u = (d * d).sum(-1)
        x = g[None] * u[..., None]
        e = torch.where(x < T, c[None] * torch.exp(-x), torch.zeros_like(x))
        g0 = e.sum(-1)
        if comps > 1:
            g1 = -(e * g[None]).sum(-1)
            g2 = (e * (g * g)[None]).sum(-1)
            radial = (4 * l + 6) * g1 + 4.0 * u * g2
        one, zero = torch.ones_like(u), torch.zeros_like(u)
        pw = []  # pw[axis][k]: k-th power
        for i in range(3):
            t = d[..., i]
            pw.append([one, t, t * t, t * t * t])

        def poly(axis, n, order):
            f = 1
            for k in range(order):
                f *= n - k
            return zero if n < order else f * pw[axis][n - order]

        for a in range(l, -1, -1):
            for b in range(l - a, -1, -1):
                k = l - a - b
                m = math.sqrt(_dfact(2 * l - 1) / (_dfact(2 * a - 1) * _dfact(2 * b - 1) * _dfact(2 * k - 1)))
                X, Y, Z = ([poly(i, n, o) for o in range(3)] for i, n in enumerate((a, b, k)))
                p = X[0] * Y[0] * Z[0]
                cols[0].append(m * p * g0)
                if comps > 1:
                    cols[1].append(m * (X[1] * Y[0] * Z[0] * g0 + 2.0 * d[..., 0] * p * g1))
                    cols[2].append(m * (X[0] * Y[1] * Z[0] * g0 + 2.0 * d[..., 1] * p * g1))
                    cols[3].append(m * (X[0] * Y[0] * Z[1] * g0 + 2.0 * d[..., 2] * p * g1))
                    lap = X[2] * Y[0] * Z[0] + X[0] * Y[2] * Z[0] + X[0] * Y[0] * Z[2]
                    cols[4].append(m * (lap * g0 + p * radial))
    return torch.stack([torch.cat(v, dim=1)[:, at] for v in cols])


def _exact_mo(mol, bits, C, r, R, w=None, comps=5):
    """mo_vgl [points, comps, mo] and, with weights, the three gradients."""
    tables = _shell_tables(mol, bits)
    P, N, K = r.shape[0], C.shape[0], C.shape[1]
    step = max(64, int(3e8 // (200 * K)) if w is not None else int(1e9 // (60 * K)))
    mo = torch.empty((P, comps, N), dtype=torch.float64, device=DEV)
    dC, dR, dr = torch.zeros_like(C), torch.zeros_like(R), torch.zeros_like(r)
    for lo in range(0, P, step):
        rr = r[lo: lo + step]
        if w is None:
            ao = _ao(tables, rr, R, comps)
        else:
            with torch.enable_grad():
                rr, RR = rr.detach().requires_grad_(True), R.detach().requires_grad_(True)
                ao = _ao(tables, rr, RR)
            ww = w[lo: lo + step].double()
            bar = torch.stack([ww[:, c].contiguous() @ C for c in range(5)])
            g = torch.autograd.grad(ao, (rr, RR), grad_outputs=bar)
            dr[lo: lo + step] = g[0]
            dR += g[1]
            ao = ao.detach()
            for c in range(5):
                dC += ww[:, c].t().contiguous() @ ao[c]
        for c in range(comps):
            mo[lo: lo + step, c] = ao[c] @ C.t()
    return mo, {"d_coef": dC, "d_elec": dr, "d_nucl": dR}


def _exact_jastrow(case, d):
    nord, kappa = case["nord"], d["kappa"]
    R, c = torch.from_numpy(d["mol"].pos).to(DEV), torch.from_numpy(d["c"]).to(DEV)
    out = []
    ne = d["r"].shape[1]
    step = max(1, int(2e7 // (ne * ne)))
    eye = torch.eye(ne, dtype=torch.bool, device=DEV)
    for lo in range(0, d["r"].shape[0], step):
        r = d["r"][lo: lo + step]
        rt = torch.exp(-kappa * (r[:, :, None, :] - r[:, None, :, :]).square().sum(-1).sqrt())
        Rt = torch.exp(-kappa * (r[:, :, None, :] - R[None, None]).square().sum(-1).sqrt())
        J, t = torch.zeros(r.shape[0], dtype=torch.float64, device=DEV), 0
        P = {}
        for p in range(2, nord + 1):
            for k in range(p):
                for l in range(p - k - (2 if k == 0 else 0) + 1):
                    if (p - k - l) % 2:
                        continue
                    m = (p - k - l) // 2
                    if (k, m) not in P:
                        power = rt.pow(k).masked_fill(eye, 0.0)
                        P[k, m] = torch.bmm(power, Rt.pow(m).contiguous())
                    J += ((Rt.pow((p - k + l) // 2) * P[k, m]).sum(1) * c[t]).sum(-1)
                    t += 1
        out.append(J)
    return torch.cat(out)


@torch.no_grad()
def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "det":
        det = torch.linalg.det(d["a"])
        return [det, torch.linalg.inv(d["a"]) * det[:, None, None]]
    if kind == "jastrow":
        return _exact_jastrow(case, d)
    if kind == "batch":
        mols = d["mols"]
        out, outs = _flat([tuple(m["w"].shape) for m in mols], torch.float64)
        flat = {k: _flat(sh, torch.float64) for k, sh in (
            ("d_coef", [m["C"].shape for m in mols]), ("d_elec", [tuple(m["r"].shape) for m in mols]),
            ("d_nucl", [m["mol"].pos.shape for m in mols]))}
        for i, m in enumerate(mols):
            mo, g = _exact_mo(m["mol"], case["bits"], torch.from_numpy(m["C"]).to(DEV), m["r"].reshape(-1, 3),
                              torch.from_numpy(m["mol"].pos).to(DEV), m["w"].reshape(-1, 5, m["C"].shape[0]))
            outs[i].copy_(mo.view(outs[i].shape))
            for k, v in g.items():
                flat[k][1][i].copy_(v.view(flat[k][1][i].shape))
        return [out, {k: v[0] for k, v in flat.items()}]
    shape = d["r"].shape
    r = d["r"].double().reshape(-1, 3)
    if kind == "train":
        C, R = d["C"].double(), d["R"].double()
    else:
        C, R = torch.from_numpy(d["C"]).to(DEV), torch.from_numpy(d["mol"].pos).to(DEV)
    if kind == "density":
        n = case["occupied"]
        mo, _ = _exact_mo(d["mol"], case["bits"], C[:n].contiguous(), r, R, comps=1)
        return (2.0 * mo[:, 0].square()).sum(-1).view(shape[:2])
    if kind == "value":
        mo, _ = _exact_mo(d["mol"], case["bits"], C, r, R, comps=1)
        return mo.view(*shape[:2], -1)
    w = d["w"].reshape(-1, 5, C.shape[0]) if "w" in d else None
    mo, g = _exact_mo(d["mol"], case["bits"], C, r, R, w)
    mo = mo.view(*shape[:2], 5, -1)
    g["d_elec"] = g["d_elec"].view(shape)
    if kind == "forward":
        return mo
    if kind == "train":
        return [g["d_coef"], g["d_nucl"], g["d_elec"]]
    return [mo, g]
