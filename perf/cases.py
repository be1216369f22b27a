"""Cases that time the library's public entry points over the range of its use.

A case is a dict of plain values:

* ``op``     what a pass runs:
    - ``step``    binning, density, solve, backward, forces, call by call (a geometry step)
    - ``replay``  the same step, with solve and backward as one call, recorded once as a HIP graph and replayed
    - ``grad``    the autograd function, forward and backward
    - ``solve``   potential and energy of a given density;  ``energy``  the energy alone
    - ``noalloc`` potential and energy without a bound workspace
* ``cell``   ``diag`` (edges la, lb, lc), ``skew`` (the same edges, sheared), ``fcc`` (rows la (0, 1, 1), ...)
* ``na, nb, nc``  the grid;  ``prec``  fp32 or fp64;  ``tuned``  whether the program has the plan tuned first
* ``sites``  ``diamond`` (lattice sites and thermal displacements) or ``uniform``, with ``atoms`` atoms
* ``nprob, shapes``  in place of a cell and a grid: a batch of that many cells, drawn as the batched workload draws them
"""
import math

import numpy as np
import torch

from paper_1209_4506_amd import hartree, inputs

A_CONV = 53.93 / 8  # diamond's conventional cell (Bohr)
SPACING = 0.1498    # grid spacing of the 360^3 workload (Bohr)
DENSITY = 8 / A_CONV**3  # atoms per cubic Bohr
LENGTHS = sorted({2**i * 3**j * 5**k * 7**m for i in range(11) for j in range(7) for k in range(5) for m in range(4)
                  if 2 <= 2**i * 3**j * 5**k * 7**m <= 1024})


def diag(op, na, nb, nc, edges, prec, sites="uniform", atoms=0, tuned=False, **more):
    return dict(op=op, cell="diag", na=na, nb=nb, nc=nc, la=float(edges[0]), lb=float(edges[1]), lc=float(edges[2]),
                prec=prec, sites=sites, atoms=atoms, tuned=tuned, **more)


def listed():
    return [
        # the smallest use: a molecule in a box, differentiated; launches and host work decide
        diag("grad", 32, 32, 32, (10, 10, 10), "fp32", atoms=8, name="grad 32^3 fp32"),
        # a small ragged cell in double precision, every call of the step on its own
        diag("step", 45, 27, 50, (12.0, 7.5, 14.0), "fp64", atoms=37, name="step 45x27x50 fp64"),
        # potential and energy of a mid-size cell whose lengths are odd 7-smooth numbers, on a plan as created
        diag("solve", 135, 168, 189, (20.2, 25.2, 28.3), "fp32", name="solve 135x168x189 fp32"),
        # a caller that may not allocate (a serving loop): the solve on the library's own scratch
        diag("noalloc", 192, 192, 192, (28.8, 28.8, 28.8), "fp32", name="noalloc 192^3 fp32"),
        # an ordinary periodic solid, 512 atoms, on a plan as created
        diag("step", 180, 180, 180, (26.96,) * 3, "fp32", "diamond", 512, name="step 180^3 fp32"),
        # cells that are not orthorhombic: diamond in its primitive cell, and a sheared cell in double precision
        dict(op="step", cell="fcc", na=160, nb=160, nc=160, la=4 * A_CONV, lb=4 * A_CONV, lc=4 * A_CONV, prec="fp32",
             sites="diamond", atoms=1024, tuned=False, name="step fcc 160^3 fp32"),
        dict(op="step", cell="skew", na=72, nb=80, nc=90, la=14.4, lb=16.0, lc=18.0, prec="fp64", sites="uniform",
             atoms=108, tuned=False, name="step skew 72x80x90 fp64"),
        # 24 uneven cells in one plan, replayed (the batched benchmark workload)
        dict(op="replay", nprob=24, shapes=1209, prec="fp32", tuned=True, name="replay batched24 fp32"),
        # 4,096 atoms on 360^3: the headline workload as it is replayed, and its double precision step
        diag("replay", 360, 360, 360, (53.93,) * 3, "fp32", "diamond", 4096, True, name="replay 360^3 fp32"),
        diag("step", 360, 360, 360, (53.93,) * 3, "fp64", "diamond", 4096, True, name="step 360^3 fp64"),
        # 16,384 atoms on a grid with factors of 7 at a coarser spacing
        diag("step", 420, 420, 210, (16 * A_CONV, 16 * A_CONV, 8 * A_CONV), "fp32", "diamond", 16384, True,
             name="step 420x420x210 fp32"),
        # the largest: 32,768 atoms on 1024^3
        diag("step", 1024, 1024, 1024, (150.0,) * 3, "fp32", "uniform", 32768, True, name="step 1024^3 fp32"),
    ]


def draw(rng):
    """One more case: cells from molecules in a box to large solids, with about the atoms per volume of a solid."""
    kind = rng.choice(["small", "diag", "diag", "solve", "skew", "batch"])
    prec = rng.choice(["fp32", "fp32", "fp64"])
    if kind == "batch":
        return dict(op=rng.choice(["replay", "step"]), nprob=rng.randint(2, 24), shapes=rng.randint(1300, 9000),
                    prec="fp32", tuned=rng.random() < 0.5)
    lo, hi = {"small": (24, 72), "diag": (72, 480), "solve": (48, 480), "skew": (32, 160)}[kind]
    base = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    n = [min(LENGTHS, key=lambda m, t=base * rng.uniform(0.75, 1.3): abs(m - t)) for _ in range(3)]
    h = SPACING * rng.uniform(0.9, 1.6)
    edges = [m * h for m in n]
    while min(edges) < 7.0:  # a box of atoms is at least this wide
        edges = [e * 1.1 for e in edges]
    atoms = max(2, int(DENSITY * edges[0] * edges[1] * edges[2] * rng.uniform(0.5, 1.5)))
    if kind == "solve":
        op = rng.choice(["solve", "energy", "noalloc"])
        if n[0] * n[1] * n[2] > (200 if prec == "fp32" else 150) ** 3 and op == "noalloc":
            op = "solve"
        return diag(op, *n, edges, prec, tuned=rng.random() < 0.3)
    if kind == "skew":
        return dict(diag("step", *n, edges, prec, "uniform", atoms), cell="skew")
    op = rng.choice(["grad", "step"]) if kind == "small" else rng.choice(["step", "replay"])
    return diag(op, *n, edges, prec, "uniform", atoms, rng.random() < (0.0 if kind == "small" else 0.5))


def problems(case):
    """Per problem: (cell rows, grid, atoms)."""
    if "nprob" in case:
        out = []
        for p in range(case["nprob"]):
            rng = np.random.default_rng(case["shapes"] * 100 + p)
            edges = rng.uniform(8.0, 40.0, 3)
            dims = tuple(int(v) for v in rng.choice(inputs.BATCH_DIMS, 3))
            out.append((np.diag(edges), dims, int(rng.integers(16, 513))))
        return out
    e = np.array([case["la"], case["lb"], case["lc"]])
    if case["cell"] == "diag":
        cell = np.diag(e)
    elif case["cell"] == "fcc":
        cell = e[:, None] * np.array([[0.0, 1.0, 1.0], [1.0, 0.0, 1.0], [1.0, 1.0, 0.0]])
    else:
        cell = np.array([[e[0], 0.0, 0.0], [0.25 * e[1], e[1], 0.0], [-0.15 * e[2], 0.2 * e[2], e[2]]])
    return [(cell, (case["na"], case["nb"], case["nc"]), case["atoms"])]


def atoms_of(case, seed):
    """Positions, charges and widths of every atom, problem by problem (host arrays)."""
    rng = np.random.default_rng([seed, 1209])
    pos, Z, sigma = [], [], []
    for cell, _, n in problems(case):
        if case.get("sites") == "diamond":
            if case["cell"] == "fcc":
                reps, basis = [int(round((n / 2) ** (1 / 3)))] * 3, np.array([[0.0, 0.0, 0.0], [0.25, 0.25, 0.25]])
            else:
                reps, basis = [int(round(v / A_CONV)) for v in np.diag(cell)], inputs._DIAMOND_BASIS
            at = np.stack(np.meshgrid(*[np.arange(r) for r in reps], indexing="ij"), -1).reshape(-1, 1, 3)
            frac = ((at + basis) / np.array(reps)).reshape(-1, 3)
            pos.append(frac @ cell + rng.normal(0.0, 0.05, (n, 3)))
            Z.append(np.full(n, 4.0))
            sigma.append(np.full(n, 0.8))
        else:
            pos.append(rng.random((n, 3)) @ cell)
            Z.append(rng.choice(np.array([1.0, 4.0, 6.0]), n))
            sigma.append(rng.uniform(0.6, 1.0, n))
    return np.concatenate(pos), np.concatenate(Z), np.concatenate(sigma)


def fields(case, seed, device):
    """Per problem: a density (``solve`` and its kin) or the loss weights times dV, in the plan's type."""
    out = []
    for p, (cell, dims, _) in enumerate(problems(case)):
        gen = torch.Generator(device=device)
        gen.manual_seed(1000003 * seed + p)
        g = torch.empty(dims, dtype=torch.float32 if case["prec"] == "fp32" else torch.float64, device=device)
        g.normal_(generator=gen)
        if case["op"] in ("solve", "energy", "noalloc"):
            # a neutral density: smooth waves over the noise of the grid
            g *= 0.01
            for x in range(3):
                t = torch.arange(dims[x], device=device, dtype=torch.float64) * (2 * math.pi / dims[x])
                wave = (torch.cos(t) + 0.5 * torch.sin(2 * t)).to(g.dtype)
                g += wave.reshape([-1 if y == x else 1 for y in range(3)])
        else:
            g *= abs(np.linalg.det(cell)) / math.prod(dims)
        out.append(g)
    return out


class State:
    """What the program holds: the plan, the inputs and the buffers it reuses."""


def prepare(case, seed):
    s = State()
    probs = problems(case)
    batched = "nprob" in case
    cells = np.stack([p[0] for p in probs])
    dims = np.array([p[1] for p in probs])
    device = torch.device("cuda:0")
    s.case = case
    s.counts = [p[2] for p in probs] if batched else None
    s.plan = hartree.Plan(cells if batched else cells[0], dims if batched else dims[0], precision=case["prec"],
                          device=device, max_atoms=max(1, sum(p[2] for p in probs)), bind=case["op"] != "noalloc")
    if case["tuned"] and case["op"] != "noalloc":
        s.plan.tune(reps=5)
    grids = fields(case, seed, device)
    grid = torch.cat([g.reshape(-1) for g in grids]) if batched else grids[0]
    del grids
    s.V = s.plan.empty_grid()
    s.E = torch.empty(len(probs), dtype=torch.float64, device=device)
    if case["op"] in ("solve", "energy", "noalloc"):
        s.rho = grid
        return s
    s.gv = grid
    s.ge = torch.ones(len(probs), dtype=torch.float64, device=device)
    s.pos, s.Z, s.sigma = (torch.tensor(v, device=device) for v in atoms_of(case, seed))
    if case["op"] == "grad":
        s.pos.requires_grad_(True)
        return s
    s.rho, s.grho = s.plan.empty_grid(), s.plan.empty_grid()
    s.gpos = torch.empty((s.pos.shape[0], 3), dtype=torch.float64, device=device)
    if case["op"] == "replay":
        s.plan.capture(lambda: step(s))
        torch.cuda.synchronize()
    return s


def step(s):
    p = s.plan
    token = p.bind_atoms(s.pos, s.Z, s.sigma, atom_counts=s.counts)
    p.splat_bound(token, out=s.rho)
    if s.case["op"] == "replay":
        p.solve_backward(s.rho, grad_v=s.gv, grad_e=s.ge, v=s.V, e_h=s.E, out=s.grho)
    else:
        p.solve(s.rho, v=s.V, e_h=s.E)
        p.backward(grad_v=s.gv, grad_e=s.ge, rho=s.rho, out=s.grho)
    p.splat_adjoint_bound(token, s.grho, out=s.gpos)


def run(s):
    op = s.case["op"]
    if op == "solve":
        return s.plan.solve(s.rho, v=s.V, e_h=s.E)
    if op == "noalloc":
        return s.plan.solve_noalloc(s.rho, s.V, e_h=s.E)
    if op == "energy":
        return (s.plan.energy(s.rho, e_h=s.E),)
    if op == "grad":
        V, E = hartree.hartree(s.pos, s.Z, s.sigma, s.plan, s.counts)
        (gpos,) = torch.autograd.grad([V, E], [s.pos], [s.gv, s.ge])
        return V, E, gpos
    if op == "replay":
        s.plan.replay()
    else:
        step(s)
    return s.rho, s.V, s.E, s.grho, s.gpos


def work(case):
    """Grids and atoms read and written once; 2.5 N log2 N per real transform, the density's and the forces' multiply-adds
    over the points within six widths of each atom."""
    real = 4 if case["prec"] == "fp32" else 8
    nbytes = flops = 0.0
    grids, transforms = {"solve": (2, 2), "noalloc": (2, 2), "energy": (1, 1), "grad": (2, 4)}.get(case["op"], (4, 4))
    for cell, dims, n in problems(case):
        pts = math.prod(dims)
        nbytes += grids * pts * real
        flops += transforms * 2.5 * pts * math.log2(max(2, pts))
        if grids > 2 or case["op"] == "grad":
            nbytes += n * (5 + 3) * 8
            inside = 1.0
            if case.get("cell", "diag") == "diag":
                for x in range(3):
                    inside *= min(dims[x], 12 * 0.8 * dims[x] / cell[x][x])
            else:
                inside = min(float(pts), 4.19 * (6 * 0.8) ** 3 * pts / abs(np.linalg.det(cell)))
            flops += 6 * n * inside
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- in 64 bits
def kernel(cell, dims, i0, i1, device):
    """4 pi / |G|^2 on planes i0 .. i1 of the half spectrum, averaged over the two signs of every Nyquist index."""
    B = 2 * math.pi * np.linalg.inv(cell).T
    idx = [torch.fft.fftfreq(dims[0], 1 / dims[0], dtype=torch.float64, device=device)[i0:i1],
           torch.fft.fftfreq(dims[1], 1 / dims[1], dtype=torch.float64, device=device),
           torch.arange(dims[2] // 2 + 1, dtype=torch.float64, device=device)]
    flipped = [torch.where(2 * v.abs() == d, -v, v) for v, d in zip(idx, dims)]
    plain = np.allclose(cell, np.diag(np.diag(cell)))
    combos = [(0, 0, 0)] if plain else [(a, b, c) for a in (0, 1) for b in (0, 1) for c in (0, 1)]
    K = 0.0
    for pick in combos:
        m = [(flipped if f else idx)[x].reshape([-1 if y == x else 1 for y in range(3)]) for x, f in enumerate(pick)]
        g2 = sum((m[0] * B[0, k] + m[1] * B[1, k] + m[2] * B[2, k]) ** 2 for k in range(3))
        K = K + torch.where(g2 > 0, 4 * math.pi / torch.where(g2 > 0, g2, 1.0), 0.0)
    return K / len(combos)


def poisson(cell, x):
    dims = tuple(x.shape)
    f = torch.fft.rfftn(x)
    for i in range(0, dims[0], 32):
        f[i:i + 32] *= kernel(cell, dims, i, min(dims[0], i + 32), x.device)
    return torch.fft.irfftn(f, s=dims)


def factors(cell, dims, pos, sigma, device):
    """Diagonal cells, per axis: the sum over images of g = exp(-d^2 / 2 sigma^2) and of g d, atoms x points."""
    out = []
    for x in range(3):
        L = cell[x][x]
        r = torch.arange(dims[x], dtype=torch.float64, device=device) * (L / dims[x])
        d0 = r[None, :] - (pos[:, x] % L)[:, None]
        reach = int(math.ceil(10.0 * float(sigma.max()) / L)) + 1
        g, gd = torch.zeros_like(d0), torch.zeros_like(d0)
        for k in range(-reach, reach + 1):
            d = d0 + k * L
            e = torch.exp(-d * d / (2 * sigma[:, None] ** 2))
            g += e
            gd += e * d
        out.append((g, gd))
    return out


def windows(cell, dims, pos, sigma):
    """Other cells, atom by atom: grid indices (flat, wrapped) and displacements of the points within ten widths."""
    device = pos.device
    A = torch.tensor(cell, device=device)
    inv = torch.linalg.inv(A.cpu()).to(device)
    frac = (pos @ inv).cpu()
    B = np.linalg.inv(cell).T
    for a in range(pos.shape[0]):
        ix = []
        for x in range(3):
            ext = 10.0 * float(sigma[a]) * np.linalg.norm(B[x]) * dims[x]
            c = float(frac[a, x]) * dims[x]
            ix.append(torch.arange(math.ceil(c - ext), math.floor(c + ext) + 1, device=device))
        d = sum((ix[x].double() / dims[x]).reshape([-1 if y == x else 1 for y in range(3)] + [1]) * A[x] for x in range(3))
        flat = ((ix[0] % dims[0])[:, None, None] * dims[1] + (ix[1] % dims[1])[None, :, None]) * dims[2] + \
            (ix[2] % dims[2])[None, None, :]
        yield a, flat.reshape(-1), (d - pos[a]).reshape(-1, 3)


def density(cell, dims, pos, Z, sigma):
    w = Z * (2 * math.pi * sigma**2) ** -1.5
    rho = torch.zeros(dims, dtype=torch.float64, device=pos.device)
    if np.allclose(cell, np.diag(np.diag(cell))):
        (gx, _), (gy, _), (gz, _) = factors(cell, dims, pos, sigma, pos.device)
        for i in range(dims[0]):
            rho[i] = torch.matmul(((w * gx[:, i])[:, None] * gy).t().contiguous(), gz)
    else:
        for a, flat, d in windows(cell, dims, pos, sigma):
            rho.view(-1).index_add_(0, flat, w[a] * torch.exp(-(d * d).sum(1) / (2 * sigma[a] ** 2)))
    return rho - Z.sum() / abs(np.linalg.det(cell))


def forces(cell, dims, pos, Z, sigma, grad):
    w = Z * (2 * math.pi * sigma**2) ** -1.5 / sigma**2
    out = torch.zeros_like(pos)
    if np.allclose(cell, np.diag(np.diag(cell))):
        (gx, dx), (gy, dy), (gz, dz) = factors(cell, dims, pos, sigma, pos.device)
        gzt, dzt = gz.t().contiguous(), dz.t().contiguous()
        gyt, dyt = gy.t().contiguous(), dy.t().contiguous()
        for i in range(dims[0]):
            s = torch.matmul(grad[i], gzt)
            row = (s * gyt).sum(0)
            out[:, 0] += dx[:, i] * row
            out[:, 1] += gx[:, i] * (s * dyt).sum(0)
            out[:, 2] += gx[:, i] * (torch.matmul(grad[i], dzt) * gyt).sum(0)
    else:
        for a, flat, d in windows(cell, dims, pos, sigma):
            g = grad.reshape(-1)[flat] * torch.exp(-(d * d).sum(1) / (2 * sigma[a] ** 2))
            out[a] = (g[:, None] * d).sum(0)
    return w[:, None] * out


def exact(case, seed):
    device = torch.device("cuda:0" if torch.cuda.is_available() else "cpu")
    probs, grids = problems(case), fields(case, seed, device)
    alone = case["op"] in ("solve", "energy", "noalloc")
    if not alone:
        pos, Z, sigma = (torch.tensor(v, device=device) for v in atoms_of(case, seed))
    got, at = [], 0
    for (cell, dims, n), field in zip(probs, grids):
        dv = abs(np.linalg.det(cell)) / math.prod(dims)
        mine = slice(at, at + n)
        rho = field.double() if alone else density(cell, dims, pos[mine], Z[mine], sigma[mine])
        V = poisson(cell, rho)
        E = 0.5 * dv * (rho * V).sum()
        if alone:
            got.append((V, E))
            continue
        grad = poisson(cell, field.double() + dv * rho)
        got.append((rho, V, E, grad, forces(cell, dims, pos[mine], Z[mine], sigma[mine], grad)))
        at += n
    batched = "nprob" in case

    def whole(k, flat):
        parts = [g[k] for g in got]
        return torch.cat([p.reshape(-1) for p in parts]) if flat else parts[0]

    if alone:
        V, E = whole(0, batched), torch.stack([g[1] for g in got])
        return (E,) if case["op"] == "energy" else (V, E)
    E = torch.stack([g[2] for g in got])
    gpos = torch.cat([g[4] for g in got])
    if case["op"] == "grad":
        return whole(1, batched), E, gpos
    return whole(0, batched), whole(1, batched), E, whole(3, batched), gpos
