"""Timed cases of the framework's main path: layered-battery systems on the GPU.

A case is one call (or one short sequence of calls) of a program that holds a
multiphysics CSR system on the device: a preconditioner application, a solve,
a Newton or time step (new matrix values, then a solve), or a training step
(new values, solve, adjoint solve, gradients).  The systems are the layered
batteries of synth/synth.c (five layers, two potentials, a pressure and one or
three species on a 2D or 3D grid), assembled here on the device from torch's
generator so that every seed gives other coefficients and right-hand sides.
"""
import math

import torch

import paper_2602_13079_amd as H

# bracket codes of ((phi_s, phi_e), ((p), (species...)))
TREES = {1: [-1, -1, 0, 1, -2, -1, 2, -2, -1, 3, -2, -2], 3: [-1, -1, 0, 1, -2, -1, 2, -2, -1, 3, 4, 5, -2, -2]}
# two children only: the voltage and the non-voltage block of the nested form
TREES2 = {1: [-1, -1, 0, 1, -2, -1, 2, 3, -2, -2], 3: [-1, -1, 0, 1, -2, -1, 2, 3, 4, 5, -2, -2]}
DIFF = (1e-3, 5e-4, 2e-3)
# Arnoldi steps that such systems take, forward and adjoint (for work())
STEPS = {False: 16, True: 28}


def case(name, op, nx, ny, nz, species=1, mixed=True, transpose=False, leaf="amg", nested=False, degree=2):
    c = dict(op=op, nx=nx, ny=ny, nz=nz, species=species, mixed=mixed, transpose=transpose, leaf=leaf,
             nested=nested, degree=degree)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one preconditioner application inside another code's Krylov loop, on a coarse 2D
        # cross-section; every field is one dense-solved level, so launches and latency are all there is
        case("apply 4k mixed", "apply", 32, 32, 0),
        # a whole small solve: 2D prototypes and parameter studies run thousands of these
        case("solve 4k fp64", "solve", 32, 32, 0, mixed=False),
        # an ordinary application on a ragged 3D grid (no dimension a multiple of a block size)
        case("apply 1M mixed ragged", "apply", 67, 61, 63),
        # the adjoint preconditioner in double precision on the six-field system of the differentiation workload
        case("apply 5.3M fp64 adjoint", "apply", 96, 96, 96, species=3, mixed=False, transpose=True),
        # the ordinary 3D solve
        case("solve 1M mixed", "solve", 64, 64, 64),
        # an axisymmetric (2D) cell, as most battery models are, double precision, odd sizes, adjoint system
        case("solve 1.4M 2D fp64 adjoint", "solve", 701, 513, 0, mixed=False, transpose=True),
        # the benchmark's solve
        case("solve 4.2M mixed", "solve", 128, 128, 64),
        # a Newton or time step: new values on the same pattern, then the solve
        case("step 4.2M mixed", "step", 128, 128, 64),
        # the same for a small ragged system in double precision, species by DD(0)-ILU(0) as the paper has them
        case("step 262k fp64 ilu", "step", 41, 37, 43, mixed=False, leaf="ilu"),
        # a training step of the differentiation workload: new values, solve, adjoint solve, value gradient
        case("train 5.3M mixed", "train", 96, 96, 96, species=3),
        # the paper's nested form (inner GMRES on the voltage and non-voltage blocks)
        case("solve 1M mixed nested", "solve", 61, 67, 59, nested=True),
        # the largest system: a full 3D battery of 25 million unknowns, six fields, planes of 256 x 256 cells
        case("solve 25M mixed", "solve", 256, 256, 64, species=3),
    ]


def draw(rng):
    """One more case: any operation, precision, direction and leaf over grids from 4 thousand unknowns up."""
    op = rng.choice(["apply", "apply", "solve", "solve", "step", "train"])
    species = rng.choice([1, 1, 3])
    two_d = rng.random() < 0.35
    mixed = rng.random() < 0.65
    transpose = op in ("apply", "solve") and rng.random() < 0.4
    leaf = rng.choice(["amg", "amg", "amg", "amg", "ilu", "jacobi"])
    nested = op == "solve" and leaf == "amg" and rng.random() < 0.15
    degree = 4 if leaf == "amg" and not nested and rng.random() < 0.15 else 2
    most = 1.5e6 if (two_d or nested or leaf == "ilu") else 6e6  # unknowns
    dof = math.exp(rng.uniform(math.log(4e3), math.log(most)))
    cells = dof / (3 + species)
    dim = 2 if two_d else 3
    side = cells ** (1.0 / dim)
    a = side * math.exp(rng.uniform(-0.3, 0.3))
    b = side * math.exp(rng.uniform(-0.3, 0.3)) if dim == 3 else cells / a
    nx, ny = max(5, round(a)), max(5, round(b))
    nz = max(5, round(cells / (nx * ny))) if dim == 3 else 0
    return case("", op, nx, ny, nz, species, mixed, transpose, leaf, nested, degree)


def _sizes(c):
    cells = c["nx"] * c["ny"] * max(1, c["nz"])
    faces = 6 if c["nz"] else 4
    nf = 3 + c["species"]
    n = cells * nf
    # entries per cell: full stencils, less the identity rows and with the couplings, to a few percent
    block = (nf - 2) * (faces + 1) + 0.8 * (faces + 1) * 2
    nnz = cells * (block + 1.2 + c["species"] * (0.8 * (faces + 1) + 0.6))
    return n, nnz, cells * block


def work(c):
    """The operator and the field blocks once per preconditioned step, vectors once; a rebuild reads the values
    once and writes each block, its transpose and its FP32 copy once."""
    n, nnz, block = _sizes(c)
    t = 4 if c["mixed"] else 8
    apply_b, apply_f = 8 * n * 2 + block * (t + 2), 2 * block * 4
    if c["op"] == "apply":
        return {"bytes": apply_b, "flops": apply_f}

    def solve(transpose):
        m = STEPS[transpose]
        step_b = apply_b + nnz * 10 + n * (t + 8)
        return m * step_b + 8 * n * m * m, m * (apply_f + 2 * nnz) + 4 * n * m * m

    b, f = solve(c["transpose"])
    if c["op"] in ("step", "train"):
        b, f = b + 8 * nnz + 2 * 12 * block, f + 6 * block
    if c["op"] == "train":
        b2, f2 = solve(True)
        b, f = b + b2 + 12 * nnz + 24 * n, f + f2 + nnz
    return {"bytes": float(b), "flops": float(f)}


# ------------------------------------------------------------------ inputs
def _harm(a, b):
    s = a + b
    return torch.where((a > 0) & (b > 0), 2.0 * a * b / torch.where(s > 0, s, torch.ones_like(s)),
                       torch.zeros_like(s))


def _rows(c, seed, dev):
    """The system by fields: for field f the list of its entries (cell offset, column's field, values, mask) in
    ascending column order, one value per cell; and the generator, for the vectors."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    dim = 3 if nz else 2
    dims = (nx, ny, nz)[:dim]
    cells = math.prod(dims)
    strides = (1, nx, nx * ny)[:dim]
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    kw = dict(device=dev, dtype=torch.float64)
    cell = torch.arange(cells, device=dev)
    x = [(cell // strides[d]) % dims[d] for d in range(dim)]
    t10, two_n = (2 * x[-1] + 1) * 10, 2 * dims[-1]
    layer = (t10 >= two_n).long() + (t10 >= 4 * two_n).long() + (t10 >= 6 * two_n).long() + (t10 >= 9 * two_n).long()
    coll, sep = (layer == 0) | (layer == 4), layer == 2
    elec = (layer == 1) | (layer == 3)
    perm = 1e-3 * 100.0 ** torch.rand(cells, generator=g, **kw)
    j0 = 0.1 * 100.0 ** torch.rand(cells, generator=g, **kw)
    pt = torch.zeros(cells, **kw)
    modes = torch.rand(4, 5, generator=g, **kw).tolist()
    for amp, k0, k1, k2, ph in modes:
        arg = torch.full((cells,), 2 * math.pi * ph, **kw)
        for d, k in zip(range(dim), (k0, k1, k2)):
            arg += 2 * math.pi * (1 + int(3 * k)) * (x[d].double() + 0.5) / dims[d]
        pt += (2 * amp - 1) * torch.sin(arg)
    zero = torch.zeros(cells, **kw)
    k_s = torch.where(coll, 1e4, torch.where(sep, 0.0, 1e2)).to(torch.float64)
    k_e = torch.where(coll, 0.0, 1.0).to(torch.float64)
    k = torch.where(elec, j0, zero)
    faces = [(d, s) for d in reversed(range(dim)) for s in (-1,)] + [(d, 1) for d in range(dim)]
    near = {}
    for d, s in faces:
        has = x[d] > 0 if s < 0 else x[d] < dims[d] - 1
        near[d, s] = (has, (cell + s * strides[d]).clamp_(0, cells - 1))

    def trans(kap):
        out = {}
        for q, (has, nb) in near.items():
            out[q] = torch.where(has, _harm(kap, kap[nb]), zero)
        return out

    t_e = trans(k_e)
    rows = []
    every = torch.ones(cells, device=dev, dtype=torch.bool)
    for f in range(3 + c["species"]):
        kap = k_s if f == 0 else k_e if f == 1 else perm if f == 2 else torch.full((cells,), DIFF[f - 3], **kw)
        tr = t_e if f == 1 else trans(kap)
        diag = zero.clone()
        for v in tr.values():
            diag += v
        if f == 0:
            diag += torch.where(x[-1] == 0, 2 * kap, zero)
        if f == 2:
            diag += torch.where(x[-1] == dims[-1] - 1, 2 * kap, zero)
        own, mig = {}, {}
        for q, (has, nb) in near.items():
            if f < 3:
                own[q] = (-tr[q], tr[q] > 0)
            else:
                u = pt - pt[nb]
                diag += torch.where(has, u.clamp(min=0), zero)
                own[q] = (torch.where(has, -tr[q] - (-u).clamp(min=0), zero), has)
                mig[q] = (-0.1 * t_e[q], t_e[q] > 0)
        if f >= 3:
            diag += 100.0
        if f == 0:
            diag = torch.where(sep, torch.ones_like(diag), diag + k)
        if f == 1:
            diag = torch.where(coll, torch.ones_like(diag), diag + k)
        entries = []

        def side(sign):
            for d, s in faces:
                if s == sign:
                    if f >= 3:
                        entries.append((s * strides[d], 1) + mig[d, s])
                    entries.append((s * strides[d], f) + own[d, s])

        side(-1)
        if f == 0:
            entries += [(0, 0, diag, every), (0, 1, -k, elec)]
        elif f == 1:
            entries += [(0, 0, -k, elec), (0, 1, diag, every)]
        elif f == 2:
            entries.append((0, 2, diag, every))
        else:
            te = sum(t_e.values())
            entries += [(0, 0, -0.5 * k, elec), (0, 1, torch.where(coll, zero, 0.5 * k + 0.1 * te), ~coll),
                        (0, f, diag, every)]
        side(1)
        rows.append(entries)
    return rows, cells, g


def _shift(n, off):
    """Slices (at the row's cell, at the column's cell) for a cell offset."""
    return (slice(0, n - off), slice(off, n)) if off >= 0 else (slice(-off, n), slice(0, n + off))


def _vectors(c, rows, cells, g, dev):
    """x_star, b = A x_star, lam_star, A^T lam_star (each entry in [-1, 1] for the starred ones)."""
    nf = len(rows)
    xs, lam = (2 * torch.rand(cells, nf, generator=g, device=dev, dtype=torch.float64) - 1 for _ in range(2))
    b, gt = torch.zeros_like(xs), torch.zeros_like(lam)
    for f, entries in enumerate(rows):
        for off, ft, v, mask in entries:
            here, there = _shift(cells, off)
            v = torch.where(mask, v, torch.zeros_like(v))[here]
            b[here, f] += v * xs[there, ft]
            gt[there, ft] += v * lam[here, f]
    return xs.view(-1), b.view(-1), lam.view(-1), gt.view(-1)


def _csr(rows, cells, dev):
    nf = len(rows)
    count = torch.stack([sum(m.to(torch.int32) for _, _, _, m in e) for e in rows], 1).view(-1)
    rowptr = torch.zeros(cells * nf + 1, device=dev, dtype=torch.int64)
    torch.cumsum(count, 0, out=rowptr[1:])
    nnz = int(rowptr[-1])
    col = torch.empty(nnz, device=dev, dtype=torch.int32)
    val = torch.empty(nnz, device=dev, dtype=torch.float64)
    cell = torch.arange(cells, device=dev)
    for f, entries in enumerate(rows):
        at = rowptr[:-1].view(cells, nf)[:, f].clone()
        for off, ft, v, mask in entries:
            p = at[mask]
            col[p] = ((cell[mask] + off) * nf + ft).to(torch.int32)
            val[p] = v[mask]
            at += mask
    return rowptr.to(torch.int32), col, val


def _system(c, seed, with_csr=True):
    dev = torch.device("cuda")
    rows, cells, g = _rows(c, seed, dev)
    xs, b, lam, gt = _vectors(c, rows, cells, g, dev)
    csr = _csr(rows, cells, dev) if with_csr else None
    field = torch.arange(len(rows), device=dev, dtype=torch.int32).repeat(cells) if with_csr else None
    return csr, field, xs, b, lam, gt


def _options(c):
    ns = c["species"]
    o = dict(precision=int(c["mixed"]), cheb_degree=c["degree"])
    if c["leaf"] != "amg":
        o["field_leaf"] = [0, 0, 0] + [2 if c["leaf"] == "ilu" else 1] * ns
    if c["nested"]:  # the paper's settings
        o.update(nested=1, restart=5, field_cheb_degree=[4, 4])
    return o, (TREES2 if c["nested"] else TREES)[ns]


def prepare(c, seed):
    (rowptr, col, val), field, xs, b, lam, gt = _system(c, seed)
    opts, tree = _options(c)
    s = dict(op=c["op"], transpose=c["transpose"], val=val, rhs=gt if c["transpose"] else b, g=gt)
    if c["op"] == "train":
        s["val"].requires_grad_(True)
        s["rhs"] = s["rhs"].requires_grad_(True)
    with torch.no_grad():
        s["solver"] = H.Solver(rowptr, col, val, field, 3 + c["species"], tree, **opts)
    return s


def run(s):
    solver = s["solver"]
    if s["op"] == "apply":
        return solver.apply(s["rhs"], transpose=s["transpose"])
    if s["op"] == "solve":
        return solver.solve(s["rhs"], transpose=s["transpose"])[:3]  # the solution, the status, the steps taken
    if s["op"] == "step":
        solver.set_values(s["val"])
        return solver.solve(s["rhs"])[:3]
    solver.set_values(s["val"])
    x = H.hbgs_solve(s["val"], s["rhs"], solver)
    grads = torch.autograd.grad(x, (s["val"], s["rhs"]), s["g"])
    return x.detach(), grads[0], grads[1]


def exact(c, seed):
    if c["op"] == "apply":
        # one dense-solved level per field: the block triangular solve itself; a whole hierarchy has no such form
        if c["leaf"] != "amg" or c["nx"] * c["ny"] * max(1, c["nz"]) > 2000:
            return None
        (rowptr, col, val), field, _, b, _, gt = _system(c, seed)
        n, nf = field.numel(), 3 + c["species"]
        a = torch.zeros(n, n, device=val.device, dtype=torch.float64)
        row = torch.repeat_interleave(torch.arange(n, device=val.device), (rowptr[1:] - rowptr[:-1]).long())
        a[row, col.long()] = val
        a, r = (a.t().contiguous(), gt) if c["transpose"] else (a, b)
        z = torch.zeros_like(r)
        for f in (reversed(range(nf)) if c["transpose"] else range(nf)):
            i = torch.nonzero(field == f).view(-1)
            z[i] = torch.linalg.solve(a[i][:, i], r[i] - a[i] @ z)
        return z
    csr, _, xs, _, lam, _ = _system(c, seed, with_csr=c["op"] == "train")
    if c["op"] != "train":
        return (lam if c["transpose"] else xs), None, None
    rowptr, col, _ = csr
    row = torch.repeat_interleave(torch.arange(xs.numel(), device=xs.device), (rowptr[1:] - rowptr[:-1]).long())
    return xs, -lam[row] * xs[col.long()], lam
