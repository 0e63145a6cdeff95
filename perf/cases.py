"""Timed cases: what a program that uses this library has it do, through the
library's public entry points, over the sizes, numberings, precisions and
options that it is used with.

Every case is a 7-point finite-volume system on an nx x ny x nz mesh, split
into px x py x pz block ranks that one plan fuses (log-uniform face
coefficients exp(U[ln kappa, 0]), walls on all sides).  `scramble` numbers each
rank's cells at random, as an unstructured mesh's cells are.  The kinds:

  spmv      y = A x, the product by itself (FP64, or the FP32 copy)
  update    one timestep's new coefficients, in device memory per rank, into
            the matrix
  grad      gradient of a loss with respect to every coefficient, from the
            solution and the adjoint solution
  vcycle    one multigrid V-cycle applied to a residual
  solve     one linear solve from x = 0
  timestep  new coefficients and a CG solve that starts from the last step's x
  adjoint   the differentiable solve, forward and backward
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2510_08536_amd as rp
from paper_2510_08536_amd.autograd import repart_solve


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _case(do, n, p, **kw):
    c = dict(do=do, nx=n[0], ny=n[1], nz=n[2], px=p[0], py=p[1], pz=p[2], kappa=1e-2, scramble=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest solve: 32^3 cells of four ranks, constant coefficients; latency and launches
        dict(_case("solve", (32, 32, 32), (1, 1, 4), kappa=1.0, tol=1e-8), name="cg_32"),
        # the pressure solve of a timestep loop at one GPU's share of a small run: 32 ranks
        dict(_case("timestep", (128, 128, 128), (4, 4, 2), tol=1e-8), name="timestep_128"),
        # the largest solve: 64 ranks, FP32 iterations under FP64 refinement
        dict(_case("solve", (256, 256, 256), (4, 4, 4), kappa=1e-3, tol=1e-11, precision="mixed"), name="mixed_256"),
        # multigrid-preconditioned CG, ragged sizes and ranks of unequal cell counts
        dict(_case("solve", (131, 117, 142), (3, 4, 2), tol=1e-8, precond="amg"), name="amg_cg_ragged"),
        # the non-symmetric momentum-type system (upper and lower differ)
        dict(_case("solve", (96, 96, 96), (2, 2, 4), tol=1e-10, method="bicgstab"), name="bicgstab_96"),
        # learning coefficients through the solve: forward, backward
        dict(_case("adjoint", (96, 96, 96), (2, 2, 4), tol=1e-8), name="adjoint_96"),
        # cells numbered without locality (unstructured mesh), 48 ranks
        dict(_case("solve", (100, 90, 95), (4, 4, 3), scramble=True, tol=1e-8), name="cg_scrambled"),
        # the largest coefficient update: 64 ranks' arrays in device memory
        dict(_case("update", (256, 256, 256), (4, 4, 4), kappa=1e-3), name="update_256"),
        # the product alone, largest size, FP64
        dict(_case("spmv", (256, 256, 256), (4, 4, 4), kappa=1e-3, dtype="float64"), name="spmv64_256"),
        # the FP32 copy's product, ragged sizes
        dict(_case("spmv", (201, 150, 177), (5, 3, 2), dtype="float32"), name="spmv32_ragged"),
        # the multigrid by itself, as a preconditioner of a caller's own iteration
        dict(_case("vcycle", (160, 160, 160), (4, 4, 3)), name="vcycle_160"),
        # coefficient gradients of a large system
        dict(_case("grad", (200, 190, 210), (3, 3, 5)), name="grad_200"),
    ]


# cells of a drawn case at least and at most, by kind
_RANGE = {"spmv": (4096, 1 << 24), "update": (4096, 1 << 24), "grad": (4096, 1 << 23), "vcycle": (4096, 1 << 22),
          "solve": (2048, 1 << 21), "timestep": (4096, 1 << 21), "adjoint": (4096, 1 << 20)}


def draw(rng):
    do = rng.choice(["spmv", "update", "grad", "vcycle", "solve", "solve", "solve", "timestep", "adjoint"])
    lo, hi = _RANGE[do]
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    s = n ** (1.0 / 3.0)
    nx = max(4, int(s * math.exp(rng.uniform(-0.4, 0.4))))
    ny = max(4, int(s * math.exp(rng.uniform(-0.4, 0.4))))
    nz = max(4, int(n / (nx * ny)))
    p = [rng.randint(1, 4) for _ in range(3)]
    c = _case(do, (nx, ny, nz), p, kappa=rng.choice([1.0, 1e-1, 1e-2, 1e-3]), scramble=rng.random() < 0.2)
    if do == "spmv":
        c["dtype"] = rng.choice(["float64", "float32"])
    if do == "update":
        c.update(lower=rng.random() < 0.3, kappa=rng.choice([1e-1, 1e-2, 1e-3]))
    if do in ("timestep", "adjoint"):
        c["tol"] = rng.choice([1e-6, 1e-8, 1e-10])
    if do == "solve":
        c["tol"] = rng.choice([1e-6, 1e-8, 1e-10])
        kind = rng.choice(["fp64", "mixed", "mixed_rr", "amg", "amg_mixed", "bicgstab", "block_jacobi", "rcm"])
        if kind in ("mixed", "mixed_rr"):
            c.update(precision=kind, tol=1e-11)
        elif kind == "amg":
            c.update(precond="amg")
        elif kind == "amg_mixed":
            c.update(precond="amg", precision="mixed", tol=1e-11)
        elif kind == "bicgstab":
            c.update(method="bicgstab", tol=1e-10)
        elif kind == "block_jacobi":
            c.update(precond="block_jacobi", block_size=rng.choice([2, 3, 4, 8]))
        elif kind == "rcm":
            c.update(order="rcm", scramble=True)
    return c


# ----------------------------------------------------------------------------
# mesh, ranks and their LDU addressing
# ----------------------------------------------------------------------------
class _Mesh:
    """Faces of the mesh, the ranks' numbering and every rank's addressing.
    Rank arrays are concatenated over the ranks; cells are in fused order."""

    def __init__(self, c, gen):
        d = gen.device
        nx, ny, nz = c["nx"], c["ny"], c["nz"]
        parts = (min(c["px"], nx), min(c["py"], ny), min(c["pz"], nz))
        self.n = n = nx * ny * nz
        self.dims = (nx, ny, nz)
        idx = torch.arange(n, device=d).view(nz, ny, nx)
        a = torch.cat([idx[:, :, :-1].reshape(-1), idx[:, :-1].reshape(-1), idx[:-1].reshape(-1)])
        b = torch.cat([idx[:, :, 1:].reshape(-1), idx[:, 1:].reshape(-1), idx[1:].reshape(-1)])
        wall = torch.cat([t.reshape(-1) for t in (idx[:, :, 0], idx[:, :, -1], idx[:, 0], idx[:, -1], idx[0], idx[-1])])
        self.a, self.b, self.wall, self.nf = a, b, wall, a.numel()
        self.R = R = parts[0] * parts[1] * parts[2]
        i, j, k = (torch.arange(m, device=d) * q // m for m, q in zip((nx, ny, nz), parts))
        rank = (i[None, None, :] + parts[0] * (j[None, :, None] + parts[1] * k[:, None, None])).reshape(-1)
        gid = torch.randperm(n, generator=gen, device=d) if c["scramble"] else torch.arange(n, device=d)
        order = torch.argsort(rank * n + gid)                   # natural id at each fused row
        self.row = torch.empty_like(order)
        self.row[order] = torch.arange(n, device=d)             # fused row of each natural id
        self.order = order
        cnt = torch.bincount(rank, minlength=R)
        ptr = torch.cat([cnt.new_zeros(1), cnt.cumsum(0)])
        local = self.row - ptr[rank]
        ra, rb, la, lb = rank[a], rank[b], local[a], local[b]
        inner = torch.nonzero(ra == rb).squeeze(1)
        own, nbr = torch.minimum(la[inner], lb[inner]), torch.maximum(la[inner], lb[inner])
        m = int(cnt.max())
        o = torch.argsort((ra[inner] * m + own) * m + nbr)
        self.face = inner[o]                                    # mesh face of each rank face
        self.fwd = la[self.face] < lb[self.face]                # its owner is the mesh face's minus side
        self.owner, self.nbr, self.frank = own[o], nbr[o], ra[self.face]
        cross = torch.nonzero(ra != rb).squeeze(1)
        e_rank, e_nrank = torch.cat([ra[cross], rb[cross]]), torch.cat([rb[cross], ra[cross]])
        e_cell, e_ncell = torch.cat([la[cross], lb[cross]]), torch.cat([lb[cross], la[cross]])
        e_face = torch.cat([cross, cross])
        e_minus = torch.arange(2 * cross.numel(), device=d) < cross.numel()
        o = torch.argsort((e_rank * R + e_nrank) * max(self.nf, 1) + e_face)
        self.if_rank, self.if_cell, self.if_nrank, self.if_ncell = e_rank[o], e_cell[o], e_nrank[o], e_ncell[o]
        self.if_face, self.if_minus = e_face[o], e_minus[o]
        self.cells = [int(v) for v in cnt]
        self.faces = [int(v) for v in torch.bincount(self.frank, minlength=R)]
        self.ifaces = [int(v) for v in torch.bincount(self.if_rank, minlength=R)]
        self.ptr = ptr

    def plan(self):
        def split(t, sizes):
            return np.split(t.to(torch.int32).cpu().numpy(), np.cumsum(sizes)[:-1])

        owner, nbr = split(self.owner, self.faces), split(self.nbr, self.faces)
        ic, ir, il = (split(t, self.ifaces) for t in (self.if_cell, self.if_nrank, self.if_ncell))
        ranks = [dict(n_cells=self.cells[r], owner=owner[r], neighbour=nbr[r], iface_cell=ic[r],
                      iface_nbr_rank=ir[r], iface_nbr_cell=il[r]) for r in range(self.R)]
        return rp.Plan(np.array(self.cells, np.int32), 0, self.R, ranks)

    def values(self, kappa, flux=None, sigma=0.0):
        """LDU values of face coefficients kappa (and upwind convection of the
        face fluxes): diag [n], upper and lower [faces], iface [ifaces]."""
        k, w = kappa[:self.nf], kappa[self.nf:]
        f = torch.zeros_like(k) if flux is None else flux
        ab, ba = -(k + torch.clamp(-f, min=0)), -(k + torch.clamp(f, min=0))
        # one axis's faces touch a cell at most once on each side, so the sum has no order to choose
        diag = torch.full((self.n,), float(sigma), dtype=torch.float64, device=k.device)
        nx, ny, nz = self.dims
        at = 0
        for count in ((nx - 1) * ny * nz, nx * (ny - 1) * nz, nx * ny * (nz - 1)):
            sl = slice(at, at + count)
            diag[self.a[sl]] -= ba[sl]
            diag[self.b[sl]] -= ab[sl]
            at += count
        at = 0
        for count in (ny * nz, ny * nz, nx * nz, nx * nz, nx * ny, nx * ny):
            diag[self.wall[at:at + count]] += w[at:at + count]
            at += count
        upper = torch.where(self.fwd, ab[self.face], ba[self.face])
        lower = torch.where(self.fwd, ba[self.face], ab[self.face])
        iface = torch.where(self.if_minus, ab[self.if_face], ba[self.if_face])
        return diag[self.order].contiguous(), upper, lower, iface

    def by_rank(self, v, lower):
        """The per-rank arrays of values(), as the update takes them."""
        d, u, l, i = v
        r = dict(diag=list(torch.split(d, self.cells)), upper=list(torch.split(u, self.faces)),
                 iface=list(torch.split(i, self.ifaces)))
        if lower:
            r["lower"] = list(torch.split(l, self.faces))
        return r

    def slots(self, v):
        """The values in receive-buffer order: per rank diag, upper, lower, interface."""
        d, u, l, i = (torch.split(t, s) for t, s in zip(v, (self.cells, self.faces, self.faces, self.ifaces)))
        return torch.cat([t for r in range(self.R) for t in (d[r], u[r], l[r], i[r])])

    def slot_entries(self):
        """(row, column) of every slot, in fused rows."""
        fo, fn = self.ptr[self.frank] + self.owner, self.ptr[self.frank] + self.nbr
        ir, ic = self.ptr[self.if_rank] + self.if_cell, self.ptr[self.if_nrank] + self.if_ncell
        dg = torch.arange(self.n, device=fo.device)
        return self.slots((dg, fo, fn, ir)), self.slots((dg, fn, fo, ic))


def _gen(seed):
    g = torch.Generator(device=_dev())
    g.manual_seed(int(seed))
    return g


def _uniform(gen, n, lo=-1.0, hi=1.0):
    return lo + (hi - lo) * torch.rand(n, generator=gen, device=gen.device, dtype=torch.float64)


def _inputs(c, seed):
    """The mesh and everything random of a case, the same for prepare and exact."""
    g = _gen(seed)
    mesh = _Mesh(c, g)
    faces = mesh.nf + mesh.wall.numel()
    kappa = torch.exp(_uniform(g, faces, math.log(c["kappa"]), 0.0)) if c["kappa"] < 1 else torch.ones(
        faces, dtype=torch.float64, device=g.device)
    flux, sigma = None, 0.0
    nonsym = c.get("method") == "bicgstab" or c.get("lower", False)
    if nonsym:
        # a rotating flow in every x-y plane (divergence-free cell by cell), largest face flux four times the
        # median coefficient, and a transient term on the diagonal
        nx, ny, nz = mesh.dims
        cm = float(kappa.median())
        X = torch.arange(nx + 1, device=g.device, dtype=torch.float64) / nx
        Y = torch.arange(ny + 1, device=g.device, dtype=torch.float64) / ny
        psi = torch.sin(math.pi * Y)[:, None] * torch.sin(math.pi * X)[None, :]
        fx = (psi[1:, 1:nx] - psi[:-1, 1:nx]).expand(nz, ny, nx - 1).reshape(-1)
        fy = -(psi[1:ny, 1:] - psi[1:ny, :-1]).expand(nz, ny - 1, nx).reshape(-1)
        flux = torch.cat([fx, fy, torch.zeros(nx * ny * (nz - 1), dtype=torch.float64, device=g.device)])
        flux = flux * (4.0 * cm / max(float(flux.abs().max()), 1e-300))
        sigma = cm
    v = mesh.values(kappa, flux, sigma)
    x, y = _uniform(g, mesh.n), _uniform(g, mesh.n)
    later = None
    if c["do"] == "timestep":
        later = mesh.values(kappa * (1.0 + 0.05 * _uniform(g, faces)))
    return mesh, v, later, x, y, nonsym


class _View:
    """A device array of the library, for torch.as_tensor (no copy)."""

    def __init__(self, ptr, n, kind):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": kind, "data": (ptr, False), "version": 2}


def _plan_array(plan, name, n, kind):
    """A tensor over one of the plan's device arrays.  The tensor holds the
    plan, whose memory it is: the array is there as long as the tensor is."""
    view = _View(plan.device_ptrs()[name], n, kind)
    view.plan = plan
    t = torch.as_tensor(view, device=_dev())
    t.plan = plan
    return t


class _State:
    pass


def _options(c):
    return {k: c[k] for k in ("tol", "precision", "precond", "method", "block_size") if k in c}


def prepare(case, seed):
    c, s = case, _State()
    mesh, v, later, x, y, nonsym = _inputs(c, seed)
    s.do, s.plan, s.x, s.y = c["do"], mesh.plan(), x, y
    s.values = mesh.by_rank(v, nonsym)
    if c.get("order"):
        s.plan.set_solve_order(c["order"])
    if s.do == "update":
        s.plan.update(**mesh.by_rank(mesh.values(torch.ones(mesh.nf + mesh.wall.numel(), dtype=torch.float64,
                                                            device=x.device)), nonsym))
        n, m = s.plan.n_rows, s.plan.n_slots
        s.out = [_plan_array(s.plan, *a) for a in (("val64", m, "<f8"), ("val32", m, "<f4"), ("dinv64", n, "<f8"),
                                                   ("dinv32", n, "<f4"))]
    elif s.do == "adjoint":
        s.slots = mesh.slots(v)
    else:
        s.plan.update(**s.values)
    if c.get("dtype") == "float32":
        s.x = x.to(torch.float32)
    if s.do == "spmv":
        s.out = torch.empty_like(s.x)
    if s.do == "vcycle" or c.get("precond") == "amg":
        s.plan.amg_setup()
    if s.do in ("solve", "timestep", "adjoint"):
        s.opts = _options(c)
    if s.do == "timestep":
        s.x0, _ = s.plan.solve(x, **s.opts)
        s.values = mesh.by_rank(later, False)
    torch.cuda.synchronize()
    return s


def run(s):
    if s.do == "spmv":
        return s.plan.spmv(s.x, s.out)
    if s.do == "update":
        s.plan.update(**s.values)
        return s.out
    if s.do == "grad":
        return s.plan.value_grad(s.x, s.y)
    if s.do == "vcycle":
        return s.plan.amg_apply(s.x)
    if s.do == "solve":
        return s.plan.solve(s.x, **s.opts)[0]
    if s.do == "timestep":
        s.plan.update(**s.values)
        return s.plan.solve(s.x, x=s.x0.clone(), **s.opts)[0]
    a, b = s.slots.detach().requires_grad_(True), s.x.detach().requires_grad_(True)
    x = repart_solve(a, b, s.plan, rp.default_opts(**s.opts))
    ga, gb = torch.autograd.grad(x, (a, b), grad_outputs=s.y)
    return x.detach(), ga, gb


# ----------------------------------------------------------------------------
# the same in 64 bits by plain torch
# ----------------------------------------------------------------------------
class _Matrix:
    """The fused matrix, at most seven entries per row, as padded rows."""

    def __init__(self, mesh, v):
        row, col = mesh.slot_entries()
        val = mesh.slots(v)
        o = torch.argsort(row * mesh.n + col)
        self.row, self.col, self.val = row[o], col[o], val[o]
        cnt = torch.bincount(self.row, minlength=mesh.n)
        start = torch.cat([cnt.new_zeros(1), cnt.cumsum(0)])
        place = torch.arange(self.row.numel(), device=row.device) - start[self.row]
        k = int(cnt.max())
        self.ec = torch.arange(mesh.n, device=row.device).repeat(k, 1)
        self.ev = torch.zeros(k, mesh.n, dtype=torch.float64, device=row.device)
        self.ec[place, self.row], self.ev[place, self.row] = self.col, self.val
        self.diag = v[0]

    def times(self, x, val=None):
        ev = self.ev if val is None else val
        y = ev[0] * x[self.ec[0]]
        for k in range(1, ev.shape[0]):
            y += ev[k] * x[self.ec[k]]
        return y


def _cg(A, b, steps=6000):
    x = torch.zeros_like(b)
    for _ in range(3):                     # restarted, so that what is left is the true residual
        r = b - A.times(x)
        z = r / A.diag
        p, rz = z.clone(), torch.dot(r, z)
        goal = 1e-28 * torch.dot(b, b)
        for k in range(steps):
            q = A.times(p)
            a = rz / torch.dot(p, q)
            x += a * p
            r -= a * q
            z = r / A.diag
            new = torch.dot(r, z)
            if k % 16 == 0 and bool(torch.dot(r, r) <= goal):
                break
            p = z + (new / rz) * p
            rz = new
    return x


def _bicgstab(A, b):
    x = torch.zeros_like(b)
    for _ in range(4):
        r = b - A.times(x)
        rh, rho, alpha, omega = r.clone(), 1.0, 1.0, 1.0
        v, p, goal = torch.zeros_like(b), torch.zeros_like(b), 1e-26 * float(torch.dot(r, r))
        if not float(torch.dot(r, r)) > 1e-32 * float(torch.dot(b, b)):
            break
        for _ in range(2000):
            new = float(torch.dot(rh, r))
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            y = p / A.diag
            v = A.times(y)
            alpha, rho = new / float(torch.dot(rh, v)), new
            s = r - alpha * v
            z = s / A.diag
            t = A.times(z)
            tt = float(torch.dot(t, t))
            omega = float(torch.dot(t, s)) / tt if tt > 0 else 0.0
            x += alpha * y + omega * z
            r = s - omega * t
            if omega == 0.0 or float(torch.dot(r, r)) <= goal:
                break
    return x


def exact(case, seed):
    c = case
    if c["do"] == "vcycle":
        return None                        # no value without the hierarchy, which is the library's own
    mesh, v, later, x, y, _ = _inputs(c, seed)
    if c["do"] == "grad":
        row, col = mesh.slot_entries()
        return -x[row] * y[col]
    A = _Matrix(mesh, later if later is not None else v)
    if c["do"] == "update":
        return [A.val, A.val, 1.0 / v[0], 1.0 / v[0]]
    if c["do"] == "spmv":
        if c["dtype"] == "float32":
            return A.times(x.to(torch.float32).double(), A.ev.to(torch.float32).double())
        return A.times(x)
    if c.get("method") == "bicgstab":
        return _bicgstab(A, x)
    u = _cg(A, x)
    if c["do"] != "adjoint":
        return u
    lam = _cg(A, y)
    row, col = mesh.slot_entries()
    return u, -lam[row] * u[col], lam


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------
def work(case):
    """Bytes: the matrix's values, its columns where the numbering has no
    pattern, and the vectors, each once per product or per iteration.  The
    iterations of a solve are estimates for meshes of these coefficients."""
    c = case
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    n = nx * ny * nz
    nnz = 7 * n - 2 * (nx * ny + ny * nz + nx * nz)
    side = n ** (1.0 / 3.0)
    slot = 8 * nnz
    index = 4 * nnz if c["scramble"] else 0
    if c["do"] == "spmv":
        v = 8 if c["dtype"] == "float64" else 4
        return {"bytes": v * nnz + index + 2 * v * n, "flops": 2 * nnz}
    if c["do"] == "update":
        read = 8 * (nnz if c.get("lower") else (nnz + n) // 2)
        return {"bytes": read + 4 * nnz + 12 * nnz + 12 * n, "flops": n}
    if c["do"] == "grad":
        return {"bytes": slot + 4 * (nnz - n) + 16 * n, "flops": nnz}
    if c["do"] == "vcycle":
        return {"bytes": 2 * 1.6 * (slot + index + 40 * n), "flops": 2 * 1.6 * 2 * nnz}
    k = {1.0: 3.0, 1e-1: 4.0, 1e-2: 5.0, 1e-3: 5.8}[c["kappa"]] * side * (1 - math.log10(c["tol"]) / 8) / 2
    v = 8
    if c.get("precision", "fp64") != "fp64":
        v, k = 4, 1.3 * k
    per = v * nnz + index + 9 * v * n
    if c["do"] == "timestep":
        k = 0.65 * k                       # the last step's solution is a start
    if c.get("method") == "bicgstab":
        k, per = 90, 2 * (slot + index) + 20 * 8 * n
    if c.get("precond") == "amg":
        k, per = 60, 4.2 * per
    total = k * per * (2 if c["do"] == "adjoint" else 1)
    return {"bytes": total, "flops": total / 8}
