"""What this framework is timed on: whole passes through its public calls.

Every case is a pass that a program built on this package makes again and again: one V-cycle as
another solver's preconditioner, a differentiable solve, a time step on a kept hierarchy, a step whose
matrix is new, a batch of systems, a discontinuous Galerkin problem.  The matrices are the ones the
repository's tests and benchmark use (first-order upwind finite differences in two and three
dimensions, P2 upwind discontinuous Galerkin on triangles), built here on the GPU; velocities, reaction
fields, mesh jitter and right-hand sides are drawn from the seed.
"""
import math

import numpy as np
import torch

import paper_1708_06065_amd as lair
from paper_1708_06065_amd.autograd import LairSolve

DEV = "cuda"
F64 = torch.float64
RTOL = 1e-10


def listed():
    return [
        # The smallest call: one V-cycle on a 64 x 64 transport grid, as the preconditioner of a
        # caller's own Krylov method.
        dict(name="cycle_64", kind="cycle", m=64, nrhs=1, precision="fp64"),
        # One gradient of a misfit with respect to source and reaction field, the hierarchy kept and
        # its diagonal replaced (forward solve, transposed solve): an optimisation step, small grid.
        dict(name="adjoint_64", kind="adjoint", m=64),
        # The same on a larger grid of odd size.
        dict(name="adjoint_193", kind="adjoint", m=193),
        # A call with default options and host arrays, splitting included: a script's first solve.
        dict(name="default_97", kind="default", m=97),
        # Steady, more diffusive flow, distance-2 neighbourhoods, flexible GMRES on a kept hierarchy.
        dict(name="fgmres_150", kind="fgmres", m=150, precision="fp64"),
        # Time stepping with a fixed matrix: one right-hand side a step, plain FP64.
        dict(name="march_73", kind="march", m=73, nrhs=1, precision="fp64"),
        # The benchmark's step: 128^3 unknowns, 16 right-hand sides, mixed precision, the splittings
        # of the grid kept while the matrix changes.
        dict(name="step_128_x16", kind="step", m=128, nrhs=16, precision="mixed", split="kept"),
        # A step from the matrix alone, split on the device, few right-hand sides, plain FP64.
        dict(name="step_80_x4_pmis", kind="step", m=80, nrhs=4, precision="fp64", split="pmis"),
        # A small batch of uneven systems (parameter study), split on the device, plain FP64.
        dict(name="batch_24_pmis", kind="batch", nsys=24, precision="fp64", split="pmis"),
        # The large batch of the repository's workloads, splittings kept, mixed precision.
        dict(name="batch_512", kind="batch", nsys=512, precision="mixed", split="kept"),
        # Recirculating advection, P2 DG, scaled by its diagonal blocks: setup and 20 cycles (the
        # steady limit is ill-posed and does not converge further).
        dict(name="dg_scaled_160", kind="dg", m=160, nodal=False, kappa=0.0, precision="fp64"),
        # The DG problem with diffusion and a reaction jump, nodal treatment, at its full size.
        dict(name="dg_nodal_256", kind="dg", m=256, nodal=True, kappa=1e-3, precision="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cycle", "adjoint", "default", "fgmres", "march", "step", "step", "batch", "dg", "dg"])
    prec = rng.choice(["fp64", "mixed"])
    if kind == "cycle":
        return dict(kind=kind, m=_log_int(rng, 24, 300), nrhs=rng.choice([1, 1, 2, 4]), precision=prec)
    if kind == "adjoint":
        return dict(kind=kind, m=_log_int(rng, 32, 256))
    if kind == "default":
        return dict(kind=kind, m=_log_int(rng, 32, 160))
    if kind == "fgmres":
        return dict(kind=kind, m=_log_int(rng, 48, 300), precision=prec)
    if kind == "march":
        return dict(kind=kind, m=_log_int(rng, 20, 112), nrhs=rng.choice([1, 1, 2, 4, 16]), precision=prec)
    if kind == "step":
        return dict(kind=kind, m=_log_int(rng, 24, 128), nrhs=rng.choice([1, 2, 4, 8, 16]), precision=prec,
                    split=rng.choice(["kept", "pmis"]))
    if kind == "batch":
        return dict(kind=kind, nsys=_log_int(rng, 6, 160), precision=prec, split=rng.choice(["kept", "pmis"]))
    nodal = rng.random() < 0.6
    return dict(kind=kind, m=_log_int(rng, 20, 200), nodal=nodal,
                kappa=rng.choice([1e-3, 1e-1]) if nodal else 0.0, precision=prec)


# ---------------------------------------------------------------------------
# Matrices
# ---------------------------------------------------------------------------
def _stencil(shape, lo, hi, diag):
    """CSR of an upwind finite difference operator on a grid of interior nodes (axis 0 fastest): row
    value diag, -lo[a] and -hi[a] for the neighbours down and up axis a; zero couplings are not stored."""
    n = math.prod(shape)
    k = torch.arange(n, device=DEV)
    stride, below, above = 1, [], []
    for a, m in enumerate(shape):
        at = (k // stride) % m
        if lo[a]:
            below.append((k - stride, at > 0, -lo[a]))
        if hi[a]:
            above.append((k + stride, at < m - 1, -hi[a]))
        stride *= m
    one = torch.ones(n, dtype=F64, device=DEV)
    entries = below[::-1] + [(k, k >= 0, None)] + above
    col = torch.stack([c for c, _, _ in entries], 1)
    keep = torch.stack([i for _, i, _ in entries], 1)
    val = torch.stack([one * (diag if v is None else v) for _, _, v in entries], 1)
    return _csr(keep, col, val)


def _csr(keep, col, val):
    """CSR of rows given as equally long lists of candidates, in column order."""
    rowptr = torch.zeros(keep.shape[0] + 1, dtype=torch.int32, device=DEV)
    rowptr[1:] = keep.sum(1).cumsum(0)
    return rowptr, col[keep].to(torch.int32), val[keep].contiguous()


def _adr_2d(m, eps, phi, c):
    """5-point upwind advection-diffusion-reaction, m x m nodes, unit speed at angle phi."""
    h = 1.0 / (m + 1)
    b, e = (math.cos(phi), math.sin(phi)), eps / (h * h)
    lo, hi = [e + max(x, 0.0) / h for x in b], [e + max(-x, 0.0) / h for x in b]
    return _stencil((m, m), lo, hi, 4 * e + (abs(b[0]) + abs(b[1])) / h + c), lo, hi


def _euler_3d(m, seed):
    """One implicit Euler step I + dt S, dt = h, of 7-point upwind advection-diffusion on m^3 nodes
    with a velocity drawn around the workloads' own."""
    rng = np.random.default_rng(seed)
    h, eps = 1.0 / (m + 1), 1e-4
    b = np.array([1.0, 0.7, 0.4]) * rng.uniform(0.8, 1.2, 3)
    b /= np.linalg.norm(b)
    e = eps / (h * h)
    lo, hi = [h * (e + max(x, 0.0) / h) for x in b], [h * (e + max(-x, 0.0) / h) for x in b]
    diag = 1.0 + h * (6 * e + float(np.abs(b).sum()) / h)
    return _stencil((m, m, m), lo, hi, diag), lo, hi, diag


def _reaction(m, g):
    """exp(xi / 2), xi a smooth cosine series with 8 x 8 normal weights (the adjoint workload's field)."""
    xs = torch.arange(1, m + 1, dtype=F64, device=DEV) / (m + 1)
    p = torch.arange(8, dtype=F64, device=DEV)
    cx = torch.cos(math.pi * xs[:, None] * p)
    xi = cx @ (torch.as_tensor(g, device=DEV) / (1 + p[:, None] ** 2 + p ** 2)) @ cx.T
    return torch.exp(0.5 * xi.T.reshape(-1)).contiguous()


def _normal(seed, *shape):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn(*shape, dtype=F64, device=DEV, generator=g)


def _p2(lam):
    """P2 basis (3 vertices, then the midpoints of edges 01, 12, 20) and its derivatives by the
    barycentric coordinates, at points lam[..., 3]."""
    l0, l1, l2 = lam[..., 0], lam[..., 1], lam[..., 2]
    val = np.stack([l0 * (2 * l0 - 1), l1 * (2 * l1 - 1), l2 * (2 * l2 - 1), 4 * l0 * l1, 4 * l1 * l2, 4 * l2 * l0], -1)
    z = np.zeros_like(l0)
    der = np.stack([np.stack(r, -1) for r in (
        (4 * l0 - 1, z, z), (z, 4 * l1 - 1, z), (z, z, 4 * l2 - 1),
        (4 * l1, 4 * l0, z), (z, 4 * l2, 4 * l1), (4 * l2, z, 4 * l0))], -2)
    return val, der


def _dg(m, kappa, nodal, seed):
    """P2 upwind DG on m x m squares cut into two triangles each, interior vertices jittered by a
    fifth of h.  nodal: velocity (y^2, cos^2(pi x / 2)), reaction 1e4 inside (1/4, 3/4)^2 and 1e-4
    outside, symmetric interior penalty for kappa, stored in dense 6 x 6 blocks.  Otherwise the
    recirculating velocity, pure advection, structural zeros dropped.  Inflow value 1."""
    h = 1.0 / m
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    i = torch.arange(m + 1, device=DEV)
    iy, ix = torch.meshgrid(i, i, indexing="ij")
    xy = torch.stack([ix, iy], -1).to(F64) * h
    move = (torch.rand(m + 1, m + 1, 2, dtype=F64, device=DEV, generator=g) - 0.5) * (0.4 * h)
    xy[1:-1, 1:-1] += move[1:-1, 1:-1]
    sw, se, nw, ne = xy[:-1, :-1], xy[:-1, 1:], xy[1:, :-1], xy[1:, 1:]
    P = torch.stack([torch.stack([sw, se, ne], 2), torch.stack([sw, ne, nw], 2)], 2).reshape(-1, 3, 2)
    E = P.shape[0]
    # the neighbour across each edge (-1: boundary) and the neighbour's number of that edge
    sq = torch.arange(m * m, device=DEV)
    x, y = sq % m, sq // m
    low = torch.stack([torch.where(y > 0, 2 * (sq - m) + 1, -1), torch.where(x < m - 1, 2 * (sq + 1) + 1, -1), 2 * sq + 1], 1)
    upp = torch.stack([2 * sq, torch.where(y < m - 1, 2 * (sq + m), -1), torch.where(x > 0, 2 * (sq - 1), -1)], 1)
    nbr = torch.stack([low, upp], 1).reshape(E, 3)
    nedge = torch.tensor([[1, 2, 0], [2, 0, 1]], device=DEV).repeat(m * m, 1)

    def velocity(p):
        if nodal:
            return torch.stack([p[..., 1] ** 2, torch.cos(0.5 * math.pi * p[..., 0]) ** 2], -1)
        return torch.stack([0.5 - p[..., 1], p[..., 0] - 0.5], -1)

    def dev(a):
        return torch.as_tensor(a, dtype=F64, device=DEV)

    d1, d2 = P[:, 1] - P[:, 0], P[:, 2] - P[:, 0]
    det = d1[:, 0] * d2[:, 1] - d1[:, 1] * d2[:, 0]
    g1 = torch.stack([d2[:, 1], -d2[:, 0]], 1) / det[:, None]
    g2 = torch.stack([-d1[:, 1], d1[:, 0]], 1) / det[:, None]
    glam = torch.stack([-g1 - g2, g1, g2], 1)                                   # [E, 3, 2]
    # volume terms, 6-point rule of degree 4
    a1, b1, w1, a2, b2, w2 = (0.108103018168070, 0.445948490915965, 0.223381589678011,
                              0.816847572980459, 0.091576213509771, 0.109951743655322)
    tq = np.array([[a1, b1, b1], [b1, a1, b1], [b1, b1, a1], [a2, b2, b2], [b2, a2, b2], [b2, b2, a2]])
    tw = dev([w1] * 3 + [w2] * 3)
    val, der = (dev(v) for v in _p2(tq))
    grad = torch.einsum("qia,eax->eqix", der, glam)
    b = velocity(torch.einsum("qa,eax->eqx", dev(tq), P))
    area = 0.5 * det
    own = -torch.einsum("eqi,qj->eij", (grad * b[:, :, None]).sum(-1) * (tw * area[:, None])[..., None], val)
    if nodal:
        cen = P.mean(1)
        gamma = torch.where(((cen > 0.25) & (cen < 0.75)).all(1), dev(1e4), dev(1e-4))
        own += torch.einsum("q,qi,qj->ij", tw, val, val) * (area * gamma)[:, None, None]
        own += kappa * torch.einsum("eqix,eqjx->eij", grad * (tw * area[:, None])[..., None, None], grad)
    # faces, 3 Gauss points
    gs = 0.5 * math.sqrt(0.6)
    s = np.array([0.5 - gs, 0.5, 0.5 + gs])
    lam = np.zeros((3, 3, 3))
    for k in range(3):
        lam[k, :, k], lam[k, :, (k + 1) % 3] = 1 - s, s
    val, der = (dev(v) for v in _p2(lam))                                       # [k, q, 6], [k, q, 6, 3]
    pa, pb = P, P[:, [1, 2, 0]]
    d = pb - pa
    length = d.norm(dim=-1)
    nrm = torch.stack([d[..., 1], -d[..., 0]], -1) / length[..., None]
    wq = dev([5 / 18, 8 / 18, 5 / 18]) * length[..., None]                      # [E, k, q]
    bn = (velocity(pa[:, :, None] + dev(s)[:, None] * d[:, :, None]) * nrm[:, :, None]).sum(-1)
    inner = nbr >= 0
    at = nbr.clamp(min=0)
    nval = val[nedge].flip(2)                                                   # the same points, seen from there
    own += torch.einsum("ekqi,kqj->eij", val * (wq * bn.clamp(min=0))[..., None], val)
    inw = wq * bn.clamp(max=0)
    off = torch.einsum("kqi,ekqj->ekij", val, nval * inw[..., None])            # [E, k, 6, 6]
    rhs = -torch.einsum("kqi,ekq->ei", val, inw * ~inner[..., None])
    if kappa:
        grad = torch.einsum("kqia,eax->ekqix", der, glam)
        dn = (grad * nrm[:, :, None, None]).sum(-1)
        dnn = (grad[at, nedge].flip(2) * nrm[:, :, None, None]).sum(-1)
        mid = 0.5 * (pa + pb)
        wall = ~inner & (mid < 1e-12).any(-1)
        half = 0.5 * inner.to(F64) + wall
        sig = 20 * kappa / length * (inner | wall)
        wk = (kappa * half)[..., None] * wq
        own -= torch.einsum("kqi,ekqj->eij", val, dn * wk[..., None])
        own -= torch.einsum("ekqi,kqj->eij", dn * wk[..., None], val)
        own += torch.einsum("ekqi,kqj->eij", val * (sig[..., None] * wq)[..., None], val)
        off -= torch.einsum("kqi,ekqj->ekij", val, dnn * wk[..., None])
        off += torch.einsum("ekqi,ekqj->ekij", dn * wk[..., None], nval)
        off -= torch.einsum("kqi,ekqj->ekij", val, nval * (sig[..., None] * wq)[..., None])
        gw = wq * wall[..., None]
        rhs += torch.einsum("kqi,ekq->ei", val, sig[..., None] * gw) - kappa * torch.einsum("ekqi,ekq->ei", dn, gw)
    # an element's blocks in column order, expanded to CSR rows
    off = off * inner[..., None, None]
    blocks = torch.cat([own[:, None], off], 1)                                  # [E, 4, 6, 6]
    ids = torch.cat([torch.arange(E, device=DEV)[:, None], torch.where(inner, nbr, E)], 1)
    ids, order = ids.sort(1)
    blocks = torch.gather(blocks, 1, order[..., None, None].expand(-1, -1, 6, 6))
    col = (6 * ids[:, None, :, None] + torch.arange(6, device=DEV)).expand(E, 6, 4, 6)
    val = blocks.permute(0, 2, 1, 3)
    if nodal:
        keep = (ids < E)[:, None, :, None] & (blocks != 0).any(-1).any(-1)[:, None, :, None]
    else:
        keep = (val != 0) | (col == (6 * torch.arange(E, device=DEV)[:, None] + torch.arange(6, device=DEV))[:, :, None, None])
    A = _csr(keep.expand(E, 6, 4, 6).reshape(6 * E, 24), col.reshape(6 * E, 24), val.reshape(6 * E, 24))
    return A, rhs.reshape(-1).contiguous()


def _batch_sizes(nsys):
    """The batch workload's grid sizes: N log-uniform in [32, 320]."""
    rng = np.random.default_rng(3)
    return [int(round(math.exp(v))) for v in rng.uniform(math.log(32), math.log(320), nsys)]


def _batch(nsys, seed):
    rng = np.random.default_rng(seed)
    got = []
    for m in _batch_sizes(nsys):
        eps, c, phi = 10.0 ** rng.uniform(-6, 0), rng.uniform(0, 1), rng.uniform(0, 2 * math.pi)
        got.append((m, _adr_2d(m, eps, phi, c), c))
    return got


def _kept(h):
    """The splittings of a hierarchy, as a program keeps them for matrices of the same structure."""
    return [torch.as_tensor(h.export(l, "cf"), device=DEV) for l in range(h.nlevels - 1)]


# ---------------------------------------------------------------------------
# States and passes
# ---------------------------------------------------------------------------
def _grid_2d(case, seed):
    """The 2-D operator of a single-system case, its couplings, and what else the seed draws."""
    m, kind = case["m"], case["kind"]
    rng = np.random.default_rng(seed)
    phi = 3 * math.pi / 16 * rng.uniform(0.8, 1.2)
    eps = {"cycle": 0.0, "adjoint": 1e-3, "default": 1e-3, "fgmres": 1e-2}[kind]
    c = _reaction(m, rng.standard_normal((8, 8))) if kind != "cycle" else 0.0
    (A, lo, hi) = _adr_2d(m, eps, phi, 0.0 if kind == "adjoint" else c)
    return A, lo, hi, c


def _shape(n, nrhs):
    return (n,) if nrhs == 1 else (n, nrhs)


def prepare(case, seed):
    kind, s = case["kind"], {"kind": case["kind"]}
    if kind in ("cycle", "adjoint", "default", "fgmres"):
        A, _, _, c = _grid_2d(case, seed)
        n = case["m"] ** 2
        b = _normal(seed, *_shape(n, case.get("nrhs", 1)))
        if kind == "cycle":
            s.update(h=lair.setup(*A, precision=case["precision"]), b=b, z=torch.empty_like(b))
        elif kind == "adjoint":
            s.update(A=A, b=b.requires_grad_(), c=c.requires_grad_(), seen=_normal(seed + 7, n),
                     opts=dict(interp="direct", reuse={}))
            LairSolve.apply(s["b"].detach(), s["c"].detach(), *A, s["opts"])
        elif kind == "default":
            s.update(A=[t.cpu().numpy() for t in A], b=b)
        else:
            s.update(h=lair.setup(*A, distance=2, interp="one_point", lump_tol=1e-3, precision=case["precision"]), b=b)
        return s
    if kind in ("march", "step"):
        A, _, _, _ = _euler_3d(case["m"], seed)
        s.update(A=A, b=_normal(seed, *_shape(case["m"] ** 3, case["nrhs"])),
                 kw=dict(interp="direct", lump_tol=1e-3, precision=case["precision"]))
        if kind == "march" or case["split"] == "kept":
            h = lair.setup(*A, **s["kw"])
            if kind == "march":
                s["h"] = h
            else:
                s["kw"]["cf_levels"] = _kept(h)
        else:
            s["kw"]["split"] = "pmis"
        return s
    if kind == "batch":
        made = _batch(case["nsys"], seed)
        s.update(A=[a for _, (a, _, _), _ in made], b=_normal(seed, sum(m * m for m, _, _ in made)),
                 kw=dict(interp="direct", lump_tol=1e-3, precision=case["precision"]))
        if case["split"] == "kept":
            s["kw"]["cf_levels"] = _kept(lair.setup_batch(s["A"], **s["kw"]))
        else:
            s["kw"]["split"] = "pmis"
        return s
    A, rhs = _dg(case["m"], case["kappa"], case["nodal"], seed)
    s.update(A=A, b=rhs, maxit=200 if case["nodal"] else 20,
             kw=dict(interp="one_point", distance=2, block_size=6, nodal=case["nodal"], precision=case["precision"]))
    s["kw"]["cf_levels"] = _kept(lair.setup(*A, **s["kw"]))
    return s


def run(s):
    kind = s["kind"]
    if kind == "cycle":
        s["z"].zero_()
        return s["h"].cycle(s["b"], s["z"])
    if kind == "adjoint":
        s["b"].grad = s["c"].grad = None
        x = LairSolve.apply(s["b"], s["c"], *s["A"], s["opts"])
        ((x - s["seen"]) ** 2).sum().backward()
        return x.detach(), s["b"].grad, s["c"].grad
    if kind == "default":
        return lair.setup(*s["A"]).solve(s["b"], rtol=RTOL)[0]
    if kind == "fgmres":
        return s["h"].solve_fgmres(s["b"], rtol=RTOL)[0]
    if kind == "march":
        return s["h"].solve(s["b"], rtol=RTOL)[0]
    if kind == "batch":
        return lair.setup_batch(s["A"], **s["kw"]).solve_batch(s["b"], rtol=RTOL)[0]
    return lair.setup(*s["A"], **s["kw"]).solve(s["b"], rtol=RTOL, maxit=s.get("maxit", 200))[0]


def work(case):
    """The matrix and the right-hand sides read once and the solutions written once; the operations
    of one product with the matrix for every right-hand side (of two, where there is a gradient)."""
    kind, m, nrhs = case["kind"], case.get("m"), case.get("nrhs", 1)
    if kind in ("march", "step"):
        n, per = m ** 3, 7
    elif kind == "batch":
        n, per = sum(k * k for k in _batch_sizes(case["nsys"])), 5
    elif kind == "dg":
        n, per = 12 * m * m, 24 if case["nodal"] else 8.3
    else:
        n, per = m * m, 3 if kind == "cycle" else 5
    vectors = 6 if kind == "adjoint" else 2
    return {"bytes": n * (12.0 * per + 4 + 8 * nrhs * vectors), "flops": 2.0 * n * per * nrhs * (2 if kind == "adjoint" else 1)}


# ---------------------------------------------------------------------------
# 64-bit references
# ---------------------------------------------------------------------------
def _block_solve(m, lo, hi, diag, f, transpose=False):
    """Direct solve of a 2-D stencil system by block elimination over the grid lines."""
    (lx, ly), (hx, hy) = (hi, lo) if transpose else (lo, hi)
    lx, hx, ly, hy = (float(v) for v in (lx, hx, ly, hy))
    f = f.reshape(m, m, -1)
    one = np.ones(m - 1)
    side = -lx * np.diag(one, -1) - hx * np.diag(one, 1)
    diag = np.broadcast_to(diag, (m * m,)).reshape(m, m)
    G, u = [], []
    for j in range(m):
        D, r = side + np.diag(diag[j]), f[j]
        if j:
            D, r = D - ly * G[-1], r + ly * u[-1]
        got = np.linalg.solve(D, np.concatenate([hy * np.eye(m), r], 1))
        G.append(got[:, :m])
        u.append(got[:, m:])
    for j in range(m - 2, -1, -1):
        u[j] = u[j] + G[j] @ u[j + 1]
    return np.concatenate(u)


def _host(t):
    return t.detach().cpu().numpy() if isinstance(t, torch.Tensor) else t


def _diag_2d(m, lo, hi, c):
    return lo[0] + hi[0] + lo[1] + hi[1] + _host(c)


def exact(case, seed):
    kind, m, nrhs = case["kind"], case.get("m"), case.get("nrhs", 1)
    if kind in ("adjoint", "default", "fgmres"):
        _, lo, hi, c = _grid_2d(case, seed)
        b = _host(_normal(seed, m * m))
        diag = _diag_2d(m, lo, hi, c)
        x = _block_solve(m, lo, hi, diag, b)[:, 0]
        if kind != "adjoint":
            return x
        lam = _block_solve(m, lo, hi, diag, 2 * (x - _host(_normal(seed + 7, m * m))), True)[:, 0]
        return x, lam, -lam * x
    if kind in ("march", "step"):
        # strongly diagonally dominant: the Jacobi iteration converges to rounding
        _, lo, hi, diag = _euler_3d(m, seed)
        b = _normal(seed, *_shape(m ** 3, nrhs)).reshape(m, m, m, nrhs)
        x = b / diag
        for _ in range(140):
            y = b.clone()
            for a in range(3):
                axis = 2 - a
                head, tail = x.narrow(axis, 0, m - 1), x.narrow(axis, 1, m - 1)
                y.narrow(axis, 1, m - 1).add_(head, alpha=lo[a])
                if hi[a]:
                    y.narrow(axis, 0, m - 1).add_(tail, alpha=hi[a])
            x = y / diag
        return x.reshape(_shape(m ** 3, nrhs))
    if kind == "batch":
        if case["nsys"] > 40:
            return None          # a direct solve of every system takes minutes
        made = _batch(case["nsys"], seed)
        b, x, at = _host(_normal(seed, sum(k * k for k, _, _ in made))), [], 0
        for k, (_, lo, hi), c in made:
            x.append(_block_solve(k, lo, hi, _diag_2d(k, lo, hi, c), b[at:at + k * k])[:, 0])
            at += k * k
        return np.concatenate(x)
    if kind == "dg" and case["nodal"] and m <= 32:
        (rowptr, col, val), rhs = _dg(m, case["kappa"], True, seed)
        n = rhs.numel()
        A = torch.zeros(n, n, dtype=F64)
        A[torch.repeat_interleave(torch.arange(n), (rowptr[1:] - rowptr[:-1]).long().cpu()), col.long().cpu()] = val.cpu()
        return torch.linalg.solve(A, rhs.cpu())
    # one cycle and a fixed number of cycles are no solution of the system, and the larger DG
    # systems are too large for a dense solve
    return None
