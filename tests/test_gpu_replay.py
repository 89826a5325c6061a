"""GPU: iterations replayed from HIP graphs against launched ones, bit for bit.

A combination of vectors is captured only after some tens of iterations, so
every case solves into the same buffers, with other work between, until the
profiler counts all the iterations of a solve as replays; a hierarchy that
never captures (graphs=False) gives the reference for each solve.  Two solves
more are then compared."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lair():
    import torch
    import paper_1708_06065_amd as lair
    assert torch.cuda.is_available()
    lair.load_library()
    return lair


def _busy(torch):
    a = torch.randn(256, 256, device="cuda")
    return float((a @ a).sum().item())


def _compare(lair, graphed, eager, b, x, seed):
    """graphed(b, x) against eager(b, x), which return info dicts (iters: of the
    solve, or of each system of a batch); new values in b for every solve."""
    import torch
    rng = np.random.default_rng(seed)
    xe = torch.zeros_like(x)
    after = 0
    for rep in range(60):
        b.copy_(torch.as_tensor(rng.standard_normal(tuple(b.shape)), device="cuda"))
        x.zero_()
        xe.zero_()
        _busy(torch)
        lair.profile_begin(["graph"])
        ig = graphed(b, x)
        replays = lair.profile_end().get("graph", {"launches": 0})["launches"]
        ie = eager(b, xe)
        torch.cuda.synchronize()
        its = np.asarray(ig["iters"])
        assert np.array_equal(its, ie["iters"]) and its.min() > 0 and ig["converged"]
        assert torch.equal(x, xe), rep
        if replays == its.max():
            after += 1
            if after == 3:
                return
    raise AssertionError("no solve was replayed")


def _vector(torch, shape, aligned):
    flat = torch.zeros(int(np.prod(shape)) + 1, dtype=torch.float64, device="cuda")
    return (flat[:-1] if aligned else flat[1:]).view(shape)


# vectors off a 16-byte boundary with several right-hand sides take the
# residual and its norms in two passes
@pytest.mark.parametrize("nrhs,aligned", [(1, True), (4, True), (4, False), (16, True)])
@pytest.mark.parametrize("ordering", ["natural", "split"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solve(lair, precision, ordering, nrhs, aligned):
    import torch
    print("case: replay", precision, ordering, nrhs, aligned, flush=True)
    w = W.implicit_euler_adr_3d(m=22, nrhs=1)
    kw = dict(interp="direct", precision=precision, ordering=ordering)
    hg, he = (lair.setup(w["rowptr"], w["col"], w["val"], graphs=g, **kw) for g in (True, False))
    shape = (w["n"],) if nrhs == 1 else (w["n"], nrhs)
    b, x = _vector(torch, shape, aligned), _vector(torch, shape, aligned)
    _compare(lair, lambda b, x: hg.solve(b, x)[1], lambda b, x: he.solve(b, x)[1], b, x, nrhs)
    hg.free()
    he.free()


# 97^2: level 0 is launched, the levels below run in one workgroup; the
# captured iterations outlive a new diagonal
@pytest.mark.parametrize("nrhs", [1, 4])
def test_transposed_solve_and_new_diagonals(lair, nrhs):
    import torch
    print("case: transposed replay", nrhs, flush=True)
    w = W.workload_c4(97)
    pos = np.flatnonzero(np.repeat(np.arange(w["n"]), np.diff(w["rowptr"])) == w["col"])
    hg, he = (lair.setup(w["rowptr"], w["col"], w["val"], graphs=g, interp="direct")
              for g in (True, False))
    assert hg.level_stats(0)["n"] > 4608
    shape = (w["n"],) if nrhs == 1 else (w["n"], nrhs)
    b, x = _vector(torch, shape, True), _vector(torch, shape, True)
    rng = np.random.default_rng(8)
    for k in range(3):
        if k:
            d = w["val"][pos] + rng.uniform(0.1, 2.0, w["n"])
            hg.update_diag(d)
            he.free()
            he = lair.setup(w["rowptr"], w["col"], w["val"], graphs=False, interp="direct")
            he.update_diag(d)
        _compare(lair, lambda b, x: hg.solve_transpose(b, x)[1],
                 lambda b, x: he.solve_transpose(b, x)[1], b, x, k)
        _compare(lair, lambda b, x: hg.solve(b, x)[1], lambda b, x: he.solve(b, x)[1], b, x, k)
    hg.free()
    he.free()


# systems that stop at different iterations, one of them above the size of a
# workgroup's levels; new diagonals renew their packed levels and blocks
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kw", [dict(interp="direct"), dict(distance=2, split="pmis")],
                         ids=["direct", "pmis"])
def test_batch_and_new_diagonals(lair, kw, precision):
    import torch
    print("case: batch replay", kw, precision, flush=True)
    rng = np.random.default_rng(9)
    systems = [W.adr_2d(m, eps, rng.uniform(0, 6), rng.uniform(0, 1))
               for m, eps in ((101, 1e-4), (12, 1e-1), (67, 1e-2), (40, 1e-3))]
    mats = [(w["rowptr"], w["col"], w["val"]) for w in systems]
    diag = np.concatenate([w["val"][np.repeat(np.arange(w["n"]), np.diff(w["rowptr"])) == w["col"]]
                           for w in systems])
    make = lambda g: lair.setup_batch(mats, graphs=g, precision=precision, **kw)
    hg, he = make(True), make(False)
    b, x = _vector(torch, (hg.n,), True), _vector(torch, (hg.n,), True)

    def solve(h):
        def run(b, x):
            info = h.solve_batch(b, x)[1]
            return dict(info, iters=info["sys_iters"])
        return run

    for k in range(3):
        if k:
            d = diag + rng.uniform(0.1, 2.0, hg.n)
            hg.update_diag(d)
            he.free()
            he = make(False)
            he.update_diag(d)
        _compare(lair, solve(hg), solve(he), b, x, k)
        # the solution of the new systems: each one's own residual
        at = 0
        for w in systems:
            n = w["n"]
            r = b[at:at + n].cpu().numpy().copy()
            xs = x[at:at + n].cpu().numpy()
            v = w["val"].copy()
            if k:
                v[np.repeat(np.arange(n), np.diff(w["rowptr"])) == w["col"]] = d[at:at + n]
            r0 = np.linalg.norm(r)
            r -= np.add.reduceat(v * xs[w["col"]], w["rowptr"][:-1])
            assert np.linalg.norm(r) <= 1e-10 * (1 + 1e-6) * r0
            at += n
    hg.free()
    he.free()

