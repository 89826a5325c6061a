"""GPU: the small levels of a cycle in one workgroup against the same levels
launched kernel by kernel.

A cycle of the allocation-free entry point on a fresh hierarchy launches
every level (the workgroup's packed operators are made by the calls that may
allocate), so it is the reference: every row is summed by as many lanes in
the same order, and the results must be equal bit for bit.  The transposed
cycle is compared with the oracle's (1e-11 of the largest entry, the
tolerance of the existing adjoint tests)."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from oracle import lair as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lair():
    import torch
    import paper_1708_06065_amd as lair
    assert torch.cuda.is_available()
    lair.load_library()
    return lair


def _adr(m):
    w = W.workload_c4(m)
    A = (sp.csr_matrix((w["val"], w["col"], w["rowptr"]), shape=(w["n"],) * 2)
         + sp.diags(w["c"])).tocsr()
    A.sort_indices()
    return dict(rowptr=A.indptr.astype(np.int32), col=A.indices.astype(np.int32), val=A.data)


# sizes: level 0 inside the workgroup, its largest row count (4,608), one
# above; a hierarchy of many levels; rows far longer than a lane's first
# entries (400 x 60 entries, 24,400 in all, and the levels below); a coarsest
# grid above one wave's rows; the nodal sweeps
CASES = {
    "transport24": (lambda: W.workload_c1(24), {}),
    "transport_4608": (lambda: W.chain_1d(4608), dict(max_coarse=10)),
    "transport_4609": (lambda: W.chain_1d(4609), dict(max_coarse=10)),
    "adr40_direct": (lambda: _adr(40), dict(interp="direct")),
    "adr61_distance2": (lambda: _adr(61), dict(distance=2, omega=0.8)),
    "long_rows": (lambda: W.random_ff_digraph(400, 60, 5), dict(interp="direct", max_coarse=20)),
    "coarse190": (lambda: _adr(20), dict(max_coarse=192)),
    "nodal": (lambda: W.workload_dgu(6, 1e-3),
              dict(distance=2, block_size=6, nodal=True)),
}


@pytest.mark.parametrize("nrhs", [1, 2, 8, 32])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", list(CASES))
def test_one_workgroup_equals_launches(lair, name, precision, nrhs):
    import torch
    print("case: tail", name, precision, nrhs, flush=True)
    make, kw = CASES[name]
    w = make()
    h = lair.setup(w["rowptr"], w["col"], w["val"], precision=precision, **kw)
    n = len(w["rowptr"]) - 1
    rng = np.random.default_rng(nrhs)
    shape = (n,) if nrhs == 1 else (n, nrhs)
    b = torch.as_tensor(rng.standard_normal(shape), device="cuda")
    x0 = torch.as_tensor(rng.standard_normal(shape), device="cuda")
    launched = h.cycle_noalloc(b, x0.clone())
    tail = h.cycle(b, x0.clone())
    assert torch.isfinite(tail).all()
    assert torch.equal(launched, tail)
    lair.profile_begin(["tail"])
    again = h.cycle_noalloc(b, x0.clone())
    h.cycle(b, torch.zeros_like(b))
    prof = lair.profile_end()
    assert prof["tail"]["launches"] == 2          # it is what ran
    assert torch.equal(launched, again)
    h.free()


@pytest.mark.parametrize("nrhs", [1, 4])
@pytest.mark.parametrize("name", ["transport24", "adr40_direct", "adr61_distance2", "long_rows"])
def test_transposed_tail_against_oracle(lair, name, nrhs):
    import torch
    print("case: transposed tail", name, nrhs, flush=True)
    make, kw = CASES[name]
    w = make()
    A = O.csr(w["rowptr"], w["col"], w["val"])
    okw = dict(kw)
    okw["interp"] = O.INTERP_DIRECT if kw.get("interp") == "direct" else O.INTERP_ONE_POINT
    omega = okw.pop("omega", 1.0)
    H = O.setup(A, **okw)
    cfl = [l.cf for l in H.levels[:-1]]
    h = lair.setup(w["rowptr"], w["col"], w["val"], cf_levels=cfl, **kw)
    n = A.shape[0]
    rng = np.random.default_rng(7)
    g = rng.standard_normal((n, nrhs))
    shape = (n,) if nrhs == 1 else (n, nrhs)
    lam = torch.zeros(shape, dtype=torch.float64, device="cuda")
    lair.profile_begin(["tail"])
    h.cycle_transpose(torch.as_tensor(g.reshape(shape), device="cuda"), lam)
    prof = lair.profile_end()
    assert prof["tail"]["launches"] == 1
    lam = lam.cpu().numpy().reshape(n, nrhs)
    for q in range(nrhs):
        ref = O.cycle_transpose(H, g[:, q], np.zeros(n), omega=omega)
        assert np.abs(lam[:, q] - ref).max() <= 1e-11 * np.abs(ref).max()
    h.free()


# one cycle of a batch from zero is x = B b whichever way it runs: the batch
# solve runs each system's small levels in a workgroup of its own, the cycle
# call launches every level over the union.  Grids of 1 to 10,201 rows: a
# system that is its coarsest grid, one whose largest level just fits a
# workgroup (67^2 = 4,489 rows) and one that does not (68^2 = 4,624)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kw", [dict(interp="direct"), dict(distance=2, omega=0.9),
                                dict(interp="direct", split="pmis", max_coarse=40),
                                dict(split="pmis", lump_tol=1e-3)],
                         ids=["direct", "distance2", "pmis", "pmis_lumped"])
@pytest.mark.parametrize("sizes", [(1, 8, 11, 23), (67, 3, 68), (101, 12, 67, 40, 40, 31)],
                         ids=["small", "edge", "uneven"])
def test_batch_workgroups_equal_launches(lair, sizes, kw, precision):
    import torch
    print("case: batch tail", sizes, kw, precision, flush=True)
    rng = np.random.default_rng(3)
    systems = [W.adr_2d(m, 10.0 ** rng.uniform(-4, -1), rng.uniform(0, 6), rng.uniform(0, 1))
               for m in sizes]
    h = lair.setup_batch([(w["rowptr"], w["col"], w["val"]) for w in systems],
                         precision=precision, **kw)
    b = torch.as_tensor(rng.standard_normal(h.n), device="cuda")
    launched = h.cycle(b, torch.zeros_like(b))
    lair.profile_begin(["tail"])
    x, info = h.solve_batch(b, maxit=1)
    prof = lair.profile_end()
    assert prof["tail"]["launches"] == 1
    assert torch.isfinite(x).all() and torch.equal(launched, x)
    for _ in range(30):           # the last of them replay a captured iteration
        again, _ = h.solve_batch(b, maxit=1)
        assert torch.equal(x, again)
    h.free()


def test_new_diagonal_reaches_every_kept_copy(lair):
    """A new diagonal leaves packed operators, transposes and captured
    iterations in place and renews their values: after three diagonals, each
    solved often enough that iterations are replayed, every solve equals that
    of a hierarchy which never met another diagonal, bit for bit."""
    import torch
    A0 = W.workload_c4(40)
    n = A0["n"]
    pos = np.flatnonzero(np.repeat(np.arange(n), np.diff(A0["rowptr"])) == A0["col"])
    rng = np.random.default_rng(1)
    diags = [A0["val"][pos] + rng.uniform(0.1, 2.0, n) for _ in range(3)]
    b = torch.as_tensor(rng.standard_normal(n), device="cuda")
    x = torch.zeros_like(b)
    for precision in ("fp64", "mixed"):
        print("case: new diagonal, kept copies", precision, flush=True)
        mk = dict(interp="direct", precision=precision)
        kept = lair.setup(A0["rowptr"], A0["col"], A0["val"], **mk)
        for k, d in enumerate(diags):
            kept.update_diag(d)
            fresh = lair.setup(A0["rowptr"], A0["col"], A0["val"], graphs=False, **mk)
            fresh.update_diag(d)
            for rep in range(5):
                for solve, ref in ((kept.solve, fresh.solve),
                                   (kept.solve_transpose, fresh.solve_transpose)):
                    x.zero_()
                    solve(b, x)
                    want, _ = ref(b)
                    assert torch.equal(x, want), (k, rep)
            z = torch.zeros_like(b)
            assert torch.equal(kept.cycle(b, z), fresh.cycle(b, torch.zeros_like(b)))
            kept.update_diag(d)       # the allocation-free cycle right after an update
            assert torch.equal(kept.cycle_noalloc(b, torch.zeros_like(b)), z)
            fresh.free()
        kept.free()
