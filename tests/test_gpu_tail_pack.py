"""GPU: packing the small levels where a lane's share of a row is longer than
what it fetches at once (16 entries), ends just before, at or after a multiple
of that, or has no entry at all; and hierarchies with more row sets than one
launch packs (32).  Cycles are compared bit for bit with launched ones
(cycle_noalloc on a hierarchy that has packed nothing), transposed ones with
the oracle's (1e-11 of the largest entry)."""
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


def _hubs(n, lengths):
    """A chain with some long rows and long columns, diagonally dominant."""
    rng = np.random.default_rng(n)
    A = sp.diags([-0.5 * np.ones(n - 1), -0.3 * np.ones(n - 1)], [1, -1]).tolil()
    for k, m in enumerate(lengths):
        i, js = (k + 1) * n // (len(lengths) + 2), rng.permutation(n)[:m]
        if k % 2:
            A[js, i] = -rng.uniform(0.01, 0.1, (m, 1))
        else:
            A[i, js] = -rng.uniform(0.01, 0.1, (1, m))
    A.setdiag(0)
    A = A.tocsr()
    A.eliminate_zeros()
    A = (A + sp.diags(np.asarray(abs(A).sum(1)).ravel() * 1.2 + 0.1)).tocsr()
    A.sort_indices()
    return A


CASES = {
    "shares of 14 to 19": (lambda: _hubs(400, (13, 14, 15, 16, 17, 18)), dict(max_coarse=20)),
    "shares of 31 to 34": (lambda: _hubs(700, (30, 31, 32, 33)), dict(max_coarse=40)),
    "rows of 500": (lambda: _hubs(2000, (500, 499, 501)), dict(max_coarse=100, interp="direct")),
    "many levels": (lambda: sp.csr_matrix((lambda w: (w["val"], w["col"], w["rowptr"]))(
        W.chain_1d(3000))), dict(max_coarse=2)),
}


@pytest.mark.parametrize("nrhs", [1, 4])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", list(CASES))
def test_pack(lair, name, precision, nrhs):
    import torch
    print("case: pack", name, precision, nrhs, flush=True)
    make, kw = CASES[name]
    A = make()
    n = A.shape[0]
    okw = dict(kw)
    okw["interp"] = O.INTERP_DIRECT if kw.get("interp") == "direct" else O.INTERP_ONE_POINT
    H = O.setup(A, **okw)
    h = lair.setup(A.indptr, A.indices, A.data, cf_levels=[l.cf for l in H.levels[:-1]],
                   precision=precision, **kw)
    assert name != "many levels" or 5 * (h.nlevels - 1) > 32
    rng = np.random.default_rng(3)
    shape = (n,) if nrhs == 1 else (n, nrhs)
    b, x0 = (torch.as_tensor(rng.standard_normal(shape), device="cuda") for _ in range(2))
    launched = h.cycle_noalloc(b, x0.clone())
    assert torch.isfinite(launched).all()
    assert torch.equal(h.cycle(b, x0.clone()), launched)
    g = b.cpu().numpy().reshape(n, nrhs)
    lam = h.cycle_transpose(b, torch.zeros_like(b)).cpu().numpy().reshape(n, nrhs)
    for q in range(nrhs if precision == "fp64" else 0):
        ref = O.cycle_transpose(H, g[:, q], np.zeros(n))
        assert np.abs(lam[:, q] - ref).max() <= 1e-11 * np.abs(ref).max()
    d = A.diagonal() * (1.0 + rng.random(n))
    h.update_diag(d)
    launched = h.cycle_noalloc(b, x0.clone())
    assert torch.equal(h.cycle(b, x0.clone()), launched)
    h.free()
