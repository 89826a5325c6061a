"""GPU: the transposed cycle where levels are launched above the workgroup that
takes the small ones, against the oracle's (1e-11 of the largest entry, the
tolerance of the other transposed cycles), before and after a new diagonal."""
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


# 97^2 = 9,409 rows (the workgroup takes levels of up to 4,608); omega other
# than one shows in the first sweep, which has a kernel of its own
@pytest.mark.parametrize("nrhs", [1, 4])
@pytest.mark.parametrize("kw", [dict(), dict(interp="direct", omega=0.8), dict(distance=2)],
                         ids=["one_point", "direct", "distance2"])
def test_against_oracle(lair, kw, nrhs):
    import torch
    print("case: transposed launches", kw, nrhs, flush=True)
    w = W.workload_c4(97)
    A = (O.csr(w["rowptr"], w["col"], w["val"]) + sp.diags(w["c"])).tocsr()
    A.sort_indices()
    okw = dict(kw)
    okw["interp"] = O.INTERP_DIRECT if kw.get("interp") == "direct" else O.INTERP_ONE_POINT
    omega = okw.pop("omega", 1.0)
    H = O.setup(A, **okw)
    h = lair.setup(A.indptr, A.indices, A.data, cf_levels=[l.cf for l in H.levels[:-1]], **kw)
    n = A.shape[0]
    assert n > 4608
    rng = np.random.default_rng(nrhs)
    g, l0 = rng.standard_normal((2, n, nrhs))
    shape = (n,) if nrhs == 1 else (n, nrhs)
    for k in range(3):
        if k:
            d = A.diagonal() * (1.0 + rng.random(n))
            h.update_diag(d)
            O.update_diag(H, d)
        lam = torch.as_tensor(l0.reshape(shape), device="cuda").clone()
        lair.profile_begin(["tail"])
        h.cycle_transpose(torch.as_tensor(g.reshape(shape), device="cuda"), lam)
        assert lair.profile_end()["tail"]["launches"] == 1
        lam = lam.cpu().numpy().reshape(n, nrhs)
        for q in range(nrhs):
            ref = O.cycle_transpose(H, g[:, q], l0[:, q].copy(), omega=omega)
            assert np.abs(lam[:, q] - ref).max() <= 1e-11 * np.abs(ref).max(), (k, q)
    h.free()
