"""GPU: the one-pass Gram-Schmidt kernels of flexible GMRES at the edges of
their range (a thread holds up to 24 basis vectors; longer bases take the
separate kernels), against the oracle's fgmres_cycle: the same number of steps
and the solution within 1e-8, the bars of the other FGMRES tests."""
import numpy as np
import pytest

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


# restarts one below, at and above the 24 vectors, and a basis that grows to
# twice that (about 50 steps at this strength threshold); 961 rows: a last
# block that is part full
@pytest.mark.parametrize("restart", [1, 23, 24, 25, 64])
@pytest.mark.parametrize("nrhs", [1, 2, 32])
def test_basis_lengths(lair, restart, nrhs):
    import torch
    print("case: gram-schmidt", restart, nrhs, flush=True)
    w = W.adr_2d(31, 1e-1, 0.5, 0.0)
    A = O.csr(w["rowptr"], w["col"], w["val"])
    kw = dict(theta=0.9, max_coarse=20)
    if restart == 1:
        kw = dict(max_coarse=20)               # steepest steps need a good cycle
    H = O.setup(A, **kw)
    h = lair.setup(w["rowptr"], w["col"], w["val"], cf_levels=[l.cf for l in H.levels[:-1]], **kw)
    rng = np.random.default_rng(restart)
    B = rng.standard_normal((961, nrhs))
    b = torch.as_tensor(B[:, 0].copy() if nrhs == 1 else B, device="cuda")
    x, info = h.solve_fgmres(b, rtol=1e-10, restart=restart, maxit=400)
    x = x.cpu().numpy().reshape(961, nrhs)
    assert info["converged"]
    steps = 0
    for q in range(0, nrhs, 7):
        xo, ito, _, _ = O.fgmres_cycle(H, B[:, q], rtol=1e-10, restart=restart, maxit=400)
        steps = max(steps, ito)
        assert np.linalg.norm(x[:, q] - xo) <= 1e-8 * np.linalg.norm(xo)
    if nrhs == 1:
        assert info["iters"] == steps
    assert info["iters"] >= steps
    h.free()
