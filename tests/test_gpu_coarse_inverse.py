"""GPU: the coarsest grid's inverse by Gauss-Jordan elimination in registers at
the edges of its range (up to 128 rows, for one grid and for the systems of a
batch)."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def lair():
    import torch
    import paper_1708_06065_amd as lair
    assert torch.cuda.is_available()
    lair.load_library()
    return lair


def _dense(n, seed):
    """A dense n x n system in CSR whose large entries stand off the diagonal,
    so that nearly every step takes its pivot from another row."""
    rng = np.random.default_rng(seed)
    M = rng.standard_normal((n, n)) / (4.0 * np.sqrt(n))
    M += np.eye(n)[rng.permutation(n)]
    A = sp.csr_matrix(M)
    return M, (A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data)


def _bound(M):
    """Gauss-Jordan's forward error, a small multiple of n eps cond(M)."""
    return 8.0 * len(M) * EPS * np.linalg.cond(M)


SIZES = [1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129]


@pytest.mark.parametrize("n", SIZES)
def test_inverse_of_one_grid(lair, n):
    import torch
    print("case: inverse", n, flush=True)
    M, csr = _dense(n, n)
    h = lair.setup(*csr, max_levels=1, max_coarse=256)
    assert h.nlevels == 1
    b = np.random.default_rng(1).standard_normal(n)
    bd = torch.as_tensor(b, device="cuda")
    x = h.cycle(bd, torch.zeros_like(bd)).cpu().numpy()
    ref = np.linalg.solve(M, b)
    assert np.linalg.norm(x - ref) <= _bound(M) * np.linalg.norm(ref)
    h.free()


def test_inverses_of_a_batch(lair):
    import torch
    print("case: inverses of a batch", flush=True)
    sys_ = [_dense(n, 100 + n) for n in SIZES]
    hb = lair.setup_batch([c for _, c in sys_], max_levels=1, max_coarse=256)
    assert hb.nlevels == 1
    b = np.random.default_rng(2).standard_normal(sum(SIZES))
    bd = torch.as_tensor(b, device="cuda")
    x = hb.cycle(bd, torch.zeros_like(bd)).cpu().numpy()
    lo = 0
    for M, _ in sys_:
        n = len(M)
        ref = np.linalg.solve(M, b[lo:lo + n])
        assert np.linalg.norm(x[lo:lo + n] - ref) <= _bound(M) * np.linalg.norm(ref), n
        lo += n
    hb.free()


@pytest.mark.parametrize("n,k", [(1, 0), (64, 63), (100, 40), (128, 127)])
def test_singular_grid_is_refused(lair, n, k):
    """Column k is zero but for an explicit zero on the diagonal."""
    print("case: singular", n, k, flush=True)
    M, _ = _dense(n, n)
    M[:, k] = 0.0
    full = (np.arange(n + 1, dtype=np.int64) * n, np.tile(np.arange(n, dtype=np.int32), n),
            M.ravel().copy())
    with pytest.raises(lair.LairError):
        lair.setup(*full, max_levels=1, max_coarse=256)
    with pytest.raises(lair.LairError):
        lair.setup_batch([_dense(5, 1)[1], full], max_levels=1, max_coarse=256)
