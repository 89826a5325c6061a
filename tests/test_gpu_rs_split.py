"""GPU: the classical first pass on the host against the oracle's, at the edges
of the sets that hold the points of one measure (64 and 4096 points a summary
word, measures of 64 and more in a heap of their own)."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import lair as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lair():
    import torch
    import paper_1708_06065_amd as lair
    assert torch.cuda.is_available()
    lair.load_library()
    return lair


def _graph(n, hubs, seed):
    """A path with random long edges; each of `hubs` points (point, dependents)
    has rows that depend on it."""
    rng = np.random.default_rng(seed)
    i = np.arange(1, n)
    rows, cols = [i, rng.integers(0, n, n // 2)], [i - 1, rng.integers(0, n, n // 2)]
    for p, d in hubs:
        rows.append(rng.choice(n, d, replace=False))
        cols.append(np.full(d, p))
    r, c = np.concatenate(rows), np.concatenate(cols)
    A = sp.csr_matrix((np.ones(len(r)), (r, c)), shape=(n, n))
    A.data[:] = -1.0
    A.setdiag(0.0)
    A.eliminate_zeros()
    A = (A + sp.diags(np.full(n, 20.0))).tocsr()
    A.sort_indices()
    return A


@pytest.mark.parametrize("n,hubs", [(1, []), (2, []), (63, []), (64, []), (65, []), (4096, []),
                                    (4097, []), (300, [(7, 61), (9, 62), (11, 63), (13, 64)]),
                                    (2000, [(5, 70), (1999, 200), (1000, 200), (3, 63)])])
def test_first_pass(lair, n, hubs):
    print("case: first pass", n, hubs, flush=True)
    A = _graph(n, hubs, n)
    h = lair.setup(A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                   max_levels=2, max_coarse=1)
    if h.nlevels > 1:
        assert np.array_equal(h.export(0, "cf"), O.rs_split(A, O.strength(A, 0.25)))
    else:
        assert n <= 2
    h.free()
