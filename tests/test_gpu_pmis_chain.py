"""GPU: the parallel splitting where decisions wait for one another in chains
longer than one launch follows."""
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


def _chain(L):
    """Point j < L depends on j - 1 only; L more rows make point j's weight
    L - j (row L + d depends on the first L - d points), so the points of the
    chain are decided one after the other: C, F, C, F, ..."""
    A = sp.lil_matrix((2 * L, 2 * L))
    for j in range(1, L):
        A[j, j - 1] = -1.0
    for d in range(L):
        A[L + d, :L - d] = -1.0
    A = (A.tocsr() + sp.diags(np.full(2 * L, 2.0 * L))).tocsr()
    A.sort_indices()
    return A


@pytest.mark.parametrize("L", [1, 2, 13, 40, 300])
def test_split_along_a_chain(lair, L):
    print("case: chain", L, flush=True)
    A = _chain(L)
    cf = O.pmis_split(A, O.strength(A, 0.25))
    assert np.array_equal(cf[:L], np.arange(L) % 2 == 0)
    h = lair.setup(A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                   interp="one_point", split="pmis", max_levels=2, max_coarse=1)
    if h.nlevels > 1:
        assert np.array_equal(h.export(0, "cf"), cf)
    else:
        assert L == 1
    h.free()
