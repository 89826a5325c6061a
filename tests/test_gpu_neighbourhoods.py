"""GPU: neighbourhoods at distance two around the size of the table that holds
their members (8 T for the team of T lanes that the longest row asks for):
below it, at it and above it, where the lists are merged instead; and the
limit of 256 merged rows."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lair():
    import torch
    import paper_1708_06065_amd as lair
    assert torch.cuda.is_available()
    lair.load_library()
    return lair


def _trees(groups, seed):
    """Per group (t, u) a C-point with t strong F-neighbours, each with u
    strong F-neighbours of its own, and one F-point that all of these share:
    N has t (u + 1) + (u > 0) members.  Points are numbered at random."""
    rng = np.random.default_rng(seed)
    n = sum(1 + t * (u + 1) + (u > 0) for t, u in groups)
    at = rng.permutation(n)
    rows, cols, sets, o = [], [], {}, 0
    cf = np.zeros(n, dtype=np.int8)
    for t, u in groups:
        c, f = at[o], at[o + 1:o + 1 + t]
        g = at[o + 1 + t:o + 1 + t + t * u].reshape(t, u)
        shared = at[o + 1 + t + t * u:o + 1 + t * (u + 1) + (u > 0)]
        o += 1 + t * (u + 1) + (u > 0)
        cf[c] = 1
        for a in range(t):
            rows.append(c)
            cols.append(f[a])
            for b in list(g[a]) + list(shared):
                rows.append(f[a])
                cols.append(b)
        sets[c] = np.sort(np.concatenate([f, g.ravel(), shared]).astype(np.int64))
    A = sp.csr_matrix((-np.ones(len(rows)), (rows, cols)), shape=(n, n))
    A = (A + sp.diags(np.full(n, 400.0))).tocsr()
    A.sort_indices()
    return A, cf, sets


# the longest row is max(t, u + 1) + 1: teams of 4 (rows up to 15), 8, 32, 64
GROUPS = {
    "T4": [(0, 0), (1, 0), (1, 3), (5, 5), (10, 2), (6, 4), (3, 9), (7, 4), (8, 6), (2, 14)],
    "T8": [(9, 6), (10, 5), (20, 2), (21, 2), (21, 3), (31, 1), (5, 1)],
    "T32": [(127, 0), (127, 1), (125, 1), (85, 2), (84, 2), (40, 40), (1, 100)],
    "T64": [(255, 0), (255, 1), (170, 2), (204, 2), (128, 3), (127, 3), (3, 200)],
}


@pytest.mark.parametrize("name", list(GROUPS))
def test_members_around_the_table(lair, name):
    print("case: neighbourhoods", name, flush=True)
    A, cf, sets = _trees(GROUPS[name], 3)
    h = lair.setup(A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                   cf_levels=[cf], distance=2, max_levels=2, max_coarse=1)
    ptr, nbr = h.export(0, "nbr_ptr"), h.export(0, "nbr")
    for k, c in enumerate(np.flatnonzero(cf == 1)):
        assert np.array_equal(nbr[ptr[k]:ptr[k + 1]], sets[c]), (name, c)
    h.free()


def test_more_than_256_rows_are_refused(lair):
    print("case: 256 neighbours", flush=True)
    A, cf, _ = _trees([(256, 0), (4, 2)], 5)
    with pytest.raises(lair.LairError, match="256"):
        lair.setup(A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                   cf_levels=[cf], distance=2, max_levels=2, max_coarse=1)
