"""GPU: direct interpolation on both sides of the row count from which a lane
takes a row: the rows of two copies of one matrix, together above it, have the
bits of the rows of one copy (and a small system), below it, where a team takes
a row."""
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


# entries per row: teams of 2, 4 and 8 lanes, rows shorter and longer than them
@pytest.mark.parametrize("offsets", [[1], [1, 2, 7], [-3, -1, 1, 2, 5, 9, 40]])
def test_same_bits(lair, offsets):
    print("case: interpolation", offsets, flush=True)
    n = 140000
    rng = np.random.default_rng(len(offsets))
    rows, cols = [], []
    for o in offsets:
        i = np.flatnonzero(rng.random(n) < 0.8)
        i = i[(i + o >= 0) & (i + o < n)]
        rows.append(i)
        cols.append(i + o)
    i = np.repeat([17, 5000, n - 1], 30)       # a few long rows
    rows.append(i)
    cols.append((i + 100 * (1 + np.arange(90))) % n)
    r, c = np.concatenate(rows), np.concatenate(cols)
    A = sp.csr_matrix((rng.uniform(-1.0, 0.4, len(r)), (r, c)), shape=(n, n))
    A.setdiag(0.0)
    A.eliminate_zeros()
    A = (A + sp.diags(rng.uniform(2.0, 3.0, n))).tocsr()
    A.sort_indices()
    cf = (rng.random(n) < 0.005).astype(np.int8)       # a coarsest grid of about 700 rows
    csr = (A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data)
    # two rows, one of them C, so that the small batch is one as well
    other = (np.array([0, 2, 4], np.int64), np.array([0, 1, 0, 1], np.int32),
             np.array([2.0, -1.0, -1.0, 2.0]))
    P = []
    for systems, types in (([csr, other], [cf, [1, 0]]), ([csr, csr], [cf, cf])):
        h = lair.setup_batch(systems, interp="direct", max_levels=2, max_coarse=1,
                             cf_levels=[np.concatenate(types).astype(np.int8)])
        P.append([np.asarray(h.export(0, "P." + x)) for x in ("rowptr", "col", "val")])
        h.free()
    (rp, cj, v), (rp2, cj2, v2) = P
    nc, nz = int(cf.sum()), int(rp[n])
    rp, cj, v = rp[:n + 1], cj[:nz], v[:nz]
    assert nz > nc
    assert np.array_equal(rp2, np.concatenate([rp, rp[1:] + nz]))
    assert np.array_equal(cj2, np.concatenate([cj, cj + nc]))
    assert np.array_equal(v2, np.concatenate([v, v]))
