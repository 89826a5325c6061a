"""GPU: the node solves at the edges of their size classes (24, 40, 72 and 104
rows), with so few nodes that one class takes them all and with more (above
1024): the rows of R are those of separate solves of the scalar rows, bit for
bit, as every entry sees the same operations in the same order."""
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


def _stars(k, sizes, seed):
    """Groups of one C-node and t F-nodes, t in `sizes`, every node of a group
    coupled with every other by entries of one magnitude (so all are strong
    and the C-node's systems have t k rows); the diagonal is no larger than
    they are, so that rows are exchanged."""
    rng = np.random.default_rng(seed)
    blocks, cf = [], []
    for t in sizes:
        n = (t + 1) * k
        blocks.append(rng.choice([-1.0, 1.0], (n, n)) * rng.uniform(0.5, 1.0, (n, n)))
        cf += [1] * k + [0] * (t * k)
    A = sp.block_diag(blocks).tocsr()
    A.sort_indices()
    return A, np.array(cf, dtype=np.int8)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("k,more,largest",
                         [(k, 0, m) for k in (2, 3, 8) for m in (24, 40, 72, 104, 128)] +
                         [(2, 1025, 40), (2, 1025, 128)])
def test_size_classes(lair, monkeypatch, k, more, largest, precision):
    print("case: node sizes", k, more, largest, precision, flush=True)
    edges = [e for e in (24, 40, 64, 72, 104, 128) if e <= largest]
    sizes = sorted({0, 1} | {max(0, e // k + d) for e in edges for d in (-1, 0, 1)
                             if k * (e // k + d) <= largest})
    if more:
        sizes += [1] * (more - len(sizes))
    A, cf = _stars(k, sizes, k)
    R = {}
    for mode in ("rows", "nodes"):
        monkeypatch.delenv("LAIR_NODAL_ROW_SOLVES", raising=False)
        if mode == "rows":
            monkeypatch.setenv("LAIR_NODAL_ROW_SOLVES", "1")
        lair.profile_begin(["local_node"])
        h = lair.setup(A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                       cf_levels=[cf], block_size=k, nodal=True, max_levels=2, max_coarse=1,
                       precision=precision)
        prof = lair.profile_end()
        assert ("local_node" in prof) == (mode == "nodes")
        assert h.level_stats(0)["s_max"] == max(sizes) * k
        R[mode] = [h.export(0, "R." + x) for x in ("rowptr", "col", "val")]
        h.free()
    for a, b in zip(R["rows"], R["nodes"]):
        assert np.array_equal(a, b)
