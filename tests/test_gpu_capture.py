"""GPU: cycles recorded into a caller's own graph.  The graph is replayed
several times with eager calls and synchronizations between, and every replay
is compared with the eager call bit for bit."""
import contextlib
import gc

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lair():
    import torch
    import paper_1708_06065_amd as lair
    assert torch.cuda.is_available()
    lair.load_library()
    return lair


@contextlib.contextmanager
def _recording(torch, graph, **kw):
    """Record into graph with the garbage collector off: hierarchies and graphs
    that earlier tests left in reference cycles wait for the device when they
    are collected, which must not happen inside a capture."""
    gc.collect()
    gc.disable()
    try:
        with torch.cuda.graph(graph, **kw):
            yield
    finally:
        gc.enable()


def _diagonals(w, k):
    """k diagonals for the workload's matrix, each larger than the last."""
    pos = np.flatnonzero(np.repeat(np.arange(w["n"]), np.diff(w["rowptr"])) == w["col"])
    rng = np.random.default_rng(2)
    return [w["val"][pos] + 2.0 * i + rng.uniform(0.1, 2.0, w["n"]) for i in range(k)]


# 40^2: every level in one workgroup; 97^2: launched levels above it
@pytest.mark.parametrize("m", [40, 97])
def test_transposed_cycle_captured_after_a_new_diagonal(lair, m):
    """Recording a transposed cycle right after a new diagonal leaves no call
    with the old diagonal's transposes: not the next eager one, and no replay."""
    import torch
    w = W.workload_c4(m)
    d1, d2 = _diagonals(w, 2)
    args = (w["rowptr"], w["col"], w["val"])
    g = torch.as_tensor(np.random.default_rng(3).standard_normal(w["n"]), device="cuda")
    fresh = lair.setup(*args, interp="direct")
    fresh.update_diag(d2)
    want = fresh.cycle_transpose(g, torch.zeros_like(g))
    h = lair.setup(*args, interp="direct")
    h.update_diag(d1)
    h.cycle_transpose(g, torch.zeros_like(g))
    h.update_diag(d2)
    torch.cuda.synchronize()
    lam = torch.zeros_like(g)
    graph = torch.cuda.CUDAGraph()
    with _recording(torch, graph):
        lam.zero_()
        h.cycle_transpose(g, lam)
    assert torch.equal(h.cycle_transpose(g, torch.zeros_like(g)), want)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(lam, want)
        assert torch.equal(h.cycle_transpose(g, torch.zeros_like(g)), want)


def test_transposes_on_a_captured_stream_are_refused(lair):
    """When the stream of the new diagonal is itself captured the call fails,
    and the eager call after it is right."""
    import torch
    w = W.workload_c4(40)
    d1, d2 = _diagonals(w, 2)
    args = (w["rowptr"], w["col"], w["val"])
    g = torch.as_tensor(np.random.default_rng(3).standard_normal(w["n"]), device="cuda")
    fresh = lair.setup(*args, interp="direct")
    fresh.update_diag(d2)
    want = fresh.cycle_transpose(g, torch.zeros_like(g))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        h = lair.setup(*args, interp="direct")
        h.update_diag(d1)
        h.cycle_transpose(g, torch.zeros_like(g))
        h.update_diag(d2)
    s.synchronize()
    lam = torch.zeros_like(g)
    graph = torch.cuda.CUDAGraph()
    with _recording(torch, graph, stream=s):
        lam.zero_()
        with pytest.raises(lair.LairError) as e:
            h.cycle_transpose(g, lam)
    assert e.value.status == -3
    del e                    # its traceback holds this frame, and so the graph
    with torch.cuda.stream(s):
        got = h.cycle_transpose(g, torch.zeros_like(g))
    s.synchronize()
    assert torch.equal(got, want)


# 40^2: every level in one workgroup; 97^2: launched levels above it.  A graph
# recorded before the workgroup's operators are packed, or after a new
# diagonal has made them old, holds launches for every level: the same bits
@pytest.mark.parametrize("nrhs", [1, 4])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("m", [40, 97])
def test_cycle_in_a_callers_graph(lair, m, precision, nrhs):
    import torch
    print("case: captured cycle", m, precision, nrhs, flush=True)
    w = W.workload_c4(m)
    args = (w["rowptr"], w["col"], w["val"])
    rng = np.random.default_rng(m)
    shape = (w["n"],) if nrhs == 1 else (w["n"], nrhs)
    b, z = torch.zeros(shape, dtype=torch.float64, device="cuda"), torch.zeros(
        shape, dtype=torch.float64, device="cuda")
    h = lair.setup(*args, interp="direct", precision=precision)

    def check(call):
        graph = torch.cuda.CUDAGraph()
        with _recording(torch, graph):
            z.zero_()
            call(b, z)
        for _ in range(3):
            b.copy_(torch.as_tensor(rng.standard_normal(shape), device="cuda"))
            graph.replay()
            torch.cuda.synchronize()
            got = z.clone()
            assert torch.equal(got, h.cycle(b, torch.zeros_like(b)))
            assert torch.isfinite(got).all()

    h.cycle_noalloc(b, z)             # the scratch array's address is known
    torch.cuda.synchronize()
    check(h.cycle_noalloc)            # recorded before anything is packed
    check(h.cycle)                    # with the workgroup
    check(h.cycle_noalloc)
    h.update_diag(_diagonals(w, 1)[0])
    check(h.cycle)                    # packed from the old diagonal
    check(h.cycle)                    # and packed again
    h.free()
