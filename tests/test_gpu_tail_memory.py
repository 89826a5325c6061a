"""GPU: the packed operators of the small levels are optional.  With an
allocation cap (LAIR_DEBUG_MAX_BYTES) that everything but the pack fits under,
cycles and solves run launch by launch and give the same bits."""
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


def _without_pack(lair, monkeypatch, make, call):
    """call(hierarchy) with all memory, and with one byte less than it holds
    afterwards, its last allocation being the pack's: both results and whether
    the second ran a tail.  (The cache is emptied before each call, so that
    equal requests hold equal blocks.)"""
    trim = lair.load_library().lair_trim
    full = make()
    trim()
    before = lair.memory()[0]
    want = call(full)
    need = lair.memory()[0] - before
    full.free()
    h = make()
    trim()
    base = lair.memory()[0]
    monkeypatch.setenv("LAIR_DEBUG_MAX_BYTES", str(base + need - 1))
    got = call(h)
    assert lair.memory()[0] < base + need - 1
    monkeypatch.delenv("LAIR_DEBUG_MAX_BYTES")
    lair.profile_begin(["tail"])
    call(h)                      # nor does it ask for the pack again
    prof = lair.profile_end()
    h.free()
    return want, got, "tail" in prof


@pytest.mark.parametrize("kind", ["cycle", "solve", "cycle_transpose", "solve_transpose"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_single_system(lair, monkeypatch, precision, kind):
    import torch
    print("case: no memory for the tail", precision, kind, flush=True)
    w = W.workload_c4(60)
    b = torch.as_tensor(np.random.default_rng(4).standard_normal(w["n"]), device="cuda")

    def call(h):
        if kind == "solve":
            return h.solve(b)[0]
        if kind == "solve_transpose":
            return h.solve_transpose(b)[0]
        return getattr(h, kind)(b, torch.zeros_like(b))

    want, got, tail = _without_pack(
        lair, monkeypatch, lambda: lair.setup(w["rowptr"], w["col"], w["val"], interp="direct",
                                              precision=precision), call)
    assert not tail and torch.equal(want, got)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch(lair, monkeypatch, precision):
    import torch
    print("case: no memory for a batch's tails", precision, flush=True)
    rng = np.random.default_rng(5)
    systems = [W.adr_2d(m, 1e-3, rng.uniform(0, 6), rng.uniform(0, 1)) for m in (71, 30, 12, 40)]
    b = torch.as_tensor(rng.standard_normal(sum(w["n"] for w in systems)), device="cuda")
    want, got, tail = _without_pack(
        lair, monkeypatch, lambda: lair.setup_batch([(w["rowptr"], w["col"], w["val"])
                                                     for w in systems],
                                                    interp="direct", precision=precision),
        lambda h: h.solve_batch(b)[0])
    assert not tail and torch.equal(want, got)
