"""GPU: a batch solve that runs out of memory (LAIR_DEBUG_MAX_BYTES) at any of
its allocations leaves a hierarchy that solves once there is memory, bit for
bit as one that never failed."""
import re

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


def _block(size):
    """Bytes the library's cache holds for a request."""
    if size > 1 << 20:
        return -(-size // (2 << 20)) * (2 << 20)
    return max(512, 1 << (size - 1).bit_length())


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_every_allocation_of_a_batch_solve(lair, monkeypatch, precision):
    import torch
    trim = lair.load_library().lair_trim
    rng = np.random.default_rng(2)
    systems = [W.adr_2d(m, 1e-3, rng.uniform(0, 6), 0.5) for m in (70, 20, 6)]
    make = lambda: lair.setup_batch([(w["rowptr"], w["col"], w["val"]) for w in systems],
                                    interp="direct", precision=precision)
    b = torch.as_tensor(rng.standard_normal(sum(w["n"] for w in systems)), device="cuda")
    h = make()
    want = h.solve_batch(b)[0]
    h.free()
    held, failed = 0, 0
    while True:
        # one more allocation fits than the time before
        h = make()
        trim()
        base = lair.memory()[0]
        monkeypatch.setenv("LAIR_DEBUG_MAX_BYTES", str(base + held))
        try:
            got = h.solve_batch(b)[0]
        except lair.LairError as e:
            assert e.status == -2
            got, text = None, str(e)
        monkeypatch.delenv("LAIR_DEBUG_MAX_BYTES")
        print("case: cap", precision, held, flush=True)
        assert got is None or torch.equal(got, want)
        assert torch.equal(h.solve_batch(b)[0], want)
        h.free()
        if got is not None:
            break
        failed += 1
        size, used = (int(v) for v in re.search(
            r"allocation of (\d+) bytes refused: (\d+) bytes in use", text).groups())
        held = used - base + _block(size)
    assert failed > 20
