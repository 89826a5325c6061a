"""GPU: many small systems run launch by launch, few of them in workgroups of
their own (the rule weighs the workgroups of a CU against the launches they
replace); either way one iteration from zero is the union's cycle, bit for
bit."""
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


# coarsest grids alone; two levels; the first with a few larger systems beside
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes,tail", [((4,) * 20, True), ((4,) * 1500, False),
                                        ((13,) * 20, True), ((13,) * 2000, False),
                                        ((4,) * 1500 + (60, 60), True)],
                         ids=["20x4", "1500x4", "20x13", "2000x13", "1500x4+2x60"])
def test_rule(lair, sizes, tail, precision):
    import torch
    print("case: batch rule", len(sizes), sizes[0], precision, flush=True)
    made = {m: W.adr_2d(m, 1e-3, 0.1 * m, 0.5) for m in set(sizes)}
    h = lair.setup_batch([(made[m]["rowptr"], made[m]["col"], made[m]["val"]) for m in sizes],
                         interp="direct", precision=precision)
    b = torch.as_tensor(np.random.default_rng(1).standard_normal(h.n), device="cuda")
    want = h.cycle(b, torch.zeros_like(b))
    lair.profile_begin(["tail"])
    x, _ = h.solve_batch(b, maxit=1)
    assert ("tail" in lair.profile_end()) == tail
    assert torch.isfinite(x).all() and torch.equal(x, want)
    h.free()
