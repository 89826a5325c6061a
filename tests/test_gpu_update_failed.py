"""GPU: a new diagonal that fails (a singular coarsest grid) leaves a
hierarchy that refuses cycles and solves, and the next one that succeeds makes
it as good as one that never failed, bit for bit, replayed iterations
included."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lair():
    import torch
    import paper_1708_06065_amd as lair
    assert torch.cuda.is_available()
    lair.load_library()
    return lair


# ones off the diagonal: with ones on it too, every row is the same
ONES = (np.arange(0, 17, 4, dtype=np.int32), np.tile(np.arange(4, dtype=np.int32), 4),
        np.where(np.eye(4, dtype=bool), 4.0, 1.0).reshape(-1))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nsys", [0, 1, 3])        # 0: lair_setup
def test_failed_update(lair, nsys, precision):
    import torch
    print("case: failed update", nsys, precision, flush=True)
    n = 4 * max(nsys, 1)
    make = (lambda: lair.setup(*ONES, precision=precision)) if nsys == 0 else \
        (lambda: lair.setup_batch([ONES] * nsys, precision=precision))
    b = torch.as_tensor(np.random.default_rng(6).standard_normal(n), device="cuda")
    x = torch.zeros_like(b)
    h = make()
    solve = (lambda h, x: h.solve(b, x)) if nsys == 0 else (lambda h, x: h.solve_batch(b, x))
    solve(h, x)                                  # a tail and a count of iterations exist
    bad = np.full(n, 4.0)
    bad[-4:] = 1.0
    with pytest.raises(lair.LairError) as e:
        h.update_diag(bad)
    assert e.value.status == -4
    calls = [lambda: h.cycle(b, x), lambda: h.cycle_noalloc(b, x), lambda: solve(h, x)]
    if nsys == 0:
        calls += [lambda: h.cycle_transpose(b, x), lambda: h.solve_transpose(b, x),
                  lambda: h.solve_fgmres(b, x)]
    x.fill_(7.0)
    for call in calls:
        with pytest.raises(lair.LairError) as e:
            call()
        assert e.value.status == -1
    torch.cuda.synchronize()
    assert bool((x == 7.0).all())
    good = np.full(n, 5.0)
    h.update_diag(good)
    fresh = make()
    fresh.update_diag(good)
    want = solve(fresh, torch.zeros_like(b))[0]
    for _ in range(30):
        x.zero_()
        assert torch.equal(solve(h, x)[0], want)


def test_gradient_after_a_failed_forward(lair):
    """A forward pass whose new diagonal fails on a kept hierarchy: the
    backward pass of the forward before it puts its own diagonal back."""
    import torch
    from paper_1708_06065_amd.autograd import LairSolve
    rp, cj, _ = (torch.as_tensor(a, device="cuda") for a in ONES)
    val0 = torch.ones(16, dtype=torch.float64, device="cuda")
    b = torch.as_tensor(np.random.default_rng(7).standard_normal(4), device="cuda")
    opts = dict(reuse={})
    LairSolve.apply(b, torch.full_like(b, 2.0), rp, cj, val0, opts)
    c = torch.full_like(b, 3.0).requires_grad_()
    x = LairSolve.apply(b, c, rp, cj, val0, opts)
    with pytest.raises(lair.LairError):
        LairSolve.apply(b, torch.zeros_like(b), rp, cj, val0, opts)
    x.sum().backward()
    A = np.ones((4, 4)) + 3.0 * np.eye(4)
    want = -np.linalg.solve(A.T, np.ones(4)) * np.linalg.solve(A, b.cpu().numpy())
    assert np.allclose(c.grad.cpu().numpy(), want, rtol=1e-9, atol=0)
