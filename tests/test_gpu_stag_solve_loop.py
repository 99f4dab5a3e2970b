"""The staggered solve's loop around the device's stopping test: what a call costs, and returns,
does not depend on the solves before it."""
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def timed(call):
    torch.cuda.synchronize()
    t = time.perf_counter()
    out = call()
    torch.cuda.synchronize()
    return time.perf_counter() - t, out


@pytest.mark.parametrize("loc", ["cell", "edge_x"])
def test_a_solve_that_needs_no_cycle_costs_the_same_after_long_solves(loc):
    """256^2: a solve from a converged guess enqueues next to nothing, whatever the cycles of the
    two solves before it (that many empty cycles take 7 to 25 times as long)."""
    from paper_2510_11152_amd import StaggeredSolver
    n = 256

    def solver():
        return StaggeredSolver(loc, n, n, 1.0 / n)

    S, T = solver(), solver()
    rng = np.random.default_rng(7)
    f = torch.from_numpy(rng.standard_normal(S.shape)).cuda()
    w = torch.zeros_like(f)
    st, long_cycles, _ = S.solve(1.0, 0.1, f, w, 1e-12, 1, 1, kmax=80)
    assert st == 0 and long_cycles >= 10
    done = w.clone()
    short, after = [], []
    for _ in range(8):
        t, (st, cycles, res) = timed(lambda: T.solve(1.0, 0.1, f, done, 1e-6, 1, 1, kmax=80))
        assert (st, cycles) == (0, 0)
        short.append(t)
        for _ in range(2):
            S.solve(1.0, 0.1, f, w.zero_(), 1e-12, 1, 1, kmax=80)
        t, again = timed(lambda: S.solve(1.0, 0.1, f, w, 1e-6, 1, 1, kmax=80))
        assert again == (st, cycles, res)
        after.append(t)
    assert min(after) < 4 * min(short), (min(after), min(short))


@pytest.mark.parametrize("tol", [1e-3, 1e-6, 1e-9])
def test_cycles_and_residual_are_those_of_the_cycle_by_cycle_loop(tol):
    """Solves that stop after any number of cycles, in an order that makes every expectation of
    the loop wrong in turn: the iterate, cycles and residual are those of single cycles."""
    from paper_2510_11152_amd import StaggeredSolver
    n = 128
    S, one = StaggeredSolver("cell", n, n, 1.0 / n), StaggeredSolver("cell", n, n, 1.0 / n)
    rng = np.random.default_rng(8)
    f = torch.from_numpy(rng.standard_normal(S.shape)).cuda()
    for scale in (1.0, 1e-4, 1.0, 1e3, 0.0, 1e-2, 1e3):
        g = f * scale
        w, v = torch.zeros_like(f), torch.zeros_like(f)
        st, cycles, res = S.solve(1.0, 0.1, g, w, tol, 2, 2, kmax=12)
        for _ in range(cycles):
            one.vcycle(1.0, 0.1, g, v, 2, 2)
        torch.cuda.synchronize()
        assert torch.equal(w, v), (scale, cycles)
        assert (st == 0) == (res <= tol) and (st == 0 or cycles == 12)
