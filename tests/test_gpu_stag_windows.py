"""The staggered sweep windows at their edges, bit for bit against the oracle: levels whose
width ends just before, at and after a window (128 columns, 116 to 120 written), with and
without windows that touch no wall, and heights around the written rows."""
import numpy as np
import pytest
import torch

from oracle import staggered as ost

pytestmark = pytest.mark.gpu

LOCS = [("cell", "neumann", ost.CELL), ("cell", "dirichlet", ost.CELL), ("edge_x", "dirichlet", ost.EDGE_X),
        ("edge_y", "dirichlet", ost.EDGE_Y)]
SIZES = [(8, 16), (116, 40), (120, 48), (124, 20), (128, 24), (232, 44), (248, 40), (250, 22), (360, 24), (376, 88)]


@pytest.mark.parametrize("loc,bc,code", LOCS)
@pytest.mark.parametrize("nx,ny", SIZES)
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 1), (3, 3)])
def test_window_edges_bitwise(loc, bc, code, nx, ny, nu1, nu2):
    from paper_2510_11152_amd import StaggeredSolver
    coarsest = ny
    while coarsest % 2 == 0 and coarsest > 4 and nx % (2 * ny // coarsest) == 0:
        coarsest //= 2
    S = StaggeredSolver(loc, nx, ny, 1.0 / nx, bc=bc, coarsest=coarsest)
    P = ost.StagProblem(code, nx, ny, 1.0 / nx, cell_bc=bc, coarsest=coarsest)
    a, c = (0.0, 1.0) if bc == "neumann" else (1.0, 0.37)
    rng = np.random.default_rng(nx * ny)
    f, w = rng.standard_normal(P.shape()), rng.standard_normal(P.shape())
    if a == 0.0:
        f -= f.mean()
    fd, wd = torch.from_numpy(f).cuda(), torch.from_numpy(w.copy()).cuda()
    for _ in range(2):
        S.vcycle(a, c, fd, wd, nu1, nu2)
        ost.vcycle(P, a, c, f, w, nu1, nu2)
    torch.cuda.synchronize()
    assert np.array_equal(wd.cpu().numpy(), w)
    if bc == "dirichlet":  # a whole solve: the norm of the last launch stops it
        st, cyc, res = S.solve(a, c, fd, wd, 0.0, nu1, nu2, kmax=1)
        ost.vcycle(P, a, c, f, w, nu1, nu2)
        ref = ost.res_norm(P, a, c, f, w)
        assert st == 1 and cyc == 1 and abs(res - ref) <= 1e-12 * ref
        assert np.array_equal(wd.cpu().numpy(), w)


# (nx, ny, coarsest): the tail alone or nearly so, from one block to rows of half blocks
TAILS = [(4, 4, 2), (8, 8, 4), (10, 6, 3), (16, 16, 2), (20, 12, 3), (32, 32, 4), (34, 32, 16), (64, 64, 4), (68, 60, 15),
         (128, 128, 4), (1024, 16, 2), (1364, 8, 2), (4096, 4, 2), (8192, 4, 2)]


@pytest.mark.parametrize("loc,bc,code", LOCS)
@pytest.mark.parametrize("nx,ny,coarsest", TAILS)
def test_tail_levels_bitwise(loc, bc, code, nx, ny, coarsest):
    from paper_2510_11152_amd import StaggeredSolver
    S = StaggeredSolver(loc, nx, ny, 1.0 / nx, bc=bc, coarsest=coarsest)
    S.set(coarse_sweeps=3)
    P = ost.StagProblem(code, nx, ny, 1.0 / nx, cell_bc=bc, coarsest=coarsest, nuc=3)
    a, c = (0.0, 1.0) if bc == "neumann" else (1.0, 0.37)
    rng = np.random.default_rng(nx + ny)
    f, w = rng.standard_normal(P.shape()), rng.standard_normal(P.shape())
    if a == 0.0:
        f -= f.mean()
    fd, wd = torch.from_numpy(f).cuda(), torch.from_numpy(w.copy()).cuda()
    for nu1, nu2 in ((2, 2), (1, 0), (0, 3)):
        S.vcycle(a, c, fd, wd, nu1, nu2)
        ost.vcycle(P, a, c, f, w, nu1, nu2)
        torch.cuda.synchronize()
        assert np.array_equal(wd.cpu().numpy(), w), (nu1, nu2)


@pytest.mark.parametrize("loc,bc,code", LOCS)
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 1), (5, 2), (3, 2)])
def test_solve_does_not_depend_on_earlier_solves(loc, bc, code, nu1, nu2):
    """Cycles enqueued on the strength of earlier solves do nothing once a solve has stopped:
    a short solve, one already converged, one cut off by kmax and one that is not finite give
    what a fresh solver gives, after two longer solves."""
    from paper_2510_11152_amd import StaggeredSolver
    from paper_2510_11152_amd._lib import FasError

    def make():
        return StaggeredSolver(loc, 256, 128, 1.0 / 256, bc=bc)

    S = make()
    a, c = (0.0, 1.0) if bc == "neumann" else (1.0, 0.37)
    g = torch.Generator(device="cuda").manual_seed(3)
    f = torch.rand(S.shape, dtype=torch.float64, device="cuda", generator=g)
    f -= f.mean()
    w0 = torch.rand(S.shape, dtype=torch.float64, device="cuda", generator=g)
    for tol, kmax in ((1e-3, 20), (1e9, 20), (1e-9, 2), (1e-9, 20)):
        fresh, w1 = make(), w0.clone()
        want = fresh.solve(a, c, f, w1, tol, nu1, nu2, kmax)
        S = make()
        for _ in range(2):
            S.solve(a, c, f, w0.clone(), 1e-9, nu1, nu2, 20)  # (V(1,1) may need more cycles)
        w2 = w0.clone()
        assert S.solve(a, c, f, w2, tol, nu1, nu2, kmax) == want
        assert torch.equal(w1, w2)
    bad = f.clone()
    bad[3, 5] = float("nan")
    w3 = w0.clone()
    with pytest.raises(FasError):
        S.solve(a, c, bad, w3, 1e-9, nu1, nu2, 20)
    assert torch.equal(w3, w0)  # not finite from the start: no cycle runs
