"""Staggered hierarchies whose coarsest level is too large for the persistent tail: its
right-hand side is formed by a launch of its own and it is smoothed between two buffers, from
the restricted iterate, by any number of sweeps; bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from oracle import staggered as ost

pytestmark = pytest.mark.gpu

LOCS = [("cell", "neumann", ost.CELL), ("cell", "dirichlet", ost.CELL), ("edge_x", "dirichlet", ost.EDGE_X),
        ("edge_y", "dirichlet", ost.EDGE_Y)]


@pytest.mark.parametrize("loc,bc,code", LOCS)
@pytest.mark.parametrize("nx,ny,coarsest", [(256, 256, 128), (4096, 8, 4), (16, 3072, 4)])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 1), (3, 1)])
@pytest.mark.parametrize("nuc", [1, 2, 3, 4, 5])
def test_large_coarsest_level_bitwise(loc, bc, code, nx, ny, coarsest, nu1, nu2, nuc):
    from paper_2510_11152_amd import StaggeredSolver
    S = StaggeredSolver(loc, nx, ny, 1.0 / nx, bc=bc, coarsest=coarsest)
    S.set(coarse_sweeps=nuc)
    P = ost.StagProblem(code, nx, ny, 1.0 / nx, cell_bc=bc, coarsest=coarsest, nuc=nuc)
    a, c = (0.0, 1.0) if bc == "neumann" else (1.0, 0.37)
    rng = np.random.default_rng(nx + ny)
    f, w = rng.standard_normal(P.shape()), rng.standard_normal(P.shape())
    if a == 0.0:
        f -= f.mean()
    fd, wd = torch.from_numpy(f).cuda(), torch.from_numpy(w.copy()).cuda()
    for _ in range(2):
        S.vcycle(a, c, fd, wd, nu1, nu2)
        ost.vcycle(P, a, c, f, w, nu1, nu2)
    torch.cuda.synchronize()
    assert np.array_equal(wd.cpu().numpy(), w)
