"""The 3D plane marches at the edges of their tiles (64 columns, 32 rows in FP64 and 48 in
FP32, segments of a computed number of planes), bit for bit against the oracle: grids one
tile wide and a little more, ragged remainders, blocks over walls and over periodic edges,
short segments, and the norm of the last pass."""
import numpy as np
import pytest
import torch

import fas_inputs as I
import oracle as O

pytestmark = pytest.mark.gpu

TD = {np.float64: torch.float64, np.float32: torch.float32}
CASES = [((64, 32, 16), 4), ((64, 40, 16), 4), ((112, 72, 24), 6), ((72, 104, 40), 10), ((160, 112, 48), 6)]


@pytest.mark.parametrize("n,coarsest", CASES)
@pytest.mark.parametrize("bc", ["neumann", "dirichlet", "periodic"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nu", [(2, 2), (1, 1), (3, 2)])
def test_march_tile_edges_bitwise(n, coarsest, bc, dtype, nu):
    from paper_2510_11152_amd import Grid
    L = (min(n) // coarsest).bit_length() - 1
    if bc == "periodic" and any((m >> L) % 2 for m in n):
        pytest.skip("periodic grids need even sizes on every level")
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.0, bc=bc, coarsest=coarsest, nuc=2)
    g = Grid(n, P.h, bc=bc, dtype=TD[dtype], coarsest=coarsest).set(coarse_sweeps=2)
    f = I.random_field(P.shape(), 31).astype(dtype)
    u = I.random_field(P.shape(), 32).astype(dtype)
    ug, fg = torch.from_numpy(u).cuda(), torch.from_numpy(f).cuda()
    for _ in range(2):
        O.vcycle(P, f, u, nu[0], nu[1])
        rel = g.vcycle(fg, ug, P.dt, nu1=nu[0], nu2=nu[1], with_residual=True)
        torch.cuda.synchronize()
        assert np.array_equal(ug.cpu().numpy(), u)
    ref = np.linalg.norm(O.residual(P, 0, f, u).astype(np.float64)) / np.linalg.norm(f.astype(np.float64))
    assert abs(rel - ref) <= 1e-10 * ref


LARGE = (176, 144, 144)  # more than bricks take, in either precision


@pytest.mark.parametrize("bc", ["neumann", "dirichlet"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_two_sweep_marches_bitwise(bc, dtype):
    from paper_2510_11152_amd import Grid
    P = O.Problem(n=LARGE, h=1.0 / 176, dt=2e-4, kappa=1.0, bc=bc, coarsest=18, nuc=2)
    g = Grid(LARGE, P.h, bc=bc, dtype=TD[dtype], coarsest=18).set(coarse_sweeps=2)
    f = I.random_field(P.shape(), 33).astype(dtype)
    u = I.random_field(P.shape(), 34).astype(dtype)
    ug = torch.from_numpy(u).cuda()
    O.vcycle(P, f, u, 2, 2)
    rel = g.vcycle(torch.from_numpy(f).cuda(), ug, P.dt, with_residual=True)
    torch.cuda.synchronize()
    assert np.array_equal(ug.cpu().numpy(), u)
    ref = np.linalg.norm(O.residual(P, 0, f, u).astype(np.float64)) / np.linalg.norm(f.astype(np.float64))
    assert abs(rel - ref) <= 1e-10 * ref


@pytest.mark.parametrize("n,coarsest,nu", [((128, 64, 32), 4, (3, 3)), (LARGE, 18, (2, 2))])
def test_mixed_marches_match_oracle(n, coarsest, nu):
    """FP32 marches that start from zero and that add into the FP64 iterate."""
    from paper_2510_11152_amd import Grid, solve_mixed
    from parity_util import check_mixed
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.0, bc="neumann", coarsest=coarsest, nuc=2)
    f = I.random_field(P.shape(), 35)
    g64 = Grid(n, P.h, coarsest=coarsest).set(coarse_sweeps=2)
    g32 = Grid(n, P.h, dtype=torch.float32, coarsest=coarsest, mixed_inner=True).set(coarse_sweeps=2)
    ug = torch.from_numpy(f).cuda()
    assert solve_mixed(g64, g32, torch.from_numpy(f).cuda(), ug, P.dt, P.kappa, None, tol=1e-9, nu1=nu[0], nu2=nu[1]) == 0
    check_mixed(P, f, f, ug.cpu().numpy(), g64.stats()["cycles"], 1e-9, nu1=nu[0], nu2=nu[1])
