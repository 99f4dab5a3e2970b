"""The brick passes of small 3D levels, bit for bit against the oracle: bricks that the level
fills in part, levels smaller than a brick's reach (on periodic grids several periods of it),
walls at each distance from a brick, one or two sweeps in each pass, and the norm."""
import numpy as np
import pytest
import torch

import fas_inputs as I
import oracle as O

pytestmark = pytest.mark.gpu

TD = {np.float64: torch.float64, np.float32: torch.float32}
CASES = [((32, 32, 32), 4), ((40, 24, 32), 6), ((28, 36, 44), 14), ((4, 64, 96), 2), ((320, 8, 8), 4), ((8, 200, 16), 4),
         ((20, 20, 60), 10), ((96, 48, 40), 10)]


@pytest.mark.parametrize("n,coarsest", CASES)
@pytest.mark.parametrize("bc", ["neumann", "dirichlet", "periodic"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_bricks_bitwise(n, coarsest, bc, dtype):
    from paper_2510_11152_amd import Grid
    L = (min(n) // coarsest).bit_length() - 1
    if bc == "periodic" and any((m >> L) % 2 for m in n):
        pytest.skip("periodic grids need even sizes on every level")
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.1, bc=bc, coarsest=coarsest, nuc=2)
    g = Grid(n, P.h, bc=bc, dtype=TD[dtype], coarsest=coarsest).set(coarse_sweeps=2)
    f = I.random_field(P.shape(), 51).astype(dtype)
    u = I.random_field(P.shape(), 52).astype(dtype)
    ug, fg = torch.from_numpy(u).cuda(), torch.from_numpy(f).cuda()
    for nu1, nu2, tr in ((2, 2, False), (1, 2, True), (2, 1, False), (1, 1, False)):
        O.vcycle(P, f, u, nu1, nu2, transposed=tr)
        rel = g.vcycle(fg, ug, P.dt, P.kappa, nu1=nu1, nu2=nu2, transposed=tr, with_residual=True)
        torch.cuda.synchronize()
        assert np.array_equal(ug.cpu().numpy(), u), (nu1, nu2, tr)
        ref = np.linalg.norm(O.residual(P, 0, f, u).astype(np.float64)) / np.linalg.norm(f.astype(np.float64))
        assert abs(rel - ref) <= 1e-10 * ref


LARGE = [((96, 64, 64), 4), ((104, 72, 88), 18), ((16, 208, 272), 4), ((8, 192, 264), 4), ((100, 84, 76), 38)]


@pytest.mark.parametrize("n,coarsest", LARGE)
@pytest.mark.parametrize("bc", ["neumann", "dirichlet", "periodic"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_large_bricks_bitwise(n, coarsest, bc, dtype):
    test_bricks_bitwise(n, coarsest, bc, dtype)


@pytest.mark.parametrize("bc", ["neumann", "periodic"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("batch", [3, 13])
def test_stacked_bricks_equal_single_solves(bc, dtype, batch):
    """13 problems of 32^3 take large bricks, one alone small ones: the same values."""
    from paper_2510_11152_amd import Grid
    n = (32, 32, 32)
    f = torch.from_numpy(I.random_field((batch,) + n, 61).astype(dtype)).cuda()
    u = torch.from_numpy(I.random_field((batch,) + n, 62).astype(dtype)).cuda()
    one = [x.clone() for x in u]
    Grid(n, 1 / 32, bc=bc, dtype=TD[dtype], batch=batch).set(kmax=3).solve_stacked(f, u, 2e-4, tol=0.0)
    g = Grid(n, 1 / 32, bc=bc, dtype=TD[dtype])
    for b in range(batch):
        for _ in range(3):
            g.vcycle(f[b], one[b], 2e-4)
    torch.cuda.synchronize()
    for b in range(batch):
        assert torch.equal(u[b], one[b]), b


def test_stacked_mixed_bricks_equal_single_solves():
    """The FP32 passes that start from zero and add into the FP64 iterate, as large bricks."""
    from paper_2510_11152_amd import Grid, solve_mixed, solve_stacked_mixed
    n, batch = (32, 32, 32), 13
    f = torch.from_numpy(I.random_field((batch,) + n, 63)).cuda()
    u = torch.zeros_like(f)
    g64 = Grid(n, 1 / 32, batch=batch)
    g32 = Grid(n, 1 / 32, dtype=torch.float32, mixed_inner=True, batch=batch)
    st, cy = solve_stacked_mixed(g64, g32, f, u, 2e-4, tol=1e-10)
    h64, h32 = Grid(n, 1 / 32), Grid(n, 1 / 32, dtype=torch.float32, mixed_inner=True)
    for b in range(batch):
        one = torch.zeros_like(f[b])
        solve_mixed(h64, h32, f[b].clone(), one, 2e-4, tol=1e-10)
        assert torch.equal(u[b], one), b
