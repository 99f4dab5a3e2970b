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
