"""2D levels narrower or lower than a block tile (128 columns, 32 or 64 rows), which the tile
passes take down to 32 x 8 cells: bit for bit against the oracle, with windows that span
several periods of a periodic level, and the sizes next to the lines of the rule."""
import numpy as np
import pytest
import torch

import fas_inputs as I
import oracle as O

pytestmark = pytest.mark.gpu

TD = {np.float64: torch.float64, np.float32: torch.float32}
CASES = [((32, 256), 16), ((28, 280), 14), ((48, 200), 6), ((112, 72), 36), ((124, 124), 62), ((64, 128), 32),
         ((1000, 8), 4), ((1000, 12), 6), ((800, 4), 2), ((130, 62), 62), ((96, 1024), 6)]


@pytest.mark.parametrize("n,coarsest", CASES)
@pytest.mark.parametrize("bc", ["neumann", "dirichlet", "periodic"])
@pytest.mark.parametrize("variable", [False, True])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_narrow_levels_bitwise(n, coarsest, bc, variable, dtype):
    from paper_2510_11152_amd import Grid
    ratio = min(n) // coarsest
    if ratio < 2:
        n, ratio = tuple(2 * m for m in n), 2
    L = ratio.bit_length() - 1
    if bc == "periodic" and any((m >> L) % 2 for m in n):
        pytest.skip("periodic grids need even sizes on every level")
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.1, bc=bc, coarsest=coarsest, nuc=2)
    g = Grid(n, P.h, bc=bc, dtype=TD[dtype], coarsest=coarsest, variable_kappa=variable).set(coarse_sweeps=2)
    kap = np.exp(0.5 * I.random_field(P.shape(), 4)).astype(dtype) if variable else None
    f = I.random_field(P.shape(), 41).astype(dtype)
    u = I.random_field(P.shape(), 42).astype(dtype)
    ug, fg = torch.from_numpy(u).cuda(), torch.from_numpy(f).cuda()
    kg = None if kap is None else torch.from_numpy(kap).cuda()
    for nu1, nu2, tr in ((2, 2, False), (1, 3, True)):
        O.vcycle(P, f, u, nu1, nu2, transposed=tr, kap=kap)
        rel = g.vcycle(fg, ug, P.dt, P.kappa, kg, nu1=nu1, nu2=nu2, transposed=tr, with_residual=True)
        torch.cuda.synchronize()
        assert np.array_equal(ug.cpu().numpy(), u), (nu1, nu2, tr)
    ref = np.linalg.norm(O.residual(P, 0, f, u, kap=kap).astype(np.float64)) / np.linalg.norm(f.astype(np.float64))
    assert abs(rel - ref) <= 1e-10 * ref
