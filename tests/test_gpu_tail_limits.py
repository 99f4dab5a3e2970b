"""The largest levels that the persistent coarse tail takes, bit for bit against the oracle:
hierarchies whose tail is a coarsest level alone (the most blocks per thread), even and with an
odd axis (half blocks), and the fullest LDS planes of each kind of grid; also as the FP32 inner
grid of a mixed solve, stacked and in a batch of unequal grids."""
import numpy as np
import pytest
import torch

import fas_inputs as I
import oracle as O

pytestmark = pytest.mark.gpu

TD = {np.float64: torch.float64, np.float32: torch.float32}

# (n, coarsest, cell kappa, dtype)
CASES = [
    ((64, 49152), 4, False, np.float32), ((64, 41600), 4, False, np.float32), ((36, 1200), 18, False, np.float32),
    ((128, 384), 64, False, np.float32), ((220, 220), 110, False, np.float32), ((204, 204), 102, False, np.float32),
    ((196, 250), 98, False, np.float32), ((250, 196), 98, False, np.float32),
    ((36, 682), 18, False, np.float64), ((576, 10912), 18, False, np.float64), ((44, 558), 22, False, np.float64),
    ((148, 166), 74, False, np.float64), ((166, 148), 74, False, np.float64),
    ((164, 242), 82, True, np.float32), ((32, 264), 4, True, np.float32),
    ((132, 150), 66, True, np.float64), ((48, 88), 6, True, np.float64),
    ((4, 6, 4094), 2, False, np.float32), ((4, 6, 2046), 2, False, np.float64),
]


@pytest.mark.parametrize("n,coarsest,variable,dtype", CASES)
@pytest.mark.parametrize("bc", ["neumann", "dirichlet", "periodic"])
def test_largest_tails_bitwise(n, coarsest, variable, dtype, bc):
    from paper_2510_11152_amd import Grid
    L = (min(n) // coarsest).bit_length() - 1
    if bc == "periodic" and any((m >> L) % 2 for m in n):
        pytest.skip("periodic grids need even sizes on every level")
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.1, bc=bc, coarsest=coarsest, nuc=3)
    g = Grid(n, P.h, bc=bc, dtype=TD[dtype], coarsest=coarsest, variable_kappa=variable).set(coarse_sweeps=3)
    kap = np.exp(0.5 * I.random_field(P.shape(), 4)).astype(dtype) if variable else None
    f = I.random_field(P.shape(), 5).astype(dtype)
    u = I.random_field(P.shape(), 6).astype(dtype)
    ug, fg = torch.from_numpy(u).cuda(), torch.from_numpy(f).cuda()
    kg = None if kap is None else torch.from_numpy(kap).cuda()
    for nu1, nu2, transposed in ((2, 2, False), (1, 2, True)):
        O.vcycle(P, f, u, nu1, nu2, transposed=transposed, kap=kap)
        g.vcycle(fg, ug, P.dt, P.kappa, kg, nu1=nu1, nu2=nu2, transposed=transposed)
        torch.cuda.synchronize()
        assert np.array_equal(ug.cpu().numpy(), u), (nu1, nu2, transposed)


@pytest.mark.parametrize("n,coarsest", [((220, 220), 110), ((196, 250), 98)])
def test_mixed_solve_with_a_large_inner_tail(n, coarsest):
    from paper_2510_11152_amd import Grid, solve_mixed
    from parity_util import check_mixed
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.0, bc="neumann", coarsest=coarsest, nuc=2)
    f = I.random_field(P.shape(), 7)
    g64 = Grid(n, P.h, coarsest=coarsest).set(coarse_sweeps=2)
    g32 = Grid(n, P.h, dtype=torch.float32, coarsest=coarsest, mixed_inner=True).set(coarse_sweeps=2)
    ug = torch.from_numpy(f).cuda()
    assert solve_mixed(g64, g32, torch.from_numpy(f).cuda(), ug, P.dt, P.kappa, None, tol=1e-9) == 0
    check_mixed(P, f, f, ug.cpu().numpy(), g64.stats()["cycles"], 1e-9)


@pytest.mark.parametrize("n,coarsest,dtype", [((220, 220), 110, np.float32), ((148, 166), 74, np.float64)])
@pytest.mark.parametrize("form", ["stacked", "uneven"])
def test_batches_with_large_tails(n, coarsest, dtype, form):
    from paper_2510_11152_amd import Grid, solve_batched
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.0, bc="neumann", coarsest=coarsest, nuc=2)
    B = 3
    f = np.stack([I.random_field(P.shape(), 8 + b) for b in range(B)]).astype(dtype)
    u = np.stack([I.random_field(P.shape(), 18 + b) for b in range(B)]).astype(dtype)
    fg, ug = torch.from_numpy(f).cuda(), torch.from_numpy(u).cuda()
    if form == "stacked":
        g = Grid(n, P.h, dtype=TD[dtype], coarsest=coarsest, batch=B).set(coarse_sweeps=2, kmax=2)
        g.solve_stacked(fg, ug, P.dt, tol=0.0)
    else:
        gs = [Grid(n, P.h, dtype=TD[dtype], coarsest=coarsest).set(coarse_sweeps=2, kmax=2) for _ in range(B)]
        solve_batched(gs, list(fg), list(ug), P.dt, tol=0.0)
    torch.cuda.synchronize()
    for b in range(B):
        for _ in range(2):
            O.vcycle(P, f[b], u[b], 2, 2)
        assert np.array_equal(ug[b].cpu().numpy(), u[b]), b
