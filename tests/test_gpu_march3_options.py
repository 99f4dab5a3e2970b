"""The 3D plane marches in every form on small levels, which their options keep on marches (a
forced segment height, one sweep per pass), and on levels and batches beyond the bricks: bit
for bit against the oracle or the same problem solved alone."""
import numpy as np
import pytest
import torch

import fas_inputs as I
import oracle as O

pytestmark = pytest.mark.gpu

TD = {np.float64: torch.float64, np.float32: torch.float32}
CASES = [((64, 32, 16), 4), ((64, 40, 16), 4), ((112, 72, 24), 6), ((72, 104, 40), 10), ((160, 112, 48), 6)]
LARGE = (176, 144, 144)  # more than bricks take, in either precision


def check_vcycle(n, coarsest, bc, dtype, nu, options, seed, cycles=2):
    from paper_2510_11152_amd import Grid
    L = (min(n) // coarsest).bit_length() - 1
    if bc == "periodic" and any((m >> L) % 2 for m in n):
        pytest.skip("periodic grids need even sizes on every level")
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.0, bc=bc, coarsest=coarsest, nuc=2)
    g = Grid(n, P.h, bc=bc, dtype=TD[dtype], coarsest=coarsest).set(coarse_sweeps=2, **options)
    f = I.random_field(P.shape(), seed).astype(dtype)
    u = I.random_field(P.shape(), seed + 1).astype(dtype)
    ug, fg = torch.from_numpy(u).cuda(), torch.from_numpy(f).cuda()
    for _ in range(cycles):
        O.vcycle(P, f, u, nu[0], nu[1])
        rel = g.vcycle(fg, ug, P.dt, nu1=nu[0], nu2=nu[1], with_residual=True)
        torch.cuda.synchronize()
        assert np.array_equal(ug.cpu().numpy(), u)
    ref = np.linalg.norm(O.residual(P, 0, f, u).astype(np.float64)) / np.linalg.norm(f.astype(np.float64))
    assert abs(rel - ref) <= 1e-10 * ref


@pytest.mark.parametrize("n,coarsest", CASES)
@pytest.mark.parametrize("bc", ["neumann", "dirichlet", "periodic"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nu", [(2, 2), (1, 1), (2, 1)])
@pytest.mark.parametrize("options", [{"seg_rows": 8}, {"seg_rows": 30}, {"march3_sweeps": 1},
                                     {"march3_sweeps": 1, "seg_rows": 10}], ids=lambda o: "-".join(map(str, o.values())))
def test_marches_on_small_levels_bitwise(n, coarsest, bc, dtype, nu, options):
    check_vcycle(n, coarsest, bc, dtype, nu, options, 31)


@pytest.mark.parametrize("nu", [(2, 2), (1, 1), (2, 1)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_marches_over_periodic_edges_bitwise(dtype, nu):
    check_vcycle(LARGE, 18, "periodic", dtype, nu, {}, 33, cycles=1)


# (n, batch, coarsest, options): the first by the default rule (9 x 64^3 FP32 are more than bricks take)
STACKS = [((64, 64, 64), 9, 4, {}), ((64, 32, 32), 3, 4, {"seg_rows": 8}), ((72, 40, 24), 4, 6, {"march3_sweeps": 1}),
          ((112, 72, 24), 3, 6, {"seg_rows": 64})]


@pytest.mark.parametrize("n,batch,coarsest,options", STACKS)
@pytest.mark.parametrize("bc", ["neumann", "periodic"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nu", [(2, 2), (1, 2)])
def test_stacked_marches_equal_single_solves(n, batch, coarsest, options, bc, dtype, nu):
    from paper_2510_11152_amd import Grid
    L = (min(n) // coarsest).bit_length() - 1
    if bc == "periodic" and any((m >> L) % 2 for m in n):
        pytest.skip("periodic grids need even sizes on every level")
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.0, bc=bc, coarsest=coarsest, nuc=2)
    f = I.random_field((batch,) + P.shape(), 61).astype(dtype)
    u0 = I.random_field((batch,) + P.shape(), 62).astype(dtype)
    fg, ug = torch.from_numpy(f).cuda(), torch.from_numpy(u0).cuda()
    g = Grid(n, P.h, bc=bc, dtype=TD[dtype], coarsest=coarsest, batch=batch).set(coarse_sweeps=2, kmax=2, **options)
    g.solve_stacked(fg, ug, P.dt, tol=0.0, nu1=nu[0], nu2=nu[1])
    one = Grid(n, P.h, bc=bc, dtype=TD[dtype], coarsest=coarsest).set(coarse_sweeps=2)
    for b in range(batch):
        us = torch.from_numpy(u0[b]).cuda()
        for _ in range(2):
            one.vcycle(fg[b], us, P.dt, nu1=nu[0], nu2=nu[1])
        torch.cuda.synchronize()
        assert torch.equal(us, ug[b]), b
    for _ in range(2):
        O.vcycle(P, f[batch - 1], u0[batch - 1], nu[0], nu[1])
    assert np.array_equal(ug[batch - 1].cpu().numpy(), u0[batch - 1])


@pytest.mark.parametrize("n,batch,coarsest,options", STACKS)
@pytest.mark.parametrize("bc", ["neumann", "periodic"])
def test_stacked_mixed_marches_equal_single_solves(n, batch, coarsest, options, bc):
    """FP32 marches that start from zero and that add into the FP64 iterate, and the FP64
    residual pass, over a batch."""
    from paper_2510_11152_amd import Grid, solve_mixed, solve_stacked_mixed
    from parity_util import check_mixed
    L = (min(n) // coarsest).bit_length() - 1
    if bc == "periodic" and any((m >> L) % 2 for m in n):
        pytest.skip("periodic grids need even sizes on every level")
    P = O.Problem(n=n, h=1.0 / n[0], dt=2e-4, kappa=1.0, bc=bc, coarsest=coarsest, nuc=2)
    f = I.random_field((batch,) + P.shape(), 63)
    fg = torch.from_numpy(f).cuda()
    ug = torch.zeros_like(fg)

    def grids(b, **opt):
        kw = {} if b is None else {"batch": b}
        return (Grid(n, P.h, bc=bc, coarsest=coarsest, **kw).set(coarse_sweeps=2, **opt),
                Grid(n, P.h, bc=bc, dtype=torch.float32, coarsest=coarsest, mixed_inner=True, **kw).set(coarse_sweeps=2, **opt))

    g64, g32 = grids(batch, **options)
    st, cy = solve_stacked_mixed(g64, g32, fg, ug, P.dt, tol=1e-10)
    assert all(s == 0 for s in st)
    h64, h32 = grids(None)
    for b in range(batch):
        us = torch.zeros_like(fg[b])
        assert solve_mixed(h64, h32, fg[b].clone(), us, P.dt, tol=1e-10) == 0
        assert h64.stats()["cycles"] == cy[b]
        assert torch.equal(us, ug[b]), b
    check_mixed(P, f[0], np.zeros_like(f[0]), ug[0].cpu().numpy(), cy[0], 1e-10)


# The first: a coarse march level (64 x 32 x 16) whose passes start in its second buffer, which
# the autotuner must not overwrite (V(2,1), one sweep per pass: three passes); the second: the
# same by the default rule (V(2,2), two sweeps: 200 x 144 x 136 below the finest).
@pytest.mark.parametrize("n,coarsest,nu,options", [((128, 64, 32), 4, (2, 1), {"march3_sweeps": 1}),
                                                   ((400, 288, 272), 34, (2, 2), {}), (LARGE, 18, (2, 2), {})])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_autotuned_marches_give_the_same_bits(n, coarsest, nu, options, dtype):
    from paper_2510_11152_amd import Grid
    shape = tuple(reversed(n))
    f = torch.from_numpy(I.random_field(shape, 65).astype(dtype)).cuda()
    ref = f.clone()
    g0 = Grid(n, 1.0 / n[0], dtype=TD[dtype], coarsest=coarsest).set(kmax=3, fused=False)
    g0.solve(f, ref, 2e-4, tol=0.0, nu1=nu[0], nu2=nu[1])
    for extra in ({}, {"autotune": True}, {"graph": True, "autotune": True}):
        g = Grid(n, 1.0 / n[0], dtype=TD[dtype], coarsest=coarsest).set(kmax=3, **options, **extra)
        for rep in range(2):  # the second solve replays the graph
            u = f.clone()
            g.solve(f, u, 2e-4, tol=0.0, nu1=nu[0], nu2=nu[1])
            torch.cuda.synchronize()
            assert torch.equal(u, ref), (extra, rep)
