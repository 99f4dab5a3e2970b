"""Host-side rules that choose a grid's kernels, checked without a GPU (grids are planned over
a workspace that nothing touches)."""
import ctypes
import itertools
import math
import os
import sys

import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2510_11152_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        pytest.fail("libfas.so is not built (run __graft_entry__.build())")
    return _lib.load()


class Planned:
    def __init__(self, lib, n, f32, coarsest, flags=0):
        self.lib, self.handle = lib, ctypes.c_void_p()
        n3 = (ctypes.c_int64 * 3)(*(list(n) + [1] * (3 - len(n))))
        need = lib.fas_workspace_size(len(n), n3, int(f32), coarsest, flags)
        assert need, (n, coarsest)
        fake = ctypes.c_void_p(1 << 20)  # never dereferenced
        assert lib.fas_grid_create(len(n), n3, 1.0, 0, int(f32), coarsest, flags, fake, need, None,
                                   ctypes.byref(self.handle)) == 0

    def __enter__(self):
        return self.handle

    def __exit__(self, *exc):
        self.lib.fas_grid_destroy(self.handle)


def tail_top_by_bytes(n, L, f32, variable):
    """First level of the tail by its budget alone: u and f of all its levels and, on a grid for
    a cell kappa, the top level's face weights (2D) or every level's kappa (3D)."""
    s, dim = 4 if f32 else 8, len(n)
    used, top = 0, L + 1
    for l in range(L, -1, -1):
        m = [x >> l for x in n]
        cells = m[0] * m[1] * (m[2] if dim == 3 else 1)
        used += (3 if variable and dim == 3 else 2) * cells * s
        faces = ((m[0] + 1) * m[1] + m[0] * (m[1] + 1)) * s if variable and dim == 2 else 0
        if used + faces > (156 if variable else 96) * 1024 or L - l + 1 > 10:
            break
        top = l
    return top


def hierarchies(f32, variable):
    """Coarsest levels of every shape up to and past the budget, one to three levels above."""
    most = (156 if variable else 96) * 1024 // (2 * (4 if f32 else 8))
    for c in range(2, int(most ** 0.5) + 1, 4):
        longest = most // c
        for m in sorted({c, c + 1, longest // 5, longest // 4, longest // 3, longest // 2} |
                        set(range(max(c, longest - 12), longest + 3))):
            if m < c:
                continue
            for L in (1, 2, 4):
                yield (c << L, m << L), c, L
                yield (m << L, c << L), c, L
    for c, m in itertools.product((2, 4, 6, 10, 18), (0, 1, 2, 5)):
        longest = most // (c * (c + m))
        for k in sorted({c + m, longest // 9, longest // 8, longest // 4, longest // 2} |
                        set(range(max(c + m, longest - 12), longest + 3))):
            if k < c + m:
                continue
            for L in (1, 2):
                yield (c << L, (c + m) << L, k << L), c, L


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("variable", [False, True])
def test_tail_holds_every_level_its_budget_admits(lib, f32, variable):
    """No level that the byte budget admits is left without planes or threads for its blocks."""
    tail_top = lib["_ZN3fas8tail_topEPK8fas_grid"]
    tail_class = lib["_ZN3fas10tail_classEPK8fas_gridi"]
    tail_top.argtypes, tail_class.argtypes = [ctypes.c_void_p], [ctypes.c_void_p, ctypes.c_int]
    seen = set()
    for n, c, L in hierarchies(f32, variable):
        with Planned(lib, n, f32, c, flags=int(variable)) as g:
            want = tail_top_by_bytes(n, L, f32, variable)
            assert tail_top(g) == want, (n, c)
            if want <= L:
                seen.add(tail_class(g, want))
    assert seen == {0, 1}


@pytest.mark.parametrize("n,coarsest", [((64, 32, 16), 4), ((96, 64, 32), 4), ((128, 128, 128), 4)])
@pytest.mark.parametrize("f32", [False, True])
def test_march_options_reach_the_levels_that_marches_take(lib, n, coarsest, f32):
    """Levels from 64 x 32 x 16 up run plane marches when an option of the marches is set: one
    sweep per pass, or a segment height; smaller levels run bricks all the same."""
    from paper_2510_11152_amd import _lib as F
    brick_ok = lib["_ZN3fas8brick_okEPK8fas_gridiiib"]
    brick_ok.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool]
    brick_ok.restype = ctypes.c_bool
    with Planned(lib, n, f32, coarsest) as g:
        def bricks(level):
            return brick_ok(g, level, 2, 2, False)
        assert bricks(0) and bricks(1)
        for opt, value, default in ((F.FAS_OPT_SEG_ROWS, 16, 0), (F.FAS_OPT_MARCH3_SWEEPS, 1, 2)):
            assert lib.fas_grid_set(g, opt, value) == F.FAS_OK
            assert not bricks(0), opt
            assert bricks(1) == (n != (128, 128, 128)), opt  # 64^3 takes marches, 32 x 16 x 8 none
            assert lib.fas_grid_set(g, opt, default) == F.FAS_OK
            assert bricks(0) and bricks(1), opt


@pytest.mark.parametrize("n,coarsest", [((64, 32, 16), 4), ((256, 256, 256), 4), ((160, 160, 160), 10), ((512, 512, 512), 4),
                                        ((64, 64, 20), 10), ((176, 144, 144), 18), ((64, 2048, 640), 4)])
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("sweeps", [1, 2])
def test_plane_march_autotuner_times_the_rules_height(lib, n, coarsest, f32, sweeps):
    """The heights that the autotuner times for plane marches start with the rule's, and no
    height at all takes fewer steps by the rule's count (rounds of blocks over 256 compute
    units times the planes that a block visits)."""
    from paper_2510_11152_amd import _lib as F
    fn = lib["_ZN3fas21fused3_seg_candidatesEPK8fas_gridiiPi"]
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    out = (ctypes.c_int * 8)()
    with Planned(lib, n, f32, coarsest) as g:
        assert lib.fas_grid_set(g, F.FAS_OPT_MARCH3_SWEEPS, sweeps) == F.FAS_OK
        heights = list(out[:fn(g, 0, sweeps, out)])
    halo = 2 * sweeps + 2
    tiles = -(-n[0] // (64 - 2 * halo)) * -(-n[1] // ((48 if f32 else 32) - 2 * halo))

    def steps(planes):
        return -(-tiles * -(-n[2] // planes) // 256) * (planes + halo + 2 * sweeps + 2)

    assert len(heights) >= 2 and len(set(heights)) == len(heights)
    assert all(4 <= h <= n[2] and h % 2 == 0 for h in heights)
    assert steps(heights[0]) == min(steps(h) for h in range(4, n[2] + 1, 2))


def test_staggered_stopping_limit(lib):
    """The limit on the squared norm that the device tests is the largest double whose norm
    passes the host's test, also where h sqrt(s2) underflows."""
    fn = lib["_ZN3fas4stag8s2_limitEdd"]
    fn.argtypes, fn.restype = [ctypes.c_double, ctypes.c_double], ctypes.c_double
    inf, big = math.inf, sys.float_info.max
    for h in (1e-300, 1e-200, 1e-170, 1e-160, 1e-3, 1 / 3, 1 / 4096, 1.0, 7.0, 1e200):
        for tol in (0.0, 5e-324, 1e-320, 1e-310, 1e-200, 1e-16, 1e-8, 0.3, 1e150, 1e300, inf):
            s2 = fn(h, tol)
            assert 0.0 <= s2 <= big and h * math.sqrt(s2) <= tol, (h, tol)
            assert s2 == big or h * math.sqrt(math.nextafter(s2, inf)) > tol, (h, tol)
    assert fn(inf, 1.0) == -1.0


# (n, coarsest, bricks in FP64, in FP32): levels that bricks fill in part (one or two axes of 4
# or 8 cells), where many bricks take longer than the per-level kernels, and full ones
THIN = [((4, 4, 8192), 2, True, True), ((4, 4, 65536), 2, False, False), ((65536, 4, 4), 2, False, False),
        ((4, 8, 16384), 2, False, True), ((8, 4, 65536), 2, False, False), ((4, 512, 512), 2, True, True),
        ((4, 1024, 2048), 2, False, False), ((2048, 4, 1024), 2, False, False), ((2048, 2048, 4), 2, False, False),
        ((8, 12, 32768), 4, True, True), ((8, 12, 131072), 4, False, False), ((8, 2048, 2048), 4, True, False),
        ((1536, 1536, 8), 4, True, True), ((32, 32, 32), 4, True, True), ((8, 8, 512), 4, True, True),
        ((16, 1024, 1024), 4, True, True), ((48, 48, 8192), 6, True, True)]


@pytest.mark.parametrize("n,coarsest,f64,f32", THIN)
def test_thin_levels_run_bricks_while_they_are_faster(lib, n, coarsest, f64, f32):
    brick_ok = lib["_ZN3fas8brick_okEPK8fas_gridiiib"]
    brick_ok.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool]
    brick_ok.restype = ctypes.c_bool
    for single, want in ((False, f64), (True, f32)):
        with Planned(lib, n, single, coarsest) as g:
            assert brick_ok(g, 0, 2, 2, False) == want, single
