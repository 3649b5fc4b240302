"""Several steps per launch in captured loops: the same bits as single steps.

A captured loop of a level whose patches have extrapolation boundaries takes
pairs of steps in one launch, and on a small level four.  State, ghosts, the other pool (the state one
step earlier), time steps and Courant numbers equal those of as many eager
single steps, bit for bit, at the edges of the pairing (1 .. 8 steps), of the
56-column segments and of the rows that a segment shares with its neighbours.
"""

import ctypes
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    import paper_1808_02638_amd as m

    return m


def _pair(ws, sizes, dtype, limiter):
    g = torch.Generator().manual_seed(7)
    mats = [(1.0 + 0.3 * k, 4.0 + k) for k in range(len(sizes))]
    patches = [dict(mx=a, my=b, dx=1 / a, dy=1.3 / b, instance=k, bc="extrap")
               for k, (a, b) in enumerate(sizes)]
    levels = [ws.Level(patches, mats, dtype=dtype, limiter=limiter) for _ in range(2)]
    for k, (a, b) in enumerate(sizes):
        q = torch.randn((3, b + 4, a + 4), generator=g, dtype=torch.float64)
        for lev in levels:
            lev.upload(k, q)
    dts = [(0.45 + 0.45 * (k % 2)) * min(1 / a, 1.3 / b) / math.sqrt(K / rho)
           for k, ((a, b), (rho, K)) in enumerate(zip(sizes, mats))]
    for lev in levels:
        lev.fill_ghosts()
        lev.set_dt(dts)
    return levels


def _same(a, b):
    torch.cuda.synchronize()  # the levels run on streams of their own
    pools = [(lev.pools[w].view(lev.dtype)) for lev in (a, b)
             for w in (lev.current_pool(), 1 - lev.current_pool())]
    for k in range(a.n):
        assert torch.isfinite(a.patch_view(pools[0], k)).all()
        assert torch.equal(a.patch_view(pools[0], k), b.patch_view(pools[2], k)), k
        assert torch.equal(a.patch_view(pools[1], k), b.patch_view(pools[3], k)), k
    for x, y in zip(a.read_dt_cfl(), b.read_dt_cfl()):
        assert np.array_equal(x, y)
    assert np.array_equal(a.patch_cfl(), b.patch_cfl())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("limiter", ["mc", "vanleer", "none"])
@pytest.mark.parametrize("sizes", [[(1, 1)], [(2, 3)], [(5, 1)], [(56, 33)], [(57, 64)],
                                   [(16, 17), (31, 8)], [(113, 18), (60, 5), (24, 200)],
                                   [(256, 255)]])
@pytest.mark.parametrize("small", [True, False])
def test_pairs_equal_single_steps(ws, small, sizes, limiter, dtype):
    # few tiles of 16 x 16 cells (one per CU in FP64): four steps per launch;
    # else pairs
    a, b = _pair(ws, sizes if small else sizes + [(400, 340)], dtype, limiter)
    a.capture(18, 0.9)
    for _ in range(2):  # a replay, with eager reads between
        a.graph_launch()
        for _ in range(18):
            b.step_auto(0.9)
        _same(a, b)


@pytest.mark.parametrize("tile", [("march", 64, 4), ("march", 64, 16), ("direct", 64, 4)])
def test_one_row_patch_has_both_ghost_sides(ws, tile):
    """MARCH tiles of a patch with one row write its ghosts above as well."""
    a, b = _pair(ws, [(70, 1)], torch.float64, "mc")
    a.set_tiling(tile[1], tile[2], variant=tile[0])
    b.set_tiling(32, 8, variant="direct")
    for lev in (a, b):
        lev.set_dt([0.2])
        for _ in range(5):
            lev.step(0.002)
    _same(a, b)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 12, 13, 16])
@pytest.mark.parametrize("shape", [(130, 77), (300, 211)])
def test_every_remainder_of_the_pairing(ws, shape, n):
    a, b = _pair(ws, [shape], torch.float64, "mc")
    a.capture(n, 0.9)
    a.graph_launch()
    for _ in range(n):
        b.step_auto(0.9)
    _same(a, b)


@pytest.mark.parametrize("dtype,limiter", [(torch.float64, "mc"), (torch.float64, "vanleer"),
                                           (torch.float32, "mc")])
@pytest.mark.parametrize("xs,ys", [([0, 3], [0, 2]), ([0, 1, 2, 5], [0, 1, 4, 5]),
                                   ([0, 57, 61, 130], [0, 2, 40, 77]), ([0, 200, 300], [0, 211])])
@pytest.mark.parametrize("periodic", [(False, False), (True, False), (False, True), (True, True)])
def test_tiled_pairs_equal_single_steps(ws, xs, ys, periodic, dtype, limiter):
    """A tiled level's pairs of steps work the domain as a whole; ghosts too."""
    g = torch.Generator().manual_seed(5)
    size = [(x1 - x0, y1 - y0) for y0, y1 in zip(ys, ys[1:]) for x0, x1 in zip(xs, xs[1:])]
    org = [(x, y) for y in ys[:-1] for x in xs[:-1]]
    dx, dy = 1 / xs[-1], 1.3 / ys[-1]
    q = [torch.randn((3, h + 4, w + 4), generator=g, dtype=torch.float64) for w, h in size]
    levels = []
    for _ in range(2):
        lev = ws.Level([dict(mx=w, my=h, dx=dx, dy=dy) for w, h in size], [(1.0, 4.0)],
                       dtype=dtype, limiter=limiter)
        lev.link(org, (xs[-1], ys[-1]), periodic=periodic)
        for k in range(lev.n):
            lev.upload(k, q[k])
        lev.fill_ghosts()
        lev.set_dt([0.4 * min(dx, dy)])
        levels.append(lev)
    a, b = levels
    a.capture(6, 0.9)
    for _ in range(2):
        a.graph_launch()
        for _ in range(6):
            b.step_auto(0.9)
        _same(a, b)


@pytest.mark.parametrize("n_steps,last", [(1, 0), (2, 0), (2, 1), (5, 0), (6, 1)])
@pytest.mark.parametrize("shape,nr", [((61, 9), 7), ((130, 77), 70), ((57, 40), 300)])
def test_traces_branches_and_sweep(ws, shape, nr, n_steps, last):
    """ws_step_traces and ws_adjoint_sweep against single calls, bit for bit."""
    mx, my = shape
    C = ws._lib
    L = C.lib()
    (a, b) = _pair(ws, [(mx, my)], torch.float64, "mc")
    dt = 0.4 * min(1 / mx, 1.3 / my) / 2.0
    at = np.random.default_rng(3).choice(mx * my, nr, replace=False)
    ij = torch.tensor(np.stack([at % mx, at // mx], 1), dtype=torch.int32, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    nb = a.mask_bytes()
    tr, tr_b = (torch.zeros((n_steps, nr), dtype=torch.float64, device="cuda") for _ in range(2))
    mk, mk_b = (torch.full((n_steps, nb), 255, dtype=torch.uint8, device="cuda")
                for _ in range(2))
    g = torch.randn((n_steps + 1, nr), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    C.check(L.ws_step_traces(a._ctx, n_steps, dt, 0, nr, p(ij), p(tr), p(mk), nb, last))
    for s in range(n_steps):
        b.step_record_masks(dt, mk_b[s])
        b.gather(0, 0, ij, tr_b[s])
    torch.cuda.synchronize()
    assert torch.equal(tr, tr_b)
    assert torch.equal(mk, mk_b)
    assert torch.equal(a.state_view(0), b.state_view(0))
    if last:
        _same(a, b)
    lam = [a.new_buffer() for _ in range(4)]
    for x in (lam[0], lam[2]):
        a.patch_view(x, 0)[0, 2:-2, 2:-2] = 0.25
    torch.cuda.synchronize()
    C.check(L.ws_adjoint_sweep(a._ctx, n_steps, dt, p(mk), nb, 0, nr, p(ij), p(g[1:]), 1, 1,
                               p(lam[0]), p(lam[1])))
    b.add_at(0, 0, ij, g[n_steps], buf=lam[2])
    for s in range(n_steps - 1, -1, -1):
        b.adjoint_step(dt, mk_b[s], lam[2], lam[3])
        b.add_at(0, 0, ij, g[s], buf=lam[3])
        lam[2], lam[3] = lam[3], lam[2]
    torch.cuda.synchronize()
    assert torch.equal(a.patch_view(lam[n_steps % 2], 0), b.patch_view(lam[2], 0))
