"""Two steps per launch in captured loops: the same bits as single steps.

A captured loop of a level whose patches have extrapolation boundaries takes
pairs of steps in one launch.  State, ghosts, the other pool (the state one
step earlier), time steps and Courant numbers equal those of as many eager
single steps, bit for bit, at the edges of the pairing (1 .. 8 steps), of the
56-column segments and of the rows that a segment shares with its neighbours.
"""

import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


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
                                   [(113, 18), (60, 5), (24, 200)], [(300, 211)]])
def test_pairs_equal_single_steps(ws, sizes, limiter, dtype):
    a, b = _pair(ws, sizes, dtype, limiter)
    a.capture(8, 0.9)
    for _ in range(2):  # a replay, with eager reads between
        a.graph_launch()
        for _ in range(8):
            b.step_auto(0.9)
        _same(a, b)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7])
def test_every_remainder_of_the_pairing(ws, n):
    a, b = _pair(ws, [(130, 77)], torch.float64, "mc")
    a.capture(n, 0.9)
    a.graph_launch()
    for _ in range(n):
        b.step_auto(0.9)
    _same(a, b)
