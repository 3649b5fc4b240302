"""Captured loops of tiled levels at the edges of what they may work as one
domain: the same bits as single steps."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    import paper_1808_02638_amd as m

    return m


def _pair(ws, shapes, cells, org, domain, dtype, dt):
    g = torch.Generator(device="cuda").manual_seed(3)
    q = [torch.randn((3, my + 4, mx + 4), generator=g, dtype=torch.float32, device="cuda")
         for mx, my in shapes]
    levels = []
    for _ in range(2):
        lev = ws.Level([dict(mx=mx, my=my, dx=dx, dy=dy)
                        for (mx, my), (dx, dy) in zip(shapes, cells)], [(1.0, 4.0)], dtype=dtype)
        lev.link(org, domain, periodic=(False, False))
        for k, t in enumerate(q):
            lev.upload(k, t)
        lev.fill_ghosts()
        lev.set_dt([dt])
        levels.append(lev)
    return levels


def _loop_is_single_steps(a, b, n):
    a.capture(n, 0.9)
    a.graph_launch()
    for _ in range(n):
        b.step_auto(0.9)
    torch.cuda.synchronize()
    for k in range(a.n):
        assert torch.equal(a.state_view(k), b.state_view(k)), k
    for x, y in zip(a.read_dt_cfl(), b.read_dt_cfl()):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("which", [0, 1])
def test_cell_sizes_equal_to_rounding(ws, which):
    """Cell sizes may differ by 1e-12 relative; every patch steps with its own."""
    cells = [[0.01, 0.02], [0.01, 0.02], [0.01, 0.02], [0.01, 0.02]]
    cells[3][which] *= 1 + 5e-13
    org = [(0, 0), (70, 0), (0, 33), (70, 33)]
    a, b = _pair(ws, [(70, 33), (60, 33), (70, 44), (60, 44)], cells, org, (130, 77),
                 torch.float64, 0.004)
    _loop_is_single_steps(a, b, 6)


@pytest.mark.parametrize("axis", ["x", "y"])
def test_domain_wider_than_tile_numbers(ws, axis):
    """More tiles along one direction of the domain than a tile's 16-bit
    position can number."""
    n, m = (8, 500000) if axis == "x" else (7, 1000000)
    one = [(m, 1) if axis == "x" else (1, m)] * n
    org = [(m * k, 0) if axis == "x" else (0, m * k) for k in range(n)]
    a, b = _pair(ws, one, [(0.01, 0.01)] * n, org, (n * m, 1) if axis == "x" else (1, n * m),
                 torch.float32, 0.004)
    _loop_is_single_steps(a, b, 6)
