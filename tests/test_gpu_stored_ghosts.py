"""Step loops read the ghosts that the state holds.

A state may be uploaded with ghosts that are not those of the boundary
condition and stepped without ``fill_ghosts``, or changed at an edge cell
between steps: the first step then reads the stored ghosts, whether it runs by
itself, in a captured loop or in ``ws_step_traces``.  Everything equals as many
single calls bit for bit.
"""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DX, DY, DT = 1 / 64, 1 / 50, 0.003


@pytest.fixture(scope="module")
def ws():
    import paper_1808_02638_amd as m

    return m


def _pair(ws, shapes, dtype=torch.float64, limiter="mc", bc="extrap", link=None):
    g = torch.Generator().manual_seed(11)
    q = [torch.randn((3, my + 4, mx + 4), generator=g, dtype=torch.float64) for mx, my in shapes]
    levels = []
    for _ in range(2):
        lev = ws.Level([dict(mx=mx, my=my, dx=DX, dy=DY, bc=bc) for mx, my in shapes],
                       [(1.0, 4.0)], dtype=dtype, limiter=limiter)
        if link:
            lev.link(*link)
        for k, t in enumerate(q):
            lev.upload(k, t)
        lev.set_dt([DT])
        levels.append(lev)
    return levels


def _same(a, b, pools=2):
    torch.cuda.synchronize()
    for w in range(pools):
        x, y = (lev.pools[lev.current_pool() ^ w].view(lev.dtype) for lev in (a, b))
        for k in range(a.n):
            assert torch.equal(a.patch_view(x, k), b.patch_view(y, k)), (w, k)
    for x, y in zip(a.read_dt_cfl(), b.read_dt_cfl()):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("n", [2, 5, 6, 9, 12, 18])
@pytest.mark.parametrize("dtype,limiter", [(torch.float64, "mc"), (torch.float32, "vanleer")])
@pytest.mark.parametrize("shapes", [[(1, 1)], [(130, 77)], [(57, 40), (16, 17)], [(400, 340)],
                                    [(113, 1), (400, 340)]])
def test_loop_from_stored_ghosts(ws, shapes, dtype, limiter, n):
    a, b = _pair(ws, shapes, dtype, limiter)
    a.capture(n, 0.9)
    a.graph_launch()
    for _ in range(n):
        b.step_auto(0.9)
    _same(a, b)


@pytest.mark.parametrize("n", list(range(1, 14)))
@pytest.mark.parametrize("periodic", [(False, False), (True, False)])
def test_tiled_loop_from_stored_ghosts(ws, periodic, n):
    xs, ys = [0, 57, 61, 130], [0, 2, 40, 77]
    shapes = [(x1 - x0, y1 - y0) for y0, y1 in zip(ys, ys[1:]) for x0, x1 in zip(xs, xs[1:])]
    org = [(x, y) for y in ys[:-1] for x in xs[:-1]]
    a, b = _pair(ws, shapes, bc=None, link=(org, (130, 77), periodic))
    a.capture(n, 0.9)
    a.graph_launch()
    for _ in range(n):
        b.step_auto(0.9)
    _same(a, b)


@pytest.mark.parametrize("shape", [(130, 77), (400, 340)])
def test_edge_cell_changed_between_loops(ws, shape):
    """A replay starts from the ghosts as the last step left them."""
    mx, my = shape
    a, b = _pair(ws, [shape])
    ij = torch.tensor([[0, 5], [mx - 1, my - 1], [3, 0]], dtype=torch.int32, device="cuda")
    val = torch.tensor([0.5, -1.5, 2.0], dtype=torch.float64, device="cuda")
    a.capture(6, 0.9)
    for _ in range(2):
        a.graph_launch()
        for _ in range(6):
            b.step_auto(0.9)
        for lev in (a, b):
            lev.add_at(0, 0, ij, val)
    _same(a, b)


@pytest.mark.parametrize("record", [True, False])
@pytest.mark.parametrize("n_steps,last", [(2, 0), (3, 1), (6, 0), (7, 1)])
def test_traces_from_stored_ghosts(ws, n_steps, last, record):
    C, L = ws._lib, ws._lib.lib()
    mx, my = 130, 77
    a, b = _pair(ws, [(mx, my)])
    # every cell within two of a side, where a step reads the ghosts
    J, I = np.divmod(np.arange(mx * my), mx)
    near = (I < 2) | (I >= mx - 2) | (J < 2) | (J >= my - 2)
    ij = torch.tensor(np.stack([I[near], J[near]], 1), dtype=torch.int32, device="cuda")
    nr, nb = ij.shape[0], a.mask_bytes()
    tr, tr_b = (torch.zeros((n_steps, nr), dtype=torch.float64, device="cuda") for _ in range(2))
    mk, mk_b = (torch.full((n_steps, nb), 255, dtype=torch.uint8, device="cuda")
                for _ in range(2))
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    torch.cuda.synchronize()
    C.check(L.ws_step_traces(a._ctx, n_steps, DT, 0, nr, p(ij), p(tr), p(mk) if record else None,
                             nb, last))
    for s in range(n_steps):
        if record:
            b.step_record_masks(DT, mk_b[s])
        else:
            b.step(DT, read_cfl=False)
        b.gather(0, 0, ij, tr_b[s])
    torch.cuda.synchronize()
    assert torch.equal(tr, tr_b)
    assert torch.equal(mk, mk_b)
    assert torch.equal(a.state_view(0), b.state_view(0))
