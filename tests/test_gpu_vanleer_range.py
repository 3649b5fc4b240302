"""van Leer's limiter at the ends of the type's range.

A wave moving right (u = p / Z, rows alike) steps up by b/2 and then by a/2
with a >> b.  The cell between the two jumps then changes by the small jump's
fluctuation and by the limited correction 2ab/(a + b) at the large one alone,
so the new p shows the quotient although a is near the largest number.  Where
the product ab overflows, so does the correction.
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N, AT, DX, DT = 130, 64, 0.1, 0.05  # c = Z = 1


@pytest.fixture(scope="module")
def ws():
    import paper_1808_02638_amd as m

    return m


def _cell(ws, dtype, a, b):
    lev = ws.Level([dict(mx=N, my=6, dx=DX, dy=DX, bc="extrap")], [(1.0, 1.0)], dtype=dtype,
                   limiter="vanleer")
    q = torch.zeros((3, 10, N + 4), dtype=torch.float64)
    q[:2, :, AT + 2] = b / 2
    q[:2, :, AT + 3:] = a / 2 + b / 2
    lev.upload(0, q)
    lev.step(DT, read_cfl=False)
    torch.cuda.synchronize()
    return lev.state_view(0)[:, 2:-2, AT + 2].double().cpu().numpy()


@pytest.mark.parametrize("dtype,a,b", [
    (torch.float32, 1.0, 0.5), (torch.float32, 8.4e37, 0.5), (torch.float32, 8.6e37, 0.5),
    (torch.float32, 1e38, 0.5), (torch.float32, 1.7e38, 0.9), (torch.float32, 3e38, 1e-3),
    (torch.float32, 1e18, 1e18), (torch.float32, 1e-3, 1e-3), (torch.float32, 1e-10, 1e-10),
    (torch.float64, 1.0, 0.5), (torch.float64, 4e307, 0.5), (torch.float64, 4.6e307, 0.5),
    (torch.float64, 1e308, 0.5), (torch.float64, 1.7e308, 1e-3), (torch.float64, 1e-100, 1e-100)])
def test_quotient_over_the_range(ws, dtype, a, b):
    nu = DT / DX
    lim = 2 * (a * (b / (a + b)))
    ref = b / 2 - nu * (0.5 * b + 0.25 * (1 - nu) * lim)
    got = _cell(ws, dtype, a, b)
    # b/2, the two terms and their factors: under ten roundings of values
    # of at most b/2 each
    tol = 5 * b * (2.0 ** -24 if dtype == torch.float32 else 2.0 ** -53)
    assert np.abs(got[0] - ref).max() <= tol, (got[0], ref)
    assert np.abs(got[1] - ref).max() <= tol, (got[1], ref)
    assert (got[2] == 0).all()


@pytest.mark.parametrize("dtype,a,b", [(torch.float32, 1e25, 1e20), (torch.float32, 2e19, 2e19),
                                       (torch.float64, 1e200, 1e150)])
def test_overflowing_product_is_infinite(ws, dtype, a, b):
    got = _cell(ws, dtype, a, b)
    assert (got[:2] == -np.inf).all(), got
