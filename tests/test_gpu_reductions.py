"""Grid-wide sums at the edges of the launch: one run of 64 sites, a ragged last block whose
padding holds NaN, fewer and more runs than wavefronts in the launch.

Tolerance: a sum of n products passes through at most about 8 n / (lanes of the launch) + 40
additions in a row, under 200 here, each rounding by 2^-53 relative to |x| |y|: 200 * 2^-53
= 2.3e-14, and 1e-13 is required."""
import numpy as np
import pytest

from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn

pytestmark = pytest.mark.gpu


def _padding(dims):
    """Mask of the padding positions of an FP64 field as doubles."""
    half = syn.volume(dims) // 2
    pad = (half + 63) // 64 * 64
    i = np.arange(pad)
    m = np.zeros((2, pad // 64, 12, 64, 2), dtype=bool)
    m[:, i // 64, :, i % 64, :] = (i >= half)[:, None, None, None]
    return m.reshape(-1)


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 6, 10), (16, 8, 8, 8), (20, 14, 18, 22)])
def test_sums_at_launch_edges(dims):
    import torch
    su3, th = syn.unit_gauge_field(dims)
    op = qdw.Op(dims, su3, th, 0.0, 1.0)
    a, b = syn.gaussian_spinor(dims, 1), syn.gaussian_spinor(dims, 2)
    x, y = op.pack(a), op.pack(b)
    mask = torch.as_tensor(_padding(dims)).cuda()
    for f in (x, y):
        f.view(torch.float64)[mask] = float("nan")
    na, nb = np.linalg.norm(a), np.linalg.norm(b)
    for _ in range(3):  # the arrival counters are back at zero after every launch
        assert abs(qdw.norm2(op, x) - na ** 2) <= 1e-13 * na ** 2
        assert abs(qdw.cdot(op, x, y) - np.vdot(a, b)) <= 1e-13 * na * nb
    # a map leaves the padding alone
    qdw.axpby(op, 1.0, x, 0.0, y)
    assert np.array_equal(op.unpack(y).cpu().numpy(), a)
