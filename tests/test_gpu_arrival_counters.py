"""Sums over an operator's fields do not depend on what an earlier reduction left in the
operator's arrival counters: two reductions at a time on one operator (which is not allowed, and
spoils their results) leave counts behind, and every later sum is right all the same.

The counters are the 33 words, one per 128 bytes, before the scalars (512 bytes) and the check
word (256 bytes) at the end of the operator's device block, which has 256 bytes of room for
its alignment."""
import numpy as np
import pytest

from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn

pytestmark = pytest.mark.gpu

WORDS = 33 * 16  # of 8 bytes


@pytest.mark.parametrize("left", [1, 5])
def test_sums_after_a_disturbed_reduction(left):
    import torch
    dims = (8, 8, 8, 8)
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 31)
    op = qdw.Op(dims, su3, th, 0.1, 1.7)
    assert op._dev_mem.data_ptr() % 256 == 0
    end = op.device_bytes - 256 - 256 - 512
    counters = op._dev_mem[end - 4352:end - 4352 + 8 * WORDS].view(torch.int64)
    psi = syn.gaussian_spinor(dims, 32)
    x, out = op.pack(psi), op.new_field()
    want = np.linalg.norm(psi) ** 2
    assert abs(qdw.norm2(op, x) - want) <= 1e-13 * want
    scratch = op.new_field()
    for scale in (2.0, 3.0):
        counters += left  # the arrivals of a launch that was cut short
        qdw.axpby(op, scale, x, 0.0, scratch)
        assert abs(qdw.norm2(op, scratch) - scale ** 2 * want) <= 1e-13 * scale ** 2 * want
    counters += left
    info = qdw.cgne_solve(op, x, out, res=1e-10, inner="f32")
    assert info["status"] > 0 and info["rel_res_true"] <= 1e-10
