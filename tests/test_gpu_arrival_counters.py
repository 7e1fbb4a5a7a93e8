"""Sums over an operator's fields after two reductions at a time on that operator. An operator is
used from one stream at a time, so those sums themselves may be wrong; what they leave in the
operator's arrival counters must not spoil the later ones. Launches of fewer workgroups than
there are counters (4^4: 3 or 6) come between larger ones."""
import threading

import numpy as np
import pytest

from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (16, 8, 8, 8)])
def test_sums_after_two_at_a_time(dims):
    import torch
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 31)
    op = qdw.Op(dims, su3, th, 0.1, 1.7)
    psi = syn.gaussian_spinor(dims, 32)
    x, y, out = op.pack(psi), op.pack(2.0 * psi), op.new_field()
    want = np.linalg.norm(psi) ** 2

    def many(field):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(200):
                qdw.norm2(op, field)

    for _ in range(2):
        threads = [threading.Thread(target=many, args=(f,)) for f in (x, y)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert abs(qdw.norm2(op, x) - want) <= 1e-13 * want
        assert abs(qdw.cdot(op, x, y) - 2.0 * want) <= 2e-13 * want
        for schur in (False, True):
            info = qdw.cgne_solve(op, x, out, res=1e-10, inner="f32", schur=schur)
            assert info["status"] > 0 and info["rel_res_true"] <= 1e-10
        info = qdw.sap_gcr_solve(op, x, out, precond="none")
        assert info["status"] > 0 and info["rel_res_true"] <= 1e-10
