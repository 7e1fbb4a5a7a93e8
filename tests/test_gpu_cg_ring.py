"""The CG iterate after k steps, for every number of directions that the solver may still hold
when it stops (it moves the iterate along four at a time), against k steps of textbook CG in
FP64 from the oracle's operator, for the whole and the reduced system.

Tolerance, relative to |x_k|: a step rounds p, q and r once and applies a rounded operator twice;
8 k u of the storage type bounds the four together (FP64: 1e-12). A lost direction would show:
each one's share of x_k is checked to be above twice that."""
import numpy as np
import pytest

import oracle
from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn
from gpu_util import make_pair, rel

pytestmark = pytest.mark.gpu

U = {"f64": 2.0 ** -53, "f32": 2.0 ** -24, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}
DIMS = (4, 4, 6, 6)


@pytest.fixture(scope="module")
def systems():
    gop, oop, _, _ = make_pair(DIMS, -0.05, 1.7, 0.3, seed=21)
    eta = syn.gaussian_spinor(DIMS, 22)
    sc = oracle.Schur(oop)
    return gop, eta, {False: (oop.normal, eta), True: (sc.normal, np.where(sc.even, eta, 0.0))}


def cg(normal, eta, k):
    """x_k and the steps alpha_l p_l that it is the sum of."""
    x, r = np.zeros_like(eta), eta.copy()
    p, rr, steps = r.copy(), np.vdot(r, r).real, []
    for _ in range(k):
        w = normal(p)
        a = rr / np.vdot(p, w).real
        steps.append(a * p)
        x, r = x + steps[-1], r - a * w
        new = np.vdot(r, r).real
        p, rr = r + (new / rr) * p, new
    return x, steps


@pytest.mark.parametrize("schur", [False, True])
@pytest.mark.parametrize("inner,steps", [("f64", (1, 2, 3, 4, 5, 6, 7, 8)), ("f32", (1, 2, 3, 4, 5, 6, 7, 8)),
                                         ("f16", (1, 2, 3, 4, 5, 6)), ("bf16", (1, 2))])
def test_iterate_after_k_steps(systems, schur, inner, steps):
    gop, eta, which = systems
    normal, src = which[schur]
    out = gop.new_field()
    for k in steps:
        want, parts = cg(normal, src, k)
        tol = 1e-12 if inner == "f64" else 8 * k * U[inner]
        assert min(np.linalg.norm(s) for s in parts) > 2 * tol * np.linalg.norm(want), (inner, k)
        info = qdw.cgne_solve(gop, gop.pack(eta), out, res=1e-14, nmx=k, inner=inner, delta=0.0, schur=schur)
        assert info["status"] == -1 and info["n_steps"] == k
        got = gop.unpack(out).cpu().numpy()
        if schur:
            got = np.where(oracle.site_parity(DIMS).reshape(-1, 1, 1) == 0, got, 0.0)
        assert rel(got, want) <= tol, (inner, k, rel(got, want), tol)
