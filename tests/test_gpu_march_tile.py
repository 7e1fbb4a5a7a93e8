"""The marching form of D, whose spatial hops inside a workgroup's tile are read from LDS, against
the plain form: tiles of several planes, tiles that end inside a row, a half-filled last tile, a
two-site direction (both neighbours one site), and launches of several fields in the default
shape. The two forms add the same nine terms of a site in another order, so they differ by a few
roundings of the largest term: 16 u relative to the largest component, and for 16-bit storage
one rounding of the output more (2 u)."""
import pytest

from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn
from gpu_util import maxrel

pytestmark = pytest.mark.gpu

U32, U = 2.0 ** -24, {"f64": 2.0 ** -53, "f32": 2.0 ** -24, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}


def tolerance(prec):
    return 16 * U[prec] if prec in ("f64", "f32") else 16 * U32 + 2 * U[prec]


def plain(op, x, prec, dag):
    keep, out = qdw.get_dw_shape(op, prec), op.new_field(prec)
    qdw.set_dw_shape(op, prec, 64, 1, 0, 0, 0)
    (qdw.dw_dag_apply if dag else qdw.dw_apply)(op, x, out, prec)
    qdw.set_dw_shape(op, prec, *keep)
    return op.unpack(out, prec).cpu().numpy()


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 6), (2, 6, 10, 6), (4, 2, 8, 16), (4, 6, 6, 26)])
@pytest.mark.parametrize("walk", [0, 1])
def test_marching_form_equals_plain_form(dims, walk):
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 71)
    op = qdw.Op(dims, su3, th, -0.05, 1.7)
    psi = syn.gaussian_spinor(dims, 72)
    for prec in U:
        x = op.pack(psi, prec)
        for dag in (False, True):
            want = plain(op, x, prec, dag)
            for ts in (64, 128) if prec != "f64" else (64,):
                for nt in (1, 2, dims[0]):
                    for pipe in (0, 1):
                        qdw.set_dw_shape(op, prec, ts, nt, pipe, walk, 1)
                        out = op.new_field(prec)
                        (qdw.dw_dag_apply if dag else qdw.dw_apply)(op, x, out, prec)
                        got = op.unpack(out, prec).cpu().numpy()
                        assert maxrel(got, want) <= tolerance(prec), (prec, dag, ts, nt, pipe)


@pytest.mark.parametrize("dims", [(24, 12, 12, 14), (6, 20, 18, 26)])
@pytest.mark.parametrize("n", [2, 3])
def test_several_fields_in_the_default_shape(dims, n):
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 73)
    op = qdw.Op(dims, su3, th, -0.05, 1.7)
    srcs = [syn.gaussian_spinor(dims, 74 + k) for k in range(n)]
    for prec in ("f64", "f32"):
        xs, outs = [op.pack(s, prec) for s in srcs], [op.new_field(prec) for _ in srcs]
        qdw.dw_apply_multi(op, xs, outs, prec)
        for x, out in zip(xs, outs):
            assert maxrel(op.unpack(out, prec).cpu().numpy(), plain(op, x, prec, False)) <= tolerance(prec), prec
