"""dw_apply_multi equals dw_apply on each field bit for bit where the default shape takes another
form or other settings for the several fields than for one:
  20 x 10^3      one field takes the form for small lattices, several march (FP64, FP32) or take
                 the plain form (16-bit storage);
  24 x 16^3      FP32 takes the pipelined hop loop for one field, the plain one for several;
  16 x 8 x 16 x 32, 32 fields   FP64 marches through 16 slices with the planes of x1 side by side.
Reading a shape and setting it again pins the default form's shape, which gives the same bits."""
import pytest

from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,n,precs", [((20, 10, 10, 10), 3, ("f64",)),
                                          ((20, 10, 10, 10), 6, ("f64", "f32", "f16", "bf16")),
                                          ((24, 16, 16, 16), 2, ("f64", "f32")),
                                          ((16, 8, 16, 32), 32, ("f64", "f32", "f16"))])
def test_several_fields_equal_single_fields(dims, n, precs):
    import torch
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 41)
    op = qdw.Op(dims, su3, th, -0.05, 1.7)
    srcs = [op.pack(syn.gaussian_spinor(dims, 42 + r)) for r in range(n)]
    for prec in precs:
        xs = [qdw.convert(op, s, "f64", op.new_field(prec), prec) for s in srcs]
        outs = [op.new_field(prec) for _ in xs]
        qdw.dw_apply_multi(op, xs, outs, prec)
        one = op.new_field(prec)
        for x, out in zip(xs, outs):
            qdw.dw_apply(op, x, one, prec)
            assert torch.equal(one, out), (prec, float((op.unpack(one, prec) - op.unpack(out, prec)).abs().max()))


@pytest.mark.parametrize("dag", [False, True])
def test_setting_the_shape_that_was_read_keeps_the_bits(dag):
    import torch
    dims = (8, 8, 8, 8)
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 43)
    op = qdw.Op(dims, su3, th, -0.05, 1.7)
    fn = qdw.dw_dag_apply if dag else qdw.dw_apply
    for prec in ("f64", "f32", "f16", "bf16"):
        x, a, b = op.pack(syn.gaussian_spinor(dims, 44), prec), op.new_field(prec), op.new_field(prec)
        fn(op, x, a, prec)
        qdw.set_dw_shape(op, prec, *qdw.get_dw_shape(op, prec))
        fn(op, x, b, prec)
        assert torch.equal(a, b), prec
