"""The two marching forms of D, with the tile's spinors in LDS and without, on either side of the
launch sizes where one takes over from the other (many small tiles: x1 slabs of a few sites),
against the plain form; the same inside the CG step, whose sums and residual update ride on
the operator; and the time of the default form where a wave per SIMD is all a launch has.

Tolerances: the forms add the same nine terms of a site in another order, a few roundings of
the largest term: 16 u relative to the largest component, and for 16-bit storage one rounding
of the output more (2 u)."""
import pytest

from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn
from gpu_util import maxrel

pytestmark = pytest.mark.gpu

U32, U = 2.0 ** -24, {"f64": 2.0 ** -53, "f32": 2.0 ** -24, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}


def tolerance(prec):
    return 16 * U[prec] if prec in ("f64", "f32") else 16 * U32 + 2 * U[prec]


def apply(op, x, prec, dag, shape=None):
    out = op.new_field(prec)
    if shape:
        qdw.set_dw_shape(op, prec, *shape)
    (qdw.dw_dag_apply if dag else qdw.dw_apply)(op, x, out, prec)
    return op.unpack(out, prec).cpu().numpy()


# 64-site units of a launch with walk 1 and nt = 1, 2, 4: 1920, 960, 480 (the last size of the
# form without the tile in FP32), 2056, 1028, 514 (FP64: beyond it) and, two ragged tiles a
# slab, 2048, 1024, 512 (a full round of FP32; the last size without the tile in FP64); with
# walk 0 the ragged last tile of 9180 sites: 576, 288, 144
@pytest.mark.parametrize("dims,walk", [((4, 480, 2, 2), 1), ((4, 514, 2, 4), 1), ((4, 256, 6, 22), 1),
                                       ((4, 18, 30, 34), 0)])
@pytest.mark.parametrize("dag", [False, True])
def test_marching_forms_equal_plain_form(dims, walk, dag):
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 81)
    op = qdw.Op(dims, su3, th, -0.05, 1.7)
    psi = syn.gaussian_spinor(dims, 82)
    for prec in U:
        x = op.pack(psi, prec)
        want = apply(op, x, prec, dag, (64, 1, 0, 0, 0))
        for ts in (64, 128) if prec != "f64" else (64,):
            for nt in (1, 2, 4):
                for pipe in (0, 1):
                    got = apply(op, x, prec, dag, (ts, nt, pipe, walk, 1))
                    assert maxrel(got, want) <= tolerance(prec), (prec, ts, nt, pipe)


@pytest.mark.parametrize("dims", [(24, 12, 12, 12), (8, 18, 30, 34)])  # FP64: 336 and 1152 units
@pytest.mark.parametrize("inner", ["f64", "f32", "f16", "bf16"])
def test_cg_on_the_marching_forms(dims, inner):
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 83)
    op = qdw.Op(dims, su3, th, 0.1, 1.7)
    eta, psi = op.pack(syn.gaussian_spinor(dims, 84)), op.new_field()
    info = qdw.cgne_solve(op, eta, psi, res=1e-10, inner=inner)
    assert info["status"] > 0 and info["rel_res_true"] <= 1e-10
    qdw.set_dw_shape(op, "f64", 64, 1, 0, 0, 0)
    t, r = op.new_field(), op.new_field()
    qdw.dw_apply(op, psi, t)
    qdw.dw_dag_apply(op, t, r)
    qdw.axpby(op, 1.0, eta, -1.0, r)
    assert qdw.norm2(op, r) ** 0.5 <= 1.01e-10 * qdw.norm2(op, eta) ** 0.5


def best_us(fn, n=50):
    import torch
    for _ in range(5):
        fn()
    best = float("inf")
    for _ in range(8):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(n):
            fn()
        e1.record()
        e1.synchronize()
        best = min(best, 1e3 * e0.elapsed_time(e1) / n)
    return best


def test_default_form_is_not_slower_than_the_plain_one():
    """56,448 sites, FP64, just past the form for small lattices: marching takes 15.9 us and the
    best plain shape 17.4 us; with the tile in LDS at one wave per SIMD marching took 19.4."""
    dims = (24, 14, 14, 12)
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 85)
    op = qdw.Op(dims, su3, th, -0.05, 1.7)
    x, y = op.pack(syn.gaussian_spinor(dims, 86)), op.new_field()
    default = best_us(lambda: qdw.dw_apply(op, x, y))
    qdw.set_dw_shape(op, "f64", 64, 1, 1, 0, 0)
    plain = best_us(lambda: qdw.dw_apply(op, x, y))
    assert default <= 1.03 * plain, (default, plain)


@pytest.mark.parametrize("dims,prec,other,was", [
    ((4, 60, 22, 54), "f64", (64, 4, 0, 0, 1), "75 against 90 us in chunks of one slice"),
    ((50, 34, 12, 50), "f32", (64, 2, 1, 0, 1), "137 against 151 us in chunks of ten slices"),
    ((38, 8, 32, 20), "f32", (64, 2, 1, 0, 1), "25.7 against 28.2 us with the plain hop loop")])
def test_default_chunk_is_not_slower_than_another(dims, prec, other, was):
    import torch
    V = syn.volume(dims)
    su3 = torch.eye(3, dtype=torch.complex128, device="cuda").expand(V, 4, 3, 3).contiguous()
    op = qdw.Op(dims, su3, torch.zeros(V, 4, dtype=torch.float64, device="cuda"), -0.05, 1.7)
    x, y = op.pack(torch.randn(V, 4, 3, dtype=torch.complex128, device="cuda"), prec), op.new_field(prec)
    default = best_us(lambda: qdw.dw_apply(op, x, y, prec), 20)
    qdw.set_dw_shape(op, prec, *other)
    assert default <= 1.03 * best_us(lambda: qdw.dw_apply(op, x, y, prec), 20), (default, was)
