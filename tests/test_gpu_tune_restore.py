"""The autotune cache restores what the tuner chose: an operator whose shape comes from the cache
runs the same D, at the same speed, as the one that was tuned, also where the tuner keeps the
default form (8^4, where no shape is as fast); an entry that does not say so pins its shape."""
import json

import pytest

from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn
from test_gpu_march_forms import best_us

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f16"])
def test_cached_operator_is_the_tuned_one(tmp_path, prec):
    import torch
    dims = (8, 8, 8, 8)
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 95)
    path = str(tmp_path / "shapes.json")
    us, out = {}, {}
    for how in ("tuned", "cached"):
        op = qdw.Op(dims, su3, th, -0.05, 1.7)
        qdw.set_dw_shape(op, prec, 64, 8, 0, 0, 0)  # whatever the operator had before
        assert qdw.autotune_cached(op, prec, 1, path) == (how, qdw.get_dw_shape(op, prec))
        x, out[how] = op.pack(syn.gaussian_spinor(dims, 96), prec), op.new_field(prec)
        us[how] = best_us(lambda: qdw.dw_apply(op, x, out[how], prec))
    assert us["cached"] <= 1.25 * us["tuned"]  # the form for small lattices takes half the time
    assert torch.equal(out["tuned"], out["cached"])


def test_default_can_be_read_and_restored(tmp_path):
    dims = (8, 8, 8, 8)
    su3, th = syn.unit_gauge_field(dims)
    op = qdw.Op(dims, su3, th, -0.05, 1.7)
    created = qdw.get_dw_shape(op)
    assert qdw.dw_shape_is_default(op)
    qdw.set_dw_shape(op, "f64", 64, 2, 0, 0, 0)
    assert not qdw.dw_shape_is_default(op) and qdw.dw_shape_is_default(op, "f32")
    qdw.default_dw_shape(op)
    assert qdw.dw_shape_is_default(op) and qdw.get_dw_shape(op) == created
    import torch
    path = str(tmp_path / "shapes.json")
    key = qdw.tune_key(dims, "f64", 1, torch.cuda.get_device_name(op.device), qdw.kernel_version())
    with open(path, "w") as fh:
        json.dump({"version": 1, "entries": {key: [64, 2, 0, 0, 0]}}, fh)
    assert qdw.autotune_cached(op, "f64", 1, path) == ("cached", (64, 2, 0, 0, 0))
    assert not qdw.dw_shape_is_default(op)
