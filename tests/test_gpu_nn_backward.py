"""The fused bf16 backward layers against the FP32-operand passes where their launches differ:
a lattice with one block of 64 sites per parity, one with fewer blocks than shares and a
ragged last block, and one with more blocks than shares of every layer, ragged too.

Tolerance: every operand of the three layers' products is rounded to bf16 (2^-9 relative);
a gradient passes through at most six such roundings one after another, each adding its
error in quadrature to sums of independent terms: sqrt(6) * 2^-9 * sqrt(2) = 7e-3 of the
norm; 3e-2 is the bar of the comparison with the oracle and is used here too."""
import numpy as np
import pytest

import oracle
from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(4, 4, 2, 4), (6, 4, 4, 6), (20, 14, 18, 22)])
def test_bf16_gradients_match_fp32_operands(dims):
    import torch
    su3, th = syn.gauge_field(dims, 0.3, 0.1, 51)
    op = qdw.Op(dims, su3, th, -0.05, 1.7)
    w = qdw.nn_weights_tensor(oracle.nn_identity_weights(seed=6, scale=0.3))
    x, g = op.pack(syn.gaussian_spinor(dims, 52)), op.pack(syn.gaussian_spinor(dims, 53))
    got = {}
    for f32 in (True, False):
        dW, gin = torch.zeros_like(w), op.new_field()
        qdw.nn_backward(op, w, x, g, dW, gin, f32_mixing=f32)
        got[f32] = qdw.nn_weights_layers(dW), op.unpack(gin).cpu().numpy()
    for a, b in zip(got[True][0], got[False][0]):
        assert np.linalg.norm(a - b) <= 3e-2 * np.linalg.norm(a)
    a, b = got[True][1], got[False][1]
    assert np.linalg.norm(a - b) <= 3e-2 * np.linalg.norm(a)
