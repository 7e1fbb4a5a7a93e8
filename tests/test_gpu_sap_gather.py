"""The plain Schwarz block solve, whose lanes gather hops and links from LDS, in every storage
type over blocks of unequal extents, of 64 to 256 sites, of 192 sites (three wavefronts) and one
site wide (both neighbours of that direction in other blocks), against the oracle: 1e-4 in FP32
storage, 1e-2 and 5e-2 in binary16 and bfloat16, whose stored values carry 2^-11 and 2^-8."""
import pytest

import oracle
from paper_2202_07388_amd import qdw
from paper_2202_07388_amd import synthetic as syn
from gpu_util import make_pair, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sdtype,tol", [("f32", 1e-4), ("f16", 1e-2), ("bf16", 5e-2)])
@pytest.mark.parametrize("dims,bs", [((8, 4, 4, 8), (4, 2, 2, 4)), ((8, 8, 8, 4), (4, 4, 4, 2)),
                                     ((8, 8, 8, 6), (4, 4, 4, 3)), ((4, 16, 8, 16), (2, 8, 2, 8)),
                                     ((8, 8, 32, 2), (4, 4, 16, 1)), ((2, 8, 8, 16), (1, 4, 4, 8))])
def test_block_shapes(dims, bs, sdtype, tol):
    gop, oop, _, _ = make_pair(dims, 0.1, 1.5, 0.3, seed=7)
    rho = syn.gaussian_spinor(dims, 8)
    phi = gop.new_field()
    qdw.sap_apply(gop, gop.pack(rho), phi, 2, 3, bs, sdtype)
    err = rel(gop.unpack(phi).cpu().numpy(), oracle.sap(oop, rho, bs, 2, 3))
    assert err <= tol, (bs, sdtype, err)
