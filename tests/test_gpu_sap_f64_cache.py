"""The plain FP64 block solver with the block operator kept on the CU (registers and LDS),
forced on and off, against the oracle: 256-site blocks, whose offsets are compile-time
constants, unequal extents, and blocks that leave lanes and LDS rows unused; both colours, and
the Schwarz cycle of two right-hand sides."""
import pytest

import synth
from oracle import solvers
from tests.helpers import clover, gauge, lattice, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,block", [((8, 8, 8, 8), (4, 4, 4, 4)), ((16, 4, 8, 8), (8, 2, 4, 4)),
                                        ((8, 6, 6, 6), (4, 3, 3, 3)), ((4, 4, 4, 4), (2, 2, 2, 2))])
@pytest.mark.parametrize("bc_t", [1, -1])
def test_plain_f64_operator_on_the_cu(dims, block, bc_t):
    m0, csw = -0.1, 1.0
    lat = lattice(dims, block, m0, csw, bc_t)
    U, A = gauge(dims), clover(dims, m0, csw)
    eta = synth.gaussian_spinor(dims, nrhs=2, seed=83)
    for cache in (1, 0, -1):
        lat.set_option("sap_cache", cache)
        for colour in (0, 1):
            zw, rw = solvers.mr_blocks(U, A, eta[0], block, colour, 4, bc_t)
            z, rho = lat.sap_block_mr(to_dev(eta[0]), colour, 4, prec="f64", eo=False)
            assert rel(to_np(z), zw) < 1e-12 and rel(to_np(rho), rw) < 1e-12, (cache, colour)
        got = to_np(lat.sap(to_dev(eta), ncy=2, nmr=3, prec="f64", eo=False))
        for r in range(2):
            assert rel(got[r], solvers.sap(U, A, eta[r], block, nmr=3, ncy=2, bc_t=bc_t)) < 1e-12, (cache, r)
