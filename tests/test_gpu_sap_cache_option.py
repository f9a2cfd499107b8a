"""The operator-cache option where the matrix-core block solver would run: 0 and 1 ask for the
vector kernel's two ways of reading the operator and get them; -1 gives the choice back.  All
three against the oracle."""
import pytest

import synth
from oracle import solvers
from tests.helpers import clover, gauge, lattice, rel, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL = {"f16": 3e-3, "bf16": 2e-2}


@pytest.mark.parametrize("prec", ["f16", "bf16"])
def test_cache_option_reaches_the_vector_kernel(prec):
    import paper_1109_4279_amd as wc
    dims, block, n = (8, 8, 16, 16), (4, 4, 4, 4), 24
    lat = lattice(dims, block)
    eta = synth.gaussian_spinor(dims, nrhs=n, seed=131)
    x = to_dev(eta)
    want = {r: solvers.mr_blocks_eo(gauge(dims), clover(dims, -0.1, 1.0), eta[r], block, 1, 4) for r in (0, n - 1)}
    for cache, tile in ((-1, 4), (0, 1), (1, 1), (-1, 4)):
        lat.set_option("sap_cache", cache)
        assert wc.sap_eo_tiles([lat], [n], prec) == [tile]
        z, rho = (to_np(t) for t in lat.sap_block_mr(x, 1, 4, prec=prec, eo=True))
        for r, (zw, rw) in want.items():
            assert rel(z[r], zw) < TOL[prec] and rel(rho[r], rw) < TOL[prec], (cache, r)
