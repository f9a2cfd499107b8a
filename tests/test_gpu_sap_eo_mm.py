"""The even/odd block solver on the matrix cores (16-bit storage, several right-hand sides):
launches of the size that selects it, at block shapes where its mapping can go wrong - full
wavefronts, a last wavefront of 6 or 1 site pairs, an odd block volume, and more border
entries than one round takes - and rhs counts that leave tiles ragged.  Checked against the
oracle (tolerances of the storage, as for the other block solvers) and against the vector
kernel, which runs the same recursion in FP32: a stored component may round to the
neighbouring 16-bit value of its site's scale, 2^-8 (BF16) or 2^-11 (FP16) of it, in a few
places; over the field the two stay within half of that."""
import numpy as np
import pytest

import synth
from oracle import solvers
from tests.helpers import clover, gauge, lattice, rel, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL = {"f16": 3e-3, "bf16": 2e-2}
SAP_TOL = {"f16": 5e-3, "bf16": 3e-2}
SAME = {"f16": 2.0 ** -12, "bf16": 2.0 ** -9}
CASES = [
    ((8, 8, 16, 16), (4, 4, 4, 4), 24),   # 8 wavefronts, 6 tiles of 4
    ((16, 4, 16, 16), (8, 2, 4, 4), 23),  # 576 border entries: two passes; a ragged tile
    ((8, 6, 12, 12), (4, 3, 3, 3), 33),   # 54 pairs, last wavefront of 6; tiles of 4 and less
    ((6, 6, 12, 12), (3, 3, 3, 3), 33),   # 81 sites: 41 pairs, one without its odd or even site
    ((8, 8, 8, 8), (2, 2, 2, 2), 9),      # 8 pairs in a wavefront, 3 tiles of 3
]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("dims,block,nrhs", CASES)
@pytest.mark.parametrize("prec", ["f16", "bf16"])
def test_matrix_core_block_solver(dims, block, nrhs, prec):
    m0, csw, bc_t = -0.1, 1.0, -1
    lat = lattice(dims, block, m0, csw, bc_t)
    U, A = gauge(dims), clover(dims, m0, csw)
    eta = synth.gaussian_spinor(dims, nrhs=nrhs, seed=81)
    check = (0, nrhs - 1)
    x = to_dev(eta)

    def run(tile):
        lat.set_tiles(prec, nr_sap_eo=tile)
        out = [to_np(t) for c in (0, 1) for t in lat.sap_block_mr(x, c, 4, prec=prec, eo=True)]
        return out + [to_np(lat.sap(x, ncy=2, nmr=3, prec=prec, eo=True))]

    got, vec = run(0), run(1)
    for colour in (0, 1):
        for r in check:
            zw, rw = solvers.mr_blocks_eo(U, A, eta[r], block, colour, 4, bc_t)
            assert rel(got[2 * colour][r], zw) < TOL[prec], (colour, r)
            assert rel(got[2 * colour + 1][r], rw) < TOL[prec], (colour, r)
    for r in check:
        want = solvers.sap(U, A, eta[r], block, nmr=3, ncy=2, eo=True, bc_t=bc_t)
        assert rel(got[4][r], want) < SAP_TOL[prec], r
    for a, b in zip(got, vec):
        assert rel(a, b) < SAME[prec]
        assert all(rel(a[r], b[r]) < 2 * SAME[prec] for r in range(nrhs))
