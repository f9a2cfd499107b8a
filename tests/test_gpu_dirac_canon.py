"""FP64 D_w on the caller's arrays (wc_apply_D / wc_apply_D_noalloc): the chunks of 256
tile-major sites that the kernel stages, at the shapes where they can go wrong - a lattice
smaller than one chunk, a ragged last chunk, several tiles in a chunk, tiles that straddle
chunks, odd block volumes and one tile per chunk - with every option, against the oracle.
Tolerance: at most 72 complex products are summed per component, 1e-13 x a few."""
import numpy as np
import pytest

import synth
from oracle import dirac
from tests.helpers import clover, gauge, lattice, maxrel, to_dev, to_np

pytestmark = pytest.mark.gpu

SHAPES = [
    ((4, 4, 4, 4), (2, 2, 2, 2)),    # one chunk, 16 tiles
    ((2, 2, 2, 2), (1, 1, 1, 1)),    # 16 sites, one-site tiles
    ((8, 6, 6, 6), (4, 3, 3, 3)),    # 108-site tiles straddling chunks, ragged last chunk
    ((6, 6, 6, 10), (3, 3, 3, 5)),   # 135-site tiles
    ((16, 4, 8, 8), (8, 2, 4, 4)),   # one 256-site tile per chunk, unequal extents
]


@pytest.mark.parametrize("dims,block", SHAPES)
@pytest.mark.parametrize("nrhs", [1, 2, 13])
def test_apply_canonical_matches_oracle(dims, block, nrhs):
    m0, csw = -0.1, 1.0
    x = synth.gaussian_spinor(dims, nrhs=nrhs, seed=91)
    U, A = gauge(dims), clover(dims, m0, csw)
    for bc_t in (1, -1):
        lat = lattice(dims, block, m0, csw, bc_t)
        for region, blk in (("full", None), ("blocks", block)):
            want = np.stack([dirac.apply_D(U, A, x[r], bc_t, blk) for r in range(nrhs)])
            wantd = np.stack([dirac.apply_Ddag(U, A, x[r], bc_t, blk) for r in range(nrhs)])
            assert maxrel(to_np(lat.apply_D(to_dev(x), region=region)), want) < 1e-13, (bc_t, region)
            assert maxrel(to_np(lat.apply_D(to_dev(x), region=region, dagger=True)), wantd) < 1e-13, (bc_t, region)
