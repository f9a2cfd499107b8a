"""The clover rows of the matrix-core block solver (288 bytes a site) take memory only in contexts
that run it, also where they are first needed by a later call or by a batch; calls before and
after agree with the vector kernel's."""
import gc

import numpy as np
import pytest

import synth
from oracle import solvers
from tests.helpers import clover, gauge, lattice, rel, to_dev, to_np

pytestmark = pytest.mark.gpu

DIMS, V = (32, 16, 16, 16), 131072
ROWS = 288 * V
SLACK = 6 << 20
EO = (576 + 144 + 8) * V  # even/odd clover in FP64, in 16 bits and its scales


def _used():
    """Device memory in use besides torch's."""
    import torch

    import paper_1109_4279_amd as wc
    gc.collect()
    wc.empty_pool()
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free - torch.cuda.memory_reserved()


def _growth(prec, nrhs, eo, tile=0):
    import torch
    lat = lattice(DIMS, (4, 4, 4, 4))
    lat.set_tiles(prec, nr_sap_eo=tile)
    x = torch.zeros((nrhs,) + DIMS + (4, 3), dtype=torch.complex128, device="cuda:0")
    before = _used()
    lat.sap(x, ncy=1, nmr=1, prec=prec, eo=eo)
    return _used() - before


@pytest.mark.parametrize("prec", ["f16", "bf16"])
def test_rows_only_where_the_kernel_runs(prec):
    for nrhs, eo, tile in ((1, True, 0), (1, False, 0), (4, True, 0), (4, True, 1)):
        _growth(prec, nrhs, eo, tile)  # what the runtime itself takes for a kernel's first launch
    assert abs(_growth(prec, 1, True) - _growth(prec, 1, False) - EO) < SLACK  # one rhs: no rows
    with_tile = _growth(prec, 4, True, tile=1)
    assert abs(_growth(prec, 4, True) - with_tile - ROWS) < SLACK  # the matrix-core kernel's


@pytest.mark.parametrize("prec", ["f16", "bf16"])
def test_rows_made_for_a_later_call(prec):
    """One context: single-rhs solve, several rhs, new clover, new block shape, a batch."""
    import paper_1109_4279_amd as wc
    tol = {"f16": 3e-3, "bf16": 2e-2}[prec]
    dims, block = (8, 8, 16, 16), (4, 4, 4, 4)
    lat = lattice(dims, block, -0.1, 1.0)
    U = gauge(dims)
    eta = synth.gaussian_spinor(dims, nrhs=24, seed=121)
    x = to_dev(eta)

    def check(blk, m0):
        assert wc.sap_eo_tiles([lat], [24], prec) == [4]
        z = to_np(lat.sap_block_mr(x, 0, 4, prec=prec, eo=True)[0])
        for r in (0, 23):
            zw, _ = solvers.mr_blocks_eo(U, clover(dims, m0, 1.0), eta[r], blk, 0, 4)
            assert rel(z[r], zw) < tol, (blk, m0, r)

    lat.solve(x[0].contiguous(), sap_prec=prec, eo=1)
    check(block, -0.1)
    from paper_1109_4279_amd import _lib
    _lib.check(_lib.load().wc_create_clover(lat._ctx, 0.2, 1.0, None))
    check(block, 0.2)
    lat.set_block((2, 4, 4, 4))
    check((2, 4, 4, 4), 0.2)
    # a batch that needs the rows of a lattice which has run single right-hand sides only
    one = lattice(dims, block, -0.1, 1.0)
    two = lattice(dims, block, -0.1, 1.0)
    for la in (one, two):
        la.solve(x[0].contiguous(), sap_prec=prec, eo=1)
    assert wc.sap_eo_tiles([one, two], [12, 12], prec) == [4, 4]
    b = [x[:12].contiguous(), x[12:].contiguous()]
    xs, st = wc.solve_batch([one, two], b, sap_prec=prec, eo=1)
    one.set_tiles(prec, nr_sap_eo=1)
    vs, sv = wc.solve_batch([one, two], b, sap_prec=prec, eo=1)
    assert max(abs(p["iters"] - q["iters"]) for p, q in zip(st, sv)) <= 1
    for p, q in zip(xs, vs):
        p, q = to_np(p), to_np(q)
        assert np.all([rel(p[r], q[r]) < 1e-8 for r in range(12)])
