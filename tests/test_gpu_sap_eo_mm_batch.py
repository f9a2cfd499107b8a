"""Which block solver a call takes, and the matrix-core one inside whole solves: that the
launches of test_gpu_sap_eo_mm are indeed its, one launch over the blocks of two lattices beside
a third of another block volume, and tiles in which some right-hand sides have nothing to do,
finish early or finish late.  Whole solves are compared with the vector kernel's (same recursion,
16-bit rounding apart: iteration counts within one, solutions within what the residuals allow)
and with the oracle's D."""
import numpy as np
import pytest

import synth
from oracle import dirac
from tests.helpers import clover, gauge, lattice, rel, to_dev, to_np
from tests.test_gpu_sap_eo_mm import CASES

pytestmark = pytest.mark.gpu

M0, CSW = -0.1, 1.0
MM = 4  # rhs per work-group of the matrix-core kernel


def _true_res(dims, b, x):
    U, A = gauge(dims), clover(dims, M0, CSW)
    return dirac.norm(b - dirac.apply_D(U, A, x)) / dirac.norm(b)


@pytest.mark.parametrize("dims,block,nrhs", CASES)
def test_the_block_solver_cases_run_on_the_matrix_cores(dims, block, nrhs):
    import paper_1109_4279_amd as wc
    lat = lattice(dims, block, M0, CSW)
    for prec in ("f16", "bf16"):
        assert wc.sap_eo_tiles([lat], [nrhs], prec) == [MM]
        assert wc.sap_eo_tiles([lat], [1], prec) == [1]
        for tile in (1, 2):
            lat.set_tiles(prec, nr_sap_eo=tile)
            assert wc.sap_eo_tiles([lat], [nrhs], prec) == [tile]
        lat.set_tiles(prec)
    for prec in ("f64", "f32"):
        assert wc.sap_eo_tiles([lat], [nrhs], prec) == [1]
    for bad in ((0, "bf16"), (-1, "f32")):
        with pytest.raises(wc.WCError):
            wc.sap_eo_tiles([lat], [bad[0]], bad[1])


@pytest.mark.timeout(300)
@pytest.mark.parametrize("prec", ["f16", "bf16"])
def test_batch_over_lattices_and_block_volumes(prec):
    import paper_1109_4279_amd as wc
    shapes = [((8, 8, 16, 16), (4, 4, 4, 4), 12), ((8, 16, 16, 16), (4, 4, 4, 4), 7), ((8, 8, 8, 8), (2, 2, 2, 2), 5)]
    lats = [lattice(d, blk, M0, CSW) for d, blk, _ in shapes]
    ns = [n for _, _, n in shapes]
    bs = [synth.gaussian_spinor(d, nrhs=n, seed=101 + i) for i, (d, _, n) in enumerate(shapes)]
    dev = [to_dev(b) for b in bs]
    assert wc.sap_eo_tiles(lats, ns, prec) == [MM, MM, 1]
    xs, st = wc.solve_batch(lats, dev, sap_prec=prec, eo=1, tol=1e-10)
    lats[0].set_tiles(prec, nr_sap_eo=1)
    assert wc.sap_eo_tiles(lats, ns, prec) == [1, 1, 1]
    vs, sv = wc.solve_batch(lats, dev, sap_prec=prec, eo=1, tol=1e-10)
    assert max(abs(a["iters"] - b["iters"]) for a, b in zip(st, sv)) <= 1
    for (d, _, n), b, x, v in zip(shapes, bs, xs, vs):
        x, v = to_np(x), to_np(v)
        assert all(rel(x[r], v[r]) < 1e-8 for r in range(n))
        for r in (0, n - 1):
            assert _true_res(d, b[r], x[r]) <= 1e-10


@pytest.mark.timeout(300)
@pytest.mark.parametrize("prec", ["f16", "bf16"])
def test_tiles_with_finished_right_hand_sides(prec):
    """Of every four rhs one is solved from nothing, one has a zero source, one starts from its
    solution and one from an approximate solution."""
    import paper_1109_4279_amd as wc
    dims, block, n = (8, 8, 16, 16), (4, 4, 4, 4), 24
    lat = lattice(dims, block, M0, CSW)
    b = synth.gaussian_spinor(dims, nrhs=n, seed=111)
    b[1::4] = 0
    src = to_dev(b)
    assert wc.sap_eo_tiles([lat], [n], prec) == [MM]
    done, _ = lat.solve(src, sap_prec="f32", eo=1, tol=1e-12)
    rough, _ = lat.solve(src, sap_prec="f32", eo=1, tol=1e-5)
    x0 = done.clone()
    x0[0::4] = 0
    x0[3::4] = rough[3::4]
    x, st = lat.solve(src, x0=x0, sap_prec=prec, eo=1, tol=1e-10)
    lat.set_tiles(prec, nr_sap_eo=1)
    v, sv = lat.solve(src, x0=x0, sap_prec=prec, eo=1, tol=1e-10)
    x, v, done = to_np(x), to_np(v), to_np(done)
    it = np.array([s["iters"] for s in st])
    assert not it[1::4].any() and not it[2::4].any()
    assert it[3::4].min() > 0 and it[0::4].min() > it[3::4].max()
    assert np.abs(it - np.array([s["iters"] for s in sv])).max() <= 1
    assert not x[1::4].any() and np.array_equal(x[2::4], done[2::4])
    for r in range(n):
        if r % 4 != 1:
            assert rel(x[r], v[r]) < 1e-8, r
    for r in (0, 3, n - 4, n - 1):
        assert _true_res(dims, b[r], x[r]) <= 1e-10, r
