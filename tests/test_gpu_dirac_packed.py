"""FP64 D_w on packed fields, the operator of the outer solvers and of their true residuals: every
rhs tile, staged in LDS or not, full and Dirichlet-block operator, D and D^dag, on blocks that fill
a tile's 256 sites and blocks that do not, against the oracle.  A tile or the staging option
selects it in wc_apply_D.  Tolerance: at most 72 complex products are summed per component."""
import ctypes
import gc

import numpy as np
import pytest

import synth
from oracle import dirac
from tests.helpers import clover, gauge, lattice, maxrel, to_dev, to_np

pytestmark = pytest.mark.gpu

M0, CSW = -0.1, 1.0
NRHS = 5  # ragged for every tile above one


@pytest.mark.parametrize("dims,block", [((8, 8, 8, 8), (4, 4, 4, 4)), ((16, 4, 8, 8), (8, 2, 4, 4)),
                                        ((8, 6, 6, 6), (4, 3, 3, 3)), ((4, 4, 4, 4), (2, 2, 2, 2))])
@pytest.mark.parametrize("bc_t", [1, -1])
def test_packed_operator_in_every_tile(dims, block, bc_t):
    x = synth.gaussian_spinor(dims, nrhs=NRHS, seed=141)
    U, A = gauge(dims), clover(dims, M0, CSW)
    want = {}
    for region, blk in (("full", None), ("blocks", block)):
        want[region, False] = np.stack([dirac.apply_D(U, A, x[r], bc_t, blk) for r in range(NRHS)])
        want[region, True] = np.stack([dirac.apply_Ddag(U, A, x[r], bc_t, blk) for r in range(NRHS)])
    lat = lattice(dims, block, M0, CSW, bc_t)
    xd = to_dev(x)
    for nr in (0, 1, 2, 3, 4):
        lat.set_tiles("f64", nr_dirac=nr)
        for stage in (-1, 0, 1):
            lat.set_option("dirac_stage", stage)
            for (region, dagger), w in want.items():
                got = to_np(lat.apply_D(xd, region=region, dagger=dagger))
                assert maxrel(got, w) < 1e-13, (nr, stage, region, dagger)


def _growth(f):
    """Device memory that f takes besides torch's."""
    import torch

    import paper_1109_4279_amd as wc

    def used():
        gc.collect()
        wc.empty_pool()
        torch.cuda.synchronize()
        free, total = torch.cuda.mem_get_info()
        return total - free - torch.cuda.memory_reserved()

    before = used()
    f()
    return used() - before


def test_tile_and_stage_select_the_packed_kernel():
    """The packed fields that it needs (and the kernel on the caller's arrays does not) appear; the
    allocation-free call agrees bit for bit either way; the autotuner's tile selects nothing."""
    import torch

    from paper_1109_4279_amd import _lib
    lib = _lib.load()
    dims, block, n = (16, 16, 16, 16), (4, 4, 4, 4), 3
    fields = 2 * n * 192 * 16 ** 4
    x = to_dev(synth.gaussian_spinor(dims, nrhs=n, seed=142))
    out = torch.empty_like(x)

    def noalloc(lat):
        y = torch.empty_like(x)
        s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        _lib.check(lib.wc_apply_D_noalloc(lat._ctx, ctypes.c_void_p(y.data_ptr()), ctypes.c_void_p(x.data_ptr()), 1,
                                          0, 0, 0, s))
        return y[0]

    for setting, packed in ((None, False), (("tile", 2), True), (("stage", 0), True), (("stage", 1), True)):
        lat = lattice(dims, block)
        if setting and setting[0] == "tile":
            lat.set_tiles("f64", nr_dirac=setting[1])
        elif setting:
            lat.set_option("dirac_stage", setting[1])
        lat.apply_D(x[:1], out=out[:1])
        got = _growth(lambda: lat.apply_D(x, out=out))
        assert abs(got - (fields if packed else 0)) < 4 << 20, setting
        assert torch.equal(noalloc(lat), lat.apply_D(x[0].contiguous()))
        if packed:  # back to the library's choice
            lat.set_tiles("f64")
            lat.set_option("dirac_stage", -1)
            assert abs(_growth(lambda: lat.apply_D(x[:2].contiguous()))) < 4 << 20
    lat = lattice(dims, block)
    lat.set_tiles("f64", nr_dirac=3)
    lat.autotune(4, prec="f64")
    assert abs(_growth(lambda: lat.apply_D(x, out=out))) < 4 << 20


def test_bench_times_the_kernel_that_apply_D_runs():
    """12 rhs on 2^4 blocks of 16^4: 131 us on the caller's arrays, 195 to 311 on packed fields."""
    import torch
    dims, n = (16, 16, 16, 16), 12
    lat = lattice(dims, (2, 2, 2, 2))
    x = torch.zeros((n,) + dims + (4, 3), dtype=torch.complex128, device="cuda:0")
    out = lat.apply_D(x)
    best = 1e9
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(50):
            lat.apply_D(x, out=out)
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) / 50)
    ms = min(lat.bench_dirac("f64", nrhs=n, iters=50) for _ in range(5))
    assert abs(ms / best - 1) < 0.2
    lat.set_tiles("f64", nr_dirac=4)
    assert min(lat.bench_dirac("f64", nrhs=n, iters=50) for _ in range(5)) > 1.5 * ms
