"""Contexts destroyed while their work is still enqueued, and while another thread captures a
stream."""
import threading

import numpy as np
import pytest

import synth
from oracle import dirac, force
from tests.helpers import clover, gauge, maxrel, to_dev, to_np

pytestmark = pytest.mark.gpu

M0, CSW = -0.1, 1.0


def _lattice(U, block):
    import paper_1109_4279_amd as wc
    return wc.Lattice(U, block=block, m0=M0, csw=CSW)


@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 1e-5)])
def test_work_enqueued_at_destruction(prec, tol):
    """Several hundred applications of D still run on one stream when their context goes; the next
    context, on another stream, is built from other links in the same memory at once."""
    import torch
    dims, block = (16, 12, 12, 12), (4, 3, 3, 3)
    other = (16, 12, 12, 12)
    U, x = to_dev(gauge(dims)), synth.gaussian_spinor(dims, nrhs=2, seed=96)
    want = np.stack([dirac.apply_D(gauge(dims), clover(dims, M0, CSW), x[r]) for r in range(2)])
    x = to_dev(x)
    U2 = torch.eye(3, dtype=torch.complex128, device="cuda:0").expand((4,) + other + (3, 3)).contiguous()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(3):
        with torch.cuda.stream(s1):
            lat = _lattice(U, block)
            out = [lat.new_spinor(2) for _ in range(40)]
            lat.apply_D(x, prec=prec, out=out[0])
            s1.synchronize()
            for k in range(400):
                lat.apply_D(x, prec=prec, out=out[k % 40])
            done = torch.cuda.Event()
            done.record()
            assert not done.query()
            del lat
            assert done.query()  # whoever takes the memory next may write it
        with torch.cuda.stream(s2):
            lat2 = _lattice(U2, block)
            y2 = lat2.apply_D(x)
        torch.cuda.synchronize()
        for y in out:
            assert maxrel(to_np(y), want) < tol
        assert torch.isfinite(torch.view_as_real(y2)).all()
        del lat2


def test_link_gradients_through_reused_scratch():
    """link_grad of two lattices in turn: the scratch of one call is the next one's, and every
    result is the oracle's."""
    cases = []
    for dims, block, seed in (((4, 4, 4, 4), (2, 2, 2, 2), 97), ((4, 4, 6, 6), (2, 2, 3, 3), 98)):
        U = gauge(dims)
        Y, X = synth.gaussian_spinor(dims, seed=seed), synth.gaussian_spinor(dims, seed=seed + 10)
        K = force.link_grad(U, X, Y, CSW)
        cases.append((_lattice(to_dev(U), block), to_dev(Y), to_dev(X), np.conj(np.swapaxes(K, -1, -2))))
    for _ in range(3):
        for lat, Y, X, want in cases:
            assert maxrel(to_np(lat.link_grad(Y, X)), want) < 1e-12


@pytest.mark.parametrize("mode", ["thread_local", "relaxed"])
def test_destroyed_by_another_thread_during_a_capture(mode):
    """A thread destroys a context while this one captures D of another context: the capture
    goes on, and its replays give D."""
    import torch
    dims, block = (8, 8, 8, 8), (4, 4, 4, 4)
    x = synth.gaussian_spinor(dims, seed=99)
    want = dirac.apply_D(gauge(dims), clover(dims, M0, CSW), x)
    U, x = to_dev(gauge(dims)), to_dev(x)
    lat, gone = _lattice(U, block), [_lattice(U, block)]
    out = lat.apply_D(x)
    gone[0].apply_D(x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode=mode):
        lat.apply_D(x, out=out)
        t = threading.Thread(target=gone.clear)
        t.start()
        t.join()
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert maxrel(to_np(out), want) < 1e-13
