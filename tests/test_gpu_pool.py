"""Device memory that passes from one context or call to the next: contexts destroyed while
their work is still enqueued, on streams of their own and from several threads, and contexts
of other sizes after them.  Every result must be what the context computes by itself."""
import threading

import numpy as np
import pytest

import synth
from oracle import dirac
from tests.helpers import clover, gauge, maxrel, to_dev, to_np

pytestmark = pytest.mark.gpu

SHAPES = [((4, 4, 4, 4), (2, 2, 2, 2)), ((8, 6, 6, 6), (4, 3, 3, 3)), ((8, 8, 8, 8), (4, 4, 4, 4))]


def _reference(dims):
    U, A = gauge(dims), clover(dims, -0.1, 1.0)
    x = synth.gaussian_spinor(dims, seed=95)
    return to_dev(U), to_dev(x), dirac.apply_D(U, A, x)


def _rounds(refs, rounds, errs):
    import torch

    import paper_1109_4279_amd as wc
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        for i in range(rounds):
            (dims, block), (U, x, want) = SHAPES[i % 3], refs[i % 3]
            lat = wc.Lattice(U, block=block, m0=-0.1, csw=1.0)
            y = lat.apply_D(x)
            z = lat.apply_D(x, prec="f32")
            g = lat.link_grad(x, x)
            del lat  # its buffers pass on with y, z and g still enqueued
            errs.append(maxrel(to_np(y), want))
            errs.append(maxrel(to_np(z), want) * 1e-8)
            errs.append(0.0 if np.isfinite(to_np(g)).all() else 1.0)


def test_contexts_in_turn_and_from_threads():
    refs = [_reference(d) for d, _ in SHAPES]
    errs = []
    _rounds(refs, 9, errs)
    threads = [threading.Thread(target=_rounds, args=(refs, 9, errs)) for _ in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(errs) == 4 * 27
    assert max(errs) < 1e-13
