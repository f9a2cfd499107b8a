"""Link derivative and force at the shapes where their kernels' mapping can go wrong: a last group
of fewer than 64 sites, odd and one-site blocks, extents of two (where the two plaquettes of a
plane share links), several right-hand sides, both boundary conditions, with and without the
clover term, against the oracle.  Tolerance: a link's derivative sums some 4 x 12 products of up to
five 3x3 matrices, 1e-13 x a few."""
import numpy as np
import pytest

import synth
from oracle import force
from tests.helpers import gauge, lattice, rel, to_dev, to_np

pytestmark = pytest.mark.gpu

SHAPES = [((2, 2, 2, 2), (1, 1, 1, 1)), ((4, 2, 2, 4), (1, 1, 1, 2)), ((6, 6, 6, 6), (3, 3, 3, 3)),
          ((2, 10, 6, 6), (1, 5, 3, 3)), ((6, 6, 6, 10), (3, 3, 3, 5)), ((8, 2, 4, 4), (4, 1, 2, 2)),
          ((16, 4, 8, 8), (8, 2, 4, 4))]


@pytest.mark.parametrize("dims,block", SHAPES)
@pytest.mark.parametrize("csw,bc_t", [(0.0, -1), (1.3, 1), (1.3, -1)])
def test_link_derivative(dims, block, csw, bc_t):
    n = 3
    U = gauge(dims)
    X, Y = (synth.gaussian_spinor(dims, nrhs=n, seed=s) for s in (151, 152))
    lat = lattice(dims, block, -0.1, csw, bc_t)
    K = [force.link_grad(U, X[r], Y[r], csw, bc_t) for r in range(n)]
    G = to_np(lat.link_grad(to_dev(Y), to_dev(X), coef=-0.7))
    assert rel(G, -0.7 * np.conj(np.swapaxes(sum(K), -1, -2))) < 5e-13
    one = to_np(lat.link_grad(to_dev(Y[1]), to_dev(X[1])))
    assert rel(one, np.conj(np.swapaxes(K[1], -1, -2))) < 5e-13


@pytest.mark.parametrize("dims,block", SHAPES[2:4])
def test_force_is_that_of_its_solutions(dims, block):
    U = gauge(dims)
    lat = lattice(dims, block, -0.1, 1.3, -1)
    F, Y, X, _ = lat.force(to_dev(synth.gaussian_spinor(dims, seed=153)), tol=1e-10, sap_prec="f32", eo=1)
    want = force.lie_force(U, force.link_grad(U, to_np(X), to_np(Y), 1.3, -1))
    assert rel(to_np(F), want) < 5e-13
