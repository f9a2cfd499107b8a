"""The rule that gives the even/odd block solver on 16-bit storage to the vector or to the
matrix-core kernel, on both sides of its lines: block volumes that let two, three and four
work-groups of the vector kernel share a CU, tiles that two, three and five right-hand sides
leave partly empty, a last round that is partly empty, and a batch in which one lattice has a
single right-hand side per block.  The expected kernel is the faster one of the half-sweeps
timed on an MI355X, where the two differ by 5 % or more."""
import pytest

pytestmark = pytest.mark.gpu

VEC, MM = 1, 4
CASES = [  # block, blocks along each axis, {rhs: kernel}
    ((4, 4, 4, 4), (4, 4, 4, 8), {3: MM, 4: MM, 8: MM}),
    ((4, 4, 4, 4), (6, 6, 6, 6), {2: VEC, 4: MM, 5: VEC}),
    ((2, 4, 4, 4), (4, 4, 4, 8), {2: VEC, 4: MM, 5: MM}),
    ((2, 4, 4, 4), (6, 6, 6, 6), {2: VEC, 3: MM, 5: MM}),
    ((2, 4, 4, 4), (8, 8, 6, 6), {2: MM, 3: MM}),
    ((4, 3, 3, 3), (6, 6, 6, 6), {2: VEC, 3: VEC, 4: MM, 5: VEC, 8: MM}),
    ((4, 3, 3, 3), (8, 8, 6, 6), {2: VEC, 3: MM, 5: MM}),
    ((3, 3, 3, 3), (8, 8, 6, 6), {2: VEC, 3: MM, 5: MM}),
    ((4, 4, 2, 2), (6, 6, 6, 6), {2: MM}),
    ((4, 4, 2, 2), (8, 8, 6, 6), {2: MM, 5: MM}),
    ((2, 2, 2, 2), (4, 4, 4, 8), {2: VEC, 5: MM}),
    ((2, 2, 2, 2), (8, 8, 8, 8), {2: MM}),
]


def _unit(block, nb):
    import torch

    import paper_1109_4279_amd as wc
    dims = tuple(b * n for b, n in zip(block, nb))
    U = torch.eye(3, dtype=torch.complex128, device="cuda:0").expand((4,) + dims + (3, 3)).contiguous()
    return wc.Lattice(U, block=block, m0=-0.1, csw=1.0)


@pytest.mark.parametrize("block,nb,want", CASES)
def test_pick_follows_the_measured_times(block, nb, want):
    import paper_1109_4279_amd as wc
    lat = _unit(block, nb)
    got = {n: wc.sap_eo_tiles([lat], [n], "bf16")[0] for n in want}
    assert got == want


def test_single_rhs_lattices_in_a_batch():
    """1152 blocks of 64 sites with one rhs each (73 us on the vector kernel, 112 on the matrix
    cores) beside 32 blocks with two."""
    import paper_1109_4279_amd as wc
    big, small = _unit((4, 4, 2, 2), (8, 8, 6, 6)), _unit((4, 4, 2, 2), (4, 4, 2, 2))
    assert wc.sap_eo_tiles([big, small], [1, 2], "bf16") == [VEC, VEC]
    assert wc.sap_eo_tiles([big, small], [4, 4], "bf16") == [MM, MM]
