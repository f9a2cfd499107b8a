"""How much device memory the library keeps of destroyed contexts: what it kept comes back on
request, and a context larger than those that follow does not shut them out of the pool."""
import gc

import pytest

pytestmark = pytest.mark.gpu

GIB = 1 << 30
SITE = 3 * 576  # bytes a site of a context without reduced-precision fields: links twice, clover


def _free():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _lattice(dims):
    import torch

    import paper_1109_4279_amd as wc
    U = torch.eye(3, dtype=torch.complex128, device="cuda:0").expand((4,) + dims + (3, 3)).contiguous()
    lat = wc.Lattice(U, m0=-0.1, csw=1.0)
    lat._U = torch.empty(0, device=U.device)  # the library has copied the links
    return lat


def test_kept_memory_comes_back_on_request():
    import paper_1109_4279_amd as wc
    gc.collect()
    _lattice((8, 8, 8, 8))  # the library's code and scratch array are loaded
    wc.empty_pool()
    assert wc.empty_pool() == 0
    before = _free()
    lat = _lattice((32, 16, 16, 16))
    need = SITE * 32 * 16 ** 3
    assert before - _free() > 0.99 * need
    del lat
    assert before - _free() > 0.99 * need  # kept
    assert wc.empty_pool() > 0.99 * need
    assert before - _free() < 8 << 20


def test_small_contexts_after_large_ones():
    import paper_1109_4279_amd as wc
    gc.collect()
    wc.empty_pool()
    lats = [_lattice((32, 24, 24, 24)) for _ in range(3)]  # 764 MB each: more than is kept
    lats.clear()
    kept = wc.empty_pool()
    assert 1.5 * GIB < kept <= 2 * GIB
    lats = [_lattice((32, 24, 24, 24)) for _ in range(3)]
    lats.clear()
    lat = _lattice((32, 16, 16, 16))
    del lat
    before = _free()
    lat = _lattice((32, 16, 16, 16))
    taken = before - _free()
    del lat
    assert taken < 8 << 20  # all of its memory was kept
    assert wc.empty_pool() <= 2 * GIB
