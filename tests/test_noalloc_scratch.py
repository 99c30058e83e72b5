"""Plans near the scratch of sb_forward_noalloc: the shorter contraction tiles of small grids write
more partials, and must not take a plan over the limit that it meets without them."""
import ctypes

import numpy as np
import pytest

LIMIT = 64 << 20


def _scratch(shape, nbins, lmax, batch=1):
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    e = np.linspace(0.0, 10.0, nbins + 1)
    prob = _lib.SbProblem(len(shape), 4, nbins, e.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), lmax, 0, 0, 0)
    sh = np.array(shape * batch, dtype=np.int64)
    h, pb, sb = ctypes.c_void_p(), ctypes.c_size_t(), ctypes.c_size_t()
    rc = lib.sb_plan_create(ctypes.byref(prob), batch, sh.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)),
                            ctypes.byref(h))
    assert rc == 0, lib.sb_last_error()
    assert lib.sb_plan_workspace(h, ctypes.byref(pb), ctypes.byref(sb)) == 0
    lib.sb_plan_destroy(h)
    return sb.value


def _sorted_even_lambdas(lmax):
    return sum((a + b + c) % 2 == 0 and c <= a + b for a in range(lmax + 1) for b in range(a, lmax + 1)
               for c in range(b, lmax + 1))


@pytest.mark.parametrize("nbins,lmax,blocks", [
    (8, 4, 256),     # fits with the short tiles: 128 cells a workgroup
    (10, 4, 64),     # fits with 512 cells only
    (10, 5, 64),
])
def test_small_grid_partials_stay_within_the_fixed_scratch(nbins, lmax, blocks):
    n = 32 ** 3
    nlam = _sorted_even_lambdas(lmax)
    nlm = (lmax + 1) * (lmax + 2) // 2
    got = _scratch((32, 32, 32), nbins, lmax)
    assert got <= LIMIT
    # density, spectrum and one gradient array (4 + 8 + 8 bytes a cell), the coefficient arrays and
    # the partials; totals, the result copy and alignment are less than another such set of partials
    part = nlam * nbins ** 3 * 8
    base = n * (4 + 8 + 8) + nlm * nbins * n * 8
    assert base + blocks * part <= got < base + 2 * blocks * part


def test_large_grids_keep_the_short_tile_rule_out():
    """64^3, 8 bins to l = 4 is past the fixed scratch either way: the partials are those of 512
    cells halved to 1024 workgroups (256 cells)."""
    n, nbins, nlm, nlam = 64 ** 3, 8, 15, _sorted_even_lambdas(4)
    part = nlam * nbins ** 3 * 8
    base = n * (4 + 8 + 8) + nlm * nbins * n * 8
    got = _scratch((64, 64, 64), nbins, 4)
    assert base + 1024 * part <= got < base + 2048 * part
