"""Fused last pass of the three-stage lengths: bin counts below, at and above its padded tiles (rows of
the missing bins have no LDS region), the packed, real and complex sums, both precisions, and more
than 12 bins on a 1024-point last axis, against the FP64 oracle."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import oracle  # noqa: E402
from fieldgen import lognormal_field, linear_edges  # noqa: E402
from parity import TOL32, TOL_SPLIT, check  # noqa: E402

pytestmark = pytest.mark.gpu


def _run(shape, edges, lmax, precision):
    from paper_2210_10206_amd import api
    d = lognormal_field(shape, seed=90, sigma=1.0)
    plan = api.Plan([shape], edges, lmax, precision=precision)
    z = plan.forward([torch.from_numpy(d).cuda()]).cpu().numpy()[0]
    plan.close()
    return d.astype(np.float64), z


@pytest.mark.parametrize("n", [96, 160, 192, 512, 1024])
@pytest.mark.parametrize("nb", [1, 5, 9, 13, 16])
def test_3d(n, nb):
    edges = linear_edges(3.9, nb)
    d, z = _run((8, 8, n), edges, 2, "fp32")
    check(z, oracle.zeta3_full(d, edges, 2).real, TOL32, print, f"8x8x{n} {nb} bins: ")


@pytest.mark.parametrize("n,nb", [(96, 10), (160, 3), (192, 14), (512, 6), (512, 11), (1024, 8), (1024, 13), (1024, 16)])
@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
def test_2d(n, nb, precision):
    if precision == "split_bf16" and n == 1024 and nb > 12:
        pytest.skip("no split form: sb_plan_create refuses it")
    edges = linear_edges(7.5, nb)
    d, z = _run((16, n), edges, 3, precision)
    check(z, oracle.zeta3_proj(d, edges, 3), TOL32 if precision == "fp32" else TOL_SPLIT, print, f"16x{n} {nb} bins {precision}: ")


@pytest.mark.parametrize("nb", [3, 10])
@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
def test_2d_parts_by_wave(nb, precision):
    """Real and imaginary sums on different waves: the smallest workgroup (4 waves) and 12 padded bins."""
    edges = linear_edges(3.9, nb)
    d, z = _run((8, 1024), edges, 3, precision)
    check(z, oracle.zeta3_proj(d, edges, 3), TOL32 if precision == "fp32" else TOL_SPLIT, print, f"8x1024 {nb} bins {precision}: ")


@pytest.mark.parametrize("n,orders,adds", [(512, 17, 32), (1024, 17, 32)])
def test_every_row_reaches_float64(n, orders, adds):
    """A constant map: every cell adds the same product to its float32 sum, so the roundings of a run of
    additions are of one sign and nothing averages out: k equal terms after one another err by at most
    (k + 1) / 2 ulps of 2^-24 of their sum.  A wave adds at most `adds` cells of a row to each of its sums
    before they go to float64 (9.8e-7 for 32; eight rows together, 7.7e-6).  Everything before the sums
    is exact: powers of two, whole numbers of cells and one rounding of density times cells."""
    from paper_2210_10206_amd import api
    shape, nb = (1024, n), 3
    edges = linear_edges(6.0, nb)
    plan = api.Plan([shape], edges, orders - 1)   # as many orders as give eight rows a workgroup
    cells = plan.bin_counts(0)
    errs = []
    for c in np.random.default_rng(11).uniform(0.5, 2.0, 16).astype(np.float32):
        z = plan.forward([torch.full(shape, float(c), dtype=torch.float32, device="cuda")]).cpu().numpy()[0]
        for b in range(nb):
            v = np.float32(c * np.float32(cells[b]))
            exact = float(np.float32(c * v)) * float(v) * shape[0] * shape[1]
            errs.append(abs(z[0, b, b].real / exact - 1))
    plan.close()
    bound = (adds + 1) / 2 * 2.0 ** -24
    print(f"{shape} constant maps: worst {max(errs):.3e} (bound {bound:.2e})", flush=True)
    assert max(errs) < bound


@pytest.mark.parametrize("n", [64, 96, 128, 160, 192, 256, 512, 1024])
@pytest.mark.parametrize("nb", [3, 7])
def test_blocks_of_eleven_rows(n, nb):
    """41 array groups of 576 rows: some eleven rows a workgroup, fewer in the last one, which ends off every
    eighth row (the two-stage lengths add to float64 there)."""
    edges = linear_edges(2.9, nb)
    d, z = _run((12, 48, n), edges, 8, "fp32")
    check(z, oracle.zeta3_full(d, edges, 8).real, TOL32, print, f"12x48x{n} {nb} bins: ")
