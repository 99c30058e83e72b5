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
