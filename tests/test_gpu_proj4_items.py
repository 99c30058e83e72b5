"""Projected 4PCF on the matrix cores: work items of general, symmetric (a, a, -2a) and real-coefficient
(m, -m, 0) triples at bin counts around their 16-pair tiles, against the FP64 oracle; partly filled
tiles and cell runs, and two fields in one launch."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import oracle  # noqa: E402
from fieldgen import lognormal_field, linear_edges  # noqa: E402
from parity import TOL32, check  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,mmax,shape", [(1, 3, (32, 24)), (2, 0, (16, 48)), (4, 2, (48, 48)), (5, 4, (64, 24)), (6, 6, (48, 64)),
                                           (7, 3, (96, 32)), (8, 4, (64, 64)), (9, 2, (64, 48)), (10, 4, (64, 96))])
def test_items(nb, mmax, shape):
    from paper_2210_10206_amd import api
    edges = linear_edges(10.5, nb)
    fields = [lognormal_field(shape, seed=50 + i, sigma=1.0) for i in range(2)]
    plan = api.Plan([shape] * 2, edges, mmax, npcf=4)
    z = plan.forward([torch.from_numpy(f).cuda() for f in fields]).cpu().numpy()
    plan.close()
    for i, f in enumerate(fields):
        _, ref = oracle.zeta4_proj(f.astype(np.float64), edges, mmax)
        check(z[i], ref, TOL32, print, f"{nb} bins m <= {mmax} field {i}: ")
