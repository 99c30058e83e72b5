"""Full 4PCF beyond l = 4 or 8 bins: the run-time matrix-core contraction against the FP64 oracle.

Bin counts at the edges of its pair tiles (4 bins a side: 1, 4 | 5, 8 | 9, 10), the smallest and
largest l, both parities, Lambda lists that mix it with the compile-time kernels (8 bins, l > 4),
cell runs that end inside a staged tile, and two fields in one launch."""
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


@pytest.mark.parametrize("nb,lmax,parity,shape,tile", [
    (1, 5, "even", (12, 16, 24), 1024), (4, 6, "odd", (16, 16, 24), 512), (5, 5, "even", (16, 24, 16), 1024),
    (8, 5, "odd", (16, 16, 24), 1024), (8, 6, "even", (24, 16, 16), 2048), (9, 0, "even", (16, 16, 16), 4096),
    (9, 4, "odd", (24, 16, 16), 1024), (10, 3, "even", (16, 16, 48), 512), (10, 5, "odd", (24, 24, 16), 1024),
    (2, 10, "even", (16, 16, 16), 1024)])
def test_run_time_contraction(nb, lmax, parity, shape, tile):
    from paper_2210_10206_amd import api
    edges = linear_edges(7.5, nb)
    fields = [lognormal_field(shape, seed=70 + i, sigma=1.0) for i in range(2)]
    plan = api.Plan([shape] * 2, edges, lmax, npcf=4, parity=parity)
    plan.set_contract_tile(tile)
    z = plan.forward([torch.from_numpy(f).cuda() for f in fields]).cpu().numpy()
    plan.close()
    for i, f in enumerate(fields):
        _, ref = oracle.zeta4_full(f.astype(np.float64), edges, lmax, parity=parity)
        check(z[i], ref.imag if parity == "odd" else ref.real, TOL32, print, f"{nb} bins lmax {lmax} {parity} field {i}: ")
