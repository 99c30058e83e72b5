"""Adjoint of plans whose kernel groups go in chunks, on the lengths of the row-pair kernel: several
launches of it, later ones adding to the direct term of the first, packed pairs and other groups in one
launch or apart.  The chunks change no operation, so gradients equal the whole plan's bit for bit; the
whole plan's is compared with the float64 gradient at some cells."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import oracle  # noqa: E402
from fieldgen import lognormal_field, linear_edges  # noqa: E402
from parity import TOL32  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 96, 128, 160, 192, 256])
@pytest.mark.parametrize("nbins", [3, 9])
def test_chunked_gradient(n, nbins):
    from paper_2210_10206_amd import api
    shape, lmax = (8, 12, n), 3   # two packed pairs, six other groups
    edges = linear_edges(3.9, nbins)
    d = lognormal_field(shape, seed=60, sigma=1.0)
    gz = np.random.default_rng(61).standard_normal((1, lmax + 1, nbins, nbins))
    dev, gdev = [torch.from_numpy(d).cuda()], torch.from_numpy(gz).cuda()
    group = nbins * d.size * 8
    got = {}
    for groups in (0, 1, 3, 5):
        plan = api.Plan([shape], edges, lmax, **({"scratch_limit": groups * group} if groups else {}))
        got[groups] = (plan.forward_raw(dev).cpu(), plan.backward(dev, gdev)[0].cpu())
        plan.close()
    for groups in (1, 3, 5):
        assert torch.equal(got[groups][0], got[0][0]) and torch.equal(got[groups][1], got[0][1]), f"{groups} groups"
    cells = np.sort(np.random.default_rng(62).choice(d.size, 24, replace=False))
    ref = oracle.grad3_full(d.astype(np.float64), edges, lmax, gz[0], cells=cells)
    err = np.max(np.abs(got[0][1].numpy().reshape(-1)[cells] - ref)) / np.max(np.abs(ref))
    print(f"{shape} {nbins} bins: gradient err {err:.3e}", flush=True)
    assert err < TOL32
