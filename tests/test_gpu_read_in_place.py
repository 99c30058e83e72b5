"""A single float32 field is read where it lies, through the whole call: at any 4-byte offset, with the
results of the same field in a buffer of its own."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

from fieldgen import lognormal_field, linear_edges  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [1, 2, 3, 5])
@pytest.mark.parametrize("kind,shape", [("full3", (16, 24, 32)), ("full3", (24, 16, 96)), ("full3", (8, 12, 256)),
                                        ("full3", (12, 8, 1024)), ("unfused", (16, 24, 32)), ("proj3", (64, 48)),
                                        ("proj3", (16, 512)), ("full4", (16, 24, 16)), ("full4_10", (16, 24, 16)),
                                        ("full4_valu", (16, 24, 16)), ("proj4", (48, 64)), ("proj4_valu", (48, 64)),
                                        ("split", (24, 16, 64)), ("proj4_split", (48, 64))])
def test_offset_field(kind, shape, offset):
    from paper_2210_10206_amd import api
    kw = dict(npcf=4 if "4" in kind else 3, fused=kind != "unfused", mfma="valu" not in kind,
              precision="split_bf16" if "split" in kind else "fp32")
    edges, lmax = linear_edges(3.9 if min(shape) < 12 else 6.0, 10 if kind.endswith("10") else 4), 3
    d = torch.from_numpy(lognormal_field(shape, seed=3, sigma=1.0)).cuda()
    buf = torch.full((d.numel() + 8,), float("nan"), device="cuda")
    view = buf[offset:offset + d.numel()].view(shape)
    view.copy_(d)
    plan = api.Plan([shape], edges, lmax, **kw)
    want, got = plan.forward_raw([d]), plan.forward_raw([view])
    assert torch.equal(got, want) and bool(torch.isfinite(got).all())   # NaN all around the field
    if kind in ("full3", "unfused", "split") and shape[-1] <= 512:
        gz = torch.from_numpy(np.random.default_rng(2).standard_normal((1, lmax + 1, 4, 4))).cuda()
        assert torch.equal(plan.backward([view], gz)[0], plan.backward([d], gz)[0])
    plan.normalize_raw([d], want)
    plan.normalize_raw([view], got)
    np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())   # (NaN where a bin has no cells)
    plan.close()
