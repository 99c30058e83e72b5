"""Calls on a stream other than the current one: a field, a result or a gradient freed right after the
call keeps its memory until the stream has passed it."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

from fieldgen import linear_edges  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["forward", "normalize", "backward"])
def test_freed_tensors_stay_until_the_stream_is_done(call):
    from paper_2210_10206_amd import api
    shape, nb = (96, 64, 96), 4
    plan = api.Plan([shape], linear_edges(8.0, nb), 2)
    field = torch.from_numpy(np.random.default_rng(1).standard_normal(shape).astype(np.float32)).cuda()
    raw = plan.forward_raw([field])
    weights = torch.ones((1, 3, nb, nb), dtype=torch.float64, device="cuda")
    want = {"forward": lambda: plan.forward_raw([field]), "normalize": lambda: raw,
            "backward": lambda: plan.backward([field], weights)[0]}[call]().clone()
    if call == "normalize":
        want = raw.clone()
        plan.normalize_raw([field], want)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(100_000_000)   # some 50 ms
    if call == "forward":
        got = plan.forward_raw([field], stream=side)
    elif call == "normalize":
        got = raw
        plan.normalize_raw([field], raw, stream=side)
    else:
        got = plan.backward([field], weights, stream=side)[0]
    held = field.data_ptr()
    del field
    other = torch.empty(shape, dtype=torch.float32, device="cuda")   # allocated, never written
    assert not side.query(), "the stream was done before the field was freed"
    assert other.data_ptr() != held
    side.synchronize()
    assert torch.equal(got, want)
    plan.close()
