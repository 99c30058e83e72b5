"""Mean gain of the transforms: the roundings of a radix's constants are the same in every transform,
so they must not add up over the passes as the roundings of the data average out.

Densities that vary along axis 0 only leave c_0 = (density * shell profile) along that axis; the gain of
the three axis-0 transforms behind it is <c, exact> / <exact, exact> - 1 with a float64 convolution,
taken over many densities: in one of 512 points the data's roundings alone scatter a transform's gain
by 8e-9."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

from fieldgen import linear_edges  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [512, 1024])
def test_long_axis_0(n):
    """The spectrum's pass along axis 0 (radices up to 16) holds float constants, each within 2^-25 =
    3.0e-8 of its value, so its gain is within 3.0e-8 too; the 32-point stages of the kernel's transform
    and of the inverse one hold pairs, which leaves the table twiddles (2e-9 each).  The scatter that the
    densities share, of the kernel's one transform, is 8e-9: two of it give 5e-8."""
    from paper_2210_10206_amd import api
    width, nb = 64, 2
    edges = linear_edges(4.0, nb)
    c = [np.fft.fftfreq(k, 1.0 / k) for k in (n, width)]
    r2 = c[0][:, None] ** 2 + c[1][None] ** 2
    plan = api.Plan([(n, width)], edges, 0, keep_coeffs=True)
    rng, num, den = np.random.default_rng(7), 0.0, 0.0
    for _ in range(32):
        f = rng.standard_normal(n).astype(np.float32)
        plan.forward([torch.from_numpy(np.repeat(f[:, None], width, axis=1).copy()).cuda()])
        for b in range(nb):
            profile = ((r2 > edges[b] ** 2) & (r2 <= edges[b + 1] ** 2)).sum(1).astype(np.float64)
            exact = np.fft.ifft(np.fft.fft(f.astype(np.float64)) * np.fft.fft(profile)).real
            got = plan.coeffs(b)[:, 0].cpu().numpy().real.astype(np.float64)
            num, den = num + got @ exact, den + exact @ exact
    plan.close()
    print(f"{n} x {width}: gain - 1 = {num / den - 1:.3e} (bound 5e-8)", flush=True)
    assert abs(num / den - 1) < 5e-8
