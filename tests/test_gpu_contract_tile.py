"""The contraction tile that a caller sets is the one that runs, on grids of every size: another number of
cells in a workgroup's float32 sums gives other bits, the same number the same bits (the projected 4PCF
adds to float64 every 64 cells, which a tile does not change)."""
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


# the compile-time kernels; the run-time one (10 bins; l > 4), 512 cells and more being several staged tiles
@pytest.mark.parametrize("nbins,lmax,parity,shape", [(8, 3, "even", (16, 16, 32)), (10, 3, "even", (16, 32, 24)),
                                                     (4, 5, "odd", (24, 16, 24)), (5, 4, "", (64, 192))])
def test_set_tile_runs(nbins, lmax, parity, shape, tmp_path):
    from paper_2210_10206_amd import api
    d, edges = lognormal_field(shape, seed=8, sigma=1.0), linear_edges(7.5, nbins)
    d64, dev = d.astype(np.float64), [torch.from_numpy(d).cuda()]
    if parity:
        ref = oracle.zeta4_full(d64, edges, lmax, parity=parity)[1]
        ref = ref.imag if parity == "odd" else ref.real
    else:
        ref = oracle.zeta4_proj(d64, edges, lmax)[1]
    new = lambda: api.Plan([shape], edges, lmax, npcf=4, parity=parity or "even")  # noqa: E731
    plan = new()
    untuned, saved = plan.forward_raw(dev).cpu().numpy(), plan.choices()
    _, (lo, hi) = plan.contract_tile()
    tiles = [c for c in (512, 1024, 2048, 4096, 8192) if lo <= c <= hi]
    seen = {}
    for c in tiles:
        plan.set_contract_tile(c)
        assert plan.contract_tile()[0] == c
        raw = plan.forward_raw(dev)
        seen[c] = raw.cpu().numpy()
        check(plan.unpack(raw)[0].cpu().numpy(), ref, TOL32, print, f"{shape} {nbins} bins tile {c}: ")
    kept = plan.choices()
    plan.set_choices(saved)   # the short tiles of a new plan again
    assert np.array_equal(plan.forward_raw(dev).cpu().numpy(), untuned)
    plan.close()
    other = new()
    other.set_choices(kept)
    assert np.array_equal(other.forward_raw(dev).cpu().numpy(), seen[tiles[-1]])
    # tuned, read back from the file, and set by hand: the same launches
    other.autotune(cache_path=str(tmp_path / "tuned.json"))
    tuned, z = other.choices(), other.forward_raw(dev).cpu().numpy()
    other.close()
    for use in (lambda p: p.autotune(cache_path=str(tmp_path / "tuned.json")), lambda p: p.set_choices(tuned)):
        p = new()
        use(p)
        assert p.choices() == tuned and np.array_equal(p.forward_raw(dev).cpu().numpy(), z)
        p.close()
    # a file without the key (it names a tile only) sets that tile
    text = (tmp_path / "tuned.json").read_text()
    start = text.index('"contract_tile": ')
    (tmp_path / "old.json").write_text(text[:start] + f'"contract_tile": {tiles[0]}' + text[text.index("}", start):])
    p = new()
    p.autotune(cache_path=str(tmp_path / "old.json"))
    p.set_choices({"fft": saved["fft"]})
    assert p.choices() == {**saved, "contract_tile": tiles[0], "short_tiles": False}
    assert np.array_equal(p.forward_raw(dev).cpu().numpy(), seen[tiles[0]])
    p.close()
    assert not parity or all(not np.array_equal(seen[a], seen[b]) for a in tiles for b in tiles if a < b)
