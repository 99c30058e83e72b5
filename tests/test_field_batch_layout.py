"""A field's sums do not depend on the fields around it: the block partials of a shape are the same for
every batch, also where the plan's scratch is near the 64 MiB of sb_forward_noalloc."""
import ctypes
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

LIMIT = 64 << 20


def _plan(lib, shapes, edges, lmax, npcf, field_batch=0):
    from paper_2210_10206_amd import _lib
    prob = _lib.SbProblem(len(shapes[0]), npcf, len(edges) - 1, edges.ctypes.data_as(ctypes.POINTER(ctypes.c_double)),
                          lmax, 0, 0, 0)
    sh = np.ascontiguousarray(np.array(shapes, dtype=np.int64).ravel())
    h, pb, sb, fb = ctypes.c_void_p(), ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_int32()
    assert lib.sb_plan_create(ctypes.byref(prob), len(shapes), sh.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)),
                              ctypes.byref(h)) == 0, lib.sb_last_error()
    assert lib.sb_plan_set_field_batch(h, field_batch) == 0
    assert lib.sb_plan_workspace(h, ctypes.byref(pb), ctypes.byref(sb)) == 0
    assert lib.sb_plan_get_field_batch(h, ctypes.byref(fb)) == 0
    return h, pb.value, sb.value, fb.value


@pytest.mark.parametrize("fields", [1, 2, 3, 4, 8])
@pytest.mark.parametrize("field_batch", [0, 1, 2, 3, 8])
def test_blocks_of_a_shape_in_every_batch(fields, field_batch):
    """24^3, 8 bins, l <= 4 (14 triples): 64 cells a workgroup, 216 partials of every value, in each batch.
    Three and four fields at once would pass 64 MiB with them, and would not with 512 cells a workgroup:
    such a plan still fits, with fewer fields at a time."""
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    n, nb, nlm, nlam, blocks = 24 ** 3, 8, 15, 14, 216
    h, _, scratch, batch = _plan(lib, [(24, 24, 24)] * fields, np.linspace(0.0, 8.0, nb + 1), 4, 4, field_batch)
    lib.sb_plan_destroy(h)
    # bytes of each field of the batch: density, spectrum, coefficient arrays, partials, totals; beside them
    # one gradient array, one result and the alignment
    each = n * (4 + 8) + nlm * nb * n * 8 + nlam * nb ** 3 * 8 * (blocks + 1)
    wanted = min(fields, field_batch or fields)
    long_blocks = wanted * (each - nlam * nb ** 3 * 8 * (blocks - 27)) + n * 8
    assert batch * each < scratch < max(batch * each + n * 8, long_blocks) + (1 << 20)
    assert batch == wanted or (long_blocks <= LIMIT < wanted * each)
    assert (scratch <= LIMIT) == (long_blocks + (1 << 18) <= LIMIT)


def _fields(shapes):
    import torch
    from fieldgen import lognormal_field
    return [torch.from_numpy(lognormal_field(s, seed=40 + i, sigma=1.0)).cuda() for i, s in enumerate(shapes)]


@pytest.mark.gpu
@pytest.mark.parametrize("npcf,nbins,lmax,shapes", [
    (4, 8, 4, [(24, 24, 24)] * 4),                          # fewer fields at a time than the batch
    (4, 10, 4, [(32, 32, 32)] * 2),                         # long tiles: one field fits only so
    (4, 10, 5, [(32, 32, 32), (24, 24, 32)]),               # one scratch layout for each shape
    (4, 5, 3, [(16, 16, 16), (32, 24, 16), (16, 16, 16)]),
    (3, 16, 8, [(16, 16, 16)] * 3 + [(12, 16, 24)]),        # blocks of the last pass held to the v arrays' room
    (3, 8, 6, [(128, 128)] * 3), (4, 5, 4, [(64, 48), (96, 96), (64, 48)])])
def test_batches_equal_single_fields(npcf, nbins, lmax, shapes):
    """One plan of all fields (its default batch, and one field at a time) against a plan for each field,
    bit for bit; sb_forward_noalloc too where it takes the plan, and a replayed graph."""
    import torch
    from paper_2210_10206_amd import _lib, api
    lib, edges, fields = _lib.load(), np.linspace(0.0, 8.0, nbins + 1), _fields(shapes)
    alone = []
    for f, s in zip(fields, shapes):
        p = api.Plan([s], edges, lmax, npcf=npcf)
        alone.append(p.forward_raw([f]).cpu().numpy()[0])
        p.close()
    for field_batch in (0, 1):
        p = api.Plan(shapes, edges, lmax, npcf=npcf, field_batch=field_batch)
        z = p.forward_raw(fields).cpu().numpy()
        assert all(np.array_equal(z[i], alone[i]) for i in range(len(fields))), f"field_batch {field_batch}"
        side, out = torch.cuda.Stream(), torch.empty((len(fields), p.zeta_doubles), dtype=torch.float64, device="cuda")
        side.wait_stream(torch.cuda.current_stream())
        for rep in range(3):
            with torch.cuda.stream(side):
                p.forward_raw(fields, out=out, graph=True)
            side.synchronize()
            assert np.array_equal(out.cpu().numpy(), z), f"replay {rep}"
            p.forward_raw(fields)
            torch.cuda.synchronize()
        p.close()
    h, pbytes, scratch, _ = _plan(lib, shapes, edges, lmax, npcf)
    persist = torch.empty(pbytes + 256, dtype=torch.uint8, device="cuda")
    s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert lib.sb_plan_bind(h, ctypes.c_void_p((persist.data_ptr() + 255) & ~255), pbytes, None, 0) == 0
    assert lib.sb_prepare(h, s) == 0
    got = torch.full((len(fields), len(alone[0])), float("nan"), dtype=torch.float64, device="cuda")
    ptrs = (ctypes.c_void_p * len(fields))(*[f.data_ptr() for f in fields])
    rc = lib.sb_forward_noalloc(h, ptrs, ctypes.c_void_p(got.data_ptr()), s)
    assert rc == (0 if scratch <= LIMIT else -3)
    if rc == 0:
        g = got.cpu().numpy()
        assert all(np.array_equal(g[i], alone[i]) for i in range(len(fields)))
    torch.cuda.synchronize()
    lib.sb_plan_destroy(h)
