"""The C-ABI library loads and exports every entry point the header declares (CPU only)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "sarabande_hip.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sb_[a-z_]+)\s*\(", text)))


def test_header_declares_the_boundary():
    names = declared_functions()
    for n in ["sb_plan_create", "sb_plan_workspace", "sb_plan_bind", "sb_prepare", "sb_forward",
              "sb_backward", "sb_zeta_size", "sb_zeta_index", "sb_bin_counts", "sb_autotune",
              "sb_forward_graph", "sb_plan_destroy", "sb_status_str", "sb_last_error"]:
        assert n in names


def test_library_exports_every_declared_symbol():
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    for n in declared_functions():
        assert hasattr(lib, n), n
        assert n in _lib.SIGNATURES, n


def _problem(ndim=3, npcf=3, edges=(0.0, 2.0, 4.0), lmax=2, prec=0, dtype=0, flags=0):
    from paper_2210_10206_amd import _lib
    import numpy as np
    e = np.asarray(edges, dtype=np.float64)
    p = _lib.SbProblem(ndim, npcf, len(e) - 1, e.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), lmax, prec, dtype,
                       flags)
    return p, e


@pytest.mark.parametrize("kw,shape,expect", [
    (dict(ndim=4), (16, 16, 16), -1),
    (dict(npcf=5), (16, 16, 16), -1),
    (dict(edges=(0.0, 3.0, 2.0)), (16, 16, 16), -1),
    (dict(edges=(-1.0, 3.0)), (16, 16, 16), -1),
    (dict(lmax=-1), (16, 16, 16), -1),
    (dict(lmax=11), (16, 16, 16), -1),
    (dict(prec=7), (16, 16, 16), -1),
    (dict(), (16, 16, 0), -1),
    (dict(), (16, 16, 14), -2),          # 14 = 2 * 7: no radix-7 pass
    (dict(npcf=4, edges=tuple(range(12))), (16, 16, 16), -2),
    (dict(flags=8), (16, 16, 16), -1),                # odd parity is a full-4PCF option
    (dict(ndim=2, npcf=4, flags=8), (16, 16, 16), -1),
])
def test_argument_validation_without_gpu(kw, shape, expect):
    """Argument errors are reported before any device call, so they can be checked on a CPU host."""
    from paper_2210_10206_amd import _lib
    import numpy as np
    lib = _lib.load()
    prob, e = _problem(**kw)
    sh = np.array(shape[:prob.ndim] if prob.ndim in (2, 3) else shape, dtype=np.int64)
    out = ctypes.c_void_p()
    rc = lib.sb_plan_create(ctypes.byref(prob), 1, sh.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)), ctypes.byref(out))
    assert rc == expect
    assert not out.value
    assert len(lib.sb_last_error()) > 0


def test_status_strings():
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    names = set()
    for s in range(-7, 1):
        name = lib.sb_status_str(s)
        assert name and name != b"unknown status"
        names.add(name)
    assert len(names) == 8
    assert lib.sb_status_str(-6) == b"non-finite input" and lib.sb_status_str(-7) == b"call out of order"
    assert lib.sb_version() >= 1


def _plan(lib, prob, shapes):
    import numpy as np
    sh = np.ascontiguousarray(np.array(shapes, dtype=np.int64).ravel())
    out = ctypes.c_void_p()
    rc = lib.sb_plan_create(ctypes.byref(prob), len(shapes), sh.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)),
                            ctypes.byref(out))
    return rc, out


def test_plan_creation_needs_no_device_and_reports_truncation():
    """Plan creation is host-only (the device tables are copied by sb_prepare into the caller's
    persistent buffer), so the layout, the exact bin counts and the box-truncation warning of
    the zero-centred kernel support can be read without a GPU."""
    import numpy as np
    import oracle
    from fieldgen import linear_edges
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    # the uneven workload's finite-difference case: 8 bins to 16 on 24^3 reaches past N/2 = 12
    for shape, edges, warn in (((24, 24, 24), linear_edges(16, 8), 1), ((64, 64, 64), linear_edges(16, 8), 0),
                               ((32, 32, 32), linear_edges(16, 8), 1), ((48, 48, 48), linear_edges(23.9, 4), 0)):
        prob, e = _problem(edges=tuple(edges), lmax=4)
        rc, h = _plan(lib, prob, [shape])
        assert rc == 0, lib.sb_last_error()
        bits = ctypes.c_uint32()
        assert lib.sb_plan_warnings(h, ctypes.byref(bits)) == 0
        assert bits.value == warn, (shape, edges[-1])
        counts = np.zeros(len(edges) - 1, dtype=np.int64)
        assert lib.sb_bin_counts(h, 0, counts.ctypes.data_as(ctypes.POINTER(ctypes.c_int64))) == 0
        assert list(counts) == list(oracle.bin_counts(shape, edges))
        pb, sbytes = ctypes.c_size_t(), ctypes.c_size_t()
        assert lib.sb_plan_workspace(h, ctypes.byref(pb), ctypes.byref(sbytes)) == 0
        assert pb.value > 0 and sbytes.value > 0
        lib.sb_plan_destroy(h)


def test_result_index_tables_match_the_oracle():
    """The Lambda list of the full 4PCF (Alg. 6 loop order) and the (m1, m2) list of the
    projected 4PCF (Alg. 8 loop order) equal the oracle's enumerations."""
    import numpy as np
    import oracle
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    for ndim, lmax, flags, want in ((3, 4, 0, oracle.lambdas(4)), (3, 4, 8, oracle.lambdas(4, parity="odd")),
                                    (2, 10, 0, oracle.mpairs(10)), (2, 3, 0, oracle.mpairs(3))):
        prob, e = _problem(ndim=ndim, npcf=4, edges=(0.0, 2.0, 4.0), lmax=lmax, flags=flags)
        rc, h = _plan(lib, prob, [(32,) * ndim])
        assert rc == 0, lib.sb_last_error()
        rows, cols = ctypes.c_int32(), ctypes.c_int32()
        tab = ctypes.POINTER(ctypes.c_int32)()
        assert lib.sb_zeta_index(h, ctypes.byref(rows), ctypes.byref(cols), ctypes.byref(tab)) == 0
        got = [tuple(tab[r * cols.value + c] for c in range(cols.value)) for r in range(rows.value)]
        assert got == [tuple(x) for x in want]
        lib.sb_plan_destroy(h)


@pytest.mark.parametrize("kw,expect", [
    (dict(prec=1, flags=2), -2),              # unfused 3PCF pair kernel: no split form
    (dict(prec=1, flags=1), -2),              # coefficients kept: the unfused path again
    (dict(prec=1, npcf=4, flags=4), -2),      # plain vector-ALU 4PCF kernel
    (dict(prec=1, npcf=4, lmax=5), -2),       # no matrix-core kernel beyond l = 4
    (dict(prec=1, ndim=2, npcf=4, flags=4), -2),
    (dict(prec=1, npcf=4), 0),                # full 4PCF on the matrix cores
])
def test_split_bf16_only_where_a_split_form_exists(kw, expect):
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    prob, e = _problem(**kw)
    rc, h = _plan(lib, prob, [(16,) * prob.ndim])
    assert rc == expect, lib.sb_last_error()
    if h.value:
        lib.sb_plan_destroy(h)


def _plan_object(shape, **kw):
    """A Plan around a handle without a device buffer (what its constructor holds before it binds any)."""
    from paper_2210_10206_amd import _lib, api
    import numpy as np
    plan = api.Plan.__new__(api.Plan)
    plan.lib, prob = _lib.load(), _problem(**kw)
    plan.ndim, plan.npcf, plan.nbins, plan.handle = kw.get("ndim", 3), kw["npcf"], prob[0].nbins, ctypes.c_void_p()
    sh = np.array(shape, dtype=np.int64)
    assert plan.lib.sb_plan_create(ctypes.byref(prob[0]), 1, sh.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)),
                                   ctypes.byref(plan.handle)) == 0
    plan._index = plan._read_index()
    return plan


def test_index_of_a_plan_without_rows():
    """Odd Lambda to l = 0: there is none, so the table is empty."""
    plan = _plan_object((16, 16, 16), npcf=4, lmax=0, flags=8)
    assert plan.zeta_index().shape == (0, 3) and plan.zeta_shape() == (0, 2, 2, 2)
    plan.lib.sb_plan_destroy(plan.handle)
    plan.handle = None


def test_index_of_a_closed_plan_is_refused():
    plan = _plan_object((16, 16, 16), npcf=3)
    plan.lib.sb_plan_destroy(plan.handle)
    plan.handle = None   # as close() leaves it
    for ask in (plan.zeta_index, plan.zeta_shape):
        with pytest.raises(RuntimeError):
            ask()


def test_autotune_and_normalize_reject_an_unbound_plan():
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    prob, e = _problem()
    rc, h = _plan(lib, prob, [(16, 16, 16)])
    assert rc == 0
    assert lib.sb_autotune(h, None, None) == -3
    ptrs = (ctypes.c_void_p * 1)(None)
    assert lib.sb_normalize(h, ptrs, None, None, None) == -1
    lib.sb_plan_destroy(h)


def test_1024_grid_plan_regenerates_kernels():
    """At 1024^3 (10 bins to 32, lmax 6) the compact kernel cache would take about 169 GB, so the
    fused 3PCF plan keeps none (regenerating each chunk's kernel planes in scratch): its
    persistent buffer holds only tables and its scratch fits one chunk of (l, m) groups."""
    import numpy as np
    from fieldgen import linear_edges
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    prob, e = _problem(edges=tuple(linear_edges(32, 10)), lmax=6)
    rc, h = _plan(lib, prob, [(1024, 1024, 1024)])
    assert rc == 0, lib.sb_last_error()
    pb, sbytes = ctypes.c_size_t(), ctypes.c_size_t()
    assert lib.sb_plan_workspace(h, ctypes.byref(pb), ctypes.byref(sbytes)) == 0
    assert pb.value < 1 << 20
    assert sbytes.value < 140 << 30
    lib.sb_plan_destroy(h)
    # the same problem at 256^3 keeps its cache: 31 kernel groups (28 (l, m) and 3 packed m = 0
    # pairs) of 10 bins, 65 stored axis-0 planes each (|c_0| <= 32); with the half store on
    # request 33 (c_0 = 0 .. 32, the rest by parity)
    for flags, planes in ((0, 65), (128, 33)):
        prob.flags = flags
        rc, h = _plan(lib, prob, [(256, 256, 256)])
        assert lib.sb_plan_workspace(h, ctypes.byref(pb), ctypes.byref(sbytes)) == 0
        size = 31 * 10 * planes * 256 * 256 * 8
        assert size <= pb.value < size + (64 << 20)
        lib.sb_plan_destroy(h)
    prob.flags = 0
    # 512^3, 16 bins to 16, lmax 10: the full cache (66 (l, m) groups x 16 bins x 33 planes, 73 GB)
    # passes the 64 GiB cap, the half one (17 planes) does not, so the plan keeps the half store
    prob16, e16 = _problem(edges=tuple(linear_edges(16, 16)), lmax=10)
    rc, h = _plan(lib, prob16, [(512, 512, 512)])
    assert rc == 0, lib.sb_last_error()
    assert lib.sb_plan_workspace(h, ctypes.byref(pb), ctypes.byref(sbytes)) == 0
    size = 71 * 16 * 17 * 512 * 512 * 8   # 66 groups and 5 packed m = 0 pairs
    assert size <= pb.value < size + (64 << 20) and pb.value < 64 << 30
    lib.sb_plan_destroy(h)
    # regeneration on request is a fused-3PCF option only
    for kw in (dict(npcf=4), dict(flags=2)):
        prob4, _ = _problem(edges=(0.0, 2.0, 4.0), lmax=2, **kw)
        prob4.flags |= 64
        rc, h = _plan(lib, prob4, [(16, 16, 16)])
        assert rc == -2 and not h.value


def test_keep_for_adjoint_layout_and_scope():
    """SB_FLAG_KEEP_FOR_ADJOINT gives every field its own region of coefficient arrays (the array
    groups of the forward: with lmax 2 the packed (0, 0) + (1, 0) pair and the four other (l, m),
    each with every bin) and the backward one more field's worth for its v arrays; it is refused
    outside the fused 3D 3PCF path and with regenerated kernels."""
    from paper_2210_10206_amd import _lib
    lib = _lib.load()
    shapes = [(16, 16, 16), (24, 24, 24), (16, 16, 16)]
    sizes = {}
    for flags in (0, 256, 256 | 16):
        prob, e = _problem(edges=(0.0, 2.0, 4.0), lmax=2, flags=flags)
        rc, h = _plan(lib, prob, shapes)
        assert rc == 0, lib.sb_last_error()
        pb, sbytes = ctypes.c_size_t(), ctypes.c_size_t()
        assert lib.sb_plan_workspace(h, ctypes.byref(pb), ctypes.byref(sbytes)) == 0
        sizes[flags] = sbytes.value
        lib.sb_plan_destroy(h)
    cells = 16 ** 3 * 2 + 24 ** 3
    for flags, nag in ((256, 5), (256 | 16, 6)):
        kept = nag * 2 * cells * 8 + nag * 2 * 24 ** 3 * 8
        assert sizes[flags] >= kept
        assert sizes[flags] - sizes[0] >= kept - 2 * 6 * 2 * 24 ** 3 * 8   # at most two fields' arrays at once before
    for kw in (dict(ndim=2), dict(npcf=4), dict(flags=2), dict(flags=64), dict(flags=1)):
        prob, _ = _problem(edges=(0.0, 2.0, 4.0), lmax=2, **kw)
        prob.flags |= 256
        rc, h = _plan(lib, prob, [(16, 16, 16)[:prob.ndim]])
        assert rc == -2 and not h.value, kw
