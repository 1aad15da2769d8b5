"""Scratch sizes, on the host alone: a scratch sized for some number of items is also used for fewer of them (the job
waves of a batch share one workspace, the tree's levels are sorted in the build's scratch, a pose may hold fewer
records than its rays allow), so no size may fall where the number of items grows."""
import ctypes as C

import pytest

from test_abi_cpu import built   # noqa: F401


def _sizes(built, name, counts, before=(), after=()):
    f = getattr(built, name)
    f.restype = C.c_size_t
    return [f(*before, C.c_int64(int(n)), *after) for n in counts]


def _around(*centres):
    """Counts on both sides of each centre, a few blocks away too."""
    return sorted({max(1, c + d) for c in centres for d in (-4097, -2049, -2048, -1, 0, 1, 2, 500, 1343, 2048, 2687, 5000)})


@pytest.mark.parametrize("key_bytes", [4, 8])
def test_sort_scratch_never_shrinks(built, key_bytes):   # noqa: F811
    n = _around(1, 2048, 1 << 20, 2 << 20, 3 << 20, 7 << 20, 64 << 20)
    b = _sizes(built, "_ZN2et15sort_temp_bytesEli", n, after=(C.c_int(key_bytes),))
    assert all(y >= x for x, y in zip(b, b[1:]))


def test_trace_scratch_never_shrinks(built):   # noqa: F811
    """Rays of a wave of a batch (no diffraction), of a pose, and triangles of a pose with diffraction."""
    n = _around(64, 16 * 5120, 64 * 5120, 1 << 20, 2 << 20, 3 << 20, 8 << 20)
    name, rest = "_ZN2et15trace_ws_layoutEllilPcPNS_7TraceWSE", (C.c_void_p(), C.c_void_p())
    for after in ((0, 0, 0), (5000, 7, 3000)):
        b = _sizes(built, name, n, after=(C.c_int64(after[0]), C.c_int32(after[1]), C.c_int64(after[2]), *rest))
        assert all(y >= x for x, y in zip(b, b[1:]))
    b = _sizes(built, name, n, before=(C.c_int64(1000),), after=(C.c_int32(7), C.c_int64(3000), *rest))
    assert all(y >= x for x, y in zip(b, b[1:]))


def test_build_scratch_never_shrinks(built):   # noqa: F811
    n = _around(2, 1 << 20, 2 << 20, 3 << 20)
    b = _sizes(built, "_ZN2et19scene_scratch_bytesEll", n, after=(C.c_int64(1000),))
    assert all(y >= x for x, y in zip(b, b[1:]))


@pytest.mark.parametrize("F,Bk", [(256, 8), (1000, 7), (256, 64)])
@pytest.mark.parametrize("flags", [0, "ET_PATH_PRODUCT", "ET_SYNTH_DIRECT"])
def test_synthesis_scratch_never_shrinks(built, F, Bk, flags):   # noqa: F811
    """Records of the paths, up to a pose's most (the workspace query) and fewer (a call on smaller paths)."""
    import paper_2602_19652_amd as et
    d = et.SimDesc(M=2, F=F, f_lo=20e3, f_hi=100e3, c=343.0, Q=3, Bk=Bk, flags=getattr(et, flags) if flags else 0)
    n = _around(64, 256 * 64, 2048, 1 << 20, 4 << 20, 8 << 20, 12 << 20)
    for name in ("_ZN2et15synth_ws_layoutEPK11et_sim_desclPcPNS_7SynthWSE", "_ZN2et19synth_bwd_ws_layoutEPK11et_sim_desclPcPNS_7SynthWSE"):
        b = _sizes(built, name, n, before=(C.byref(d),), after=(C.c_void_p(), C.c_void_p()))
        assert all(y >= x for x, y in zip(b, b[1:]))
