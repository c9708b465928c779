"""FlashSCA's binned backward, C ABI (CPU only): the workspace size and the
checks that run before any HIP call."""
import ctypes

import numpy as np
import pytest

import paper_2607_10071_amd as fb
from paper_2607_10071_amd import GridSpec, ScaValue, ZBins

S = fb.STATUS
BASE = 0x7F0000000000   # fake device addresses, 2^36 bytes apart
LEVELS = ((116, 200), (58, 100), (29, 50), (15, 25))


def structs(B=1, N=6, C=256, heads=8, dtype="f32", X=200, Y=200, levels=LEVELS, data=BASE):
    z = np.asarray((-4.5, -2.2, 0.2, 2.5), np.float32)
    n = len(levels)
    lh = (ctypes.c_int32 * 8)(*[h for h, _ in levels], *([0] * (8 - n)))
    lw = (ctypes.c_int32 * 8)(*[w for _, w in levels], *([0] * (8 - n)))
    v = ScaValue(data, fb.DTYPE_CODES[dtype], B, N, C, heads, n, lh, lw, 900, 1600)
    g = GridSpec(-51.2, 0.512, X, -51.2, 0.512, Y, 1e-5, 0)
    return v, g, ZBins(z.ctypes.data_as(ctypes.POINTER(ctypes.c_float)), 4), z


def size(P=8, **kw):
    v, g, zb, _z = structs(**kw)
    out = ctypes.c_uint64()
    rc = fb._lib().flashsca_backward_workspace_size(ctypes.byref(v), ctypes.byref(g),
                                                    ctypes.byref(zb), P, ctypes.byref(out))
    return rc, out.value


def call(P=8, ws=BASE + (9 << 36), ws_bytes=1 << 40, gv=BASE + (5 << 36), gv_dtype="f32", **kw):
    v, g, zb, _z = structs(**kw)
    a = lambda k: ctypes.c_void_p(BASE + (k << 36))
    return fb._lib().flashsca_backward_ws(
        ctypes.byref(v), a(1), ctypes.byref(g), ctypes.byref(zb), P, a(2), a(3), a(4),
        ctypes.c_void_p(gv), fb.DTYPE_CODES[gv_dtype], a(6), a(7), ctypes.c_void_p(ws),
        ctypes.c_uint64(ws_bytes), ctypes.c_void_p(0))


@pytest.mark.parametrize("kw,status", [
    (dict(C=40 * 8), "ERR_UNSUPPORTED"),                  # head rows of 40 channels
    (dict(C=12, heads=4), "ERR_UNSUPPORTED"),
    (dict(X=0), "ERR_UNSUPPORTED"),                       # nothing to sum
    (dict(N=0), "ERR_UNSUPPORTED"),
    (dict(X=2000, Y=2000), "ERR_UNSUPPORTED"),            # more than 2^28 points
    (dict(levels=((1 << 15, 4),)), "ERR_UNSUPPORTED"),
    (dict(P=6), "ERR_SHAPE"),
])
def test_shapes_without_a_binned_form(kw, status):
    assert size(**kw)[0] == S[status]
    assert call(**kw) == S[status]


def test_workspace_size_and_checks():
    rc, need = size()
    pts = 200 * 200 * 8 * 32
    assert rc == S["OK"] and 2 * pts * 16 < need < 4 * pts * 16   # records, slices, tables
    assert size(dtype="bf16")[1] > need    # a float32 gradient for tiles that are scattered
    assert call(ws_bytes=need - 1) == S["ERR_SCRATCH"]
    assert call(ws=0) == S["ERR_NULLPTR"]
    assert call(ws=BASE + (9 << 36) + 16) == S["ERR_ALIGN"]
    assert call(ws=BASE + (4 << 36)) == S["ERR_ALIAS"]
    assert call(gv=BASE + (5 << 36) + 2) == S["ERR_ALIGN"]
    assert call(gv_dtype="bf16") == S["ERR_DTYPE"]        # neither float32 nor the value's
    assert call(gv=BASE + (4 << 36)) == S["ERR_ALIAS"]
    lib = fb._lib()
    assert lib.flashsca_backward_workspace_size(None, None, None, 8, None) == S["ERR_NULLPTR"]
    assert lib.flashsca_backward_ws(*([None] * 4), 8, *([None] * 4), 0, None, None, None, 0,
                                    None) == S["ERR_NULLPTR"]


def test_python_method_argument():
    v, g, zb, _z = structs()
    with pytest.raises(ValueError):
        fb._sca_workspace_bytes(*map(ctypes.byref, (v, g, zb)), 8, "sorted", 1, True)
    big = fb.SCA_BINNED_MIN_POINTS
    assert fb._sca_workspace_bytes(*map(ctypes.byref, (v, g, zb)), 8, "auto", big - 1, True) == -1
    assert fb._sca_workspace_bytes(*map(ctypes.byref, (v, g, zb)), 8, "auto", big, None) == -1
    assert fb._sca_workspace_bytes(*map(ctypes.byref, (v, g, zb)), 8, "auto", big, True) == size()[1]
    assert fb._sca_workspace_bytes(*map(ctypes.byref, (v, g, zb)), 8, "scatter", big, True) == -1
    # nothing to bin without a value gradient: no workspace
    assert fb._sca_workspace_bytes(*map(ctypes.byref, (v, g, zb)), 8, "binned", big, None) == -1
    assert fb._sca_workspace_bytes(*map(ctypes.byref, (v, g, zb)), 8, "binned", 1, True) == size()[1]


def best(P=8, gv_dtype="f32", **kw):
    v, g, zb, _z = structs(**kw)
    out = ctypes.c_uint64()
    rc = fb._lib().flashsca_backward_workspace_best(ctypes.byref(v), ctypes.byref(g),
                                                    ctypes.byref(zb), P, fb.DTYPE_CODES[gv_dtype],
                                                    ctypes.byref(out))
    assert rc == S["OK"]
    return out.value


@pytest.mark.parametrize("kw,binned", [
    (dict(), True),                                            # BEVFormer-base
    (dict(X=32, Y=32), True), (dict(X=31, Y=32), False),       # from 2^18 points on
    (dict(C=320), False),                                      # not served
    (dict(N=12), True),
    # points per query and head, head widths, cameras
    (dict(levels=((116, 200),), P=4), False), (dict(levels=((116, 200),), P=8), True),
    (dict(levels=((58, 100),), P=8, C=64), False), (dict(levels=((58, 100),), P=16, C=64), True),
    (dict(levels=((58, 100),), P=8, C=64, dtype="bf16"), False),
    (dict(levels=((58, 100),), P=8, C=64, dtype="bf16", gv_dtype="bf16"), True),
    (dict(levels=((58, 100),), P=12, N=2), False), (dict(levels=((58, 100),), P=32, N=2), True),
    # maps of few bins
    (dict(levels=((14, 56),), P=32), False), (dict(levels=((17, 39),), P=32), True),
    (dict(levels=((16, 44),), P=16, X=75, Y=80), False), (dict(levels=((16, 44),), P=16), True),
    (dict(levels=((16, 44),), P=32, X=75, Y=80), True),
    # points per bin
    (dict(B=4, X=40, Y=40), False), (dict(B=4, X=64, Y=64), True),
    (dict(B=4, X=40, Y=40, dtype="bf16"), False),              # a float32 gradient
    (dict(B=4, X=40, Y=40, dtype="bf16", gv_dtype="bf16"), True),
    # coarse grids under wide maps
    (dict(P=32, X=40, Y=40), False), (dict(P=32, X=64, Y=64), True),
])
def test_where_the_binned_form_is_taken(kw, binned):
    assert best(**kw) == (size(**{k: t for k, t in kw.items() if k != "gv_dtype"})[1] if binned
                          else 0)


def test_best_size_refuses_what_the_call_refuses():
    v, g, zb, _z = structs()
    out = ctypes.c_uint64()
    call = fb._lib().flashsca_backward_workspace_best
    ref = [ctypes.byref(t) for t in (v, g, zb)]
    assert call(*ref, 8, fb.DTYPE_CODES["f32"], None) == S["ERR_NULLPTR"]
    assert call(*ref, 8, fb.DTYPE_CODES["bf16"], ctypes.byref(out)) == S["ERR_DTYPE"]
    assert call(*ref, 6, fb.DTYPE_CODES["f32"], ctypes.byref(out)) == S["ERR_SHAPE"]
