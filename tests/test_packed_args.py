"""The binding's packed C structures (CPU only): byte for byte the ctypes
structures, over random values of each field; values past a field's type go
through the structures themselves."""
import ctypes

import numpy as np
import pytest

import paper_2607_10071_amd as fb


def raw(s):
    return bytes(memoryview(s).cast("B"))


def test_packed_structures_match_the_ctypes_ones():
    rng = np.random.default_rng(0)
    for _ in range(50):
        ints = [int(v) for v in rng.integers(-2**31, 2**31, 12)]
        g = fb.BevGrid(*(float(v) if k % 3 != 2 else ints[k] for k, v in
                         enumerate(rng.standard_normal(6) * 50)), depth_eps=float(rng.random()))
        z = rng.standard_normal(int(rng.integers(1, 40))).astype(np.float32)
        z.flags.writeable = bool(rng.integers(2))
        ptr = int(rng.integers(0, 2**47))
        reduce = ("mean", "sum")[int(rng.integers(2))]
        args = (ints[:5], int(rng.integers(3)), ptr, ints[5:7], g, z, reduce)
        for a, b in zip(fb._packed(*args), fb._structs(*args)):
            n = 12 if isinstance(b, fb.ZBins) else len(a)   # the rest is padding
            assert a[:n] == raw(b)[:n]
        levels = [tuple(map(int, rng.integers(1, 300, 2))) for _ in range(int(rng.integers(1, 9)))]
        args = (ints[:4], 1, ptr, ints[4], levels, ints[5:7], g, z, reduce)
        for a, b in zip(fb._sca_packed(*args), fb._sca_structs(*args)):
            n = 12 if isinstance(b, fb.ZBins) else len(a)
            assert a[:n] == raw(b)[:n]


def test_values_past_the_c_types_take_the_structures():
    z = np.zeros(2, np.float32)
    g = fb.BevGrid(-1e300, 1.0, 4, 0.0, 1.0, 4)          # float32 overflow: infinity there
    # float32 overflow is an infinity either way
    a = fb._packed((1, 1, 2, 2, 4), 0, 0, (4, 4), g, z, "mean")
    assert a[1] == raw(fb._structs((1, 1, 2, 2, 4), 0, 0, (4, 4), g, z, "mean")[1])
    # an integer past 32 bits wraps in the structure
    a = fb._packed((1, 1, 2, 2, (1 << 32) + 4), 0, 0, (4, 4), g, z, "mean")
    assert not isinstance(a[0], bytes)
    assert fb._packed_call("flashbev_sample_vt", "PPPPPP")(a[0], 0, a[1], a[2], 0, 0) == \
        fb.STATUS["ERR_VALUE"]
    with pytest.raises(ValueError):
        fb._sca_packed((1, 1, 4, 4), 0, 0, 1, [(1, 1)] * 9, (4, 4), g, z, "mean")
    with pytest.raises(KeyError):
        fb._packed((1, 1, 2, 2, 4), 0, 0, (4, 4), g, z, "max")


def test_empty_heights_have_an_address():
    assert isinstance(fb._address(np.zeros(0, np.float32)), int)
    assert fb._packed_call("flashbev_sample_vt", "PPPPPP")(None, 0, None, None, 0, 0) == \
        fb.STATUS["ERR_NULLPTR"]


def test_gradient_types_of_the_gather_form():
    import ctypes
    z = np.zeros(2, np.float32)
    f, g, zb = fb._packed((1, 1, 2, 2, 4), fb.DTYPE_CODES["bf16"], 0, (4, 4),
                          fb.BevGrid(-1, 1, 4, -1, 1, 4), z, "mean")
    call = fb._packed_call("flashbev_sample_vt_backward_ws_as", "PPPPPPiPQP")
    base = 0x7F0000000000
    args = lambda grad, code, ws: (f, base, g, zb, base + 4096, grad, code, ws, 1 << 20, 0)
    S = fb.STATUS
    assert call(*args(base + 8192, fb.DTYPE_CODES["f16"], base + (1 << 24))) == S["ERR_DTYPE"]
    assert call(*args(base + 8193, fb.DTYPE_CODES["bf16"], base + (1 << 24))) == S["ERR_ALIGN"]
    assert call(*args(base + 8194, fb.DTYPE_CODES["f32"], base + (1 << 24))) == S["ERR_ALIGN"]
    # a 16-bit gradient of 32 bytes right before the output gradient is no overlap
    assert call(*args(base + 4096 - 32, fb.DTYPE_CODES["bf16"], base + (1 << 24) + 1)) == S["ERR_ALIGN"]
    assert call(*args(base + 4096 - 30, fb.DTYPE_CODES["bf16"], base + (1 << 24))) == S["ERR_ALIAS"]
    assert call(None, *args(0, 0, 0)[1:]) == S["ERR_NULLPTR"]


def test_packed_calls_belong_to_the_loaded_library():
    # the phase-clock tool loads another build of the library and goes back
    from paper_2607_10071_amd import phases
    address = lambda: ctypes.cast(fb._packed_call("flashbev_sample_vt", "PPPPPP"),
                                  ctypes.c_void_p).value
    of = lambda lib: ctypes.cast(lib["flashbev_sample_vt"], ctypes.c_void_p).value
    plain_path, plain = fb._LIB_PATH, fb._lib()
    assert address() == of(plain)
    try:
        fb._LIB_PATH, fb._LIB = phases.LIB_PATH, None
        assert address() == of(fb._lib()) != of(plain)
    finally:
        fb._LIB_PATH, fb._LIB = plain_path, plain
    assert address() == of(plain)
