"""GPU parity of the FlashSCA backward's binned form against the CPU oracle,
with the bars of test_gpu_sca_backward (the value gradient's covers float32
addition in any order).  The shapes are those where the form can go wrong:
each head width it serves, maps whose sides are on, above and below the bin
size (7 x 7 pixels), bins summed whole and in slices, points spread over more
bins than a tile's table holds, more records than the workspace does, and
output gradients that are not finite.  A 16-bit value gradient must be the
float32 one rounded once.
"""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_sca_backward import _dev, _g, assert_bwd_parity, small

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    import paper_2607_10071_amd as m
    return m


def run(fb, inst, g, device, dtype=None, want=("value", "offsets", "logits")):
    """The binned form through the C ABI, its outputs prefilled with NaN and
    its workspace with ones."""
    import ctypes
    import torch

    wl = inst.wl
    v, l2i, off, lg = _dev(inst, device)
    gt = torch.from_numpy(g).to(device)
    z = fb._z_array(inst.z)
    st = fb._sca_structs(v.shape, fb._dtype_code(v), v.data_ptr(), wl.heads, wl.levels,
                         (wl.img_h, wl.img_w), fb.grid_of(wl), z, "mean")
    need = ctypes.c_uint64()
    rc = fb._lib().flashsca_backward_workspace_size(*(ctypes.byref(t) for t in st), wl.P,
                                                    ctypes.byref(need))
    assert rc == 0, fb.status_string(rc)
    ws = torch.full((need.value,), 255, dtype=torch.uint8, device=device)
    out = {"value": torch.full((wl.B, wl.N, wl.S, wl.C), float("nan"), device=device,
                               dtype=dtype or torch.float32),
           "offsets": torch.full(tuple(off.shape), float("nan"), device=device),
           "logits": torch.full(tuple(lg.shape), float("nan"), device=device)}
    p = lambda k: ctypes.c_void_p(out[k].data_ptr() if k in want else 0)
    rc = fb._lib().flashsca_backward_ws(
        ctypes.byref(st[0]), ctypes.c_void_p(l2i.data_ptr()), ctypes.byref(st[1]),
        ctypes.byref(st[2]), wl.P, ctypes.c_void_p(off.data_ptr()),
        ctypes.c_void_p(lg.data_ptr()), ctypes.c_void_p(gt.data_ptr()), p("value"),
        fb._dtype_code(out["value"]), p("offsets"), p("logits"), ctypes.c_void_p(ws.data_ptr()),
        ctypes.c_uint64(need.value), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, fb.status_string(rc)
    torch.cuda.synchronize()
    # records, -, scattered tiles, full, slices, bins in slices
    misc = ws[:24].view(torch.int32).cpu().numpy()
    return {k: (t if k in want else None) for k, t in out.items()}, misc


def check(fb, inst, device, what, full=False, scattered=None, half=False):
    wl = inst.wl
    print(f"[case] sca binned {what} value={inst.value.shape} {wl.dtype} heads={wl.heads} "
          f"P={wl.P} X={wl.X} Y={wl.Y}", flush=True)
    g = _g(wl)
    out, misc = run(fb, inst, g, device)
    assert bool(misc[3]) == full
    if scattered is not None:
        assert (misc[2] > 0) == scattered
    ref = oracle.sca_backward_instance(inst, g, "mean")
    assert_bwd_parity({k: t.cpu().numpy() for k, t in out.items()}, ref, wl, what)
    if half:
        # against the oracle too: float32 sums may differ in order between calls
        import torch
        dt = {"f16": torch.float16, "bf16": torch.bfloat16}[wl.dtype]
        h, _ = run(fb, inst, g, device, dt)
        a = h["value"].float().cpu().numpy().astype(np.float64)
        u = 2.0 ** -11 if wl.dtype == "f16" else 2.0 ** -8
        tiny = 2.0 ** -25 if wl.dtype == "f16" else 0.0   # half a subnormal step
        K = np.repeat(ref["value_terms"], wl.C // wl.heads, axis=-1) + 16.0
        tol = K * 2.0 ** -24 * ref["value_scale"] * 1.01 + u * np.abs(ref["value"]) * 1.01 + tiny
        assert np.all(np.abs(a - ref["value"]) <= tol)
        assert np.array_equal(h["offsets"].cpu().numpy(), out["offsets"].cpu().numpy())
    return misc


@pytest.mark.parametrize("D", [8, 16, 24, 32, 48, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_binned_head_widths(fb, device, D, dtype):
    inst = small(20, C=D * 4, heads=4, dtype=dtype, X=11, Y=9, P=8, Z=4)
    check(fb, inst, device, f"D={D} {dtype}", half=dtype != "f32")


@pytest.mark.parametrize("levels", [((7, 7), (14, 28)), ((8, 15), (15, 29)), ((6, 13), (13, 27)),
                                    ((1, 1), (1, 40), (40, 1))])
def test_binned_map_edges(fb, device, levels):
    # offsets around and past every border of the maps
    inst = small(21, levels=levels, C=64, heads=2, P=16, Z=2, X=12, Y=10)
    rng = np.random.default_rng(21)
    h, w = levels[-1]
    inst.offsets[...] = (rng.uniform(-1.3, 1.3, inst.offsets.shape) * (w, h)).astype(np.float32)
    check(fb, inst, device, f"edges {levels}")


def crowded(seed, D=32, dtype="f32"):
    """Bins of several slices of records each."""
    return small(seed, levels=((5, 11), (20, 44)), C=2 * D, heads=2, dtype=dtype, P=32, Z=4, X=48,
                 Y=40, dx=1.0, dy=1.0)


@pytest.mark.parametrize("D,dtype", [(32, "f32"), (32, "bf16"), (8, "f32"), (16, "f16"), (24, "f32"),
                                     (48, "bf16"), (64, "f32")])
def test_binned_shared_bins(fb, device, D, dtype):
    # slices summed by a wavefront each and joined: one channel slice (8 to 32
    # channels) and two (48 and 64)
    misc = check(fb, crowded(22, D, dtype), device, f"shared bins D={D} {dtype}",
                 half=dtype != "f32")
    assert misc[4] > misc[5] > 0   # slices, bins in slices


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_binned_tile_beyond_its_table(fb, device, dtype):
    inst = small(23, levels=((116, 200), (116, 200), (116, 200)), C=128, heads=4, dtype=dtype,
                 P=16, Z=4, X=16, Y=16)
    rng = np.random.default_rng(23)
    inst.offsets[...] = rng.uniform(-150.0, 150.0, inst.offsets.shape).astype(np.float32)
    check(fb, inst, device, f"scattered tiles {dtype}", scattered=True, half=dtype == "f16")


def test_binned_tiles_beyond_their_tables_cost_little(fb, device):
    """Tiles of far more bins than a table holds are given up when theirs is
    full: a call of nothing else takes 1.5 times the scatter form's time (840
    us), where it took 6 times as much while every point searched the full
    table.  The bound lies between."""
    import torch

    inst = small(30, levels=((116, 200), (58, 100), (29, 50)), C=64, heads=4, P=64, Z=4, X=24, Y=24)
    rng = np.random.default_rng(30)
    inst.offsets[...] = rng.uniform(-150.0, 150.0, inst.offsets.shape).astype(np.float32)
    wl = inst.wl
    v, l2i, off, lg = _dev(inst, device)
    gt = torch.from_numpy(_g(wl)).to(device)
    us = {}
    for method in ("scatter", "binned"):
        times = []
        for k in range(12):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            fb.sca_backward(v, l2i, inst.z, fb.grid_of(wl), (wl.img_h, wl.img_w), wl.levels,
                            wl.heads, off, lg, gt, method=method)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3)
        us[method] = float(np.median(times[2:]))
    print(f"[case] spread tiles scatter {us['scatter']:.0f} us, binned {us['binned']:.0f} us",
          flush=True)
    assert us["binned"] < 4.0 * us["scatter"]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_binned_more_records_than_workspace(fb, device, dtype):
    # every camera the same: each seen query has N hits
    inst = small(24, N=8, C=64, heads=2, dtype=dtype, P=4, Z=2, X=9, Y=20, x_min=4.0, dx=2.0,
                 y_min=-10.0, dy=1.0)
    inst.lidar2img[:] = inst.lidar2img[:, :1]
    check(fb, inst, device, f"full {dtype}", full=True, half=dtype == "bf16")


def test_binned_room_for_many_cameras(fb, device):
    # a ring of 24 cameras: more than two records per point
    inst = small(31, B=1, N=24, levels=((32, 88),), C=64, heads=2, P=4, Z=4, X=40, Y=36, x_min=-40.0,
                 dx=2.0, y_min=-36.0, dy=2.0)
    wl = inst.wl
    misc = check(fb, inst, device, "24 cameras")
    assert misc[0] > 2 * wl.B * wl.Q * wl.heads * wl.L * wl.P


def test_binned_points_without_value_gradient(fb, device):
    inst = small(25, C=64, heads=2)
    g = _g(inst.wl)
    out, _ = run(fb, inst, g, device, want=("offsets", "logits"))
    ref = oracle.sca_backward_instance(inst, g, "mean")
    assert_bwd_parity({k: (t.cpu().numpy() if t is not None else None) for k, t in out.items()},
                      ref, inst.wl, "no value gradient")


def test_binned_degenerate_inputs(fb, device):
    inst = small(26, C=64, heads=2)
    inst.offsets[:, : inst.wl.Q // 2] = 1e9
    inst.offsets[:, inst.wl.Q // 2:, :, :, ::2] = np.nan
    check(fb, inst, device, "far and NaN offsets")


@pytest.mark.parametrize("case,D,dtype", [("whole", 8, "f32"), ("whole", 32, "bf16"),
                                          ("whole", 48, "f32"), ("slices", 24, "f32"),
                                          ("slices", 32, "f32"), ("slices", 64, "f16")])
def test_binned_gradient_that_is_not_finite(fb, device, case, D, dtype):
    """Infinite and NaN elements of the output gradient reach the elements that
    their points touch, and no other (the matrix rows multiply them by the zero
    weights of every pixel near by)."""
    import torch

    inst = crowded(29, D, dtype) if case == "slices" else small(29, C=4 * D, heads=4, dtype=dtype)
    wl = inst.wl
    print(f"[case] sca binned not finite {case} D={D} {dtype}", flush=True)
    g = _g(wl)
    # single elements of a few queries that a camera sees
    seen = np.argwhere(oracle.sca_backward_instance(inst, np.ones_like(g))["point_terms"]
                       .reshape(wl.B, wl.Q, -1).sum(-1) > 0)
    rng = np.random.default_rng(29)
    bad = np.zeros_like(g)
    for k, (b, q) in enumerate(seen[rng.choice(len(seen), 3, replace=False)]):
        bad[b, q, rng.integers(wl.C)] = (np.inf, -np.inf, np.nan)[k]
    rest = np.where(bad == 0, g, np.float32(0))
    touched = oracle.sca_backward_instance(inst, (bad != 0).astype(np.float32))["value_scale"] > 0
    assert touched.any() and not touched.all()
    ref = oracle.sca_backward_instance(inst, rest)
    for dt in {torch.float32, synth.to_storage(inst.value[:1], dtype).dtype}:
        out, misc = run(fb, inst, np.where(bad == 0, g, bad), device, dt)
        assert (misc[4] > 0) == (case == "slices")
        v = out["value"].float().cpu().numpy()
        assert not np.isfinite(v[touched]).any()
        v[touched] = ref["value"][touched]
        if dt == torch.float32:
            assert_bwd_parity({"value": v}, ref, wl, f"not finite {case} D={D}")
        else:
            assert np.isfinite(v).all()


def test_binned_large_call_is_the_default(fb, device):
    """sca_backward takes the binned form by itself for many points, and its
    gradients agree with the scatter form's."""
    import torch
    inst = small(27, levels=((29, 50), (15, 25)), C=256, heads=8, P=8, Z=4, X=64, Y=64, x_min=-32.0,
                 dx=1.0, y_min=-32.0, dy=1.0)
    wl = inst.wl
    assert wl.B * wl.Q * wl.heads * wl.L * wl.P >= fb.SCA_BINNED_MIN_POINTS
    v, l2i, off, lg = _dev(inst, device)
    g = _g(wl)
    gt = torch.from_numpy(g).to(device)
    args = (v, l2i, inst.z, fb.grid_of(wl), (wl.img_h, wl.img_w), wl.levels, wl.heads, off, lg, gt)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats(device)
    base = torch.cuda.memory_allocated(device)
    a = fb.sca_backward(*args)
    outs = sum(t.numel() * 4 for t in a.values())
    assert torch.cuda.max_memory_allocated(device) > base + outs   # the workspace
    torch.cuda.synchronize()
    ref = oracle.sca_backward_instance(inst, g, "mean")
    assert_bwd_parity({k: t.cpu().numpy() for k, t in a.items()}, ref, wl, "auto")
    b = fb.sca_backward(*args, method="scatter")
    assert_bwd_parity({k: t.cpu().numpy() for k, t in b.items()}, ref, wl, "scatter")


def test_binned_slices_of_bins_barely_above_a_slice(fb, device):
    """Bins of about 1100 records take two slices of 1024 each: the workspace
    has the slots for all of them, and the call is not left to the scatter
    form."""
    inst = small(28, B=1, N=1, levels=((70, 105),), C=64, heads=8, P=32, Z=4, X=64, Y=64, x_min=2.0,
                 dx=0.25, y_min=-2.0, dy=0.0625)
    wl = inst.wl
    # one wide camera along x sees every query near the middle of the image,
    # and the points lie evenly over the map around it: 1114 a bin
    inst.lidar2img[0, 0] = np.array([[wl.img_w / 2, -1, 0, 0], [wl.img_h / 2, 0, -1, 0], [1, 0, 0, 0],
                                     [0, 0, 0, 1]], np.float32)
    h, w = wl.levels[0]
    rng = np.random.default_rng(28)
    inst.offsets[...] = (rng.uniform(-0.5, 0.5, inst.offsets.shape) * (w, h)).astype(np.float32)
    misc = check(fb, inst, device, "two slices a bin")
    pts = wl.B * wl.Q * wl.heads * wl.L * wl.P
    assert misc[4] > 2 * pts // 1024 + 64   # more than full slices of the most records there can be
