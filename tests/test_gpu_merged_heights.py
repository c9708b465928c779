"""GPU parity of the forward where consecutive heights share their taps and
are merged into one record: dense heights in any order, repeated heights,
passes of several height chunks and of several cells, maps of one row or
column, ragged grids and every storage type, against the CPU oracle with
test_gpu_parity's bars.  The grids have the cell groups from which merging is
taken (2048), and spacings well below it; each test asserts that it is taken
(non-finite heights, whose spacing says nothing, go without).
"""
import numpy as np
import pytest

import synth
import test_gpu_parity as tp
from test_gpu_parity import small

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    import paper_2607_10071_amd as m
    return m


def check_instance(fb, inst, device, reduce="mean", what="", path="merged"):
    wl = inst.wl
    assert fb.launch_path(inst.features.shape, wl.dtype, inst.z, fb.grid_of(wl),
                          (wl.img_h, wl.img_w), reduce) == path
    tp.check_instance(fb, inst, device, reduce, what)


@pytest.mark.parametrize("dtype,C", [("f32", 16), ("f32", 32), ("f32", 80), ("bf16", 64), ("f16", 33),
                                     ("bf16", 7)])
@pytest.mark.parametrize("N,Z", [(6, 24), (1, 65), (2, 64)])
def test_dense_heights(fb, device, dtype, C, N, Z):
    inst = small(N=N, C=C, dtype=dtype, X=133, Y=129, half=50.0, Z=Z)
    check_instance(fb, inst, device, what=f"dense {dtype} C={C} N={N} Z={Z}")


@pytest.mark.parametrize("order", ["descending", "repeated", "shuffled", "bunches", "nonfinite"])
def test_height_orders(fb, device, order):
    inst = small(C=32, X=160, Y=111, half=50.0, Z=40)
    z = np.array(inst.z)
    rng = np.random.default_rng(3)
    if order == "descending":
        z = z[::-1]
    elif order == "repeated":
        z = np.repeat(z[::8], 8)
    elif order == "shuffled":   # neighbouring pairs swapped: runs break and resume
        z = z.reshape(-1, 2)[:, ::-1].reshape(-1)
    elif order == "bunches":
        z = np.concatenate([np.sort(rng.uniform(a, a + 0.05, 10)) for a in (-4, -1, 0, 2)])
    else:
        z[7], z[20] = np.nan, np.inf
    inst.z = np.ascontiguousarray(z.astype(np.float32))
    check_instance(fb, inst, device, what=order,
                   path="culled" if order == "nonfinite" else "merged")


@pytest.mark.parametrize("H,W", [(1, 44), (16, 1), (1, 1), (2, 2)])
def test_thin_maps(fb, device, H, W):
    wl = small(C=32, X=130, Y=130, half=50.0, Z=20).wl.with_(H=H, W=W)
    check_instance(fb, synth.make_workload(wl), device, what=f"{H} x {W} map")


@pytest.mark.parametrize("reduce", ["mean", "sum"])
def test_batch_and_reduce(fb, device, reduce):
    check_instance(fb, small(B=3, C=64, dtype="bf16", X=81, Y=83, half=40.0, Z=32), device, reduce,
                   what=f"batch {reduce}")
