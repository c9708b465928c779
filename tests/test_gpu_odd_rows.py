"""GPU parity where feature rows are not whole 16-byte vectors and the last
vector is moved back to end with its row: row lengths around the widths where
that is taken (128 bytes forward, 256 bytes of float32 gradient backward),
every remainder, wide rows with several vectors per lane, a base address off
16 bytes, and the last pixel of the maps; forward and gather-form backward
against the CPU oracle with test_gpu_parity's and test_gpu_backward's bars."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_backward import check as check_backward
from test_gpu_parity import RTOL, assert_parity, check_instance, small

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    import paper_2607_10071_amd as m
    return m


@pytest.mark.parametrize("dtype,C", [("f32", 31), ("f32", 33), ("f32", 34), ("f32", 35), ("f32", 63),
                                     ("f32", 65), ("f32", 99), ("f32", 255), ("f32", 257),
                                     ("f32", 513), ("f32", 1021), ("bf16", 62), ("bf16", 66),
                                     ("f16", 70), ("bf16", 250), ("f16", 514), ("bf16", 65)])
def test_odd_rows(fb, device, dtype, C):
    inst = small(B=2, C=C, dtype=dtype, X=19, Y=17, Z=5)
    check_instance(fb, inst, device, what=f"odd rows {dtype} C={C}")
    check_backward(fb, inst, device, what=f"odd rows {dtype} C={C}", prefill=float("nan"))


@pytest.mark.parametrize("dtype,C,shift", [("f32", 80, 1), ("f32", 33, 3), ("bf16", 64, 2),
                                           ("bf16", 66, 1), ("f16", 128, 4)])
def test_unaligned_base(fb, device, dtype, C, shift):
    """Features ``shift`` elements into an allocation."""
    import torch
    inst = small(C=C, dtype=dtype, X=19, Y=17)
    wl = inst.wl
    ft = synth.to_storage(inst.features, dtype).to(device)
    room = torch.zeros(ft.numel() + shift, dtype=ft.dtype, device=device)
    room[shift:] = ft.reshape(-1)
    out = fb.sample_vt(room[shift:].view(ft.shape), torch.from_numpy(
        np.ascontiguousarray(inst.lidar2img)).to(device), inst.z, fb.grid_of(wl),
        (wl.img_h, wl.img_w))
    r, s, _ = oracle.run_instance(inst, "mean")
    assert_parity(out.cpu().numpy(), r, s, RTOL[dtype], f"{dtype} C={C} shift={shift}")
