"""The gather-form backward writing a 16-bit gradient: bit for bit its float32
gradient rounded once (the form sums in a fixed order), over row widths of
each vector width, one and two rows per group, and odd channel counts."""
import numpy as np
import pytest

import synth
from test_gpu_parity import small, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    import paper_2607_10071_amd as m
    return m


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("C", [1, 6, 33, 64, 128, 300, 1024])
def test_gradient_in_the_features_type(fb, device, dtype, C):
    import torch
    inst = small(B=2, N=3, C=C, dtype=dtype, X=21, Y=23, Z=5)
    wl = inst.wl
    ft, l2i = to_dev(inst, device)
    g = torch.from_numpy(np.random.default_rng(C).standard_normal((wl.B, C, wl.X, wl.Y))
                         .astype(np.float32)).to(device)
    g[0, 0, :2] = 1e30   # overflows half
    args = (l2i, inst.z, fb.grid_of(wl), (wl.img_h, wl.img_w))
    ref = fb.sample_vt_backward(g, *args, ft.shape, wl.dtype).to(ft.dtype)
    x = ft.clone().requires_grad_(True)
    out = fb.sample_vt_autograd(x, *args)
    (got,) = torch.autograd.grad(out, [x], g)
    assert got.dtype == ft.dtype and got.shape == ft.shape
    assert torch.equal(got.view(torch.int16), ref.view(torch.int16))
    assert bool((ref != 0).any())
    # the scatter form's gradient still comes in the features' type
    out = fb.sample_vt_autograd(x, *args, method="scatter")
    assert torch.autograd.grad(out, [x], g)[0].dtype == ft.dtype


@pytest.mark.parametrize("C,dtype", [(32, "f32"), (80, "bf16"), (129, "f32"), (256, "f16")])
@pytest.mark.parametrize("Z", [3, 8, 37])
def test_shared_heights(fb, device, C, dtype, Z):
    """Small maps under a grid of many voxels: several wavefronts share a pixel
    group's heights where the workspace has room, one has them all otherwise.
    Both against the oracle, and the 16-bit gradient the float32 one rounded."""
    import torch
    from test_gpu_backward import assert_bwd_parity, oracle_backward
    inst = small(N=4, C=C, dtype=dtype, X=90, Y=70, Z=Z, half=40.0, img=(64, 176), stride=16)
    wl = inst.wl
    ft, l2i = to_dev(inst, device)
    g = np.random.default_rng(C + Z).standard_normal((wl.B, C, wl.X, wl.Y)).astype(np.float32)
    gt = torch.from_numpy(g).to(device)
    args = (l2i, inst.z, fb.grid_of(wl), (wl.img_h, wl.img_w))
    ref, scale, terms = oracle_backward(inst, g)
    shared = fb.sample_vt_backward(gt, *args, ft.shape, wl.dtype)
    need = fb.backward_workspace_size(ft.shape, wl.dtype, inst.z, fb.grid_of(wl),
                                      (wl.img_h, wl.img_w))
    ws = torch.empty(need, dtype=torch.uint8, device=device)
    alone = fb.sample_vt_backward(gt, *args, ft.shape, wl.dtype, workspace=ws)
    torch.cuda.synchronize()
    for what, got in (("shared", shared), ("alone", alone)):
        assert_bwd_parity(got.cpu().numpy(), ref, scale, terms, f"{what} C={C} Z={Z}")
    assert not torch.equal(shared, alone)   # sums in another order
    x = ft.clone().requires_grad_(True)
    (got,) = torch.autograd.grad(fb.sample_vt_autograd(x, *args), [x], gt)
    assert torch.equal(got, shared.to(ft.dtype))
