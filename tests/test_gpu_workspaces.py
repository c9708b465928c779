"""Device workspaces of the backwards: how much of a caller's own is used."""
import ctypes

import numpy as np
import pytest

import synth
import test_gpu_backward as tb
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    import paper_2607_10071_amd as m
    return m


class VT:
    """A backward on small maps under many voxels, where heights are shared by
    several wavefronts if the workspace has the room."""

    def __init__(self, fb, device):
        import torch
        wl = tp.small(C=128, X=200, Y=200, half=50.0, Z=8).wl.with_(H=16, W=44)
        self.inst = synth.make_workload(wl)
        self.g = tb._grad_out(wl)
        self.grid, self.img = fb.grid_of(wl), (wl.img_h, wl.img_w)
        self.shape, self.dtype = self.inst.features.shape, wl.dtype
        self.gt = torch.from_numpy(self.g).to(device)
        self.l2i = torch.from_numpy(np.ascontiguousarray(self.inst.lidar2img)).to(device)
        self.need = fb.backward_workspace_size(self.shape, wl.dtype, self.inst.z, self.grid,
                                               self.img)
        out = ctypes.c_uint64()
        f, g, zb = fb._packed(self.shape, fb.DTYPE_CODES[wl.dtype], 0, self.img, self.grid,
                              fb._z_array(self.inst.z), "mean")
        assert fb._packed_call("flashbev_backward_workspace_best", "PPPP")(
            f, g, zb, ctypes.byref(out)) == 0
        self.best = out.value
        assert self.best > self.need
        self.args = (self.gt, self.l2i, self.inst.z, self.grid, self.img, self.shape, wl.dtype)

    def check(self, grad, what):
        ref, scale, terms = tb.oracle_backward(self.inst, self.g)
        tb.assert_bwd_parity(grad.float().cpu().numpy(), ref, scale, terms, what)


def test_a_larger_workspace_is_used_up_to_the_minimum(fb, device):
    """flashbev_sample_vt_backward_ws touches the minimum only: an arena may
    hold the gradient behind it, and the sums' order does not depend on its
    size.  The same for sample_vt_backward's ``workspace``."""
    import torch
    c = VT(fb, device)
    n = int(np.prod(c.shape))
    arena = torch.full((c.best + 4 * n,), 255, dtype=torch.uint8, device=device)
    grad = arena[c.need:c.need + 4 * n].view(torch.float32).view(c.shape)
    rc = fb.sample_vt_backward_ws_raw(c.shape, c.dtype, c.l2i.data_ptr(), c.inst.z, c.grid, c.img,
                                      c.gt.data_ptr(), grad.data_ptr(), arena.data_ptr(),
                                      arena.numel(), stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0, fb.status_string(rc)
    c.check(grad, "arena")
    assert bool((arena[c.need + 4 * n:] == 255).all())
    least = torch.empty(c.need, dtype=torch.uint8, device=device)
    a = fb.sample_vt_backward(*c.args, workspace=least)
    assert torch.equal(a, grad)
    grad.fill_(7.0)
    b = fb.sample_vt_backward(*c.args, grad_features=grad, workspace=arena)
    assert torch.equal(a, b)
