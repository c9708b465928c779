"""Device workspaces of the backwards: how much of a caller's own is used, what
happens where the device has no room for one, and which stream holds it."""
import ctypes

import numpy as np
import pytest

import oracle
import synth
import test_gpu_backward as tb
import test_gpu_parity as tp
import test_gpu_sca_backward as ts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    import paper_2607_10071_amd as m
    return m


@pytest.fixture
def room(monkeypatch):
    """room(n): from here on torch.empty raises OutOfMemoryError where more
    than n bytes of its tensors would be alive."""
    import torch
    import weakref

    kept = torch.empty
    live = [0]

    def limit(n):
        def empty(*a, **kw):
            t = kept(*a, **kw)
            size = t.numel() * t.element_size()
            if live[0] + size > n:
                raise torch.cuda.OutOfMemoryError(f"{live[0]} + {size} > {n} bytes")
            live[0] += size
            weakref.finalize(t, lambda: live.__setitem__(0, live[0] - size))
            return t
        monkeypatch.setattr(torch, "empty", empty)
    return limit


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


class SCA:
    """A FlashSCA backward of enough points for the binned form."""

    def __init__(self, fb, device, dtype="f32"):
        import torch
        self.inst = ts.small(27, levels=((29, 50), (15, 25)), C=256, heads=8, P=8, Z=4, X=64, Y=64,
                             x_min=-32.0, dx=1.0, y_min=-32.0, dy=1.0, dtype=dtype)
        wl = self.wl = self.inst.wl
        assert wl.B * wl.Q * wl.heads * wl.L * wl.P >= fb.SCA_BINNED_MIN_POINTS
        self.v, self.l2i, self.off, self.lg = ts._dev(self.inst, device)
        self.g = ts._g(wl)
        self.gt = torch.from_numpy(self.g).to(device)
        self.args = (self.v, self.l2i, self.inst.z, fb.grid_of(wl), (wl.img_h, wl.img_w),
                     wl.levels, wl.heads, self.off, self.lg, self.gt)
        st = fb._sca_structs(self.v.shape, fb._dtype_code(self.v), 0, wl.heads, wl.levels,
                             (wl.img_h, wl.img_w), fb.grid_of(wl), fb._z_array(self.inst.z), "mean")
        self.need = fb._sca_workspace_bytes(*map(ctypes.byref, st), wl.P, "auto", self.lg.numel(),
                                            True)
        assert self.need > 0

    def check(self, r, what):
        ref = oracle.sca_backward_instance(self.inst, self.g, "mean")
        ts.assert_bwd_parity({k: t.cpu().numpy() for k, t in r.items()}, ref, self.wl, what)


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


@pytest.mark.parametrize("call", ["plain", "prepared", "bf16"])
def test_gather_backward_without_room_for_shared_heights(fb, device, room, call):
    """Memory for the gradient and the smallest workspace is enough."""
    import torch
    c = VT(fb, device)
    grad = torch.empty(c.shape, device=device)
    size = grad.numel() * 4
    assert c.best > c.need + size
    if call == "prepared":
        room(c.need)
        fb.prepare_sample_vt_backward(*c.args, grad)()
    elif call == "plain":
        room(c.need + size)
        grad = fb.sample_vt_backward(*c.args)
    else:
        least = torch.empty(c.need, dtype=torch.uint8, device=device)
        want = fb.sample_vt_backward(*c.args[:6], "bf16", workspace=least).bfloat16()
        room(c.need + size // 2)
        grad = fb._sample_vt_backward(*c.args[:6], "bf16", None, "mean", None, "gather", None,
                                      torch.bfloat16)
    torch.cuda.synchronize()
    if call == "bf16":
        assert grad.dtype == torch.bfloat16
        assert torch.equal(grad, want)
    else:
        c.check(grad, f"no room, {call}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sca_backward_without_room_for_a_workspace(fb, device, room, dtype):
    """Memory for the float32 gradients alone is enough (the scatter form)."""
    import torch
    c = SCA(fb, device, dtype)
    room(max(c.need, 4 * (c.v.numel() + c.off.numel() + c.lg.numel())))
    r = fb._sca_backward(*c.args, None, None, None, ("value", "offsets", "logits"), "mean", None,
                         "auto", c.v.dtype)
    torch.cuda.synchronize()
    assert r["value"].dtype == c.v.dtype
    if dtype == "f32":
        c.check(r, "no room")


@pytest.mark.parametrize("op", ["vt", "vt prepared", "sca", "sca prepared"])
def test_a_workspace_belongs_to_the_stream_of_its_call(fb, device, op, monkeypatch):
    """A call on another stream than the current one: its workspace is neither
    a block that the current stream's work may still be using nor one that the
    current stream is given next, when the other may still be using it."""
    import torch
    c = SCA(fb, device) if op.startswith("sca") else VT(fb, device)
    size = c.need if op.startswith("sca") else c.best
    out = [torch.empty(t, device=device) for t in
           ((c.v.shape, c.off.shape, c.lg.shape) if op == "sca prepared" else (c.shape,) if op.startswith("vt") else ())]
    s = torch.cuda.Stream(device)
    kept, seen = torch.empty, []

    def empty(*a, **kw):
        t = kept(*a, **kw)
        if kw.get("dtype") is torch.uint8:
            seen.append(t.data_ptr())
        return t

    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    block = torch.empty(size, dtype=torch.uint8, device=device)
    freed = block.data_ptr()
    del block   # the current stream's pool holds a block of the workspace's size
    with monkeypatch.context() as m:
        m.setattr(torch, "empty", empty)
        if op == "vt":
            r = fb.sample_vt_backward(*c.args, grad_features=out[0], stream=s)
        elif op == "sca":
            r = fb.sca_backward(*c.args, stream=s)
        elif op == "vt prepared":
            r = out[0]
            fb.prepare_sample_vt_backward(*c.args, r, stream=s)()
        else:
            r = dict(zip(("value", "offsets", "logits"), out))
            fb.prepare_sca_backward(*c.args, *out, stream=s)()
    assert len(seen) == 1 and seen[0] != freed
    after = [torch.empty(size, dtype=torch.uint8, device=device) for _ in range(2)]
    assert seen[0] not in [t.data_ptr() for t in after]
    s.synchronize()
    c.check(r, op)


@pytest.mark.parametrize("op", ["vt", "sca"])
def test_a_workspace_on_the_default_stream_by_its_address(fb, device, op):
    """stream=0 (the default stream's address) from within another stream: the
    workspace comes from the default stream's pool, which is given it again."""
    import torch
    c = SCA(fb, device) if op == "sca" else VT(fb, device)
    size = c.need if op == "sca" else c.best
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    block = torch.empty(size, dtype=torch.uint8, device=device)
    mine = block.data_ptr()
    del block   # in the default stream's pool, next in line for this size
    seen = []
    kept = fb._workspace

    def workspace(*a):
        t = kept(*a)
        seen.append(t.data_ptr())
        return t

    side = torch.cuda.Stream(device)
    side.wait_stream(torch.cuda.current_stream(device))
    fb._workspace = workspace
    try:
        with torch.cuda.stream(side):
            r = fb.sca_backward(*c.args, stream=0) if op == "sca" else \
                fb.sample_vt_backward(*c.args, stream=0)
    finally:
        fb._workspace = kept
    assert seen == [mine]
    torch.cuda.synchronize()
    c.check(r, f"{op}, stream 0")
