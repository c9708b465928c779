"""The phase-clock tool: a log without records is an error (CPU), and both of
its runs record every wavefront of the kernels that have the clock (GPU), also
in a process that has called the operators through the plain library."""
import numpy as np
import pytest

import synth
from paper_2607_10071_amd import phases


@pytest.mark.parametrize("table", [phases.phase_table, phases.sca_backward_table])
def test_a_log_without_records_is_an_error(table):
    with pytest.raises(RuntimeError, match="no wavefront"):
        table(np.zeros((8, phases.SLOTS), np.int64))


@pytest.mark.gpu
def test_forward_clock(device):
    import paper_2607_10071_amd as fb
    import torch

    wl = synth.config("tiny")
    inst = synth.make_workload(wl)
    feats = synth.to_storage(inst.features, wl.dtype).to(device)
    l2i = torch.from_numpy(np.ascontiguousarray(inst.lidar2img)).to(device)
    plain = fb._lib()
    fb.sample_vt(feats, l2i, inst.z, fb.grid_of(wl), (wl.img_h, wl.img_w))
    (r,) = phases.run(["tiny"], calls=1, device=device)
    assert r["waves"] == r["launch"]["workgroups"] * (r["launch"]["threads"] // 64)
    assert r["outputs_bitwise_equal"]
    assert fb._lib() is plain


@pytest.mark.gpu
def test_sca_backward_clock(device):
    (r,) = phases.run_sca_backward([8], calls=1, device=device)
    assert r["waves"] == r["launch"]["workgroups"] * (r["launch"]["threads"] // 64)
    assert abs(sum(s["share"] for s in r["steps_us_per_wave"].values()) - 1.0) < 0.01
