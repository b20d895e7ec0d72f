"""Forward passes over whole rows in workgroups of eight waves (at most 256 row groups): numbers of 32-step chunks around the
four slots of their inputs, lengths of whole slices and others, the edges of a chunk, fewer states, the exact hold; what the backward
pass takes from them, whole and in segments (the sums of whose step sizes they leave); the last grid that they take and the
first that they do not; calls on both sides of the line."""
import numpy as np
import pytest

from paper_2312_00752_amd import workloads as wl
from tests import util
from tests import test_gpu_ragged

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("batch,seqlen,dim,dstate,zoh", [
    (1, 8, 64, 16, False), (2, 32, 70, 16, False), (1, 33, 64, 7, False), (1, 64, 3, 16, True), (1, 72, 66, 2, False), (2, 96, 64, 16, False),
    (1, 97, 40, 16, True), (1, 104, 130, 12, False), (1, 119, 64, 1, False), (3, 120, 65, 16, True), (1, 127, 64, 16, False),
    (48, 257, 250, 16, False), (40, 520, 256, 9, False), (64, 136, 193, 16, True), (56, 295, 256, 16, False)])
def test_whole_rows(io, batch, seqlen, dim, dstate, zoh):
    test_gpu_ragged.test_ragged_rows(io, batch, seqlen, dim, dstate, zoh)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("segments,batch,seqlen,dim,dstate,zoh", [
    (5, 96, 583, 65, 16, False), (5, 192, 584, 2, 7, False), (7, 192, 1283, 1, 16, True), (7, 144, 779, 3, 16, False), (7, 192, 1344, 2, 16, False),
    (5, 176, 777, 1, 4, False), (3, 160, 777, 2, 12, True)])
def test_sums_of_segments(io, segments, batch, seqlen, dim, dstate, zoh):
    """Whole forward, backward in several segments, the last of them shorter or as long: each reads the sums of the others' step sizes."""
    assert test_gpu_ragged._segments(batch, seqlen, dim, dstate) == segments and not util.in_segments(io, batch, seqlen, dim, dstate, zoh)
    test_gpu_ragged.test_ragged_rows(io, batch, seqlen, dim, dstate, zoh)


@pytest.mark.parametrize("groups", [256, 257])
@pytest.mark.parametrize("io,seqlen", [("f32", 136), ("bf16", 131)])
def test_last_grid(io, seqlen, groups):
    """Bare calls (no gate, no softplus, no skip, nothing lent) on both sides of the line."""
    import torch
    from oracle import ss_oracle as orc
    from paper_2312_00752_amd import binding as B
    w = wl.make_scan_inputs(groups, seqlen, 20, 16, io=io, seed=groups)
    w["delta"] = np.abs(w["delta"]) * 0.1
    if io == "bf16":
        w["delta"] = torch.from_numpy(w["delta"]).to(torch.bfloat16).float().numpy()
    g = util.upload(w)
    out, h_last = B.ss_scan_fwd(g["u"], g["delta"], g["A"], g["B"], g["C"], return_last_state=True)
    torch.cuda.synchronize()
    ref = orc.scan_fwd(w["u"], w["delta"], w["A"], w["B"], w["C"])
    util.assert_close(out, ref["out"], io, "out")
    util.assert_close(h_last, ref["h_last"], io, "h_last")


# with few states the four-wave kernels are done sooner, and short segments of the exact hold cost less than they are modelled to
@pytest.mark.parametrize("io,groups,seqlen,dstate,zoh", [
    ("bf16", 136, 3072, 4, False), ("bf16", 136, 3072, 8, False), ("f32", 1, 192, 16, True), ("bf16", 8, 192, 3, True), ("f32", 80, 320, 16, True),
    ("f32", 80, 320, 4, False), ("bf16", 1, 2048, 16, False)])
def test_faster_in_segments(io, groups, seqlen, dstate, zoh):
    assert util.in_segments(io, 1, seqlen, 64 * groups, dstate, zoh)


@pytest.mark.parametrize("io,groups,seqlen,dstate,zoh", [
    ("bf16", 136, 3072, 16, False), ("bf16", 160, 1536, 4, False), ("bf16", 160, 1536, 8, False), ("f32", 1, 192, 16, False), ("f32", 144, 320, 16, True),
    ("f32", 104, 320, 4, False)])
def test_faster_whole(io, groups, seqlen, dstate, zoh):
    assert not util.in_segments(io, 1, seqlen, 64 * groups, dstate, zoh)
