"""Rows that are not whole 16-byte pieces: the edges of slices, chunks, blocks and segments, forward and backward,
with NaN around every input (nothing outside a row may enter a result) and a pattern around every output
(nothing outside a row may be written)."""
import numpy as np
import pytest

from paper_2312_00752_amd import workloads as wl
from tests import util
from tests.test_gpu_bwd import GRADS, ORACLE_NAME

pytestmark = pytest.mark.gpu

PAD = 64   # elements before and after a tensor
PATTERN = 7.0


def _guarded(shape, dtype, fill):
    import torch
    n = int(np.prod(shape))
    pool = torch.full((n + 2 * PAD,), fill, dtype=dtype, device="cuda")
    return pool, pool[PAD: PAD + n].view(shape)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("batch,seqlen,dim,dstate,zoh", [
    (2, 8, 65, 16, False), (1, 9, 3, 16, False), (2, 15, 70, 5, False), (1, 17, 64, 3, False), (1, 31, 1, 16, True),
    (2, 33, 33, 16, False), (1, 47, 100, 9, True), (2, 63, 64, 20, False), (1, 65, 129, 16, False),
    (1, 95, 66, 16, False), (1, 130, 64, 7, False),
    # split sequences: the last segment ends inside a slice, a block, a chunk
    (1, 2049, 40, 16, False), (1, 2055, 64, 4, False), (1, 2079, 70, 16, True), (1, 4091, 30, 18, False)])
def test_ragged_rows(io, batch, seqlen, dim, dstate, zoh):
    import torch
    from oracle import ss_oracle as orc
    from paper_2312_00752_amd import binding as B
    w = wl.make_scan_inputs(batch, seqlen, dim, dstate, io=io, seed=400 + seqlen)
    rng = np.random.default_rng(seqlen)
    w["h0"] = rng.normal(size=(batch, dim, dstate)).astype(np.float32)
    w["dh_last"] = rng.normal(size=(batch, dim, dstate)).astype(np.float32)
    g = util.upload(w)
    for k in ("u", "delta", "z", "B", "C", "dout"):
        pool, view = _guarded(g[k].shape, g[k].dtype, float("nan"))
        view.copy_(g[k])
        g[k] = view
    tio = g["u"].dtype
    outs = {k: _guarded((batch, dim, seqlen), tio, PATTERN) for k in ("out", "du", "ddelta", "dz")}
    outs.update({k: _guarded((batch, dstate, seqlen), torch.float32, PATTERN) for k in ("dB", "dC")})
    f32 = dict(dtype=torch.float32, device="cuda")
    grads = {k: outs[k][1] for k in ("du", "ddelta", "dz", "dB", "dC")}
    grads.update(dA=torch.empty((dim, dstate), **f32), dD=torch.empty(dim, **f32), ddelta_bias=torch.empty(dim, **f32),
                 dh0=torch.empty((batch, dim, dstate), **f32))
    code = B.SS_BF16 if io == "bf16" else B.SS_F32
    ws = torch.full((B.ss_workspace_bytes(batch, dim, seqlen, dstate, io_dtype=code),), 0x7f, dtype=torch.uint8, device="cuda")
    kw = dict(Dskip=g["Dskip"], z=g["z"], delta_bias=g["delta_bias"], h0=g["h0"], delta_softplus=True, exact_zoh=zoh)
    args = (g["u"], g["delta"], g["A"], g["B"], g["C"])
    out, h_last = B.ss_scan_fwd(*args, return_last_state=True, workspace=ws, out=outs["out"][1], **kw)
    B.ss_scan_bwd(g["dout"], *args, ws, dh_last=g["dh_last"], want_dh0=True, grads=grads, **kw)
    torch.cuda.synchronize()
    okw = dict(Dskip=w["Dskip"], z=w["z"], bias=w["delta_bias"], h0=w["h0"], softplus=True, exact_zoh=zoh)
    oargs = (w["u"], w["delta"], w["A"], w["B"], w["C"])
    rf = orc.scan_fwd(*oargs, **okw)
    rb = orc.scan_bwd(*oargs, w["dout"], dh_last=w["dh_last"], **okw)
    exact = dstate <= 16   # more states round the running sum to the io type between passes
    util.assert_close(out, rf["out"], io, "out", exact_inputs=exact)
    util.assert_close(h_last, rf["h_last"], io, "h_last", exact_inputs=exact)
    for k in GRADS:
        util.assert_close(grads[k], rb[ORACLE_NAME.get(k, k)], io, k, exact_inputs=exact)
    for k, (pool, view) in outs.items():
        assert bool((pool[:PAD] == PATTERN).all()) and bool((pool[PAD + view.numel():] == PATTERN).all()), k


def _segments(batch, seqlen, dim, dstate):
    """How many segments a call is split into, from the size of its scratch: per segment 17 floats a row, and
    B and C once in whole 32-step chunks (each block rounded up to 256 bytes)."""
    from paper_2312_00752_amd import binding as B
    up = lambda n: (n + 255) // 256 * 256
    rows = batch * dim
    bc = up(batch * ((dstate + 15) // 16 * 16) * ((seqlen + 31) // 32 * 32) * 2 * 4)
    left = B.ss_workspace_bytes(batch, dim, seqlen, dstate, for_backward=False, io_dtype=B.SS_F32, has_z=False) - bc
    return next(n for n in range(1, 4097) if left == (n > 1) * (up(n * rows * 64) + up(n * rows * 4)))


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("segments,batch,seqlen,dim,dstate,zoh", [
    (2, 1, 193, 70, 16, False), (2, 1, 197, 40, 4, False), (3, 1, 257, 65, 16, True), (5, 1, 513, 40, 3, False),
    (6, 2, 699, 33, 18, False), (9, 1, 1025, 70, 16, True), (16, 1, 1985, 70, 16, False), (16, 3, 1937, 130, 7, False)])
def test_ragged_rows_in_few_segments(io, segments, batch, seqlen, dim, dstate, zoh):
    """Up to sixteen segments every workgroup works its incoming state out itself: one, several and all fifteen aggregates.  (The
    forward pass of the shapes in two or three segments goes over whole rows; those below are its own.)"""
    assert _segments(batch, seqlen, dim, dstate) == segments
    test_ragged_rows(io, batch, seqlen, dim, dstate, zoh)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("segments,batch,seqlen,dim,dstate,zoh", [
    # more than 16 states, the exact hold in short segments, more than 256 row groups
    (2, 1, 193, 70, 18, False), (2, 1, 200, 40, 20, False), (3, 1, 192, 66, 16, True), (3, 1, 192, 40, 5, True),
    (3, 320, 904, 2, 16, False), (3, 320, 907, 1, 7, False), (3, 320, 905, 2, 3, True)])
def test_few_segments_of_the_forward_pass(io, segments, batch, seqlen, dim, dstate, zoh):
    assert _segments(batch, seqlen, dim, dstate) == segments and util.in_segments(io, batch, seqlen, dim, dstate, zoh)
    test_ragged_rows(io, batch, seqlen, dim, dstate, zoh)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("batch,seqlen,dim,dstate,zoh", [
    (257, 8, 2, 16, False), (257, 9, 2, 3, False), (130, 33, 65, 16, False), (257, 40, 3, 4, False), (257, 47, 1, 7, True), (257, 63, 2, 16, False),
    (257, 88, 2, 6, True), (257, 95, 3, 2, False), (257, 97, 1, 8, False), (260, 104, 2, 16, True), (129, 123, 66, 13, False)])
def test_rows_of_more_groups_than_units(io, batch, seqlen, dim, dstate, zoh):
    """More than 256 row groups, unsplit: the four-wave forward kernel with one, two and four slots per lane and the exact hold, on and
    off eight steps, ending in an even and in an odd chunk."""
    test_ragged_rows(io, batch, seqlen, dim, dstate, zoh)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("batch,dim,seqlen,width", [(2, 3, 9, 4), (1, 2, 11, 3), (3, 5, 15, 2), (1, 4, 509, 4), (2, 3, 517, 4),
                                                    (1, 2, 1021, 1)])
def test_ragged_convolution(io, batch, dim, seqlen, width):
    import torch
    from oracle import conv_oracle as cv
    from paper_2312_00752_amd import binding as B
    w = wl.make_conv_inputs(batch, dim, seqlen, width, io, seed=seqlen)
    tio = torch.bfloat16 if io == "bf16" else torch.float32
    g = {}
    for k in ("x", "dout"):
        pool, g[k] = _guarded(w[k].shape, tio, float("nan"))
        g[k].copy_(torch.from_numpy(w[k]))
    wt, bias = torch.from_numpy(w["w"]).cuda(), torch.from_numpy(w["bias"]).cuda()
    pool, out = _guarded(w["x"].shape, tio, PATTERN)
    B.ss_conv_fwd(g["x"], wt, bias, out=out)
    grads = B.ss_conv_bwd(g["dout"], g["x"], wt, bias)
    torch.cuda.synchronize()
    ref, rg = cv.conv_fwd(w["x"], w["w"], w["bias"], None, True), cv.conv_bwd(w["x"], w["w"], w["dout"], w["bias"], None, True)
    util.assert_close(out, ref["out"], io, "out")
    for k in ("dx", "dw", "dbias"):
        util.assert_close(grads[k], rg[k], io, k)
    assert bool((pool[:PAD] == PATTERN).all()) and bool((pool[PAD + out.numel():] == PATTERN).all())
