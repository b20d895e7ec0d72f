"""Time-invariant B / C with a workgroup per compute unit (256) and with more: the backward kernels built for one and
for two workgroups per unit, real and complex state, rows of whole 16-byte pieces and others, against the oracles."""
import numpy as np
import pytest

from oracle import complex_oracle as cx
from tests import test_gpu_complex as gc
from tests import test_gpu_fixed_bc as gf
from tests import util

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 256, 24, 3), ("bf16", 256, 21, 3), ("f32", 257, 21, 3), ("bf16", 129, 40, 66)]


@pytest.mark.parametrize("bfix,cfix", gf.MODES)
@pytest.mark.parametrize("io,batch,seqlen,dim", SHAPES)
def test_real(io, batch, seqlen, dim, bfix, cfix):
    gf.test_fixed_bc_forward_and_backward(io, batch, seqlen, dim, 16, False, bfix, cfix)


@pytest.mark.parametrize("bfix,cfix", gf.MODES)
@pytest.mark.parametrize("io,batch,seqlen,dim", SHAPES)
def test_complex(io, batch, seqlen, dim, bfix, cfix):
    import torch
    from paper_2312_00752_amd import binding as B
    dstate = 8
    w = gc._workload(io, batch, seqlen, dim, dstate, 700 + seqlen, True)
    del w["h0"], w["dh_last"]
    rng = np.random.default_rng(701)
    for name, fixed in (("B", bfix), ("C", cfix)):
        if fixed:
            w[name] = (rng.normal(size=(dim, dstate)) + 1j * rng.normal(size=(dim, dstate))).astype(np.complex64)
    g = gc._upload(w | {"h0": w["A"], "dh_last": w["A"]})   # the two are not used
    code = B.SS_BF16 if io == "bf16" else B.SS_F32
    ws = torch.empty(B.ss_workspace_bytes(batch, dim, seqlen, dstate, io_dtype=code, b_fixed=bfix, c_fixed=cfix,
                                          complex_state=True), dtype=torch.uint8, device="cuda")
    kw = dict(Dskip=g["Dskip"], z=g["z"], delta_bias=g["delta_bias"], delta_softplus=True, complex_state=True)
    args = (g["u"], g["delta"], g["A"], g["B"], g["C"])
    out, _ = B.ss_scan_fwd(*args, workspace=ws, **kw)
    grads = B.ss_scan_bwd(g["dout"], *args, ws, **kw)
    torch.cuda.synchronize()
    # The oracle has no time-invariant mode: channel by channel on broadcast copies.  A selective operand's gradient
    # is a sum over the channels.
    sel = {k: 0.0 for k in ("B", "C")}
    ref = {k: [] for k in ("out", "du", "ddelta", "dz", "dA", "dB", "dC", "dD", "dbias")}
    for d in range(dim):
        s = slice(d, d + 1)
        full = {k: np.broadcast_to(w[k][d][None, :, None], (batch, dstate, seqlen)) if w[k].ndim == 2 else w[k] for k in ("B", "C")}
        okw = dict(Dskip=w["Dskip"][s], z=w["z"][:, s], bias=w["delta_bias"][s], softplus=True)
        oargs = (w["u"][:, s], w["delta"][:, s], w["A"][s], full["B"], full["C"])
        ref["out"].append(cx.scan_fwd(*oargs, **okw)["out"])
        rb = cx.scan_bwd(*oargs, w["dout"][:, s], **okw)
        for k in ("B", "C"):
            ref["d" + k].append(rb["d" + k].sum(axis=(0, 2))[None])
            sel[k] = sel[k] + rb["d" + k]
        for k in ("du", "ddelta", "dz", "dA", "dD", "dbias"):
            ref[k].append(rb[k])
    cat = lambda k, axis: np.concatenate(ref[k], axis=axis)
    util.assert_close(out, cat("out", 1), io, "out")
    for k in ("du", "ddelta", "dz"):
        util.assert_close(grads[k], cat(k, 1), io, k)
    util.assert_close(grads["dA"], gc._pairs_last(cat("dA", 0)), io, "dA")
    util.assert_close(grads["dD"], cat("dD", 0), io, "dD")
    util.assert_close(grads["ddelta_bias"], cat("dbias", 0), io, "ddelta_bias")
    for k, fixed in (("B", bfix), ("C", cfix)):
        want = gc._pairs_last(cat("d" + k, 0)) if fixed else gc._pairs_before_time(sel[k])
        util.assert_close(grads["d" + k], want, io, "d" + k)
