"""Rows of 2^23 steps and more, whose 64-row tiles do not fit 31-bit offsets: the kernels that address every row on its
own and read B and C from the repacked copy, with a split sequence, forward and backward, against the oracle."""
import numpy as np
import pytest

from paper_2312_00752_amd import workloads as wl
from tests import util
from tests.test_gpu_bwd import GRADS, ORACLE_NAME

pytestmark = pytest.mark.gpu

LONG = 1 << 23   # 64 rows of as many floats: 2^31 bytes


@pytest.mark.parametrize("io,seqlen,dim,dstate,zoh", [("f32", LONG, 2, 2, False), ("bf16", LONG + 5, 1, 3, False), ("f32", LONG + 3, 1, 2, True)])
def test_long_rows(io, seqlen, dim, dstate, zoh):
    import torch
    from oracle import ss_oracle as orc
    from paper_2312_00752_amd import binding as B
    w = wl.make_scan_inputs(1, seqlen, dim, dstate, io=io, seed=23)
    rng = np.random.default_rng(24)
    w["h0"] = rng.normal(size=(1, dim, dstate)).astype(np.float32)
    w["dh_last"] = rng.normal(size=(1, dim, dstate)).astype(np.float32)
    g = util.upload(w)
    ws = torch.empty(B.ss_workspace_bytes(1, dim, seqlen, dstate, io_dtype=B.SS_BF16 if io == "bf16" else B.SS_F32),
                     dtype=torch.uint8, device="cuda")
    kw = dict(Dskip=g["Dskip"], z=g["z"], delta_bias=g["delta_bias"], h0=g["h0"], delta_softplus=True, exact_zoh=zoh)
    args = (g["u"], g["delta"], g["A"], g["B"], g["C"])
    out, h_last = B.ss_scan_fwd(*args, return_last_state=True, workspace=ws, **kw)
    grads = B.ss_scan_bwd(g["dout"], *args, ws, dh_last=g["dh_last"], want_dh0=True, **kw)
    torch.cuda.synchronize()
    okw = dict(Dskip=w["Dskip"], z=w["z"], bias=w["delta_bias"], h0=w["h0"], softplus=True, exact_zoh=zoh, nthreads=dim)
    oargs = (w["u"], w["delta"], w["A"], w["B"], w["C"])
    ref = orc.scan_fwd(*oargs, **okw)
    util.assert_close(out, ref["out"], io, "out")
    util.assert_close(h_last, ref["h_last"], io, "h_last")
    ref = orc.scan_bwd(*oargs, w["dout"], dh_last=w["dh_last"], **okw)
    for k in GRADS:
        util.assert_close(grads[k], ref[ORACLE_NAME.get(k, k)], io, k)
