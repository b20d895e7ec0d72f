"""A step size that is not a number stays one in every kernel: the results that depend on it are NaN and no others, forward,
backward (whole and split sequences, odd lengths, exact zero-order hold, general kernels) and one token at a time, as in the oracle."""
import numpy as np
import pytest

from oracle import ss_oracle as orc
from paper_2312_00752_amd import workloads as wl
from tests import util
from tests.test_gpu_bwd import GRADS, ORACLE_NAME

pytestmark = pytest.mark.gpu


def _same(got, ref, io, name):
    """NaN in the same places, and close everywhere else."""
    import torch
    ref = np.asarray(ref, np.float64)
    nan = np.isnan(ref)
    where = torch.from_numpy(nan).to(got.device)
    assert torch.equal(torch.isnan(got), where), (name, int(torch.isnan(got).sum()), int(nan.sum()))
    if not nan.all():
        util.assert_close(torch.where(where, torch.zeros_like(got), got), np.where(nan, 0.0, ref), io, name)


@pytest.mark.parametrize("io,batch,seqlen,dim,dstate,zoh", [
    ("f32", 2, 200, 70, 16, False), ("bf16", 2, 200, 70, 16, False), ("bf16", 2, 203, 70, 16, False), ("bf16", 1, 136, 64, 4, False),
    ("f32", 2, 200, 70, 8, True), ("f32", 2, 72, 9, 20, False),
    ("f32", 1, 4096, 64, 16, False), ("bf16", 1, 4099, 70, 8, False), ("bf16", 1, 4096, 64, 16, True)])   # split
def test_scan(io, batch, seqlen, dim, dstate, zoh):
    import torch
    from paper_2312_00752_amd import binding as B
    w = wl.make_scan_inputs(batch, seqlen, dim, dstate, io=io, seed=300 + seqlen)
    w["delta"][0, dim // 2, seqlen // 2] = np.nan
    g = util.upload(w)
    code = B.SS_BF16 if io == "bf16" else B.SS_F32
    ws = torch.empty(B.ss_workspace_bytes(batch, dim, seqlen, dstate, io_dtype=code), dtype=torch.uint8, device="cuda")
    kw = dict(Dskip=g["Dskip"], z=g["z"], delta_bias=g["delta_bias"], delta_softplus=True, exact_zoh=zoh)
    out, h_last = B.ss_scan_fwd(g["u"], g["delta"], g["A"], g["B"], g["C"], return_last_state=True, workspace=ws, **kw)
    grads = B.ss_scan_bwd(g["dout"], g["u"], g["delta"], g["A"], g["B"], g["C"], ws, **kw)
    torch.cuda.synchronize()
    okw = dict(Dskip=w["Dskip"], z=w["z"], bias=w["delta_bias"], softplus=True, exact_zoh=zoh)
    ref_f = orc.scan_fwd(w["u"], w["delta"], w["A"], w["B"], w["C"], **okw)
    ref_b = orc.scan_bwd(w["u"], w["delta"], w["A"], w["B"], w["C"], w["dout"], **okw)
    _same(out, ref_f["out"], io, "out")
    _same(h_last, ref_f["h_last"], io, "h_last")
    for k in GRADS:
        if grads.get(k) is not None:
            _same(grads[k], ref_b[ORACLE_NAME.get(k, k)], io, k)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("batch,dim,dstate", [(3, 70, 16), (3, 70, 5), (70, 64, 16)])
def test_step(io, batch, dim, dstate):
    import torch
    from paper_2312_00752_amd import binding as B
    w = wl.make_step_inputs(batch, dim, dstate, 1, io=io, seed=7)
    t = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in w.items() if isinstance(v, np.ndarray)}
    bf = torch.bfloat16 if io == "bf16" else torch.float32
    one = lambda k: t[k][0].contiguous().to(bf)
    delta = one("delta")
    delta[1, 3] = float("nan")
    h = torch.zeros(batch, dim, dstate, device="cuda")
    out = B.ss_step(h, one("u"), delta, t["A"], one("B"), one("C"), Dskip=t["Dskip"], z_t=one("z"), delta_bias=t["delta_bias"],
                    delta_softplus=True)
    torch.cuda.synchronize()
    where = torch.zeros(batch, dim, dtype=torch.bool, device="cuda")
    where[1, 3] = True
    assert torch.equal(torch.isnan(out), where)
    assert torch.equal(torch.isnan(h), where[:, :, None].expand_as(h))


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("batch", [2, 6])
def test_layer_token(io, batch):
    """Through the projections: a channel of the step-size weights without a value."""
    import torch
    from paper_2312_00752_amd import binding as B
    dim, dstate, rank = 72, 16, 8
    w = wl.make_layer_inputs(batch, 1, dim, dstate, io, seed=8, rank=rank)
    bf = torch.bfloat16 if io == "bf16" else torch.float32
    t = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in w.items() if isinstance(v, np.ndarray)}
    weights = [t["conv_w"], t["conv_b"], t["W_x"].to(bf), t["W_dt"].to(bf), t["dt_bias"], t["A"], t["Dskip"]]
    weights[3][5] = float("nan")
    code = B.SS_BF16 if io == "bf16" else B.SS_F32
    scratch = torch.empty(B.ss_layer_step_scratch_bytes(batch, dim, dstate, rank, code), dtype=torch.uint8, device="cuda")
    h, cs = torch.zeros(batch, dim, dstate, device="cuda"), torch.zeros(batch, dim, 3, device="cuda", dtype=bf)
    x, z = (t[k][..., 0].contiguous().to(bf) for k in ("x", "z"))
    out = B.ss_layer_step(h, cs, x, z, *weights, scratch=scratch)
    torch.cuda.synchronize()
    where = torch.zeros(batch, dim, dtype=torch.bool, device="cuda")
    where[:, 5] = True
    assert torch.equal(torch.isnan(out), where)
    assert torch.equal(torch.isnan(h), where[:, :, None].expand_as(h))
