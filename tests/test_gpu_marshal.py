"""The compiled marshalling and the Python one beneath it make the same calls: same results bit for bit, same errors, and
calls that the compiled one does not serve (views that are not contiguous, wrong types, CPU tensors) raise as before."""
import pytest

pytestmark = pytest.mark.gpu


def _step_args(io, nb=3, nd=40, nn=16, seed=0):
    import torch
    g = torch.Generator().manual_seed(seed)
    t = lambda *s, dt=torch.float32: torch.randn(s, generator=g).to(dt).cuda()
    return dict(h=t(nb, nd, nn), u_t=t(nb, nd, dt=io), delta_t=t(nb, nd, dt=io), A=-t(nd, nn).abs(), B_t=t(nb, nn, dt=io), C_t=t(nb, nn, dt=io),
                Dskip=t(nd), z_t=t(nb, nd, dt=io), delta_bias=t(nd), delta_softplus=True)


class _Nothing:
    """Serves no call."""
    def __getattr__(self, name):
        return lambda *a: None


@pytest.mark.parametrize("optional", [True, False])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_same_results(monkeypatch, io, optional):
    import torch
    from paper_2312_00752_amd import binding as B
    dt = torch.float32 if io == "f32" else torch.bfloat16
    code = B.SS_F32 if io == "f32" else B.SS_BF16
    nb, nd, nl, nn = 2, 70, 72, 16

    def calls():
        a = _step_args(dt)
        if not optional:
            a.update(Dskip=None, z_t=None, delta_bias=None)
        res = [B.ss_step(**a), a["h"]]
        g = torch.Generator().manual_seed(5)
        t = lambda *s, d=torch.float32: torch.randn(s, generator=g).to(d).cuda()
        s = dict(u=t(nb, nd, nl, d=dt), delta=t(nb, nd, nl, d=dt), A=-t(nd, nn).abs(), Bmat=t(nd, nn), Cmat=t(nb, nn, nl, d=dt))
        kw = dict(Dskip=t(nd), z=t(nb, nd, nl, d=dt), delta_bias=t(nd), h0=t(nb, nd, nn)) if optional else {}
        ws = torch.empty(B.ss_workspace_bytes(nb, nd, nl, nn, io_dtype=code, has_z=optional, b_fixed=True), dtype=torch.uint8, device="cuda")
        out, last = B.ss_scan_fwd(**s, delta_softplus=True, return_last_state=optional, workspace=ws, **kw)
        assert (last is not None) == optional
        res += [out] + ([last] if optional else [])
        grads = B.ss_scan_bwd(t(nb, nd, nl, d=dt), s["u"], s["delta"], s["A"], s["Bmat"], s["Cmat"], ws, delta_softplus=True,
                              want_dh0=optional, dh_last=t(nb, nd, nn) if optional else None, **kw)
        assert list(grads) == ["du", "ddelta", "dz", "dB", "dC", "dA", "dD", "ddelta_bias", "dh0"]
        res += [v for k, v in grads.items() if v is not None and k != "dC"]   # dC is added up by atomics
        assert all(grads[k].is_contiguous() for k in ("du", "ddelta")) and [k for k, v in grads.items() if v is None] == (
            [] if optional else ["dz", "dD", "ddelta_bias", "dh0"])
        torch.cuda.synchronize()
        return res

    served = calls()
    monkeypatch.setattr(B, "_native", _Nothing())
    for x, y in zip(served, calls()):
        assert torch.equal(x, y)


@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_same_layer_results(monkeypatch, io):
    import torch
    from paper_2312_00752_amd import binding as B
    dt = torch.float32 if io == "f32" else torch.bfloat16
    code = B.SS_F32 if io == "f32" else B.SS_BF16
    nb, nd, nl, nn, R, W = 2, 72, 40, 16, 8, 4

    def calls():
        g = torch.Generator().manual_seed(6)
        t = lambda *s, d=torch.float32: (0.3 * torch.randn(s, generator=g)).to(d).cuda()
        p = [t(nd, W), t(nd), t(R + 2 * nn, nd, d=dt), t(nd, R, d=dt), t(nd), -t(nd, nn).abs(), t(nd)]
        x, z = t(nb, nd, nl, d=dt), t(nb, nd, nl, d=dt)
        scratch = torch.empty(B.ss_layer_scratch_bytes(nb, nd, nl, nn, R, W, code, True), dtype=torch.uint8, device="cuda")
        saved = torch.empty(B.ss_layer_saved_bytes(nb, nd, nl, nn, R, W, code), dtype=torch.uint8, device="cuda")
        out = B.ss_layer_fwd(x, z, *p, scratch=scratch, saved=saved)
        grads = B.ss_layer_bwd(t(nb, nd, nl, d=dt), x, z, *p, scratch=scratch, saved=saved)
        assert list(grads) == ["dx", "dz", "dconv_w", "dconv_b", "dW_x", "dW_dt", "ddt_bias", "dA", "dD"]
        res = [out, grads["dz"], grads["ddt_bias"], grads["dA"], grads["dD"]]   # the others follow from sums by atomics
        out, h, win = B.ss_layer_fwd(x, z, *p, scratch=scratch, return_states=True)
        step = torch.empty(B.ss_layer_step_scratch_bytes(nb, nd, nn, R, code), dtype=torch.uint8, device="cuda")
        res += [out, h.clone(), win.clone(), B.ss_layer_step(h, win, t(nb, nd, d=dt), t(nb, nd, d=dt), *p, scratch=step), h, win]
        torch.cuda.synchronize()
        return res

    served = calls()
    monkeypatch.setattr(B, "_native", _Nothing())
    for x, y in zip(served, calls()):
        assert x.dtype == y.dtype and torch.equal(x, y)


def test_what_is_not_served(monkeypatch):
    import torch
    from paper_2312_00752_amd import binding as B
    for change, error in (({"u_t": lambda t: t.cpu()}, ValueError), ({"A": lambda t: t.t()}, ValueError), ({"h": lambda t: t.double()}, TypeError),
                          ({"B_t": lambda t: t[:, :8].contiguous()}, ValueError), ({"u_t": lambda t: t.half()}, TypeError)):
        a = _step_args(torch.float32)
        for k, f in change.items():
            a[k] = f(a[k])
        with pytest.raises(error):
            B.ss_step(**a)
    a = _step_args(torch.float32)
    base = torch.zeros(a["h"].numel() + 1, device="cuda")
    a["h"] = base[1:].view(a["h"].shape)   # off 16 bytes: the library's own error
    with pytest.raises(B.SsError) as e:
        B.ss_step(**a)
    assert e.value.code == B.SS_ERR_ALIGN
    # a subclass goes through the Python marshalling
    class Sub(torch.Tensor):
        pass
    a, b = _step_args(torch.float32), _step_args(torch.float32)
    b["u_t"] = b["u_t"].as_subclass(Sub)
    assert torch.equal(B.ss_step(**a), B.ss_step(**b).as_subclass(torch.Tensor))
    # under vmap a tensor has no memory of its own
    a = _step_args(torch.float32)
    with pytest.raises(RuntimeError):
        torch.vmap(lambda z: B.ss_step(**{**a, "z_t": z}))(a["z_t"][None].expand(2, -1, -1))
