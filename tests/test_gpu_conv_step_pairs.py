"""One token of the convolution with two channels per thread (width 4, an even number of channels) and with one, from any element on,
against the step in float64; nothing around the tensors changes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("nb,nd,width", [(1, 2, 4), (3, 130, 4), (2, 131, 4), (5, 64, 3), (257, 4, 4)])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_step(io, nb, nd, width, off):
    import torch
    from paper_2312_00752_amd import binding as B
    dt = torch.float32 if io == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(nd + off)

    def at(*shape, d=dt):   # from element `off` of a larger buffer
        n = 1
        for k in shape:
            n *= k
        buf = torch.full((n + off + 9,), 77.0, dtype=d, device="cuda")
        buf[off:off + n] = torch.randn(n, generator=g).to(d).cuda()
        return buf, buf[off:off + n].view(shape)

    (bs, state), (bx, x), (bw, w), (bb, bias), (bo, out) = at(nb, nd, width - 1), at(nb, nd), at(nd, width, d=torch.float32), at(nd, d=torch.float32), at(nb, nd)
    for use_bias, silu in ((True, True), (False, False)):
        win = torch.cat([state.double().cpu(), x.double().cpu()[:, :, None]], dim=2)
        v = (win * w.double().cpu()).sum(2) + (bias.double().cpu() if use_bias else 0.0)
        ref = v * torch.sigmoid(v) if silu else v
        size = (win * w.double().cpu()).abs().sum(2) + (bias.double().cpu().abs() if use_bias else 0.0)
        B.ss_conv_step(state, x, w, bias if use_bias else None, silu=silu, out_t=out)
        torch.cuda.synchronize()
        # four float32 roundings of sums bounded by `size`, a sigmoid to 1e-6 of its value (its argument's rounding included), the io rounding
        bound = 4 * 2.0 ** -24 * size * 1.2 + 4e-6 * (ref.abs() + size) + (2.0 ** -8 * ref.abs() if io == "bf16" else 0.0)
        assert ((out.double().cpu() - ref).abs() <= bound).all()
        assert torch.equal(state.double().cpu(), win[:, :, 1:])
    for buf, t in ((bs, state), (bx, x), (bo, out)):
        assert (buf[:off] == 77.0).all() and (buf[off + t.numel():] == 77.0).all()
