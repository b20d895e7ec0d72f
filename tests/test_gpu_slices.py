"""Rows off eight steps in the kernels for complex state and time-invariant B / C: slices read in one access from inside the row, the
last one shifted into place; rows shorter than a slice, one step more and less, values next to the row that must not be used."""
import pytest

from tests import test_gpu_fixed_bc as gf
from tests import test_gpu_fixed_bc_grids as grids

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seqlen", [1, 2, 3, 4, 5, 7, 9, 15, 19, 20, 21, 31, 33, 65])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_every_remainder(io, seqlen):
    for bfix, cfix in gf.MODES:
        gf.test_fixed_bc_forward_and_backward(io, 2, seqlen, 66, 13, False, bfix, cfix)
    grids.test_complex(io, 2, seqlen, 3, False, False)
    grids.test_complex(io, 1, seqlen, 5, True, False)


@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_infinite_neighbours_stay_out(io):
    """Selective B of 13 steps with infinities in the next batch entry's rows, which lie behind the rows read here."""
    import torch
    from paper_2312_00752_amd import binding as B
    dt = torch.float32 if io == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(3)
    t = lambda *s, d=torch.float32: torch.randn(s, generator=g).to(d).cuda()
    nb, nd, nl, nn = 2, 5, 13, 16
    u, delta, Bm, A, C = t(nb, nd, nl, d=dt), t(nb, nd, nl, d=dt), t(nb, nn, nl, d=dt), -t(nd, nn).abs(), t(nd, nn)
    want, _ = B.ss_scan_fwd(u, delta, A, Bm, C, delta_softplus=True)
    u[1], Bm[1] = float("inf"), float("inf")
    got, _ = B.ss_scan_fwd(u, delta, A, Bm, C, delta_softplus=True)
    torch.cuda.synchronize()
    assert torch.equal(want[0], got[0]) and not torch.isfinite(got[1]).any()
