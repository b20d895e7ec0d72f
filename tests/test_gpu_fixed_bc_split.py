"""Time-invariant B / C with the sequence split across workgroups: the aggregate passes and the partial sums per
segment, real, exact zero-order hold and complex, whole slices and others, more than 16 states, against the oracles.  Every call
here is cut."""
import pytest

from paper_2312_00752_amd import binding as B
from tests import test_gpu_fixed_bc as gf
from tests import test_gpu_fixed_bc_grids as grids
from tests.test_split_plan_cpu import segments

pytestmark = pytest.mark.gpu

# few rows: cut into segments of 64 steps and up, the last one short, the carry inside (16) and beyond (17) one batch
REAL = [("f32", 1, 331, 70, 16, False), ("bf16", 2, 1032, 65, 9, False), ("bf16", 1, 2049, 30, 16, True), ("f32", 1, 456, 40, 24, False),
        ("f32", 2, 1152, 64, 16, True)]
COMPLEX = [("f32", 1, 264, 3), ("bf16", 2, 331, 4)]
# more than one workgroup per compute unit after the cut: the backward kernels that leave room for two
MANY = [("f32", 100, 512, 1), ("bf16", 100, 512, 2), ("f32", 120, 331, 2), ("bf16", 120, 331, 1)]


def _segments(io, batch, seqlen, dim, dstate, bfix, cfix, more=0):
    import torch  # noqa: F401  (before the library: both bring a HIP runtime, and the library's launches need torch's)
    return segments(batch, seqlen, dim, B.SS_BF16 if io == "bf16" else B.SS_F32, B.SS_B_FIXED * bfix | B.SS_C_FIXED * cfix | more, dstate)


@pytest.mark.parametrize("bfix,cfix", gf.MODES)
@pytest.mark.parametrize("io,batch,seqlen,dim,dstate,zoh", REAL)
def test_real(io, batch, seqlen, dim, dstate, zoh, bfix, cfix):
    assert _segments(io, batch, seqlen, dim, dstate, bfix, cfix, B.SS_EXACT_ZOH_B * zoh) > 1
    gf.test_fixed_bc_forward_and_backward(io, batch, seqlen, dim, dstate, zoh, bfix, cfix)


@pytest.mark.parametrize("bfix,cfix", gf.MODES)
@pytest.mark.parametrize("io,batch,seqlen,dim", COMPLEX)
def test_complex(io, batch, seqlen, dim, bfix, cfix):
    assert _segments(io, batch, seqlen, dim, 8, bfix, cfix, B.SS_COMPLEX_STATE) > 1
    grids.test_complex(io, batch, seqlen, dim, bfix, cfix)


@pytest.mark.parametrize("bfix,cfix", gf.MODES)
@pytest.mark.parametrize("io,batch,seqlen,dim", MANY)
def test_more_than_a_workgroup_per_unit(io, batch, seqlen, dim, bfix, cfix):
    for more, dstate in ((0, 13), (B.SS_COMPLEX_STATE, 8)):
        nseg = _segments(io, batch, seqlen, dim, dstate, bfix, cfix, more)
        assert nseg > 1 and batch * nseg > 256
    gf.test_fixed_bc_forward_and_backward(io, batch, seqlen, dim, 13, False, bfix, cfix)
    grids.test_complex(io, batch, seqlen, dim, bfix, cfix)
