"""Time-invariant B / C with the sequence split across workgroups: the aggregate passes and the partial sums per
segment, real, exact zero-order hold and complex, whole slices and others, more than 16 states, against the oracles."""
import pytest

from tests import test_gpu_fixed_bc as gf
from tests import test_gpu_fixed_bc_grids as grids

pytestmark = pytest.mark.gpu

# few rows: cut into segments of 64 steps and up, the last one short, the carry inside (16) and beyond (17) one batch
REAL = [("f32", 1, 331, 70, 16, False), ("bf16", 2, 1032, 65, 9, False), ("bf16", 1, 2049, 30, 16, True), ("f32", 1, 456, 40, 24, False),
        ("f32", 2, 1152, 64, 16, True)]
COMPLEX = [("f32", 1, 264, 3), ("bf16", 2, 331, 4)]


@pytest.mark.parametrize("bfix,cfix", gf.MODES)
@pytest.mark.parametrize("io,batch,seqlen,dim,dstate,zoh", REAL)
def test_real(io, batch, seqlen, dim, dstate, zoh, bfix, cfix):
    gf.test_fixed_bc_forward_and_backward(io, batch, seqlen, dim, dstate, zoh, bfix, cfix)


@pytest.mark.parametrize("bfix,cfix", gf.MODES)
@pytest.mark.parametrize("io,batch,seqlen,dim", COMPLEX)
def test_complex(io, batch, seqlen, dim, bfix, cfix):
    grids.test_complex(io, batch, seqlen, dim, bfix, cfix)
