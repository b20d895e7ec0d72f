"""A handed-over window that is not finite reaches the tap gradients of the steps that see it and no others: rows that start on
and off a whole 32-bit word (the latter's first slice begins a step before the row), without SiLU, against the oracle."""
import numpy as np
import pytest

from oracle import conv_oracle as cv
from paper_2312_00752_amd.workloads import make_conv_inputs
from tests import test_gpu_conv as conv
from tests.util import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("at", [0, 1, 2])
@pytest.mark.parametrize("seqlen", [9, 513, 1025, 1039])
def test_window_with_infinities(seqlen, at, io):
    w = make_conv_inputs(1, 4, seqlen, 4, io, seed=seqlen)
    w["state_in"][:, :, at] = np.inf
    out, _, g = conv._run(w, silu=False, with_state=True)
    ref = cv.conv_fwd(w["x"], w["w"], w["bias"], w["state_in"], False)["out"]
    rg = cv.conv_bwd(w["x"], w["w"], w["dout"], w["bias"], w["state_in"], False)
    for got, want, name in ((out, ref, "out"), (g["dx"], rg["dx"], "dx"), (g["dw"], rg["dw"], "dw"), (g["dbias"], rg["dbias"], "dbias")):
        got = got.float().cpu().numpy()
        finite = np.isfinite(want)
        np.testing.assert_array_equal(np.isfinite(got), finite, err_msg=name)
        assert_close(np.where(finite, got, 0.0), np.where(finite, want, 0.0), io, name)
