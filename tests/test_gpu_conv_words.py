"""Rows of 16-bit elements that start off a whole 32-bit word, whose slices, above 1024 steps, start one step before the row: lengths
around a slice and around a wave's 512 steps, with and without a handed-over window, forward and backward against the oracle."""
import pytest

from paper_2312_00752_amd.workloads import make_conv_inputs
from tests import test_gpu_conv as conv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("with_state", [False, True])
@pytest.mark.parametrize("width", [2, 3, 4])
@pytest.mark.parametrize("seqlen", [9, 15, 17, 505, 511, 513, 1023, 1025, 1031, 1033, 1535, 1537, 2047])
def test_conv_rows_off_a_word(seqlen, width, with_state):
    conv._check(make_conv_inputs(2, 3, seqlen, width, "bf16", seed=seqlen + width), with_state=with_state)
