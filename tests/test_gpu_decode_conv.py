"""Single-token steps with the convolution formed inside the first projection (up to four entries, an even number of
channels): the smallest widths, parts of the contraction that end inside a step, are empty, or take two rounds of staging."""
import pytest

from tests import test_gpu_layer as layer

pytestmark = pytest.mark.gpu


# (batch, seqlen, dim, dstate, rank)
@pytest.mark.parametrize("io,shape", [
    ("bf16", (4, 14, 8, 16, 8)), ("bf16", (3, 14, 34, 5, 9)), ("bf16", (1, 14, 130, 16, 10)), ("bf16", (4, 14, 6152, 16, 16)),
    ("f32", (4, 14, 8, 16, 8)), ("f32", (1, 14, 18, 16, 8)), ("f32", (3, 14, 3086, 3, 20)),
    ("f32", (1, 14, 5120, 3, 20)), ("f32", (2, 14, 4608, 16, 20)),
    ("bf16", (5, 14, 130, 16, 10)), ("f32", (4, 14, 129, 16, 10)), ("f32", (2, 14, 4610, 16, 20))])   # the three launches
def test_decode_conv(io, shape):
    layer.test_layer_prompt_then_token_by_token(io, shape)
