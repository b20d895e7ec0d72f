"""Single-token steps of the layer on the matrix cores at widths and ranks that are no whole number of their
pieces (16 bytes of a row) or steps (32 bf16 or 16 float contraction indices), in both io types: a prompt, then
token by token, against the parallel mode of the oracle over the whole sequence."""
import pytest

from tests import test_gpu_layer as layer

pytestmark = pytest.mark.gpu


# (batch, seqlen, dim, dstate, rank)
@pytest.mark.parametrize("io,shape", [
    ("bf16", (2, 20, 100, 16, 12)), ("bf16", (5, 16, 35, 7, 9)), ("bf16", (9, 16, 776, 16, 25)),
    ("bf16", (2, 14, 9, 3, 255)), ("bf16", (1, 14, 8, 1, 8)), ("bf16", (130, 14, 1100, 16, 35)),
    ("f32", (1, 14, 100, 16, 256)), ("f32", (17, 24, 161, 12, 23)), ("f32", (2, 16, 1108, 16, 66)),
    ("f32", (3, 14, 33, 16, 31)), ("f32", (1, 14, 8, 2, 8)), ("f32", (234, 13, 1040, 16, 33)),
    # fewer than eight of either, more than 256 ranks: the general products
    ("f32", (2, 14, 40, 3, 7)), ("bf16", (2, 14, 7, 16, 12)), ("bf16", (2, 14, 20, 16, 264))])
def test_decode_sizes(io, shape):
    layer.test_layer_prompt_then_token_by_token(io, shape)


@pytest.mark.parametrize("rank", [8, 6])
def test_refused_step_leaves_the_states_alone(rank):
    import torch
    from paper_2312_00752_amd import binding as B
    nb, nd, nn, bf = 3, 64, 16, torch.bfloat16
    r = lambda *s, dtype=torch.float32: torch.randn(s, device="cuda").to(dtype)
    h = r(nb * nd * nn + 1)[1:].view(nb, nd, nn)   # four bytes off
    conv_state = r(nb, nd, 3, dtype=bf)
    keep_h, keep_conv = h.clone(), conv_state.clone()
    scratch = torch.empty(B.ss_layer_step_scratch_bytes(nb, nd, nn, rank, B.SS_BF16), dtype=torch.uint8, device="cuda")
    with pytest.raises(B.SsError) as e:
        B.ss_layer_step(h, conv_state, r(nb, nd, dtype=bf), r(nb, nd, dtype=bf), r(nd, 4), r(nd), r(rank + 2 * nn, nd, dtype=bf),
                        r(nd, rank, dtype=bf), r(nd), -r(nd, nn).abs(), r(nd), scratch)
    torch.cuda.synchronize()
    assert e.value.code == B.SS_ERR_ALIGN
    assert torch.equal(h, keep_h) and torch.equal(conv_state, keep_conv)
