"""Single-token steps in two launches (up to four entries; the last launch slides the convolution's window): replayed from a
HIP graph, and against the same entries inside a larger call, which takes three."""
import numpy as np
import pytest

from paper_2312_00752_amd.workloads import make_layer_inputs

pytestmark = pytest.mark.gpu

PARAMS = ("conv_w", "conv_b", "W_x", "W_dt", "dt_bias", "A", "Dskip")


class _Decode:
    def __init__(self, w, batch):
        import torch
        from paper_2312_00752_amd import binding as B
        self.B, io = B, torch.bfloat16 if w["io"] == "bf16" else torch.float32
        _, self.steps, dim, dstate, rank, _ = w["shape"]
        t = {k: torch.from_numpy(np.ascontiguousarray(w[k])).cuda() for k in PARAMS + ("x", "z")}
        self.weights = [t[k].to(io) if k.startswith("W_") else t[k] for k in PARAMS]
        self.x, self.z = (t[k].to(io)[:batch].permute(2, 0, 1).contiguous() for k in ("x", "z"))
        code = B.SS_BF16 if w["io"] == "bf16" else B.SS_F32
        self.scratch = torch.empty(B.ss_layer_step_scratch_bytes(batch, dim, dstate, rank, code), dtype=torch.uint8, device="cuda")
        self.h = torch.zeros(batch, dim, dstate, device="cuda")
        self.window = torch.zeros(batch, dim, 3, device="cuda", dtype=io)
        self.out = torch.zeros(self.steps, batch, dim, device="cuda", dtype=io)

    def clear(self):
        for v in (self.h, self.window, self.out):
            v.zero_()

    def run(self):
        for i in range(self.steps):
            self.B.ss_layer_step(self.h, self.window, self.x[i], self.z[i], *self.weights, scratch=self.scratch, out_t=self.out[i])

    def results(self):
        return [v.clone() for v in (self.out, self.h, self.window)]


def _equal(a, b):
    import torch
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("batch", [1, 2, 4])
def test_replayed_from_a_graph(io, batch):
    import torch
    d = _Decode(make_layer_inputs(batch, 9, 256, 16, io, seed=50 + batch, rank=8), batch)
    d.run()                                 # eager
    torch.cuda.synchronize()
    want = d.results()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            d.run()
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        d.clear()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert _equal(d.results(), want)


@pytest.mark.parametrize("io,dim,dstate,rank", [("bf16", 256, 16, 8), ("bf16", 1030, 9, 33), ("f32", 256, 16, 8), ("f32", 3082, 16, 12),
                                              ("bf16", 6152, 16, 16), ("f32", 4090, 16, 12)])
@pytest.mark.parametrize("batch", [1, 3, 4])
def test_same_bits_as_three_launches(io, dim, dstate, rank, batch):
    import torch
    w = make_layer_inputs(6, 5, dim, dstate, io, seed=60, rank=rank)
    few, many = _Decode(w, batch), _Decode(w, 6)
    few.run()
    many.run()
    torch.cuda.synchronize()
    out, h, window = many.results()
    assert _equal(few.results(), [out[:, :batch], h[:batch], window[:batch]])
