"""The calls whose speed matters to a user of this framework, with the sizes they have in use.

A case is a dict of plain values.  Its ``kind`` says which public entry point one pass goes through:

  scan_train     autograd.selective_scan forward and the gradients of all inputs (complex state, which
                 the autograd front-end does not take: binding.ss_scan_fwd, then binding.ss_scan_bwd)
  scan_fwd       binding.ss_scan_fwd without gradients, the last state returned (prompt of a model
                 that brings its own projections)
  scan_step      binding.ss_step, one token
  layer_train    autograd.selective_ssm_layer forward and the gradients of all inputs
  layer_prefill  binding.ss_layer_fwd with the states handed over to generation
  layer_step     binding.ss_layer_step, one token

Values and distributions are those of paper_2312_00752_amd/workloads.py (S4D-real A, step-size bias from
softplus^-1 of [1e-3, 1e-1], fan-in scaled weights, unit normal activations), drawn on the GPU.
"""
import math

import torch

from paper_2312_00752_amd import autograd
from paper_2312_00752_amd import binding as B
from paper_2312_00752_amd import workloads

# options of the scan beside shape and dtype
_PLAIN = {"gate": True, "h_last": False, "zoh": False, "complex": False, "fixed": "", "symbols": False}


def _case(kind, batch, seqlen, dim, dtype, dstate=16, **options):
    c = {"kind": kind, "batch": batch, "seqlen": seqlen, "dim": dim, "dstate": dstate, "dtype": dtype}
    if kind.startswith("scan"):
        c.update(_PLAIN)
    c.update(options)
    return c


def _named(name, case):
    return {"name": name, **case}


def listed():
    return [
        # generation, one token of one layer at inner width 4096: a single user, then a served batch
        _named("layer_step_b1", _case("layer_step", 1, 1, 4096, "bf16")),
        _named("layer_step_b64", _case("layer_step", 64, 1, 4096, "bf16")),
        # the recurrence alone, for a model with its own convolution and projections (workloads.STEP_CONFIG)
        _named("scan_step_b64", _case("scan_step", 64, 1, 4096, "bf16")),
        # the five workloads of workloads.CONFIGS, forward and backward: the smallest (latency and launches), ...
        _named("scan_tiny_fp32", _case("scan_train", 1, 256, 64, "f32", h_last=True)),
        # ... language-model layers at context 2048, ...
        _named("scan_130m_bf16", _case("scan_train", 8, 2048, 1536, "bf16")),
        _named("scan_1p4b_bf16", _case("scan_train", 8, 2048, 4096, "bf16")),
        # ... a long context and a DNA sequence of 2^20 symbols
        _named("scan_2p8b_long_bf16", _case("scan_train", 2, 16384, 5120, "bf16")),
        _named("scan_genomics_fp32", _case("scan_train", 1, 1048576, 256, "f32", symbols=True)),
        # Eq. 4 as the paper prints it: the exact zero-order hold, on a layer of the smaller width
        _named("scan_zoh_bf16", _case("scan_train", 8, 2048, 1536, "bf16", zoh=True)),
        # training of the whole layer
        _named("layer_train_1p4b_bf16", _case("layer_train", 8, 2048, 4096, "bf16")),
        # next-token training on documents of 2048 tokens: inputs are tokens 0 .. 2046
        _named("layer_train_l2047_bf16", _case("layer_train", 8, 2047, 1536, "bf16")),
        # prompts have any length
        _named("layer_prefill_l1531_bf16", _case("layer_prefill", 4, 1531, 4096, "bf16")),
    ]


def _log_int(rng, low, high):
    return min(high, max(low, int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))))


def _length(rng, low, high):
    """Half of them multiples of 64 (contexts of training runs), half as they come (prompts, documents)."""
    n = _log_int(rng, low, high)
    return max(low, n // 64 * 64) if rng.random() < 0.5 and n >= 64 else n


def _width(rng, low, high):
    """Inner widths: mostly multiples of 64, some of 16, a few as they come."""
    n, r = _log_int(rng, low, high), rng.random()
    step = 64 if r < 0.7 else (16 if r < 0.9 else 1)
    return max(low, n // step * step)


# token * channels * states of a drawn training case at most; the listed ones reach 4.3e9
_MOST_TRAIN = {"scan": 1.1e9, "layer": 8e8}


def _shrink(c, most):
    """Halve batch, then length, then width until the case fits."""
    while c["batch"] * c["seqlen"] * c["dim"] * c["dstate"] > most:
        key = "batch" if c["batch"] > 1 else ("seqlen" if c["seqlen"] > 1024 else "dim")
        c[key] = max(1, c[key] // 2)
    return c


def draw(rng):
    kind = rng.choice(("scan_train", "scan_train", "scan_train", "scan_fwd", "scan_step", "layer_train", "layer_train",
                       "layer_prefill", "layer_prefill", "layer_step"))
    dtype = "bf16" if rng.random() < 0.7 else "f32"
    if kind.endswith("step"):
        return _case(kind, _log_int(rng, 1, 256), 1, _width(rng, 256, 5120), dtype)
    if kind == "layer_train":
        c = _case(kind, _log_int(rng, 1, 16), _length(rng, 128, 4096), _width(rng, 256, 5120), dtype)
        return _shrink(c, _MOST_TRAIN["layer"])
    if kind == "layer_prefill":
        c = _case(kind, _log_int(rng, 1, 16), _length(rng, 16, 16384), _width(rng, 256, 5120), dtype)
        return _shrink(c, _MOST_TRAIN["layer"])
    dstate = rng.choice((1, 4, 8, 16, 16, 16, 16, 16, 16, 32, 64))
    c = _case(kind, _log_int(rng, 1, 16), _length(rng, 64, 65536), _width(rng, 64, 5120), dtype, dstate)
    c["gate"] = rng.random() < 0.8
    c["symbols"] = dtype == "f32" and c["seqlen"] >= 8192
    c["h_last"] = kind == "scan_fwd" or rng.random() < 0.3
    variant = rng.random()   # the ablations: B-bar rule, time-invariant B and C, complex state
    if variant < 0.1:
        c["zoh"] = True
    elif variant < 0.2:
        c["fixed"] = rng.choice(("B", "C", "BC"))
    elif variant < 0.3:
        c["complex"] = True
        c["dstate"] = min(c["dstate"], 32)
    return _shrink(c, _MOST_TRAIN["scan"] / (4 if variant < 0.3 else 1))


# ---- inputs ----------------------------------------------------------------------------------------
class _Draws:
    """Tensors on the GPU from one generator, in a fixed order."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, *shape, dtype=torch.float32):
        return torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32).to(dtype)

    def uniform(self, low, high, *shape, dtype=torch.float32):
        return torch.empty(shape, device="cuda", dtype=torch.float32).uniform_(low, high, generator=self.g).to(dtype)

    def symbols(self, nb, nd, nl):
        """A random sequence over four symbols, embedded, with a little noise."""
        table = self.normal(nd, 4)
        u = 0.02 * self.normal(nb, nd, nl)
        for b in range(nb):
            u[b] += table[:, torch.randint(0, 4, (nl,), generator=self.g, device="cuda")]
        return u

    def step_bias(self, dim):
        return torch.log(torch.expm1(self.uniform(1e-3, 1e-1, dim)))


def _decay(dim, dstate):
    """A[d,n] = -(n+1)."""
    return (-torch.arange(1, dstate + 1, device="cuda", dtype=torch.float32)).expand(dim, dstate).contiguous()


def _code(case):
    return B.SS_BF16 if case["dtype"] == "bf16" else B.SS_F32


def _io(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _scan_inputs(case, r):
    nb, nl, nd, nn, io = case["batch"], case["seqlen"], case["dim"], case["dstate"], _io(case)
    c2 = (2,) if case["complex"] else ()
    u = r.symbols(nb, nd, nl).to(io) if case["symbols"] else r.normal(nb, nd, nl, dtype=io)
    s = {"u": u, "delta": r.normal(nb, nd, nl, dtype=io),
         "z": r.normal(nb, nd, nl, dtype=io) if case["gate"] else None, "delta_bias": r.step_bias(nd),
         "Dskip": r.normal(nd)}
    for name in ("B", "C"):
        fixed = name in case["fixed"]
        s[name] = r.normal(nd, nn, *c2) if fixed else r.normal(nb, nn, *c2, nl, dtype=io)
    if case["complex"]:   # S4D-Lin: A_n = -1/2 + n i
        n = torch.arange(nn, device="cuda", dtype=torch.float32)
        s["A"] = torch.stack((torch.full_like(n, -0.5), n), dim=-1).expand(nd, nn, 2).contiguous()
    else:
        s["A"] = _decay(nd, nn)
    return s


def _layer_inputs(case, r):
    nd, nn, io, width = case["dim"], case["dstate"], _io(case), 4
    rank = workloads.layer_rank(nd)
    k, kd, kr = width ** -0.5, nd ** -0.5, rank ** -0.5
    return {"conv_w": r.uniform(-k, k, nd, width), "conv_b": r.uniform(-k, k, nd),
            "W_x": r.uniform(-kd, kd, rank + 2 * nn, nd, dtype=io), "W_dt": r.uniform(-kr, kr, nd, rank, dtype=io),
            "dt_bias": r.step_bias(nd), "A": _decay(nd, nn), "Dskip": r.normal(nd)}


def _scratch(nbytes):
    return torch.empty(max(256, nbytes), dtype=torch.uint8, device="cuda")


_LAYER_ORDER = ("x", "z", "conv_w", "conv_b", "W_x", "W_dt", "dt_bias", "A", "Dskip")


def prepare(case, seed):
    r = _Draws(seed)
    kind, nb, nl, nd, nn, io, code = (case["kind"], case["batch"], case["seqlen"], case["dim"], case["dstate"], _io(case),
                                      _code(case))
    state = {"case": case}
    if kind == "scan_train":
        t = _scan_inputs(case, r)
        state["dout"] = r.normal(nb, nd, nl, dtype=io)
        if case["complex"]:
            state["ws"] = _scratch(B.ss_workspace_bytes(nb, nd, nl, nn, True, code, case["gate"], "B" in case["fixed"],
                                                        "C" in case["fixed"], complex_state=True))
        else:
            for v in t.values():
                if v is not None:
                    v.requires_grad_(True)
        state["t"] = t
    elif kind == "scan_fwd":
        state["t"] = _scan_inputs(case, r)
        state["ws"] = _scratch(B.ss_workspace_bytes(nb, nd, nl, nn, False, code, case["gate"], "B" in case["fixed"],
                                                    "C" in case["fixed"], complex_state=case["complex"]))
    elif kind == "scan_step":
        state["t"] = {"h": 0.3 * r.normal(nb, nd, nn), "u_t": r.normal(nb, nd, dtype=io), "delta_t": r.normal(nb, nd, dtype=io),
                      "A": _decay(nd, nn), "B_t": r.normal(nb, nn, dtype=io), "C_t": r.normal(nb, nn, dtype=io),
                      "Dskip": r.normal(nd), "z_t": r.normal(nb, nd, dtype=io), "delta_bias": r.step_bias(nd)}
    else:
        t = _layer_inputs(case, r)
        rank, width = t["W_dt"].shape[1], t["conv_w"].shape[1]
        if kind == "layer_step":
            t.update(h=0.3 * r.normal(nb, nd, nn), conv_state=r.normal(nb, nd, width - 1, dtype=io),
                     x_t=r.normal(nb, nd, dtype=io), z_t=r.normal(nb, nd, dtype=io))
            state["scratch"] = _scratch(B.ss_layer_step_scratch_bytes(nb, nd, nn, rank, code))
        else:
            t.update(x=r.normal(nb, nd, nl, dtype=io), z=r.normal(nb, nd, nl, dtype=io))
            if kind == "layer_train":
                state["dout"] = r.normal(nb, nd, nl, dtype=io)
                for v in t.values():
                    v.requires_grad_(True)
            else:
                state["scratch"] = _scratch(B.ss_layer_scratch_bytes(nb, nd, nl, nn, rank, width, code, False))
        state["t"] = t
    return state


# ---- one pass ----------------------------------------------------------------------------------------
def _run_scan_train(case, state):
    t, dout = state["t"], state["dout"]
    if case["complex"]:
        kw = dict(Dskip=t["Dskip"], z=t["z"], delta_bias=t["delta_bias"], delta_softplus=True, complex_state=True)
        out, h_last = B.ss_scan_fwd(t["u"], t["delta"], t["A"], t["B"], t["C"], return_last_state=case["h_last"],
                                    workspace=state["ws"], **kw)
        g = B.ss_scan_bwd(dout, t["u"], t["delta"], t["A"], t["B"], t["C"], state["ws"], **kw)
        return [v for v in (out, h_last, *g.values()) if v is not None]
    res = autograd.selective_scan(t["u"], t["delta"], t["A"], t["B"], t["C"], t["Dskip"], t["z"], t["delta_bias"],
                                  delta_softplus=True, exact_zoh=case["zoh"], return_last_state=case["h_last"])
    out, last = (res[0], [res[1].detach()]) if case["h_last"] else (res, [])
    grads = torch.autograd.grad(out, [v for v in t.values() if v is not None], dout)
    return [out.detach(), *last, *grads]


def run(state):
    case, t = state["case"], state["t"]
    kind = case["kind"]
    if kind == "scan_train":
        return _run_scan_train(case, state)
    if kind == "scan_fwd":
        return B.ss_scan_fwd(t["u"], t["delta"], t["A"], t["B"], t["C"], Dskip=t["Dskip"], z=t["z"], delta_bias=t["delta_bias"],
                             delta_softplus=True, return_last_state=True, workspace=state["ws"], save_for_bwd=False,
                             exact_zoh=case["zoh"], complex_state=case["complex"])
    if kind == "scan_step":
        out = B.ss_step(t["h"], t["u_t"], t["delta_t"], t["A"], t["B_t"], t["C_t"], Dskip=t["Dskip"], z_t=t["z_t"],
                        delta_bias=t["delta_bias"], delta_softplus=True)
        return out, t["h"]
    if kind == "layer_step":
        out = B.ss_layer_step(t["h"], t["conv_state"], t["x_t"], t["z_t"], t["conv_w"], t["conv_b"], t["W_x"], t["W_dt"],
                              t["dt_bias"], t["A"], t["Dskip"], state["scratch"])
        return out, t["h"], t["conv_state"]
    args = [t[k] for k in _LAYER_ORDER]
    if kind == "layer_prefill":
        return B.ss_layer_fwd(*args, scratch=state["scratch"], return_states=True)
    out = autograd.selective_ssm_layer(*args)
    return (out.detach(), *torch.autograd.grad(out, args, state["dout"]))


# ---- what a pass cannot do without -------------------------------------------------------------------
def work(case):
    """Inputs read once, outputs written once; flops as the formulas have them: per token, channel and real
    state 4 multiply-adds and an exponential forward and 12 and one backward, the convolution 2 W per element
    and pass, a projection product 2 per multiply-add (once forward, twice backward)."""
    kind, nb, nl, nd, nn = case["kind"], case["batch"], case["seqlen"], case["dim"], case["dstate"]
    esz = 2 if case["dtype"] == "bf16" else 4
    tc = nb * nl * nd
    if kind.startswith("scan"):
        slots = nn * (2 if case["complex"] else 1)
        gate = int(case["gate"])
        state = 4 * nb * nd * slots
        bc = sum(4 * nd * slots if name in case["fixed"] else esz * nb * nl * slots for name in ("B", "C"))
        par = 4 * nd * (slots + 2)
        if kind == "scan_step":
            return {"bytes": tc * esz * 4 + bc + par + 2 * state, "flops": 9 * tc * slots}
        fwd = tc * esz * (3 + gate) + bc + par + (state if case["h_last"] else 0)
        if kind == "scan_fwd":
            return {"bytes": fwd, "flops": 9 * tc * slots}
        return {"bytes": fwd + tc * esz * (3 + gate) + bc + par, "flops": 34 * tc * slots}
    rank, width = workloads.layer_rank(nd), 4
    weights = esz * nd * (2 * rank + 2 * nn)
    par = 4 * nd * (width + 3 + nn)
    products = 2 * tc * (2 * rank + 2 * nn)
    if kind == "layer_step":
        return {"bytes": tc * esz * 3 + weights + par + 8 * nb * nd * nn + 2 * esz * nb * nd * (width - 1),
                "flops": 9 * tc * nn + products + 2 * width * tc}
    if kind == "layer_prefill":
        return {"bytes": tc * esz * 3 + weights + par + 4 * nb * nd * nn + esz * nb * nd * (width - 1),
                "flops": 9 * tc * nn + products + 2 * width * tc}
    return {"bytes": tc * esz * 6 + 2 * (weights + par), "flops": 34 * tc * nn + 3 * products + 6 * width * tc}


def tolerance(case):
    """About four times the largest relative error of any output against the same pass in 64 bits (measured
    at 512 steps, width 128 to 1024, and on the 2^20-step case): float32 1.8e-6 (A's gradient over 2^20 steps);
    bf16 2.4e-3 for the scan, 2.8e-3 for the layer, which rounds u, [r;B;C] and delta between its kernels, and
    3.4e-3 with more than 16 states, which round the running sum once per sixteen."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["kind"].startswith("layer"):
        return {"rel": 1.2e-2}
    return {"rel": 1.4e-2 if case["dstate"] > 16 else 1e-2}
