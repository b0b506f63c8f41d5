"""Performance cases of the MoE++ layer forward: what a program that uses this library has
it do, from one decoded token to the largest prefill batch, through the public entry points
(`Layer.layer_forward`, `layer_forward_static`, a chain of layers linked by the gating
residual).

A case is a dict of plain values; `listed()` are the fixed ones, `draw(rng)` gives one more of
the same ranges.  `prepare` makes the inputs and what a program keeps (the layer context and
the packed expert weights), `run` is one pass, `exact` the same outputs in float64 without
this library.
"""
import math

import torch

from paper_2410_07348_amd import binding

DEVICE = "cuda:0"
WEIGHT_STD = 0.02          # all weights and constant vectors
BIAS_STD = 0.5             # router bias "normal"

# Layer widths of the repository's workloads: the layers of the paper's models (768 / 2048,
# 1536 / 4096) and the benchmark's small, mid and large layers.
WIDTHS = ((768, 2048), (1024, 2048), (2048, 1408), (1536, 4096), (4096, 5632))

DEFAULTS = dict(n_ffn=16, n_zero=1, n_copy=1, n_const=2, k=2, act="bf16", residual=True,
                bias="none", gamma=0.0, tau=0.0, entry="layer", layers=1)


def _case(**kw):
    c = dict(DEFAULTS)
    c.update(kw)
    return c


def listed():
    return [
        # one token of one sequence being decoded, through a layer of the paper's 1B model:
        # launches and latency are everything
        _case(name="decode_1", T=1, D=768, F=2048),
        # a decoding batch in a serving loop that may not allocate: static scratch, the
        # outputs are the loop's own buffers
        _case(name="decode_static_16", T=16, D=4096, F=5632, entry="static"),
        # the benchmark's small-batch workload: 64 sequences decode together
        _case(name="smallbatch_64", T=64, D=4096, F=5632),
        # one prompt (or a mixed prefill and decode batch) of an odd length: some 80 rows per
        # expert, between a weight stream and a matrix product
        _case(name="prompt_777", T=777, D=4096, F=5632),
        # the float32 layer of the tests and the benchmark's tiny workload
        _case(name="tiny_f32", T=256, D=128, F=256, n_ffn=4, act="f32"),
        # a float32 layer of the paper's 0.6B model over one sequence: what a user runs to check a model
        _case(name="sequence_f32", T=2048, D=768, F=2048, n_ffn=8, act="f32"),
        # widths that are not multiples of the tiles, top-3, first layer (no gating residual)
        _case(name="odd_widths", T=1999, D=1000, F=1416, n_ffn=8, k=3, residual=False),
        # the benchmark's small workload: 4 sequences of 2048
        _case(name="small", T=8192, D=1024, F=2048, n_ffn=8),
        # four layers of the paper's 2B model (32 + 8 experts), linked by the gating residual
        _case(name="chain_2b", T=4096, D=768, F=2048, n_ffn=32, n_const=6, entry="chain", layers=4),
        # the benchmark's mid workload: 8 sequences of 2048, ragged groups
        _case(name="mid", T=16384, D=2048, F=1408, bias="normal"),
        # skewed routing (half of the slots on zero-computation experts, one hot expert) with
        # the expert capacities and the load-balance statistics of training
        _case(name="skew_capacity", T=16384, D=2048, F=1408, bias="skew", gamma=1.1, tau=0.75),
        # the benchmark's default workload: 8 sequences of 4096, the largest
        _case(name="large", T=32768, D=4096, F=5632),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _ffn_flops(c):
    slots = c["T"] * c["k"] * c["n_ffn"] / (c["n_ffn"] + c["n_zero"] + c["n_copy"] + c["n_const"])
    return 6.0 * c["D"] * c["F"] * slots * c["layers"]


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(("decode", "decode", "serve", "serve", "prefill", "prefill", "f32", "odd"))
    n_ffn = rng.choice((4, 8, 16, 16, 32))
    zc = rng.choice(((1, 1, 2), (1, 1, 2), (1, 1, 6), (0, 0, 0)))
    c = _case(n_ffn=n_ffn, n_zero=zc[0], n_copy=zc[1], n_const=zc[2], k=rng.choice((1, 2, 2, 2, 4)),
              residual=rng.random() < 0.75, bias=rng.choice(("none", "none", "normal")))
    if kind in ("decode", "serve", "prefill"):
        D, F = rng.choice(WIDTHS)
        T = _log_int(rng, *{"decode": (1, 64), "serve": (65, 1024), "prefill": (1025, 32768)}[kind])
        if kind == "decode" and rng.random() < 0.25:
            c["entry"] = "static"
        if kind == "prefill" and rng.random() < 0.25:
            c.update(gamma=1.1, tau=0.75)
        if kind == "prefill" and rng.random() < 0.25:
            c.update(entry="chain", layers=3)
        limit = 7.0e12
    else:
        c["act"] = "f32" if kind == "f32" else "bf16"
        D, F = 8 * _log_int(rng, 8, 128), 8 * _log_int(rng, 8, 256)
        T = _log_int(rng, 1, 2048 if kind == "f32" else 4096)
        limit = 4.0e10
    c.update(D=D, F=F, T=T)
    if c["entry"] != "layer":
        c["bias"] = "none"
    flops = _ffn_flops(c)
    if flops > limit:                      # as costly as the largest listed case at most
        c["T"] = max(1, int(c["T"] * limit / flops))
    return c


def _n(c):
    return c["n_ffn"] + c["n_zero"] + c["n_copy"] + c["n_const"]


def _router_bias(c, gen):
    if c["bias"] == "none":
        return None
    if c["bias"] == "normal":
        return torch.randn(_n(c), generator=gen, device=DEVICE) * BIAS_STD
    # "skew": zero-computation experts take about half of the slots, FFN expert 0 four times
    # the mean load of the others
    b = torch.zeros(_n(c), device=DEVICE)
    b[c["n_ffn"]:] = 0.861
    b[0] = 0.752
    return b


def _logits(t, x, prev):
    """G(x) of the tokens x in float64 (Eq.2, Eq.6); prev: G(x_prev) or None."""
    f64 = torch.float64
    gate = x.to(f64) @ t["W_g"].to(f64).t()
    if prev is not None:
        gate = gate + prev.to(f64) @ t["W_res"].to(f64).t()
    if t["bias"] is not None:
        gate = gate + t["bias"].to(f64)
    return gate


TIE = 1e-5        # logits closer than this are in an order that float32 summation may decide


def _settle_ties(c, t, prev):
    """Two correct routers may send a token to different experts where the logits at the top-k
    boundary differ by less than float32 summation noise; its output is then another one.  Such
    tokens (a handful among 10^5) get x -> -x, as likely a draw as x, so that outputs can be
    compared.  Returns the logits."""
    gate = _logits(t, t["x"], prev)
    if c["k"] < _n(c):
        for _ in range(3):
            v = torch.topk(gate, c["k"] + 1, dim=1).values
            near = torch.nonzero(v[:, -2] - v[:, -1] < TIE).reshape(-1)
            if near.numel() == 0:
                break
            t["x"][near] = -t["x"][near]
            gate[near] = _logits(t, t["x"][near], None if prev is None else prev[near])
    return gate


def _layers(c, gen):
    """The inputs of the case's layers and their logits in float64, one after the other."""
    gate = None
    for j in range(c["layers"]):
        t = _tensors(c, gen)
        prev = None if t["W_res"] is None else t["prev_gate"] if j == 0 else gate
        gate = _settle_ties(c, t, prev)
        yield t, gate


def _tensors(c, gen):
    """The inputs of one layer, from the generator alone: activations and expert weights in the
    layer's type, router-side tensors in float32."""
    act = torch.bfloat16 if c["act"] == "bf16" else torch.float32
    T, D, F, N, nc = c["T"], c["D"], c["F"], _n(c), c["n_const"]

    def normal(shape, std, dtype=torch.float32):
        return (torch.randn(shape, generator=gen, device=DEVICE) * std).to(dtype)

    def experts(rows, cols):
        w = torch.empty((c["n_ffn"], rows, cols), dtype=act, device=DEVICE)
        for e in range(c["n_ffn"]):
            w[e] = normal((rows, cols), WEIGHT_STD, act)
        return w

    t = {"x": normal((T, D), 1.0, act), "W_g": normal((N, D), WEIGHT_STD),
         "prev_gate": normal((T, N), 1.0) if c["residual"] else None,
         "W_res": normal((N, N), WEIGHT_STD) if c["residual"] else None,
         "const_vecs": normal((nc, D), WEIGHT_STD, act) if nc else None,
         "W_c": normal((nc, 2, D), WEIGHT_STD) if nc else None,
         "w1": experts(F, D), "w3": experts(F, D), "w2": experts(D, F)}
    t["bias"] = _router_bias(c, gen)
    return t


def _capacity(c):
    """Eq.8 with T k assignments, for every expert."""
    per_eta = c["gamma"] * c["T"] * c["k"] / (c["tau"] * c["n_ffn"] + _n(c) - c["n_ffn"])
    return [math.ceil((c["tau"] if i < c["n_ffn"] else 1.0) * per_eta - 1e-9) for i in range(_n(c))]


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    layer = binding.Layer(c["T"], c["D"], c["F"], c["n_ffn"], c["n_zero"], c["n_copy"], c["n_const"],
                          k=c["k"], act=c["act"], device=DEVICE)
    state = {"case": c, "layer": layer, "layers": []}
    for t, _ in _layers(c, gen):
        t["experts"] = layer.pack_experts(t.pop("w1"), t.pop("w3"), t.pop("w2"))
        layer.set_router_bias(t["bias"])
        state["layers"].append(t)
    if c["gamma"] > 0.0:
        layer.set_capacity(layer.capacity(c["T"], c["gamma"], c["tau"]))
        layer.set_balance(c["tau"])
    if c["entry"] == "static":
        state["out"] = torch.empty((c["T"], c["D"]), dtype=layer.act_dtype, device=DEVICE)
        state["gate"] = torch.empty((c["T"], _n(c)), dtype=torch.float32, device=DEVICE)
    return state


def run(state):
    c, layer = state["case"], state["layer"]
    if c["entry"] == "static":
        t = state["layers"][0]
        binding.layer_forward_static(layer.desc, t["x"], t["prev_gate"], t["W_g"], t["W_res"],
                                     t["experts"], t["const_vecs"], t["W_c"], c["k"], state["out"],
                                     state["gate"])
        return [{"out": state["out"], "gate": state["gate"]}]
    results = []
    for j, t in enumerate(state["layers"]):
        # layer j > 0 of a chain takes the logits of the layer before it
        prev = None if t["W_res"] is None else t["prev_gate"] if j == 0 else results[-1]["gate"]
        out, gate = layer.layer_forward(t["x"], prev, t["W_g"], t["W_res"], t["experts"],
                                        t["const_vecs"], t["W_c"])
        results.append({"out": out, "gate": gate})
    if c["tau"] > 0.0:
        results[-1]["balance"] = layer.get_balance()
    return results


def _touched(c):
    """FFN experts that receive at least one slot, expected."""
    return c["n_ffn"] * (1.0 - (1.0 - 1.0 / _n(c)) ** (c["T"] * c["k"]))


def work(case):
    c = dict(DEFAULTS, **case)
    b = 2 if c["act"] == "bf16" else 4
    T, D, F, N, nc = c["T"], c["D"], c["F"], _n(c), c["n_const"]
    share = 0.5 if c["bias"] == "skew" else c["n_ffn"] / N
    rows = T * c["k"] * share
    bytes_ = (2 * T * D * b                                   # x, out
              + T * N * 4 * (2 if c["residual"] else 1)       # logits in and out
              + (N + 2 * nc) * D * 4 + nc * D * b             # router, constant experts
              + (N * N * 4 if c["residual"] else 0)
              + 3.0 * _touched(c) * D * F * b)                # weights of the selected experts
    flops = 6.0 * D * F * rows + 2.0 * T * D * (N + 2 * nc)
    return {"bytes": bytes_ * c["layers"], "flops": flops * c["layers"]}


def tolerance(case):
    # bf16 layers: two correct kernel families (other summation order, h and yffn rounded to
    # bf16) differ by 2e-3 to 3e-3 of the output; float32 layers: float32 sums in another order
    return {"rel": 1e-2} if case.get("act", "bf16") == "bf16" else {"rel": 2e-6}


def _exact_layer(c, t, gate):
    f64 = torch.float64
    n_ffn, n_zero, n_copy, nc, N = c["n_ffn"], c["n_zero"], c["n_copy"], c["n_const"], _n(c)
    T, k = c["T"], c["k"]
    x = t["x"].to(f64)
    prob = torch.softmax(gate, dim=1)
    top = torch.topk(gate, k, dim=1).indices                  # [T, k], descending
    weight = torch.gather(prob, 1, top)
    counts = torch.bincount(top.reshape(-1), minlength=N)
    keep = torch.ones((T, k), dtype=torch.bool, device=x.device)
    if c["gamma"] > 0.0:                                      # an expert keeps its first cap slots
        for i, cap in enumerate(_capacity(c)):
            mine = (top == i).reshape(-1)
            rank = torch.cumsum(mine.to(torch.int64), 0) - 1
            keep &= ~(mine & (rank >= cap)).reshape(T, k)
    coef = torch.zeros((T, N), dtype=f64, device=x.device).scatter_(1, top, weight * keep)
    out = x * coef[:, n_ffn + n_zero:n_ffn + n_zero + n_copy].sum(1, keepdim=True)
    for j in range(nc):
        w = coef[:, N - nc + j:N - nc + j + 1]
        a = torch.softmax(x @ t["W_c"][j].to(f64).t(), dim=1)
        out += w * (a[:, :1] * x + a[:, 1:] * t["const_vecs"][j].to(f64))
    for e in range(n_ffn):
        tok = torch.nonzero(((top == e) & keep).any(dim=1)).reshape(-1)
        if tok.numel() == 0:
            continue
        xe = x[tok]
        z = xe @ t["w1"][e].to(f64).t()
        h = z * torch.sigmoid(z) * (xe @ t["w3"][e].to(f64).t())
        out[tok] += coef[tok, e:e + 1] * (h @ t["w2"][e].to(f64).t())
    result = {"out": out, "gate": gate}
    if c["tau"] > 0.0:
        f = counts.to(f64) / T
        p = prob.mean(dim=0)
        eta = torch.full((N,), c["tau"], dtype=f64, device=x.device)
        eta[:n_ffn] = 1.0
        result["balance"] = {"f": f, "P": p, "loss": (eta * f * p).sum().reshape(1)}
    return result


def exact(case, seed):
    c = dict(DEFAULTS, **case)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    return [_exact_layer(c, t, gate) for t, gate in _layers(c, gen)]
