"""The work a user of this framework has it do, as timed cases.

A Dyad layer stands in for ``torch.nn.Linear``, so what a program calls is a
feed-forward block (``DyadFF``) or a single layer (``DyadLinear``), in a
training step (forward, then every gradient through autograd) or at inference.
The cases take both modules through the range of this repository's workloads:
the OPT-125m / OPT-350m feed-forward shapes, the width/block sweep, the wide
pair 8192 -> 32768, the widths n_dyad does not divide; one token to a training
batch; odd token counts; every variant; bf16 and fp32.

Kinds:
  ff_step      DyadFF forward + backward (input, weight and bias gradients)
  linear_step  DyadLinear forward + backward
  ff_infer     DyadFF under no_grad
  linear_infer DyadLinear under no_grad
"""
from __future__ import annotations

import math

import torch

import paper_2312_06881_amd  # noqa: F401  (libdyad binding)
from paper_2312_06881_amd.nn import DyadFF, DyadLinear

_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, kind, n_in, n_out, n_dyad, variant, tokens, dtype="bf16"):
    return {"name": name, "kind": kind, "n_in": n_in, "n_out": n_out, "n_dyad": n_dyad,
            "variant": variant, "tokens": tokens, "dtype": dtype}


def listed():
    return [
        # OPT-125m pretraining, 8 sequences of 2048: the block the paper times
        _case("opt125m_train", "ff_step", 768, 3072, 4, "IT", 16384),
        # OPT-350m pretraining, same batch
        _case("opt350m_train", "ff_step", 1024, 4096, 4, "DT", 16384),
        # a wider block at n_dyad 8 on a smaller batch
        _case("d2048_train", "ff_step", 2048, 8192, 8, "OT", 8192),
        # an attention projection of a 4096-wide model in training
        _case("d4096_proj_train", "linear_step", 4096, 4096, 4, "IT", 8192),
        # the wide pair in training: the largest amount of work
        _case("wide_train", "ff_step", 8192, 32768, 16, "DT", 8192),
        # the wide pair decoding for 16 sequences: a stream of the weights
        _case("wide_decode", "ff_infer", 8192, 32768, 16, "IT", 16),
        # the wide pair on a short prefill or a large decode batch
        _case("wide_prefill", "ff_infer", 8192, 32768, 16, "OT", 256),
        # OPT-125m inference on a prompt of odd length
        _case("opt125m_prefill", "ff_infer", 768, 3072, 4, "DT", 2047),
        # one attention projection for one token: the smallest call
        _case("proj_decode", "linear_infer", 768, 768, 4, "OT", 1),
        # widths that n_dyad does not divide (zero-padded blocks of 154 / 615)
        _case("opt125m_D5_train", "ff_step", 768, 3072, 5, "IT", 8192),
        # n_dyad 6 with a ragged batch
        _case("opt125m_D6_train", "ff_step", 768, 3072, 6, "OT", 5000),
        # fp32, the paper's own training precision
        _case("opt125m_f32_train", "linear_step", 768, 3072, 4, "IT", 4096, "f32"),
    ]


# widths of the workloads: (d, ffn)
_FF = [(768, 3072), (1024, 4096), (2048, 8192), (4096, 16384), (8192, 32768)]
_MAX_FLOPS = 24.0 * 8192 * 8192 * 32768 / 16      # wide_train


def draw(rng):
    kind = rng.choice(["ff_step", "ff_step", "linear_step", "ff_infer", "linear_infer"])
    dtype = "f32" if kind == "linear_step" and rng.random() < 0.25 else "bf16"
    n_in, n_out = rng.choice(_FF[:3] if dtype == "f32" else _FF)
    if kind.startswith("linear"):
        # projections d -> d, and each of the two layers of a block
        n_in, n_out = rng.choice([(n_in, n_in), (n_in, n_out), (n_out, n_in)])
    # n_dyad: the paper's 4 and 8 most often; 3, 5 and 6 at the OPT-125m widths
    n_dyad = rng.choice([2, 4, 4, 4, 8, 8, 16])
    if max(n_in, n_out) <= 3072 and rng.random() < 0.3:
        n_dyad = rng.choice([3, 5, 6])
    per_token = (24.0 if kind == "ff_step" else 12.0 if kind == "linear_step" else
                 8.0 if kind == "ff_infer" else 4.0) * n_in * n_out / n_dyad
    hi = min(16384.0, _MAX_FLOPS / per_token, 8192.0 if dtype == "f32" else 16384.0)
    lo = 512.0 if kind.endswith("step") else 1.0
    tokens = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if tokens > 64 and rng.random() < 0.5:
        tokens = tokens // 64 * 64               # half of the larger batches are round, half ragged
    return {"kind": kind, "n_in": n_in, "n_out": n_out, "n_dyad": n_dyad,
            "variant": rng.choice(["IT", "OT", "DT"]), "tokens": tokens, "dtype": dtype}


def _layers(case):
    """(n_in, n_out) of each layer of the case."""
    a, b = case["n_in"], case["n_out"]
    return [(a, b), (b, a)] if case["kind"].startswith("ff") else [(a, b)]


def _inputs(case, seed):
    """x, the upstream gradient (training) and the parameters of each layer, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt, D = _TORCH[case["dtype"]], case["n_dyad"]

    def normal(shape, std):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dt)

    layers = _layers(case)
    x = normal((case["tokens"], layers[0][0]), 1.0)
    dy = normal((case["tokens"], layers[-1][1]), 1.0) if case["kind"].endswith("step") else None
    params = []
    for n_in, n_out in layers:
        shape = (D, -(-n_out // D), -(-n_in // D))
        params.append((normal(shape, 0.02), normal(shape, 0.02), normal((n_out,), 0.02)))
    return x, dy, params


def prepare(case, seed):
    x, dy, params = _inputs(case, seed)
    dt = _TORCH[case["dtype"]]
    if case["kind"].startswith("ff"):
        m = DyadFF(case["n_in"], case["n_out"], case["n_dyad"], case["variant"], device="cuda", dtype=dt)
        mods = [m.fc1, m.fc2]
    else:
        m = DyadLinear(case["n_in"], case["n_out"], case["n_dyad"], case["variant"], device="cuda", dtype=dt)
        mods = [m]
    with torch.no_grad():
        for mod, (w1, w2, b) in zip(mods, params):
            mod.w1.copy_(w1)
            mod.w2.copy_(w2)
            mod.bias.copy_(b)
    if dy is None:
        return {"module": m, "x": x}
    leaves = [x.requires_grad_(True)]
    for mod in mods:
        leaves += [mod.w1, mod.w2, mod.bias]
    return {"module": m, "x": x, "dy": dy, "leaves": leaves}


def run(state):
    if "dy" not in state:
        with torch.no_grad():
            return state["module"](state["x"])
    y = state["module"](state["x"])
    return (y.detach(),) + torch.autograd.grad(y, state["leaves"], state["dy"])


def work(case):
    M, D = case["tokens"], case["n_dyad"]
    e = 2 if case["dtype"] == "bf16" else 4
    layers = _layers(case)
    train = case["kind"].endswith("step")
    flops = sum(4.0 * M * a * b / D for a, b in layers) * (3 if train else 1)
    weights = sum(2 * D * (-(-a // D)) * (-(-b // D)) + b for a, b in layers)
    acts = M * (layers[0][0] + layers[-1][1])          # x in, y out
    # training also reads dy, writes dx, and writes a gradient of every parameter
    return {"bytes": e * (acts + weights) * (2 if train else 1), "flops": flops}


def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    # about four times the error against 64 bits: one bf16 rounding of an fp32 sum in a
    # layer; in a block the activation between the layers is rounded as well
    if case["kind"].startswith("linear"):
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 1e-2, "max": 5e-2}


# ---- the same in 64 bits, from the dense weight -----------------------------------

def _maps(n_in, n_out, D, variant):
    """Flat positions in the padded dense [D*bo, D*bi] weight of every stored entry [D][bo][bi]."""
    bo, bi = -(-n_out // D), -(-n_in // D)
    i = torch.arange(D, device="cuda").view(D, 1, 1)
    j = torch.arange(bo, device="cuda").view(1, bo, 1)
    k = torch.arange(bi, device="cuda").view(1, 1, bi)
    out_t, in_t = variant in ("OT", "DT"), variant in ("IT", "DT")
    rows = D * bo
    cols = D * bi
    pos1 = (i * bo + j) * cols + (i * bi + k)
    r2 = j * D + i if out_t else i * bo + j
    c2 = k * D + i if in_t else i * bi + k
    return pos1, r2 * cols + c2, rows, cols


def _dense(w1, w2, n_in, n_out, variant):
    pos1, pos2, rows, cols = _maps(n_in, n_out, w1.shape[0], variant)
    W = torch.zeros(rows * cols, dtype=torch.float64, device="cuda")
    W[pos1.flatten()] += w1.double().flatten()
    W[pos2.flatten()] += w2.double().flatten()
    return W.view(rows, cols)[:n_out, :n_in].contiguous()


def _weight_grads(dz, x, D, variant):
    n_out, n_in = dz.shape[1], x.shape[1]
    pos1, pos2, rows, cols = _maps(n_in, n_out, D, variant)
    G = torch.zeros((rows, cols), dtype=torch.float64, device="cuda")
    G[:n_out, :n_in] = dz.t().contiguous() @ x
    G = G.flatten()
    return G[pos1], G[pos2], dz.sum(0)


def exact(case, seed):
    x, dy, params = _inputs(case, seed)
    layers, variant, D = _layers(case), case["variant"], case["n_dyad"]
    x = x.double()
    W = [_dense(w1, w2, a, b, variant) for (w1, w2, _), (a, b) in zip(params, layers)]
    b = [p[2].double() for p in params]
    h = x @ W[0].t() + b[0]
    if len(layers) == 1:
        if dy is None:
            return h
        dy = dy.double()
        return (h, dy @ W[0]) + _weight_grads(dy, x, D, variant)
    cdf = 0.5 * torch.erfc(-h / math.sqrt(2.0))
    a = h * cdf
    y = a @ W[1].t() + b[1]
    if dy is None:
        return y
    dy = dy.double()
    dh = (dy @ W[1]) * (cdf + h * torch.exp(-0.5 * h * h) / math.sqrt(2.0 * math.pi))
    return (y, dh @ W[0]) + _weight_grads(dh, x, D, variant) + _weight_grads(dy, a, D, variant)
