"""The calls that a program built on this library makes, at the sizes it makes them: what its speed is measured on.

A case is one FFN layer (or a stack of them) and one way of driving it through paper_2312_11514_amd.Layer:

  kind "step"    Layer.step: one whole step for `batch` tokens of independent streams (decode)
  kind "tokens"  Layer.step_tokens: one speculative verification pass of `batch` consecutive tokens, `keep` accepted
  kind "calls"   the four separate calls predict -> update_window -> load_bundles -> sparse_ffn
  kind "ffn"     Layer.sparse_ffn alone on a cache that stays as it is (`static`: Layer.sparse_ffn_static)

`steps` consecutive steps make a pass.  restart = True: the pass is a new sequence, it begins with Layer.reset on an
empty cache.  restart = False: the sequence goes on where the last pass stopped (a stored stream, walked round).
graph = True: the step is captured once into a HIP graph with staging buffers and replayed, as a serving loop does.
hint = True: Layer.set_expected_rows was told the mean number of cached rows, as bench.py does.

Weights and streams are those of workloads/__init__.py, made on the GPU: W ~ N(0, 1/d), AR(1) tokens, biases that let
a fraction p of the neurons fire.  The ReLU'd projection is part low-rank, so that the rank-r predictor foresees most
of the neurons that fire.
"""
import functools
import math

import numpy as np
import torch

import paper_2312_11514_amd as lif

STREAM = 48            # steps of the stored stream of a sequence that goes on
PREDICTOR_CORR = 0.9   # correlation of the predictor's logit with the true pre-activation

_BASE = {"kind": "step", "d": 4096, "F": 16384, "rank": 128, "k": 5, "p": 0.03, "rho": 0.9, "dtype": "f16", "glu": False,
         "gate": False, "batch": 1, "keep": 0, "capacity": 8192, "shrink": False, "full": False, "static": False,
         "layers": 1, "steps": 1, "restart": False, "graph": False, "hint": True}


def _case(name, **changes):
    c = dict(_BASE, name=name)
    c.update(changes)
    return c


def listed():
    return [
        # the smallest layer (bench workload C1, fp32), one token at a time: what a call costs when there is no data
        _case("tiny_f32_token", d=256, F=1024, rank=32, k=4, p=0.05, dtype="f32", capacity=1024, hint=False),
        # the headline: one decode token of an OPT-6.7B-shaped layer (C2), launched from the host
        _case("opt_token"),
        # one decode token of a Falcon-7B-shaped layer (C3: rows that are no power of two)
        _case("falcon_token", d=4544, F=18176, p=0.07, rho=0.85, capacity=9088),
        # one decode token of a Llama-2-7B-shaped gated layer (C4), replayed from a graph as a serving loop does
        _case("llama_token_graph", F=11008, rank=256, k=4, p=0.10, glu=True, capacity=11008, graph=True),
        # the same layer serving eight streams at once (C4 batch 8)
        _case("llama_batch8", F=11008, rank=256, k=4, p=0.10, glu=True, batch=8, capacity=11008),
        # gate projection resident in HBM as the exact predictor (N4)
        _case("llama_gate_token", F=11008, rank=256, k=4, p=0.10, gate=True, capacity=11008),
        # a new sequence under a memory limit: dynamic window, 10 % active, cache of 25 % of the rows (N1)
        _case("opt_dynamic_sequence", p=0.10, k=8, capacity=4096, shrink=True, steps=24, restart=True),
        # a new sequence decoded by speculative verification passes of five tokens, four accepted (N2)
        _case("opt_speculative_sequence", kind="tokens", batch=5, keep=4, steps=12, restart=True),
        # one token through stacked OPT layers, one graph per token (C5 with fewer layers)
        _case("opt_stack8_graph", layers=8, graph=True),
        # the FFN alone on a warm cache, from the host (a caller that does its own cache management, no allocation)
        _case("opt_ffn", kind="ffn", static=True),
        # the FFN alone, eight tokens over a cache that holds most of a gated layer, every bundle read completely
        _case("llama_ffn_batch8_full", kind="ffn", F=11008, rank=256, k=4, p=0.35, glu=True, batch=8, capacity=11008, full=True),
        # four separate calls, fp32, ragged sizes, a small batch, no row-count hint
        _case("ragged_f32_calls", kind="calls", d=1288, F=5000, rank=68, k=3, p=0.06, dtype="f32", batch=3, capacity=4000,
              hint=False),
    ]


def _log(rng, lo, hi, step):
    return max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step + 0.5) * step)


def draw(rng):
    """A layer of any shape between the listed extremes, driven in any of the ways above."""
    most = max(_cost(c) for c in listed())
    while True:
        c = dict(_BASE)
        c["kind"] = rng.choice(["step", "step", "step", "tokens", "calls", "ffn"])
        c["dtype"] = rng.choice(["f16", "f16", "f16", "f32"])
        e, v = (2, 8) if c["dtype"] == "f16" else (4, 4)
        c["d"] = _log(rng, 256, 5120, v)
        c["F"] = _log(rng, 1024, 20480, 64 if c["kind"] == "tokens" else 8)
        c["rank"] = _log(rng, 32, 768, v)
        c["k"] = rng.randint(1, 10)
        c["p"] = round(math.exp(rng.uniform(math.log(0.02), math.log(0.35 if c["kind"] == "ffn" else 0.12))), 4)
        c["rho"] = round(rng.uniform(0.8, 0.95), 3)
        shape = rng.choice(["plain", "plain", "glu"] + (["gate"] if c["kind"] != "ffn" else []))
        c["glu"], c["gate"] = shape == "glu", shape == "gate"
        c["batch"] = 1 if c["kind"] in ("step", "ffn") and rng.random() < 0.6 else rng.randint(2, 8)
        if c["kind"] == "tokens":
            c["keep"] = rng.randint(1, c["batch"])
        c["full"] = rng.random() < 0.25
        c["static"] = c["kind"] == "ffn" and rng.random() < 0.5
        c["hint"] = rng.random() < 0.7
        c["graph"] = c["kind"] in ("step", "ffn") and rng.random() < 0.4
        c["layers"] = rng.choice([1, 1, 1, 2, 4]) if c["kind"] == "step" else 1
        if c["kind"] != "ffn" and not c["graph"] and rng.random() < 0.4:
            c["restart"], c["steps"] = True, rng.randint(4, 24)
        held, mask = _rates(c)[0], _rates(c)[3]
        if c["kind"] != "ffn" and rng.random() < 0.25:      # a cache too small for the window
            c["shrink"], c["capacity"] = True, min(c["F"], int(0.7 * held + 3 * mask) + 64)
        else:
            c["capacity"] = min(c["F"], int(2.5 * held) + 256)
        scratch = 4 * c["batch"] * (c["capacity"] + 64 + 32 * c["d"])
        if c["batch"] * c["d"] * e > 64 * 1024 or (c["static"] and scratch > lif.load_library().lif_static_scratch_bytes()):
            continue
        if c["layers"] * c["F"] * _vectors(c) * c["d"] * e <= 600e6 and _cost(c) <= most:
            return c


def _vectors(c):
    return 3 if c["glu"] else 2


@functools.lru_cache(maxsize=None)
def _simulate(k, p, rho, batch, keep, exact):
    """Rows held, rows added and rows that fire per step, and rows of one step's mask, each per neuron of the layer.
    A neuron's logit along the stream is an AR(1) process: the rates of many of them."""
    z0 = float(torch.distributions.Normal(0.0, 1.0).icdf(torch.tensor(1.0 - p, dtype=torch.float64)))
    r, n, s = np.random.RandomState(7), 4096, math.sqrt(1.0 - rho * rho)
    steps, streams, per = k + 10, (1 if keep else batch), (batch if keep else 1)
    advance = keep if keep else 1
    z, noise = r.standard_normal((2, streams, n))
    logits, pre = [], []
    for _ in range(steps * advance + per):
        corr = 1.0 if exact else PREDICTOR_CORR
        logits.append((z > z0))
        pre.append((corr * z + math.sqrt(1.0 - corr * corr) * noise > z0))
        z, noise = rho * z + s * r.standard_normal((streams, n)), rho * noise + s * r.standard_normal((streams, n))
    before, window, held, added, fire, mask = np.zeros(n, bool), [], [], [], [], []
    for t in range(steps):
        at = range(t * advance, t * advance + per)
        now = [logits[i].any(axis=0) for i in at]
        window = (window + now[:advance])[-k:]
        union = np.any(window + now, axis=0)
        if t >= k:
            held.append(union.mean())
            added.append((union & ~before).mean())
            fire.append((union & np.any([pre[i].any(axis=0) for i in at], axis=0)).mean())
            mask.append(np.any(now, axis=0).mean())
        before = union
    return tuple(float(np.mean(v)) for v in (held, added, fire, mask))


def _rates(c):
    held, added, fire, mask = (v * c["F"] for v in _simulate(c["k"], c["p"], c["rho"], c["batch"], c["keep"], c["gate"]))
    if c["shrink"]:
        part = min(1.0, c["capacity"] / max(held, 1.0))
        held, fire = held * part, fire * part
    return held, added, fire, mask


def _parts(c):
    """Per step and layer: bytes that cross the host link, bytes of HBM traffic, operations."""
    e = 2 if c["dtype"] == "f16" else 4
    d, b, g = c["d"], c["batch"], _vectors(c)
    held, added, fire, _ = _rates(c)
    down = held if c["full"] else fire
    hbm = held * (g - 1) * d * e + down * d * e + 2 * b * d * e
    flops = 2.0 * b * d * (held * (g - 1) + down)
    if c["kind"] == "ffn":
        return 0.0, hbm, flops
    if c["gate"]:
        hbm, flops = hbm + c["F"] * d * e, flops + 2.0 * b * d * c["F"]
    else:
        hbm, flops = hbm + (d + c["F"]) * c["rank"] * e, flops + 2.0 * b * (d + c["F"]) * c["rank"]
    hbm += b * c["F"] / 8 + (c["k"] + 2) * c["F"] / 8
    link = added * g * d * e                                # read from the host, written to the cache
    return link, hbm + link, flops


def _cost(c):
    link, hbm, flops = _parts(c)
    return c["layers"] * c["steps"] * (10.0 + link / 50e3 + hbm / 4e6 + flops / 1e8)


def work(case):
    link, hbm, flops = _parts(case)
    n = case["layers"] * case["steps"]
    return {"bytes": n * (link + hbm), "flops": n * flops}


def tolerance(case):
    # y: fp32 accumulation, rounded once to the storage type; masks, ids, counts and cache rows are exact
    return {"rel": 1e-3, "max": 1e-2} if case["dtype"] == "f16" else {"rel": 1e-5, "max": 1e-4}


def _make_layer(c, g, dev):
    d, F, r, dt = c["d"], c["F"], c["rank"], torch.float16 if c["dtype"] == "f16" else torch.float32
    z = float(torch.distributions.Normal(0.0, 1.0).icdf(torch.tensor(1.0 - c["p"], dtype=torch.float64)))

    def gaussian(*shape, var):
        return torch.randn(shape, generator=g, device=dev) * math.sqrt(var)

    A = B = cc = None
    w = gaussian(F, d, var=1.0 / d)                         # the ReLU'd projection
    if not c["gate"]:
        A = gaussian(r, d, var=1.0 / d).to(dt)
        B = gaussian(r, F, var=1.0 / r).to(dt)
        w = math.sqrt(1.0 - PREDICTOR_CORR ** 2) * w + PREDICTOR_CORR * (B.float().t().contiguous() @ A.float())
        cc = -z * B.float().norm(dim=0)
    w = w.to(dt)
    b = -z * w.float().norm(dim=1)
    vectors = [w] if not (c["glu"] or c["gate"]) else [w, gaussian(F, d, var=1.0 / d).to(dt)] if c["glu"] else \
        [gaussian(F, d, var=1.0 / d).to(dt)]
    vectors.append(gaussian(F, d, var=1.0 / d).to(dt))
    host = torch.empty((F, len(vectors) * d), dtype=dt, pin_memory=True)
    host.copy_(torch.cat(vectors, dim=1))
    lay = lif.Layer(d_model=d, d_ffn=F, rank=r, window_k=c["k"], capacity_rows=c["capacity"], max_batch=c["batch"],
                    glu=c["glu"], dtype=c["dtype"], ffn_mode=lif.FFN_FULL_BUNDLE if c["full"] else lif.FFN_SKIP_DEAD,
                    shrink_window=c["shrink"], predictor=lif.PRED_GATE if c["gate"] else lif.PRED_LOWRANK, threshold=0.0,
                    A=w if c["gate"] else A, B=B, c=cc, b=b, host_bundles=host)
    for t in (lay.matrix, lay.bias, lay.masks, lay.step_mask, lay.added, lay.removed, lay.n_added, lay.n_removed):
        t.zero_()                                           # what lies past the counts is compared too
    lay.pointers.fill_(-1)
    return lay


def _one(c, lay, x, y):
    if c["kind"] == "step":
        lay.step(x, y, c["batch"])
    elif c["kind"] == "tokens":
        lay.step_tokens(x, y, c["batch"], c["keep"])
    elif c["kind"] == "calls":
        lay.step_calls(x, y, c["batch"])
    elif c["static"]:
        lay.sparse_ffn_static(x, y, c["batch"])
    else:
        lay.sparse_ffn(x, y, c["batch"])


def prepare(case, seed):
    c, dev = case, torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    layers = [_make_layer(c, g, dev) for _ in range(c["layers"])]
    # the token stream: AR(1), one stream per token of the batch (consecutive tokens of one stream for "tokens")
    n = c["steps"] if c["restart"] else STREAM
    streams, advance = (1, c["keep"]) if c["kind"] == "tokens" else (c["batch"], 1)
    noise = torch.randn((n * advance + c["batch"], streams, c["d"]), generator=g, device=dev)
    x, s = noise.clone(), math.sqrt(1.0 - c["rho"] ** 2)
    for t in range(1, len(x)):
        x[t] = c["rho"] * x[t - 1] + s * noise[t]
    x = x.to(layers[0].tdtype)
    if c["kind"] == "tokens":
        xs = [x[t * advance:t * advance + c["batch"], 0].contiguous() for t in range(n)]
    else:
        xs = [x[t].contiguous() for t in range(n)]
    y = torch.zeros((c["steps"], c["layers"], c["batch"], c["d"]), dtype=x.dtype, device=dev)
    st = {"case": c, "layers": layers, "x": xs, "y": y, "at": 0, "graph": None,
          "y_of": [[y[t, l] for l in range(c["layers"])] for t in range(c["steps"])]}
    # the sequence so far: fills the caches, and tells the mean number of rows in use
    for lay in layers:
        lay.reset()
        for t in range(n):
            if c["kind"] == "ffn":
                lay.step(xs[t], st["y_of"][0][0], c["batch"])
            else:
                _one(c, lay, xs[t], st["y_of"][0][0])
        if lay.state()["error"]:
            raise RuntimeError("the cache is too small for the stream")
        if c["hint"]:
            got = lay.counters()
            rows = lay.state()["num_used"] if c["kind"] == "ffn" else got["ffn_rows"] / got["ffn_calls"]
            lay.set_expected_rows(int(1.15 * rows))
    if c["graph"]:
        st["x_stage"] = xs[0].clone()
        torch.cuda.synchronize()
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            for l, lay in enumerate(layers):
                _one(c, lay, st["x_stage"], st["y_of"][0][l])
    return st


def run(state):
    c, layers, xs = state["case"], state["layers"], state["x"]
    if c["restart"]:
        for lay in layers:
            lay.reset()
        state["at"] = 0
    for t in range(c["steps"]):
        x = xs[state["at"]]
        state["at"] = (state["at"] + 1) % len(xs)
        if state["graph"] is not None:
            state["x_stage"].copy_(x)
            state["graph"].replay()
        else:
            for lay, y in zip(layers, state["y_of"][t]):
                _one(c, lay, x, y)
    out = {"y": state["y"]}
    if c["kind"] != "ffn":                                  # the updated caches, and what the last step reported
        for l, lay in enumerate(layers):
            out["layer%d" % l] = {"matrix": lay.matrix, "pointers": lay.pointers, "bias": lay.bias, "mask": lay.step_mask,
                                  "n_added": lay.n_added, "n_removed": lay.n_removed}
    return out
