"""Performance cases: the calls that a program around this library makes, at the sizes and options it is used with.

Five kinds of work, told apart by `kind`:
  linear   one projection, called the plain way (`gwq.linear`, which allocates its result)
  decode   one token of `m` sequences through `layers` decoder layers: q/k/v grouped, o, the gated pair and the down
           projection on its result (seven single calls where activations are bfloat16); calls prepared once and
           replayed from one HIP graph, as a generation loop does
  prefill  the seven products of a decoder layer on `m` > 16 rows, called the plain way
  pack     quantising a layer: `gwq.pack` of its q, gate and down matrices, then `gwq.quality` of each
  score    calibrating one matrix: the mean of its weight gradient over two samples of `m` tokens (`gwq.score`)
Shapes are those of the 7B and 70B layers of the benchmark and the tests; `draw` spreads over the sizes around them.
"""
import math

import torch

import paper_2411_00850_amd as gwq

# What the draws stay below: the work of the largest listed case of each kind.
_MOST_WEIGHTS = {"linear": 230e6, "decode": 600e6, "prefill": 600e6, "pack": 110e6, "score": 45e6}
_MOST_FLOPS = {"prefill": 0.6e12, "score": 0.3e12}


def listed():
    b7 = dict(hidden=4096, kv=4096, ffn=11008)
    b70 = dict(hidden=8192, kv=1024, ffn=28672)
    fmt = dict(bits=4, group=128, ppm=10000, scores="free", dtype="float16")
    return [
        # the smallest call: one projection for one token, host path included
        dict(name="linear_1", kind="linear", n=4096, k=4096, m=1, **fmt),
        # single-stream generation on the 7B shapes: the benchmark's own configuration, four layers of the model
        dict(name="decode_1", kind="decode", layers=4, m=1, **b7, **fmt),
        # the group size that the method's paper uses, a few sequences at once
        dict(name="decode_4_group16", kind="decode", layers=2, m=4, **b7, **dict(fmt, group=16)),
        # 3-bit weights, a small batch
        dict(name="decode_8_int3", kind="decode", layers=2, m=8, **b7, **dict(fmt, bits=3)),
        # the largest decode batch
        dict(name="decode_16", kind="decode", layers=2, m=16, **b7, **fmt),
        # a model that computes in bfloat16, an odd number of sequences
        dict(name="decode_11_bf16", kind="decode", layers=2, m=11, **b7, **dict(fmt, dtype="bfloat16")),
        # single-stream generation on the 70B shapes, outliers clustered in few columns
        dict(name="decode_1_70b", kind="decode", layers=1, m=1, **b70, **dict(fmt, scores="columns")),
        # a short prompt (or a batch too large for decode) on the 70B shapes
        dict(name="prefill_64_70b", kind="prefill", m=64, **b70, **dict(fmt, scores="columns")),
        # an odd prompt length at 3 bits and the paper's group size
        dict(name="prefill_301_int3_group16", kind="prefill", m=301, **b7, **dict(fmt, bits=3, group=16)),
        # a full prompt on the 7B shapes: the benchmark's prefill configuration
        dict(name="prefill_2048", kind="prefill", m=2048, **b7, **fmt),
        # quantising a 7B layer from FP32 scores
        dict(name="pack_7b", kind="pack", hidden=4096, ffn=11008, score_type="float32", bits=4, group=128, ppm=10000, scores="free"),
        # calibrating the down projection of a 7B layer
        dict(name="score_2048", kind="score", n=4096, k=11008, m=2048),
    ]


def _log_int(rng, low, high):
    """Whole number from low to high, even over the logarithm."""
    return min(high, max(low, int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))))


def _width(rng, low, high):
    """A row length: a multiple of 128."""
    return 128 * _log_int(rng, low // 128, high // 128)


def draw(rng):
    while True:
        kind = rng.choice(["linear", "decode", "decode", "decode", "prefill", "prefill", "pack", "score"])
        fmt = dict(bits=rng.choice([4, 4, 3]), group=rng.choice([128, 128, 64, 32, 16]), ppm=rng.choice([10000, 10000, 5000, 1000]),
                   scores=rng.choice(["free", "columns"]), dtype="float16")
        if fmt["group"] == 128 and rng.random() < 0.3:
            fmt["dtype"] = "bfloat16"
        hidden, ffn = _width(rng, 1024, 8192), _width(rng, 2048, 28672)
        kv = rng.choice([hidden, max(128, hidden // 4), max(128, hidden // 8)])
        if kind == "linear":
            case = dict(kind=kind, n=_log_int(rng, 257, 50000), k=_width(rng, 1024, 16384), m=_log_int(rng, 1, 300), **fmt)
        elif kind == "decode":
            case = dict(kind=kind, layers=rng.randint(1, 4), m=_log_int(rng, 1, 16), hidden=hidden, kv=kv, ffn=ffn, **fmt)
        elif kind == "prefill":
            case = dict(kind=kind, m=_log_int(rng, 17, 3000), hidden=hidden, kv=kv, ffn=ffn, **fmt)
        elif kind == "pack":
            del fmt["dtype"]
            case = dict(kind=kind, hidden=hidden, ffn=ffn, score_type=rng.choice(["float32", "float32", "float16"]), **fmt)
        else:
            case = dict(kind=kind, n=_log_int(rng, 129, 16384), k=_width(rng, 1024, 16384), m=_log_int(rng, 100, 3000))
        if work(case)["flops"] > _MOST_FLOPS.get(kind, 1e18):
            continue
        if case.get("layers", 1) * sum(n * k for n, k in _matrices(case)) <= _MOST_WEIGHTS[kind]:
            return case


def _matrices(case):
    """(N, K) of the matrices of one layer (or of the single one): q, k, v, o, gate, up, down."""
    if case["kind"] in ("linear", "score"):
        return [(case["n"], case["k"])]
    h, f = case["hidden"], case["ffn"]
    if case["kind"] == "pack":
        return [(h, h), (f, h), (h, f)]
    return [(h, h), (case["kv"], h), (case["kv"], h), (h, h), (f, h), (f, h), (h, f)]


def _weight(n, k, gen):
    """FP16 [n, k]: 0.02 * Student-t(df=4), eight input columns x20."""
    z = torch.randn((n, k), generator=gen, device="cuda")
    u = (1 - torch.rand((n, k), generator=gen, device="cuda")) * (1 - torch.rand((n, k), generator=gen, device="cuda"))
    w = z.mul_(0.02).div_(u.log_().mul_(-0.5).clamp_(min=1e-6).sqrt_())
    cols = torch.randperm(k, generator=gen, device="cuda")[:8]
    w[:, cols] *= 20.0
    return w.clamp_(-3e4, 3e4).half()


def _score(w, how, ppm, gen):
    """FP32 scores: |N(0,1)| * |W|, or ("columns") a share of ppm of the entries raised, 60 % of them in 1 % of the columns."""
    n, k = w.shape
    if how == "free":
        return torch.randn((n, k), generator=gen, device="cuda").abs_().mul_(w.abs())
    share = torch.full((k,), 0.4 * ppm * 1e-6, device="cuda")
    share[torch.randperm(k, generator=gen, device="cuda")[:max(1, k // 100)]] = min(1.0, 60.0 * ppm * 1e-6)
    s = torch.rand((n, k), generator=gen, device="cuda")
    return s.add_(torch.rand((n, k), generator=gen, device="cuda").lt_(share), alpha=2.0)


def _activations(m, k, gen, dtype, hot=False):
    """[m, k] ~ N(0,1); `hot`: 0.1 % of the channels x50."""
    x = torch.randn((m, k), generator=gen, device="cuda")
    if hot:
        x[:, torch.randperm(k, generator=gen, device="cuda")[:max(1, k // 1000)]] *= 50.0
    return x.to(dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, shapes = case["kind"], _matrices(case)
    if kind == "score":
        n, k, m = case["n"], case["k"], case["m"]
        samples = [(_activations(m, n, gen, torch.float16).mul_(0.01), _activations(m, k, gen, torch.float16, hot=True)) for _ in range(2)]
        return dict(kind=kind, samples=samples, out=torch.empty((n, k), device="cuda"))

    def packed(n, k):
        w = _weight(n, k, gen)
        return gwq.pack(w, _score(w, case["scores"], case["ppm"], gen), case["bits"], case["ppm"], group=case["group"])

    if kind == "pack":
        pairs = []
        for n, k in shapes:
            w = _weight(n, k, gen)
            pairs.append((w, _score(w, case["scores"], case["ppm"], gen).to(getattr(torch, case["score_type"]))))
        return dict(kind=kind, pairs=pairs, bits=case["bits"], ppm=case["ppm"], group=case["group"])
    m, dtype = case["m"], getattr(torch, case["dtype"])
    if kind in ("linear", "prefill"):
        xs = {k: _activations(m, k, gen, dtype, hot=kind == "prefill") for k in sorted({k for _, k in shapes})}
        layers = [packed(n, k) for n, k in shapes]
        return dict(kind=kind, linear=gwq.linear if dtype is torch.float16 else gwq.linear_bf16, calls=[(p, xs[p.K]) for p in layers])
    calls, outs, keep = [], [], []
    for _ in range(case["layers"]):
        q, k, v, o, gate, up, down = ps = [packed(n, k) for n, k in shapes]
        x1, x2, x3 = (_activations(m, case["hidden"], gen, dtype) for _ in range(3))
        if dtype is torch.float16:
            y = [torch.empty((m, p.N), dtype=dtype, device="cuda") for p in (q, k, v, o, gate, down)]
            calls += [gwq.prepare_linear_batch([q, k, v], [x1] * 3, y[:3]), gwq.prepare_linear(o, x2, y[3]),
                      gwq.prepare_linear_gate_up(gate, up, x3, y[4]), gwq.prepare_linear(down, y[4], y[5])]
            keep.append((ps, x1, x2, x3))
        else:
            y = [torch.empty((m, p.N), dtype=dtype, device="cuda") for p in ps]
            x4 = _activations(m, case["ffn"], gen, dtype)
            calls += [lambda p=p, x=x, out=out: gwq.linear_bf16(p, x, out=out) for p, x, out in zip(ps, (x1, x1, x1, x2, x3, x3, x4), y)]
            keep.append((ps, x1, x2, x3, x4))
        outs += y
    for call in calls:                                  # once outside the capture, as every program that captures does
        call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for call in calls:
            call()
    return dict(kind=kind, graph=graph, calls=calls, outs=outs, keep=keep)


def run(state):
    kind = state["kind"]
    if kind == "decode":
        state["graph"].replay()
        return state["outs"]
    if kind in ("linear", "prefill"):
        return [state["linear"](p, x) for p, x in state["calls"]]
    if kind == "score":
        (dy0, x0), (dy1, x1) = state["samples"]
        gwq.score(dy0, x0, out=state["out"], alpha=0.5)
        return gwq.score(dy1, x1, out=state["out"], alpha=0.5, beta=1.0)
    got = []
    for w, s in state["pairs"]:
        p = gwq.pack(w, s, state["bits"], state["ppm"], group=state["group"])
        merit = gwq.quality(p, w, s)
        groups = p.N * (p.K // p.group)                 # the arrays' padding is never written
        got.append([p.qweight, p.scales[:groups], p.zeros[:groups], p.row_ptr, p.col_idx[:p.n_outliers], p.out_val[:p.n_outliers], merit])
    return got


def _packed_bytes(case, n, k):
    outliers = math.ceil(case["ppm"] * n * k / 1e6)
    return n * (k // 128) * (64 if case["bits"] == 4 else 52) + 3 * n * (k // case["group"]) + 4 * outliers + 4 * (n + 1)


def work(case):
    kind, shapes = case["kind"], _matrices(case)
    if kind == "score":
        n, k, m = case["n"], case["k"], case["m"]
        return {"bytes": 2 * 2 * m * (n + k) + 4 * n * k, "flops": 2 * 2 * m * n * k}
    if kind == "pack":                                  # weights and scores read, the packed layer and three numbers written
        score_bytes = 4 if case["score_type"] == "float32" else 2
        return {"bytes": sum(n * k * (2 + score_bytes) + _packed_bytes(case, n, k) + 24 for n, k in shapes), "flops": 0}
    m, layers = case["m"], case.get("layers", 1)
    outliers = [math.ceil(case["ppm"] * n * k / 1e6) for n, k in shapes]
    nbytes = sum(_packed_bytes(case, n, k) for n, k in shapes)
    if kind == "linear":
        nbytes += 2 * m * (case["n"] + case["k"])
    else:                                               # inputs of q/k/v, o, gate/up and down; outputs (gate and up are one)
        h, f = case["hidden"], case["ffn"]
        pair = 1 if kind == "decode" and case["dtype"] == "float16" else 2
        nbytes += 2 * m * (3 * h + f) + 2 * m * (h + 2 * case["kv"] + h + pair * f + h)
    return {"bytes": layers * nbytes, "flops": layers * (2 * m * sum(n * k for n, k in shapes) + 2 * m * sum(outliers))}


def tolerance(case):
    """About four times the distance of a correct result from the fp64 product of the same packed layer, as measured."""
    if case["kind"] == "pack":                          # whole numbers and FP16 bits are exact; the merits are fp64 sums in some order
        return {"rel": 1e-10, "differ": 0.0}
    if case["kind"] == "score":                         # FP32 sums of exact products over m: 2.9e-7, largest difference 1.9e-5
        return {"rel": 2e-6, "max": 1e-4}
    if case["dtype"] == "bfloat16":                     # the bfloat16 store alone: 1.7e-3; weights rounded to bfloat16 for m > 16
        return {"rel": 8e-3, "max": 4e-2}
    return {"rel": 1.5e-3, "max": 1e-2}                 # 2.0e-4 (one product) to 4.9e-4 (down on the gated pair), 2.4e-3
