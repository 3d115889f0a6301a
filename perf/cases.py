"""Performance cases of the selective FFN framework: what its users run, over the sizes they run.

Every case goes through the public functions of ``paper_2607_18081_amd``. Layers, activations
and active sets follow the synthetic recipe of the benchmark: weights N(0, 0.02), activations
N(0, 1), per-token active sets drawn without replacement from the loaded slots with Zipf
(rank^-1.1) popularity. Kinds:

``ffn``     one layer, B tokens with a set of k active slots each (decode, batch, prefill)
``stage``   consecutive layers of a decode stack, one token, captured once in a HIP graph and
            replayed per token, as a serving loop does
``dynset``  the dynamic active set of a prompt of T tokens
``scores``  Eq. 1 profiler scores of T tokens over a full layer, accumulated into the file's sums
``topk``    per-token top-k of a score matrix
"""
import math

import numpy as np
import torch

import paper_2607_18081_amd as si

DEV = "cuda:0"
W_STD = 0.02
ZIPF = 1.1
DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
FLAGS = {"": 0, "exact_h": si.FLAG_EXACT_H}
EPS = 1e-5


def listed():
    return [
        # the smallest call: a tiny float32 layer, one token (launches and latency)
        dict(name="tiny_f32_decode", kind="ffn", B=1, d=256, L=512, k=128, dt="f32", hot=0,
             flags=""),
        # the ordinary decode step: 7B-shape layer, 70% of 11008 neurons loaded, 20% active
        dict(name="decode_7b", kind="ffn", B=1, d=4096, L=7706, k=2202, dt="bf16", hot=0,
             flags=""),
        # four concurrent decode streams over the same layer
        dict(name="decode_7b_x4", kind="ffn", B=4, d=4096, L=7706, k=2202, dt="bf16", hot=0,
             flags=""),
        # a pipeline stage of the 8B-shape stack: 4 of its 32 layers, replayed per token
        dict(name="stage_8b", kind="stage", layers=4, d=4096, L=8602, k=2150, dt="bf16"),
        # batch-16 decode with the shared hot core of a common prompt
        dict(name="batch16_7b", kind="ffn", B=16, d=4096, L=7706, k=2202, dt="bf16", hot=1101,
             flags=""),
        # an odd-sized serving batch of the 13B-shape layer in IEEE half, the paper's storage type
        dict(name="batch45_13b_f16", kind="ffn", B=45, d=5120, L=9677, k=3456, dt="f16", hot=0,
             flags=""),
        # a short ragged prompt over the 8B-shape layer with h kept at 16 significant bits
        dict(name="prefill200_8b_exact", kind="ffn", B=200, d=4096, L=8602, k=2150, dt="bf16",
             hot=0, flags="exact_h"),
        # the benchmark's prefill: 512 tokens of the 13B-shape layer
        dict(name="prefill512_13b", kind="ffn", B=512, d=5120, L=9677, k=3456, dt="bf16", hot=0,
             flags=""),
        # a long prompt in IEEE half over the 7B-shape layer
        dict(name="prefill2048_7b_f16", kind="ffn", B=2048, d=4096, L=7706, k=2202, dt="f16",
             hot=0, flags=""),
        # the dynamic set of a 512-token prompt (30% static, 40% of 13824 neurons in all)
        dict(name="dynset512_13b", kind="dynset", T=512, d=5120, L=9677, n_static=4147,
             n_total=5530, dt="bf16"),
        # one profiling call: 512 tokens over the whole 8B-shape layer
        dict(name="scores512_8b", kind="scores", T=512, d=4096, L=14336, dt="bf16"),
        # the active sets of 16 tokens picked from their scores
        dict(name="topk16_7b", kind="topk", B=16, L=7706, k=2202),
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["ffn1", "ffn4", "ffn_b", "ffn_b", "ffn_p", "ffn_p", "stage", "dynset",
                       "scores", "topk", "f32"])
    # widths of the named configurations as often as odd multiples of 8
    d = rng.choice([2048, 3072, 4096, 5120]) if rng.random() < 0.5 else _log_int(rng, 512, 8192, 8)
    n = _log_int(rng, 2 * d, min(4 * d, 16384))
    L = int(n * rng.uniform(0.5, 0.8))
    k = max(1, int(n * rng.uniform(0.1, 0.3)))
    dt = rng.choice(["bf16", "bf16", "f16"])
    ffn = dict(kind="ffn", d=d, L=L, k=k, dt=dt, hot=0, flags="")
    if kind == "f32":
        d = _log_int(rng, 128, 2048, 4)
        L = int(4 * d * rng.uniform(0.5, 0.8))
        return dict(ffn, B=rng.randint(1, 8), d=d, L=L, k=max(1, int(L * rng.uniform(0.1, 0.4))),
                    dt="f32")
    if kind == "ffn1":
        return dict(ffn, B=1)
    if kind == "ffn4":
        return dict(ffn, B=rng.randint(2, 4))
    if kind == "ffn_b":
        return dict(ffn, B=_log_int(rng, 5, 127), hot=rng.choice([0, k // 2]))
    if kind == "ffn_p":
        # at most the work of the largest listed case
        top = min(2048, int(2048 * 4096 * 7706 / (d * L)))
        return dict(ffn, B=_log_int(rng, 128, max(129, top)), flags=rng.choice(["", "", "exact_h"]))
    if kind == "stage":
        return dict(kind="stage", layers=rng.randint(2, 5), d=min(d, 5120), L=L, k=k, dt="bf16")
    if kind == "topk":
        return dict(kind="topk", B=_log_int(rng, 1, 512), L=L, k=k)
    T = _log_int(rng, 128, max(129, min(1024, int(512 * 5120 * 9677 / (d * L)))))
    if kind == "dynset":
        return dict(kind="dynset", T=T, d=d, L=L, n_static=int(0.4 * L), n_total=int(0.57 * L),
                    dt=dt)
    return dict(kind="scores", T=T, d=d, L=L, dt=dt)


# ---- inputs ------------------------------------------------------------------------------------

def _normal(g, dtype, std, *shape):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=g)


def _sets(g, B, L, k, hot):
    """CSR active sets: k slots a token, sampled with Zipf popularity (Efraimidis-Spirakis keys),
    the `hot` most popular slots in every token's set."""
    rank = torch.randperm(L, generator=g, device=DEV).double() + 1.0
    u = torch.rand((B, L), generator=g, device=DEV, dtype=torch.float64).clamp_min(1e-300)
    keys = u.log() * rank.pow(ZIPF)
    if hot:
        keys[:, rank <= hot] = math.inf
    idx = torch.topk(keys, k, dim=1).indices.sort(dim=1).values
    off = torch.arange(0, (B + 1) * k, k, dtype=torch.int32, device=DEV)
    return off, idx.to(torch.int32).reshape(-1).contiguous()


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    kind = case["kind"]
    s = {"case": case}
    if kind == "topk":
        # activations of a SwiGLU layer: a product of two normal factors
        a = _normal(g, torch.float32, 1.0, case["B"], case["L"])
        s["scores"] = torch.nn.functional.silu(a) * _normal(g, torch.float32, 1.0, *a.shape)
        return s
    dtype = DTYPES[case["dt"]]
    d, L = case["d"], case["L"]
    if kind == "stage":
        s["layers"] = []
        for _ in range(case["layers"]):
            off, idx = _sets(g, 1, L, case["k"], 0)
            s["layers"].append((_normal(g, dtype, W_STD, L, 2, d), _normal(g, dtype, W_STD, L, d),
                                off, idx))
        s["x"] = _normal(g, dtype, 1.0, 1, d)
        s["ws"] = torch.empty(max(256, si.selective_ffn_workspace(1, case["k"], L, d)),
                              dtype=torch.uint8, device=DEV)
        s["xs"] = [torch.empty_like(s["x"]) for _ in range(case["layers"])]
        s["ys"] = [torch.empty((1, d), dtype=torch.float32, device=DEV) for _ in s["layers"]]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _stage(s)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _stage(s)
        return s
    s["gate_up"] = _normal(g, dtype, W_STD, L, 2, d)
    if kind == "ffn":
        s["down"] = _normal(g, dtype, W_STD, L, d)
        s["x"] = _normal(g, dtype, 1.0, case["B"], d)
        s["off"], s["idx"] = _sets(g, case["B"], L, case["k"], case["hot"])
    else:
        s["x"] = _normal(g, dtype, 1.0, case["T"], d)
        if kind == "dynset":
            s["static"] = torch.randperm(L, generator=g, device=DEV)[: case["n_static"]].to(
                torch.int32)
        else:
            s["scores"] = torch.zeros(L, dtype=torch.float64, device=DEV)
    return s


# ---- one pass ----------------------------------------------------------------------------------

def _stage(s):
    """One token through the stage: each layer after the first normalises the pair (x, y) of the
    one before; the last pair leaves as the next stage's input."""
    x = s["x"]
    for i, (gu, dn, off, idx) in enumerate(s["layers"]):
        if i == 0:
            si.selective_ffn(x, off, idx, gu, dn, y=s["ys"][0], workspace=s["ws"])
        else:
            si.selective_ffn_resnorm(x, s["ys"][i - 1], off, idx, gu, dn, eps=EPS,
                                     x_out=s["xs"][i - 1], y=s["ys"][i], workspace=s["ws"])
            x = s["xs"][i - 1]
    si.residual_rmsnorm(x, s["ys"][-1], eps=EPS, out=s["xs"][-1])


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "ffn":
        return si.selective_ffn(s["x"], s["off"], s["idx"], s["gate_up"], s["down"],
                                flags=FLAGS[case["flags"]])
    if kind == "stage":
        s["graph"].replay()
        return {"x": s["xs"], "y": s["ys"]}
    if kind == "dynset":
        out, counts = si.dynamic_set(s["x"], s["gate_up"], s["static"], case["n_total"],
                                     case["n_total"])
        return {"slots": out, "counts": counts}
    if kind == "scores":
        return si.profile_scores(s["x"], s["gate_up"], scores=s["scores"])
    return si.select_topk(s["scores"], case["k"])


# ---- what a pass cannot do without ---------------------------------------------------------------

def _union(B, L, k, hot):
    """Expected size of the union of B sampled sets: slot i is in a set with probability
    1 - exp(-t w_i), t such that the probabilities add up to k."""
    w = np.arange(hot + 1, L + 1, dtype=np.float64) ** -ZIPF
    need = k - hot
    if need <= 0 or B == 1:
        return float(k)
    lo, hi = 0.0, 1.0
    while np.sum(-np.expm1(-hi * w)) < need and hi < 1e12:
        hi *= 2.0
    for _ in range(60):
        t = 0.5 * (lo + hi)
        lo, hi = (t, hi) if np.sum(-np.expm1(-t * w)) < need else (lo, t)
    return hot + float(np.sum(-np.expm1(-B * hi * w)))


def work(case):
    kind = case["kind"]
    if kind == "topk":
        return {"bytes": case["B"] * (case["L"] + case["k"]) * 4, "flops": 0}
    d, L = case["d"], case["L"]
    es = 4 if case["dt"] == "f32" else 2
    if kind == "ffn":
        B, k = case["B"], case["k"]
        rows = _union(B, L, k, case["hot"])
        return {"bytes": rows * 3 * d * es + B * d * (es + 4) + B * k * 4,
                "flops": 6.0 * d * k * B}
    if kind == "stage":
        n = case["layers"]
        return {"bytes": n * (case["k"] * (3 * d * es + 4) + d * (es + 8)),
                "flops": n * 6.0 * d * case["k"]}
    T = case["T"]
    out = 4 * (L + case["n_total"]) if kind == "dynset" else 16 * L
    return {"bytes": 2 * L * d * es + T * d * es + out, "flops": 4.0 * T * L * d}


def tolerance(case):
    kind = case["kind"]
    if kind == "topk":
        return "exact"
    if kind == "dynset":
        # tokens whose alpha-th keys tie within float32 rounding may rank them the other way
        return {"rel": 1e-5, "differ": 0.005}
    if kind == "scores":
        return {"rel": 1e-5}
    if kind == "stage":
        # x is rounded to bf16 between layers: a last-bit difference in a sum can flip a rounding
        # (1.2e-3 to 2e-3 from the 64-bit chain after four layers)
        return {"rel": 8e-3}
    if case["B"] < 128 or case["flags"] == "exact_h":
        return {"rel": 1e-5}    # 32-bit sums; from 5 tokens h as a 16-bit hi + lo pair (2.6e-6)
    # h as one 16-bit value: 1.7e-3 from the 64-bit result in bf16, 2.1e-4 in half
    return {"rel": 7e-3 if case["dt"] == "bf16" else 8.4e-4}


# ---- the same in 64 bits -------------------------------------------------------------------------

def _ffn64(x, off, idx, gate_up, down):
    B, L = x.shape[0], gate_up.shape[0]
    x = x.double()
    h = torch.nn.functional.silu(x @ gate_up[:, 0].double().t()) * \
        (x @ gate_up[:, 1].double().t())
    mask = torch.zeros((B, L), dtype=torch.bool, device=DEV)
    tok = torch.repeat_interleave(torch.arange(B, device=DEV), (off[1:] - off[:-1]).long())
    mask[tok, idx.long()] = True
    return torch.where(mask, h, 0.0) @ down.double()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("topk", "dynset"):
        return None                            # slots and counts: no computed numbers
    s = prepare(case, seed)
    if kind == "ffn":
        return _ffn64(s["x"], s["off"], s["idx"], s["gate_up"], s["down"])
    if kind == "stage":
        # only the first layer's sums: after it x is rounded to bf16, and the distance from a
        # 64-bit chain tells which elements lay beside a rounding boundary, not how exact the
        # sums are (2e-6 to 8e-6 in the first x from one seed to the next)
        gu, dn, off, idx = s["layers"][0]
        none = [None] * (case["layers"] - 1)
        return {"x": [None] + none, "y": [_ffn64(s["x"], off, idx, gu, dn)] + none}
    x = s["x"].double()
    a = torch.nn.functional.silu(x @ s["gate_up"][:, 0].double().t()) * \
        (x @ s["gate_up"][:, 1].double().t())
    return a.abs().sum(dim=0)
