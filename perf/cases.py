"""The calls this library is timed and compared on, through its public Python
entry points: synchronisation rounds of every kind, the standalone statistics,
one GPU's share of a round, and the workers' inner AdamW step, from a few
thousand parameters (where launches and host work count) to the 1.1B-parameter
round (88 GB of traffic).

A case is a dict of plain values:
  kind    "round" (fused outer step), "stats" (round_stats), "int8" and "bf16"
          (the round with that payload), "share" (payload, shard step and reset
          of one GPU of k), "inner" (AdamW step of k workers)
  n, k    parameters and workers
  dtype   replica type, "f32" or "bf16"
  stats, reset   the outer step's flags ("inner": stats = the norms are read back)
  mean    int8 / bf16: the received mean is written out as well
  copy    inner: the BF16 compute copy is written as well
  spread  buffers from the library's spread allocator instead of torch's
"""
import math

import numpy as np
import torch

import paper_2609_36662_amd as al

EPS = 1e-12
CHUNK = 1 << 24          # elements per chunk of the 64-bit reference; a multiple of the codec block
BLOCK = 4096             # INT8 codec block
GPT2_SMALL = 124_439_808
LLAMA_1B1 = 1_100_048_384
# Selected interval of 750 steps against 500: rho, and the corrected coefficients
# of a base (0.7, 0.9).
RHO = 1.4914
MU = 0.9 ** RHO
ETA = 0.7 * RHO * (1 - MU) / (1 - 0.9)
# Inner AdamW, the C4 settings.
LR, BETA1, BETA2, ADAM_EPS, DECAY, CLIP, STEP = 4e-4, 0.9, 0.95, 1e-8, 0.1, 1.0, 1000
NORMS = (0.5, 2.0, 0.9, 4.0)   # gradient norms about the clipping threshold


def _case(name, kind, n, k, dtype="f32", stats=True, reset=True, mean=False, copy=False, spread=False):
    c = {"kind": kind, "n": n, "k": k, "dtype": dtype, "stats": stats, "reset": reset, "mean": mean, "copy": copy,
         "spread": spread}
    return dict(c, name=name) if name else c


def listed():
    return [
        # an adapter or a test model: the round is launches and host work
        _case("round 10k k2 f32", "round", 10_007, 2),
        # the smallest configuration of the repository's own bench
        _case("round tiny k4 f32", "round", 1 << 20, 4),
        # GPT-2 small, eight workers
        _case("round gpt2 k8 f32", "round", GPT2_SMALL, 8),
        # the headline round: 1.1B parameters, eight workers, buffers placed by the library
        _case("round 1.1b k8 f32", "round", LLAMA_1B1, 8, spread=True),
        # sixteen workers with bf16 replicas, 215M parameters (the pretraining size), a ragged count
        _case("round 215m k16 bf16", "round", 215_000_003, 16, dtype="bf16"),
        # the controller's statistics on their own (a drift check between synchronisations), ragged
        _case("stats 30m k8 bf16", "stats", 30_000_001, 8, dtype="bf16", reset=False),
        # the INT8 payload with sixteen workers, the encoded mean kept for distribution
        _case("int8 gpt2 k16 f32", "int8", GPT2_SMALL, 16, mean=True),
        # the INT8 payload with bf16 replicas that the trainer resets itself, a ragged last block
        _case("int8 215m k8 bf16", "int8", 215_000_003, 8, dtype="bf16", reset=False),
        # the BF16 payload of the main runs, the received mean kept
        _case("bf16 gpt2 k8 f32", "bf16", GPT2_SMALL, 8, mean=True),
        # one GPU of eight at 1.1B: payload, shard step, reset of its replica
        _case("share 1.1b k8 f32", "share", LLAMA_1B1, 8),
        # the inner optimiser of four workers, clipped, with the BF16 compute copies
        _case("inner gpt2 k4 copy", "inner", GPT2_SMALL, 4, copy=True),
        # the same on a tiny model, asynchronous (norms not read back)
        _case("inner tiny k4", "inner", 1 << 20, 4, stats=False),
    ]


def draw(rng):
    """A case of the same ranges: sizes over their logarithm from 5,000 parameters to a quarter of the headline round's
    traffic, any worker count the paper or the tests use, odd and ragged sizes among them."""
    kind = rng.choice(["round", "round", "round", "stats", "int8", "int8", "bf16", "share", "inner", "inner"])
    k = rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 8, 12, 16])
    if kind == "inner":
        k = min(k, 8)
    dtype = rng.choice(["f32", "bf16"])
    flags = [rng.random() < p for p in (0.8, 0.7, 0.4, 0.5)]
    c = _case("", kind, 1, k, dtype=dtype if kind != "inner" else "f32", stats=flags[0] or kind in ("stats", "share"),
              reset=flags[1] and kind not in ("stats", "inner"), mean=flags[2] and kind in ("int8", "bf16"),
              copy=flags[3] and kind == "inner")
    most = 22e9 / work(c)["bytes"]
    n = int(math.exp(rng.uniform(math.log(5e3), math.log(most))))
    c["n"] = n - n % rng.choice([1, 1, 4, 4096]) if n > 8192 else n
    return c


# ------------------------------------------------------------------- inputs --
def _normal(out, std, seed, role, k=0):
    g = torch.Generator(device=out.device)
    g.manual_seed((seed * 1_000_003 + role * 101 + k) & 0x7FFF_FFFF_FFFF_FFFF)
    torch.randn(out.shape, generator=g, device=out.device, dtype=torch.float32, out=out)
    return out.mul_(std)


def _shard(c):
    """Parameters of the first GPU's shard: n / k rounded up to whole runs of 8."""
    return min(c["n"], (c["n"] + c["k"] - 1) // c["k"] + 7 & ~7)


def _round_buffers(c, alloc):
    rdt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    t = alloc([torch.float32] * 2 + [rdt] * c["k"])
    return {"theta": t[0], "momentum": t[1], "replicas": t[2:]}


def _fill_round(c, seed, b):
    """theta ~ N(0, 0.02), momentum ~ N(0, 1e-4), replicas theta + 0.7 s + 0.3 e_k with s, e_k ~ N(0, 1e-3): the
    endpoints of workers that drift mostly together."""
    _normal(b["theta"], 0.02, seed, 1)
    _normal(b["momentum"], 1e-4, seed, 2)
    base = _normal(torch.empty_like(b["theta"]), 0.7e-3, seed, 3).add_(b["theta"])
    e = torch.empty_like(base)
    for k, r in enumerate(b["replicas"]):
        r.copy_(_normal(e, 0.3e-3, seed, 4, k).add_(base))
    return b


def _share_inputs(c, seed, dev):
    n, ns = c["n"], _shard(c)
    one = dict(c, k=1)
    b = _round_buffers(one, lambda dts: [torch.empty(n, dtype=d, device=dev) for d in dts])
    _fill_round(one, seed, b)
    base = _normal(torch.empty(ns, device=dev), 0.7e-3, seed, 5)
    e = torch.empty_like(base)
    b["payloads"] = [_normal(e, 0.3e-3, seed, 6, k).add_(base).to(torch.bfloat16) for k in range(c["k"])]
    b["momentum"] = b["momentum"][:ns].clone()   # a GPU keeps its own shard of the momentum
    return b


def _inner_inputs(c, seed, dev):
    n = c["n"]
    b = {"params": [], "exp_avg": [], "exp_avg_sq": [], "grads": []}
    for k in range(c["k"]):
        b["params"].append(_normal(torch.empty(n, device=dev), 0.02, seed, 7, k))
        b["exp_avg"].append(_normal(torch.empty(n, device=dev), 1e-4, seed, 8, k))
        b["exp_avg_sq"].append(_normal(torch.empty(n, device=dev), 1e-4, seed, 9, k).square_())
        b["grads"].append(_normal(torch.empty(n, device=dev), NORMS[k % 4] / math.sqrt(n), seed, 10, k))
    return b


def prepare(case, seed):
    c, n, dev = case, case["n"], "cuda"
    ctx = al.autoloco_create(0)
    s = {"case": c, "ctx": ctx}
    if c["kind"] == "inner":
        s.update(_inner_inputs(c, seed, dev))
        s["coeffs"] = al.make_adamw_coeffs(LR, STEP, BETA1, BETA2, ADAM_EPS, DECAY, CLIP)
        s["copy"] = [torch.empty(n, dtype=torch.bfloat16, device=dev) for _ in range(c["k"])] if c["copy"] else None
        return s
    s["coeffs"] = al.make_coeffs(MU, ETA, RHO, True)
    s["flags"] = (al.FUSE_STATS if c["stats"] else 0) | (al.FUSE_RESET if c["reset"] else 0)
    if c["kind"] == "share":
        s.update(_share_inputs(c, seed, dev))
        s["shard"] = s["theta"][:_shard(c)]
        s["payload"] = torch.empty(n, dtype=torch.bfloat16, device=dev)
        return s
    if c["spread"]:
        s.update(_fill_round(c, seed, _round_buffers(c, lambda dts: al.spread_tensors(ctx, n, dts)[0])))
    else:
        s.update(_fill_round(c, seed, _round_buffers(c, lambda dts: [torch.empty(n, dtype=d, device=dev) for d in dts])))
    s["mean"] = s["scales"] = None
    if c["mean"]:
        s["mean"] = torch.empty(n, dtype=torch.int8 if c["kind"] == "int8" else torch.bfloat16, device=dev)
        if c["kind"] == "int8":
            s["scales"] = torch.empty((n + BLOCK - 1) // BLOCK, device=dev)
    return s


# ---------------------------------------------------------------------- run --
def _stats(st, k):
    return None if st is None else [st.D, st.C, st.disagreement, st.sq_mean] + st.sq_norm[:k] + st.sq_dev[:k]


def run(s):
    c = s["case"]
    ctx, k = s["ctx"], c["k"]
    if c["kind"] == "inner":
        st = al.autoloco_inner_adamw(ctx, s["params"], s["exp_avg"], s["exp_avg_sq"], s["grads"], s["coeffs"],
                                     model_bf16=s["copy"], stats=c["stats"])
        return {"params": s["params"], "exp_avg": s["exp_avg"], "exp_avg_sq": s["exp_avg_sq"], "copy": s["copy"],
                "norms": None if st is None else st.grad_norm[:k]}
    if c["kind"] == "share":
        norm = al.autoloco_rank_payload(ctx, s["theta"], s["replicas"][0], s["payload"])
        mean = al.autoloco_shard_step(ctx, s["shard"], s["momentum"], s["payloads"], s["coeffs"])
        if c["reset"]:
            al.autoloco_broadcast_reset(ctx, s["theta"], s["replicas"])
        return {"payload": s["payload"], "theta": s["theta"], "momentum": s["momentum"], "replicas": s["replicas"],
                "stats": [norm, mean]}
    if c["kind"] == "stats":
        return {"stats": _stats(al.autoloco_round_stats(ctx, s["theta"], s["replicas"], EPS), k)}
    a = (ctx, s["theta"], s["momentum"], s["replicas"], s["coeffs"], s["flags"], EPS)
    if c["kind"] == "int8":
        st = al.autoloco_outer_step_int8(*a, mean_codes=s["mean"], mean_scales=s["scales"])
    elif c["kind"] == "bf16":
        st = al.autoloco_outer_step_bf16(*a, mean_bf16=s["mean"])
    else:
        st = al.autoloco_outer_step(*a)
    return {"theta": s["theta"], "momentum": s["momentum"], "replicas": s["replicas"], "mean": s["mean"],
            "scales": s["scales"], "stats": _stats(st, k)}


def work(case):
    c, n, k = case, case["n"], case["k"]
    r = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "inner":
        # theta, m, v in and out and the gradient once; about 15 operations an element
        return {"bytes": n * k * (28 + (2 if c["copy"] else 0)), "flops": 15 * n * k}
    if c["kind"] == "share":
        # payload: theta and the replica in, 2 bytes out; shard: theta and momentum in and out, k payloads in; reset
        return {"bytes": n * (4 + r + 2) + _shard(c) * (16 + 2 * k) + (n * (4 + r) if c["reset"] else 0),
                "flops": 4 * n + _shard(c) * (k + 8)}
    if c["kind"] == "stats":
        return {"bytes": n * (4 + k * r), "flops": 6 * n * k}
    out = 0 if not c["mean"] else 2 if c["kind"] == "bf16" else 1 + 4 / BLOCK
    return {"bytes": n * (16 + k * r * (2 if c["reset"] else 1) + out),
            "flops": n * k * ((6 if c["stats"] else 2) + (6 if c["kind"] == "int8" else 0))}


def tolerance(case):
    """fp32 elements carry a few roundings of 2^-24 and the sums are fp64 over fp32 terms: 4e-7 covers four times what is
    seen.  A bf16 output (replica, mean, copy) flips to its neighbour where the fp32 value before it moves over a tie:
    2^-8 of the element, on a share of them near 2^-16."""
    narrow = case["dtype"] == "bf16" or case["copy"] or case["kind"] in ("bf16", "share")
    return {"rel": 1e-4, "max": 1e-2} if narrow else {"rel": 4e-7, "max": 4e-5}


# ------------------------------------------------------------ 64-bit values --
def _bf16(x):
    return x.float().to(torch.bfloat16).double()


def _codec(x):
    """Encode and decode blocks of BLOCK elements (the last one padded): decoded values and the block scales."""
    m = x.numel()
    pad = -m % BLOCK
    b = torch.nn.functional.pad(x, (0, pad)).view(-1, BLOCK)
    top = b.abs().amax(1, keepdim=True)
    scale = torch.where(top == 0, torch.ones_like(top), (top / 127).clamp_min(2.0 ** -126))
    return (torch.round(b / scale).clamp_(-127, 127) * scale).view(-1)[:m], scale.view(-1)


def _step(theta, v, mean):
    dt = mean / RHO
    vn = MU * v + dt
    return theta - ETA * (dt + MU * vn), vn


def exact(case, seed):
    c, n, k, dev = case, case["n"], case["k"], "cuda"
    if c["kind"] == "inner":
        b = _inner_inputs(c, seed, dev)
        norms = [math.sqrt(sum(float(g[i:i + CHUNK].double().square().sum()) for i in range(0, n, CHUNK)))
                 for g in b["grads"]]
        out = {"params": [], "exp_avg": [], "exp_avg_sq": []}
        for j in range(k):
            coef = min(1.0, CLIP / (norms[j] + 1e-6))
            g = b["grads"][j].double().mul_(coef)
            m = b["exp_avg"][j].double().mul_(BETA1).add_(g, alpha=1 - BETA1)
            v = b["exp_avg_sq"][j].double().mul_(BETA2).addcmul_(g, g, value=1 - BETA2)
            p = b["params"][j].double().mul_(1 - LR * DECAY)
            den = v.sqrt().div_(math.sqrt(1 - BETA2 ** STEP)).add_(ADAM_EPS)
            p.addcdiv_(m, den, value=-LR / (1 - BETA1 ** STEP))
            for name, x in (("params", p), ("exp_avg", m), ("exp_avg_sq", v)):
                out[name].append(x)
        out["copy"] = out["params"] if c["copy"] else None
        out["norms"] = norms if c["stats"] else None
        return out
    if c["kind"] == "share":
        b, ns = _share_inputs(c, seed, dev), _shard(c)
        payload = b["theta"].double() - b["replicas"][0].double()
        norm = float(payload.square().sum())
        mean = _bf16(sum(p.double() for p in b["payloads"]) / k)
        theta = b["theta"].double()
        theta[:ns], v = _step(theta[:ns].clone(), b["momentum"].double(), mean)
        return {"payload": payload, "theta": theta, "momentum": v,
                "replicas": [theta] if c["reset"] else [b["replicas"][0]], "stats": [norm, float(mean.square().sum())]}
    b = _fill_round(c, seed, _round_buffers(c, lambda dts: [torch.empty(n, dtype=d, device=dev) for d in dts]))
    sums = torch.zeros(2 * k + 1, dtype=torch.float64, device=dev)
    f64 = dict(dtype=torch.float64, device=dev)
    step = c["kind"] != "stats"
    theta, mom = (torch.empty(n, **f64), torch.empty(n, **f64)) if step else (None, None)
    means, scales = [], []
    for i in range(0, n, CHUNK):
        at = slice(i, min(n, i + CHUNK))
        th = b["theta"][at].double()
        d = [th - r[at].double() for r in b["replicas"]]
        if c["kind"] == "int8":
            mean, sc = _codec(sum(_codec(x)[0] for x in d) / k)
            scales.append(sc)
        elif c["kind"] == "bf16":
            mean = _bf16(sum(_bf16(x) for x in d) / k)
        else:
            mean = sum(d) / k
        if c["mean"] and c["kind"] == "bf16":
            means.append(mean.to(torch.bfloat16))
        for j, x in enumerate(d):
            sums[j] += x.square().sum()
            sums[k + j] += (x - mean).square_().sum()
        sums[2 * k] += mean.square().sum()
        if step:
            theta[at], mom[at] = _step(th, b["momentum"][at].double(), mean)
        del d
    s = sums.tolist()
    big_d = sum(s[:k]) / k
    stats = [big_d, k * s[2 * k] / (big_d + EPS), sum(s[k:2 * k]) / k, s[2 * k]] + s[:2 * k]
    if not step:
        return {"stats": stats}
    return {"theta": theta, "momentum": mom, "replicas": [theta] * k if c["reset"] else b["replicas"],
            "mean": torch.cat(means).double() if means else None,
            "scales": torch.cat(scales) if c["mean"] and scales else None, "stats": stats if c["stats"] else None}
