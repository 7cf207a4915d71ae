"""What this library is timed on: one pass of a stitched plan, or of a planned program, through the public
entry points, on device tensors.

Families and the ranges they stand for (sizes spread over their logarithm, half of them odd):

  layernorm       LayerNorm forward, fp32 / bf16 / fp16, 64 .. 32768 rows of 256 .. 8192
  softmax         scale + mask + softmax, the mask full or a key padding shared by heads and queries,
                  fp32 / fp16 / bf16, 16 .. 1024 keys
  attention       QK^T -> scale -> mask -> softmax -> PV (-> gate -> residual, log-sum-exp), fp16 / bf16,
                  1 .. 128 queries and 16 .. 128 keys per batch element, head dim 32 / 64 / 128
  gelu_layernorm  bias + GELU + residual + LayerNorm, bf16 / fp16 / fp32, as layernorm
  layernorm_bwd   dx, dgamma, dbeta, fp32, 256 .. 32768 rows of 128 .. 4096
  log_softmax     over a vocabulary, fp32 / bf16, 64 .. 4096 rows of 8192 .. 131072
  clip            gradients of a layer clipped by their global norm: a graph cut into several kernels by the
                  fusion planner

Calls that move less than SMALL bytes go through Plan.launch with the tensors at hand, as an eager program's
calls do; larger ones through arguments bound once, as a training or serving loop's do.
"""
import math

import torch

from paper_1911_11576_amd import BoundArgs, FusedProgram, Plan
from workloads import graphs

DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}
EPS = 1e-5
SMALL = 24 << 20
LARGEST = 400 << 20          # bytes of a drawn case


def listed():
    return [
        # one LayerNorm over a few hundred tokens: nothing but the latency of a call
        {"name": "layernorm_small", "family": "layernorm", "dtype": "f32", "rows": 256, "cols": 768},
        # the LayerNorm of a wide layer over a training batch
        {"name": "layernorm_wide", "family": "layernorm", "dtype": "bf16", "rows": 8192, "cols": 4096},
        # attention scores of 64 x 16 heads x 128 queries with a full mask
        {"name": "softmax_full_mask", "family": "softmax", "dtype": "f32", "b": 64, "h": 16, "q": 128, "s": 128, "mask": "full"},
        # image patches plus one token: rows of an odd length, the mask shared by heads and queries
        {"name": "softmax_key_padding", "family": "softmax", "dtype": "f16", "b": 32, "h": 12, "q": 197, "s": 197, "mask": "key_padding"},
        # causal self-attention over short sequences, batch x heads in one launch
        {"name": "attention_causal", "family": "attention", "dtype": "f16", "b": 4096, "q": 64, "s": 64, "d": 64, "causal": True, "mask": "", "extras": False},
        # one new token per sequence against a cache of keys and values, padded keys masked
        {"name": "attention_decode", "family": "attention", "dtype": "f16", "b": 4096, "q": 1, "s": 128, "d": 64, "causal": False, "mask": "key", "extras": False},
        # an attention block with gate, residual and log-sum-exp kept for the backward pass, odd length
        {"name": "attention_block", "family": "attention", "dtype": "bf16", "b": 1536, "q": 100, "s": 100, "d": 64, "causal": True, "mask": "key", "extras": True},
        # the tail of a Transformer layer, forward
        {"name": "gelu_layernorm", "family": "gelu_layernorm", "dtype": "bf16", "rows": 16384, "cols": 1024},
        # LayerNorm backward over a training batch: row and column reductions in one plan
        {"name": "layernorm_bwd", "family": "layernorm_bwd", "dtype": "f32", "rows": 32768, "cols": 1024},
        # ... of a wide layer
        {"name": "layernorm_bwd_wide", "family": "layernorm_bwd", "dtype": "f32", "rows": 4096, "cols": 4096},
        # log-probabilities over a vocabulary of an odd size
        {"name": "log_softmax_vocabulary", "family": "log_softmax", "dtype": "f32", "rows": 512, "cols": 50257},
        # gradient clipping over the eight tensors of a layer
        {"name": "clip_by_global_norm", "family": "clip", "dtype": "f32", "width": 1024, "inner": 4096, "layers": 1},
    ]


def _between(rng, lo, hi, step=1):
    """A size from lo to hi, even over the logarithm; half of them multiples of 64 (where the range allows), the others any."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5 and hi >= 128:
        n = max(64, n // 64 * 64)
    n = max(lo, min(hi, n))
    return max(step, n // step * step)


def _rows_within(rng, lo, hi, bytes_per_row):
    return _between(rng, lo, max(lo, min(hi, LARGEST // bytes_per_row)))


def draw(rng):
    family = rng.choice(["layernorm", "softmax", "attention", "gelu_layernorm", "layernorm_bwd", "log_softmax", "clip"])
    if family in ("layernorm", "gelu_layernorm"):
        dtype = rng.choice(["f32", "bf16", "f16"])
        cols = _between(rng, 256, 8192)
        return {"family": family, "dtype": dtype, "rows": _rows_within(rng, 64, 32768, 3 * SIZE[dtype] * cols), "cols": cols}
    if family == "softmax":
        dtype, mask = rng.choice(["f32", "f16", "bf16"]), rng.choice(["full", "key_padding"])
        s, h = _between(rng, 16, 1024), rng.choice([8, 12, 16])
        b = rng.randint(1, 64)
        b = max(1, min(b, LARGEST // (3 * SIZE[dtype] * h * s * s)))
        return {"family": family, "dtype": dtype, "b": b, "h": h, "q": s, "s": s, "mask": mask}
    if family == "attention":
        d, s = rng.choice([32, 64, 128]), _between(rng, 16, 128)
        q = 1 if rng.random() < 0.3 else s if rng.random() < 0.6 else _between(rng, 16, 128)
        extras = q > 1 and rng.random() < 0.4
        return {"family": family, "dtype": rng.choice(["f16", "bf16"]), "b": _rows_within(rng, 96, 8192, 8 * d * (q + s)), "q": q, "s": s, "d": d,
                "causal": q == s and q > 1 and rng.random() < 0.6, "mask": rng.choice(["", "key"]), "extras": extras}
    if family == "layernorm_bwd":
        cols = _between(rng, 128, 4096)
        return {"family": family, "dtype": "f32", "rows": _rows_within(rng, 256, 32768, 12 * cols), "cols": cols}
    if family == "log_softmax":
        dtype, cols = rng.choice(["f32", "bf16"]), _between(rng, 8192, 131072)
        return {"family": family, "dtype": dtype, "rows": _rows_within(rng, 64, 4096, 2 * SIZE[dtype] * cols), "cols": cols}
    width = _between(rng, 256, 2048, 4)
    return {"family": family, "dtype": "f32", "width": width, "inner": width * rng.choice([2, 3, 4]), "layers": rng.choice([1, 2])}


# ---------------------------------------------------------------- shapes, work

def _clip_shapes(c):
    w, i = c["width"], c["inner"]
    return [(w, w), (w,), (w, w), (w,), (w, i), (i,), (i, w), (w,)] * c["layers"]


def _ops(c):
    f = c["family"]
    if f == "layernorm":
        return graphs.layernorm_fwd(c["rows"], c["cols"], c["dtype"], EPS)
    if f == "gelu_layernorm":
        return graphs.bias_gelu_residual_layernorm(c["rows"], c["cols"], c["dtype"], EPS)
    if f == "softmax":
        return graphs.scaled_masked_softmax((c["b"], c["h"], c["q"], c["s"]), 0.125, c["mask"], c["dtype"])
    if f == "attention":
        x = c["extras"]
        return graphs.attention_block(c["b"], c["q"], c["s"], c["d"], c["dtype"], causal=c["causal"], mask=c["mask"] or None, gate=x, residual=x, lse=x)
    if f == "layernorm_bwd":
        return graphs.layernorm_bwd(c["rows"], c["cols"])
    if f == "log_softmax":
        return graphs.log_softmax((c["rows"], c["cols"]), c["dtype"])
    return graphs.clip_by_global_norm(_clip_shapes(c), 1.0)


def work(c):
    """Every group input read once, every output written once; of the operations, the dots (two per product) and a handful
    per element of the rest.  Clipping reads the gradients twice: no factor is known before the last of them is read."""
    clip = c["family"] == "clip"
    total = 0
    for op in _ops(c):
        if op.kind in ("parameter", "output"):
            total += math.prod(op.shape) * SIZE[op.dtype] * (2 if clip and op.kind == "parameter" else 1)
    dots = 4 * c["b"] * c["q"] * c["s"] * c["d"] // (2 if c["causal"] else 1) if c["family"] == "attention" else 0
    return {"bytes": total, "flops": max(dots, total)}


def tolerance(c):
    """About four times the distance from the 64-bit result: fp32 5e-8 .. 8e-8 (sums in another order add as much again,
    and a drawn norm over 10^7 terms more), fp16 2e-4 .. 3e-4, bf16 1.7e-3 .. 2.4e-3 (one rounding at the store, one of the
    attention weights); of single values, a rounding that falls the other way and what the weights' rounding adds."""
    if c["dtype"] == "f32":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 8e-3, "max": 3e-2} if c["dtype"] == "bf16" else {"rel": 1e-3, "max": 4e-3}


# ---------------------------------------------------------------- inputs and passes

def _inputs(c, seed):
    """The group's inputs in parameter order, rounded to their storage types."""
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    dt = DT[c["dtype"]]

    def normal(*shape, mean=0.0, std=1.0, dtype=dt):
        return (torch.randn(*shape, device="cuda:0", generator=gen) * std + mean).to(dtype)

    def uniform(*shape, dtype=dt):
        return torch.rand(*shape, device="cuda:0", generator=gen).to(dtype)

    def padding(*shape, dtype=dt):     # a tenth of the keys padded away
        return torch.where(torch.rand(*shape, device="cuda:0", generator=gen) < 0.1, -1e4, 0.0).to(dtype)

    f = c["family"]
    if f == "layernorm":
        n, k = c["rows"], c["cols"]
        return [normal(n, k), normal(k, mean=1.0, std=0.2), normal(k, std=0.1)]
    if f == "gelu_layernorm":
        n, k = c["rows"], c["cols"]
        return [normal(n, k), normal(k, std=0.02), normal(n, k), normal(k, mean=1.0, std=0.02), normal(k, std=0.02)]
    if f == "softmax":
        shape = (c["b"], c["h"], c["q"], c["s"])
        return [normal(*shape, std=2.0), padding(*(shape if c["mask"] == "full" else (c["b"], 1, 1, c["s"])))]
    if f == "attention":
        b, q, s, d = c["b"], c["q"], c["s"], c["d"]
        ins = [normal(b, q, d), normal(b, s, d), normal(b, s, d)]
        if c["mask"]:
            ins.append(padding(b, 1, s, dtype=torch.float32))
        return ins + ([uniform(b, q, d), normal(b, q, d)] if c["extras"] else [])
    if f == "layernorm_bwd":
        n, k = c["rows"], c["cols"]
        dy, x = normal(n, k), normal(n, k)
        mean = x.mean(dim=1)
        rstd = torch.rsqrt(x.var(dim=1, unbiased=False) + EPS)
        return [dy, x, normal(k, mean=1.0, std=0.02), mean, rstd]
    if f == "log_softmax":
        return [normal(c["rows"], c["cols"], std=3.0)]
    return [normal(*shape, std=0.01) for shape in _clip_shapes(c)]


def prepare(case, seed):
    ops, ins = _ops(case), _inputs(case, seed)
    if case["family"] == "clip":
        program = FusedProgram(ops)
        program.bind(ins)
        return {"program": program, "ins": ins}
    outs = [torch.empty(op.shape, dtype=DT[op.dtype], device="cuda:0") for op in ops if op.kind == "output"]
    state = {"plan": Plan(ops), "ins": ins, "outs": outs, "bound": None}
    if work(case)["bytes"] >= SMALL:
        state["bound"] = BoundArgs(ins, outs)
        state["stream"] = torch.cuda.current_stream().cuda_stream
    return state


def run(state):
    if "program" in state:
        return state["program"].run_bound()
    if state["bound"] is not None:
        state["plan"].launch_bound(state["bound"], state["stream"])
    else:
        state["plan"].launch(state["ins"], state["outs"])
    return state["outs"]


# ---------------------------------------------------------------- the same in 64 bits, plain torch

def _layernorm(r, gamma, beta):
    c = r - r.mean(dim=1, keepdim=True)
    return c * torch.rsqrt((c * c).mean(dim=1, keepdim=True) + EPS) * gamma + beta


def exact(case, seed):
    ins = [t.double() for t in _inputs(case, seed)]
    f = case["family"]
    if f == "layernorm":
        return [_layernorm(*ins)]
    if f == "gelu_layernorm":
        x, bias, res, gamma, beta = ins
        h = x + bias
        gelu = 0.5 * h * (1.0 + torch.tanh(0.7978845608028654 * (h + 0.044715 * h ** 3)))
        return [_layernorm(gelu + res, gamma, beta)]
    if f == "softmax":
        return [torch.softmax(ins[0] * 0.125 + ins[1], dim=-1)]
    if f == "attention":
        q, k, v = ins[:3]
        z = torch.matmul(q, k.transpose(1, 2).contiguous()) * case["d"] ** -0.5
        if case["mask"]:
            z = z + ins[3]
        if case["causal"]:
            above = torch.ones(case["q"], case["s"], dtype=torch.bool, device=z.device).triu(1)
            z = z.masked_fill(above, -math.inf)
        o = torch.matmul(torch.softmax(z, dim=-1), v)
        if not case["extras"]:
            return [o]
        return [o * ins[-2] + ins[-1], torch.logsumexp(z, dim=-1)]
    if f == "layernorm_bwd":
        dy, x, gamma, mean, rstd = ins
        rstd = rstd[:, None]
        xhat = (x - mean[:, None]) * rstd
        g = dy * gamma
        dx = (g - g.mean(dim=1, keepdim=True) - xhat * (g * xhat).mean(dim=1, keepdim=True)) * rstd
        return [dx, (dy * xhat).sum(dim=0), dy.sum(dim=0)]
    if f == "log_softmax":
        return [torch.log_softmax(ins[0], dim=-1)]
    norm = torch.sqrt(sum((t * t).sum() for t in ins))
    return [t / torch.clamp(norm, min=1.0) for t in ins]
