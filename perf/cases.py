"""Timed workloads of the stage library: what a pipeline runtime has one stage do in one iteration.

A case is one stage and one iteration on it: F of every microbatch, then B and W of every microbatch (or any
other legal order), then stage_grad_reduce.  `prepare` makes what a training program holds between iterations
(parameters, arena, handle, the tensors that arrive from the neighbour stages), `run` is the iteration, and its
outputs are everything the iteration produces: the outputs and input gradients of all microbatches and the
reduced parameter gradients.

The model widths are the five workloads of `stage_inputs` and smaller or mixed ones of the same families;
microbatch counts are reduced so that several copies fit one card (the tasks of a microbatch do not depend on
how many there are).  Segment lengths of a microbatch are separated by ",", microbatches by "|".
"""
from __future__ import annotations

import math

import torch

import paper_2605_18750_amd as R
import stage_inputs as SI

DEVICE = "cuda:0"

# Defaults of a case; the entries of listed() and draw() state what differs.
BASE = dict(layers=1, hidden=4096, q_heads=32, kv_heads=32, head_dim=128, ffn=11008, dtype="bf16", mlp="swiglu",
            causal=True, norm="rms", bias=False, rope=False, qk_norm=False, w_std=0.02, x_std=1.0, streams=1,
            order="drain", tokens="4096")


def _case(shape=None, **kw):
    c = dict(BASE)
    if shape is not None:
        c.update(layers=shape.n_layers, hidden=shape.hidden, q_heads=shape.n_q_heads, kv_heads=shape.n_kv_heads,
                 head_dim=shape.head_dim, ffn=shape.ffn, dtype=shape.dtype, mlp=shape.mlp_kind, causal=shape.causal,
                 x_std=shape.x_std, w_std=shape.w_std)
    c.update(kw)
    return c


def listed():
    img = SI.VISION_TOKENS_PER_IMAGE
    return [
        # The smallest stage of the repository, in fp32: bring-up, numerical debugging, unit tests of a runtime.
        # Every kernel is short, so launches and host work count.
        _case(SI.TINY, name="tiny_fp32", tokens="128|128|128|128"),
        # fp32 at a size someone trains a small model with, ragged packed samples and grouped heads.
        _case(name="fp32_packed", layers=2, hidden=1024, q_heads=16, kv_heads=4, head_dim=64, ffn=2752, dtype="fp32",
              tokens="300,724|517"),
        # A small bf16 stage with ragged microbatches: the many-small-calls end of the bf16 path.
        _case(name="small_bf16", layers=2, hidden=512, q_heads=8, kv_heads=2, head_dim=64, ffn=1536, w_std=0.04,
              tokens="300,477|100|33,64,1|129"),
        # The language stage, the workload the benchmark quotes.
        _case(SI.LANGUAGE, name="language_4k", tokens="4096|4096"),
        # The same stage with the short microbatches of fine-tuning or of a long pipeline cut into many microbatches.
        _case(SI.LANGUAGE, name="language_short", tokens="512|77,223|256|419"),
        # Text plus image tokens: microbatches of one iteration differ by a factor of eight, some hold two samples.
        _case(SI.MULTIMODAL, name="multimodal", tokens="1093|6136|791,1032|2815"),
        # The widest stage, grouped query heads.
        _case(SI.WIDE_GQA, name="wide_gqa", tokens="4096"),
        # Image encoder as stated: bidirectional, head dimension 80, GELU.
        _case(SI.VISION, name="vision", tokens="|".join([",".join([str(img)] * 8)] * 2)),
        # The image encoder with its tasks issued in a random ready order over three streams, as a readiness-driven
        # runtime issues them, with fewer images per microbatch.
        _case(SI.VISION, name="vision_ready_order", layers=4, tokens="|".join([",".join([str(img)] * 3)] * 4), streams=3,
              order="ready"),
        # The encoder variant with LayerNorm and projection biases on images of different sizes.
        _case(SI.VISION, name="vision_layernorm_bias", layers=4, norm="layer", bias=True,
              tokens="256,1024,784,577|1024,196,900"),
        # The language stage with head norms and rotary embedding and grouped heads, two packed samples.
        _case(SI.LANGUAGE, name="language_qknorm_rope", layers=2, kv_heads=8, qk_norm=True, rope=True,
              tokens="1500,548|2048"),
        # Many short samples packed into one microbatch (instruction data): attention over 20 segments.
        _case(name="packed_short", layers=2, hidden=2048, q_heads=32, kv_heads=8, head_dim=64, ffn=5632,
              tokens="201,64,333,97,412,150,38,275,511,120,89,166,240,73,301,55,190,128,402,251"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cut(rng, total, most):
    """`total` tokens cut into up to `most` ragged segments."""
    n = rng.randint(1, max(1, min(most, total // 24)))
    cuts = sorted(rng.sample(range(1, total), n - 1)) if n > 1 else []
    return ",".join(str(b - a) for a, b in zip([0] + cuts, cuts + [total]))


def draw(rng):
    """One more case of the ranges above: small to large stages, both types, all variants, ragged token counts."""
    kind = rng.choice(["fp32", "small", "language", "language", "multimodal", "wide", "vision", "vision", "packed"])
    order = rng.choice(["drain", "drain", "ready"])
    c = _case(order=order, streams=1 if order == "drain" else rng.choice([1, 2, 3]))
    tokens_lo, tokens_hi, segments, microbatches = 32, 4096, 2, rng.randint(1, 4)
    if kind == "fp32":
        kv = rng.choice([1, 2, 4])
        c.update(dtype="fp32", layers=rng.randint(1, 2), hidden=_log_int(rng, 64, 1024) // 4 * 4, kv_heads=kv,
                 q_heads=kv * rng.choice([1, 2, 4]), head_dim=rng.choice([16, 32, 64, 128]), ffn=_log_int(rng, 48, 2752) // 4 * 4,
                 w_std=0.05, x_std=rng.choice([0.02, 1.0]), mlp=rng.choice(["swiglu", "gelu"]), causal=rng.random() < 0.7,
                 norm=rng.choice(["rms", "rms", "layer"]), bias=rng.random() < 0.3, rope=rng.random() < 0.4,
                 qk_norm=rng.random() < 0.3)
        tokens_hi, segments = 1024, 4
    elif kind == "small":
        kv = rng.choice([2, 4, 8])
        c.update(layers=rng.randint(1, 4), hidden=_log_int(rng, 128, 1536) // 64 * 64, kv_heads=kv,
                 q_heads=kv * rng.choice([1, 2, 4]), head_dim=rng.choice([64, 128]), ffn=_log_int(rng, 192, 4096) // 64 * 64,
                 w_std=0.03, mlp=rng.choice(["swiglu", "swiglu", "gelu"]), rope=rng.random() < 0.4, bias=rng.random() < 0.3,
                 norm=rng.choice(["rms", "rms", "layer"]))
        tokens_hi, segments = 2048, 8
    elif kind in ("language", "multimodal"):
        c.update(layers=rng.randint(1, 4), kv_heads=rng.choice([8, 32]), rope=rng.random() < 0.3, qk_norm=rng.random() < 0.2)
        tokens_hi, segments = (6144, 2) if kind == "multimodal" else (4096, 4)
    elif kind == "wide":
        c.update(layers=rng.randint(1, 2), hidden=8192, q_heads=64, kv_heads=8, ffn=28672)
        microbatches = 1
    elif kind == "vision":
        layer_norm = rng.random() < 0.4
        c.update(layers=rng.randint(2, 8), hidden=1280, q_heads=16, kv_heads=16, head_dim=80, ffn=5120, mlp="gelu",
                 causal=False, norm="layer" if layer_norm else "rms", bias=layer_norm)
        tokens_lo, tokens_hi, segments = 400, 6272, 12
    else:
        kv = rng.choice([4, 8])
        c.update(layers=rng.randint(1, 4), hidden=_log_int(rng, 1024, 4096) // 128 * 128, kv_heads=kv,
                 q_heads=kv * rng.choice([2, 4]), head_dim=rng.choice([64, 128]), ffn=_log_int(rng, 2048, 11008) // 128 * 128,
                 rope=rng.random() < 0.5)
        tokens_hi, segments = 4096, 32
    c["tokens"] = "|".join(_cut(rng, _log_int(rng, tokens_lo, tokens_hi), segments) for _ in range(microbatches))
    # no more work than the largest listed case, fp32 held to what its lower rate allows
    limit = 2.5e11 if c["dtype"] == "fp32" else 4.0e13
    while work(c)["flops"] > limit:
        if "|" in c["tokens"]:
            c["tokens"] = c["tokens"].rsplit("|", 1)[0]
        else:
            total = sum(int(v) for v in c["tokens"].split(","))
            c["tokens"] = _cut(rng, max(2, total // 2), segments)
    return c


def _segments(case):
    """cu_seqlens of every microbatch."""
    out = []
    for mb in case["tokens"].split("|"):
        cu = [0]
        for n in mb.split(","):
            cu.append(cu[-1] + int(n))
        out.append(cu)
    return out


def _config(case):
    cus = _segments(case)
    return R.stage_config(
        n_layers=case["layers"], hidden=case["hidden"], n_q_heads=case["q_heads"], n_kv_heads=case["kv_heads"],
        head_dim=case["head_dim"], ffn=case["ffn"], max_tokens=max(cu[-1] for cu in cus), n_microbatches=len(cus),
        max_segments=max(len(cu) - 1 for cu in cus),
        dtype=R.STAGE_DTYPE_FP32 if case["dtype"] == "fp32" else R.STAGE_DTYPE_BF16,
        mlp_kind=R.STAGE_MLP_SWIGLU if case["mlp"] == "swiglu" else R.STAGE_MLP_GELU, causal=int(case["causal"]),
        norm_kind=int(case["norm"] == "layer"), norm_eps=1e-5, rope=int(case["rope"]), rope_base=10000.0,
        bias=int(case["bias"]), qk_norm=int(case["qk_norm"]))


class Iteration:
    """One stage with the device buffers a training program keeps for it and the tensors of one iteration."""

    def __init__(self, case, seed):
        self.handle = None
        self.cfg = cfg = _config(case)
        self.cus = _segments(case)
        M, dt = len(self.cus), torch.float32 if case["dtype"] == "fp32" else torch.bfloat16
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(seed)

        def normal(shape, std):
            return torch.empty(shape, dtype=dt, device=DEVICE).normal_(0.0, std, generator=gen)

        param_bytes, grad_bytes, arena_bytes = R.stage_query(cfg)
        self.params = normal(param_bytes // (4 if dt == torch.float32 else 2), case["w_std"])
        for layer in range(cfg.n_layers):
            for which in (R.STAGE_P_G1, R.STAGE_P_G2, R.STAGE_P_GQ, R.STAGE_P_GK):     # gains are 1 + N(0, w_std)
                off, (rows, cols) = R.stage_param_layout(cfg, layer, which)
                self.params[off:off + rows * cols] += 1.0
        # zeroed: the alignment gaps between the parameter tensors are part of the flat gradient buffer
        self.arena = torch.zeros(arena_bytes, dtype=torch.uint8, device=DEVICE)
        self.grad = torch.zeros(grad_bytes // 4, dtype=torch.float32, device=DEVICE)
        self.xs = [normal((cu[-1], cfg.hidden), case["x_std"]) for cu in self.cus]
        self.dys = [normal((cu[-1], cfg.hidden), case["x_std"]) for cu in self.cus]
        self.ys = [torch.empty_like(x) for x in self.xs]
        self.dxs = [torch.empty_like(x) for x in self.xs]
        # one stream: the caller's current one; several: streams of the runtime, ordered against the current one
        self.streams = [torch.cuda.Stream() for _ in range(case["streams"])] if case["streams"] > 1 else None
        if case["order"] == "ready":
            self.order = SI.ready_order(M, SI.BASE_SEED)
        else:
            self.order = [("F", j) for j in range(M)] + [t for j in range(M) for t in (("B", j), ("W", j))]
        self.handle = R.stage_create(cfg, self.params, self.arena, arena_bytes)

    def __del__(self):
        if self.handle is not None:
            torch.cuda.synchronize()
            R.stage_destroy(self.handle)
            self.handle = None


def prepare(case, seed):
    return Iteration(case, seed)


def run(state):
    current = torch.cuda.current_stream()
    streams = state.streams or [current]
    if state.streams:
        for s in streams:
            s.wait_stream(current)
    for i, (kind, j) in enumerate(state.order):
        s = streams[i % len(streams)]
        if kind == "F":
            R.stage_F(state.handle, j, state.xs[j], state.cus[j], state.ys[j], s)
        elif kind == "B":
            R.stage_B(state.handle, j, state.dys[j], state.dxs[j], s)
        else:
            R.stage_W(state.handle, j, s)
    R.stage_grad_reduce(state.handle, state.grad, streams[0])
    if state.streams:
        for s in streams:
            current.wait_stream(s)
    return {"y": state.ys, "dx": state.dxs, "grad": state.grad}


def work(case):
    """Matrix products of F, B and W (2 flops per multiply-add) and attention over the unmasked pairs, no
    recomputation; parameters, inputs and output gradients read once, outputs and gradients written once."""
    H, d, F = case["hidden"], case["head_dim"], case["ffn"]
    nq, nkv = case["q_heads"], case["kv_heads"]
    per_token = H * (nq + 2 * nkv) * d + nq * d * H + (3 if case["mlp"] == "swiglu" else 2) * H * F
    cus = _segments(case)
    tokens = sum(cu[-1] for cu in cus)
    pairs = sum((b - a) * (b - a + 1) / 2 if case["causal"] else (b - a) ** 2 for cu in cus for a, b in zip(cu, cu[1:]))
    size = 4 if case["dtype"] == "fp32" else 2
    flops = case["layers"] * (6.0 * tokens * per_token + 12.0 * d * nq * pairs)
    return {"bytes": case["layers"] * per_token * (size + 4.0) + 4.0 * tokens * H * size, "flops": flops}


def tolerance(case):
    """Measured: the fp32 path against the same layers in 64 bits 1.1e-6 (largest value 1.2e-5), the bf16 path against
    the fp32 path on the same values 2e-3 to 9e-3 (largest 0.33, in gradients near zero), more with depth and width."""
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 2e-2, "max": 0.6}
