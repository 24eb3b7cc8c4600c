"""Workloads of the Recurrent Transformer layer library: what its users call, at the sizes they call it with.

Six kinds of work, all through the binding of the C entry points:

    decode     rt_decode_step: one position over a cache the caller holds, one layer
    generate   one generated token of a stack: rt_embed_rows, rt_decode_step per layer, rt_lm_head
    prefill    rt_layer_prefill: a whole sequence through one layer
    stack      a prompt through a stack: rt_embed_rows, rt_stack_prefill, rt_lm_head
    parallel   the layer without its sequential loop: rt_transformer_layer (source "x") or, in a training step that
               kept only the layer's output, rt_layer_recompute (source "z")
    backward   rt_layer_backward: gradients of the input and of every parameter

Matrices are N(0, 0.02^2), inputs N(0, 1) (as in the benchmark's workloads), gains 1 + N(0, 0.1^2); cached keys have
the norm that the layer's per-head normalisation gives them, cached values the spread that its projection gives them.
Heads are 64 wide and the hidden width of the MLP is 4 d throughout.
"""
import math

import torch

from paper_2604_21215_amd import binding

DEVICE = "cuda:0"
VOCAB = 32768
MATRICES = ("Wq", "Wk", "Wv", "Wo", "W1", "W2")
GAINS = ("g_attn", "g_mlp", "g_kv", "g_q", "g_k")


def listed():
    return [
        # the smallest call: one sequence, the first tokens of a generation, a small layer
        dict(name="decode_first_tokens", kind="decode", dtype="bf16", B=1, t=37, d=512, alibi=0.0, scale=1.0),
        # one token of eight conversations through twelve layers, embedding and read-out included
        dict(name="generate_12_layers", kind="generate", dtype="bf16", B=8, t=1500, d=1024, layers=12),
        # a serving batch: 200 sequences that share a step
        dict(name="decode_serving_batch", kind="decode", dtype="bf16", B=200, t=511, d=1024, alibi=0.0, scale=1.0),
        # the fp32 layer of the first benchmark configuration
        dict(name="prefill_f32", kind="prefill", dtype="f32", B=1, N=256, d=128, alibi=0.0, scale=1.0),
        # shaped like a 150M-parameter model with its positional bias; ragged batch and length
        dict(name="prefill_768_ragged", kind="prefill", dtype="bf16", B=5, N=1000, d=768, alibi=8.0, scale=1.0),
        # the headline configuration: shaped like a 300M-parameter model
        dict(name="prefill_headline", kind="prefill", dtype="bf16", B=8, N=2048, d=1024, alibi=0.0, scale=1.0),
        # two points of the paper's latency table (N = 512): a middling odd batch and the largest
        dict(name="prefill_batch_100", kind="prefill", dtype="bf16", B=100, N=512, d=1024, alibi=0.0, scale=0.125),
        dict(name="prefill_batch_1024", kind="prefill", dtype="bf16", B=1024, N=512, d=1024, alibi=0.0, scale=0.125),
        # a prompt of 4096 tokens through the twelve-layer stack
        dict(name="stack_12_layers", kind="stack", dtype="bf16", B=4, N=4096, d=1024, layers=12),
        # the layer with every pair known in advance, at the headline shape
        dict(name="transformer_layer", kind="parallel", dtype="bf16", B=8, N=2048, d=1024, source="x", alibi=0.0, scale=1.0),
        # gradients: long sequences in a small batch, and a training batch of the paper's sequence length
        dict(name="backward_long", kind="backward", dtype="bf16", B=8, N=2048, d=1024, alibi=0.0, scale=0.125),
        dict(name="backward_batch", kind="backward", dtype="bf16", B=48, N=512, d=1024, alibi=0.0, scale=0.125),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("decode", "generate", "prefill", "prefill", "stack", "parallel", "backward"))
    d = rng.choice((256, 512, 768, 1024, 1024))
    alibi, scale = rng.choice((0.0, 0.0, 8.0)), rng.choice((1.0, 0.125))
    f32 = rng.random() < 0.15
    if kind == "decode":
        B = _log(rng, 1, 256)
        return dict(kind=kind, dtype="f32" if f32 and B <= 16 else "bf16", B=B, t=_log(rng, 1, min(4000, 262144 // B)), d=d,
                    alibi=alibi, scale=scale)
    if kind == "generate":
        return dict(kind=kind, dtype="bf16", B=_log(rng, 1, 32), t=_log(rng, 16, 2000), d=d, layers=rng.randint(2, 12))
    if kind == "prefill":
        if f32:
            return dict(kind=kind, dtype="f32", B=rng.randint(1, 4), N=_log(rng, 32, 512), d=rng.choice((128, 256, 384)), alibi=alibi,
                        scale=scale)
        B = _log(rng, 1, 1024)
        # softmax weights are sharp without scaling: large batches take the scaled logits of the latency table
        return dict(kind=kind, dtype="bf16", B=B, N=_log(rng, 64, min(2048, 524288 // B)), d=d, alibi=alibi,
                    scale=scale if B <= 16 else 0.125)
    if kind == "stack":
        return dict(kind=kind, dtype="bf16", B=rng.randint(1, 8), N=_log(rng, 128, 2048), d=d, layers=rng.randint(2, 12))
    if kind == "parallel":
        B = _log(rng, 1, 16)
        return dict(kind=kind, dtype="bf16", B=B, N=_log(rng, 64, 2048), d=d, source=rng.choice(("x", "z")), alibi=alibi, scale=scale)
    # gradients of the gains through unscaled (sharp) softmax weights are differences of large sums: scaled logits
    if f32:
        return dict(kind=kind, dtype="f32", B=rng.randint(1, 2), N=_log(rng, 32, 256), d=rng.choice((128, 256)), alibi=alibi,
                    scale=0.125)
    B = _log(rng, 1, 48)
    return dict(kind=kind, dtype="bf16", B=B, N=_log(rng, 64, min(2048, 24576 // B)), d=d, alibi=alibi, scale=0.125)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


class _Draws:
    def __init__(self, case, seed):
        self.g = torch.Generator(device=DEVICE)
        self.g.manual_seed(int(seed))
        self.dtype = _dtype(case)

    def normal(self, *shape, std=1.0, mean=0.0):
        return (torch.randn(shape, generator=self.g, device=DEVICE) * std + mean).to(self.dtype)

    def layer(self, d):
        w = {n: self.normal(*s, std=0.02) for n, s in
             zip(MATRICES, ((d, d), (d, d), (d, d), (d, d), (4 * d, d), (d, 4 * d)))}
        w.update({n: self.normal(d, std=0.1, mean=1.0) for n in GAINS})
        return w, binding.make_weights(w)

    def cache(self, cap, B, d):
        K = self.normal(cap, B, d // 64, 64)
        for rows in K.split(256):   # per-head normalisation: mean square 1
            rows.div_(rows.float().square().mean(-1, keepdim=True).sqrt_().to(rows.dtype))
        return K, self.normal(cap, B, d // 64, 64, std=0.02 * math.sqrt(d))


def prepare(case, seed):
    r = _Draws(case, seed)
    kind, B, d = case["kind"], case["B"], case["d"]
    H, layers = d // 64, case.get("layers", 1)
    n = case.get("N") or case["t"] + 1
    td = _dtype(case)
    # the twelve-layer stacks scale the residual branches by 1 / sqrt(L) (Sec. 2)
    ctx = binding.RTContext(d, H, 4 * d, B, n, case["dtype"], resid_scale=1.0 / math.sqrt(layers), attn_scale=case.get("scale", 1.0),
                            rms_eps=1e-6, stream=torch.cuda.current_stream().cuda_stream, alibi_max_bias=case.get("alibi", 0.0),
                            reserve_stack_layers=layers if kind == "stack" else 0,
                            reserve={"parallel": binding.RT_RESERVE_LOOP_FREE, "backward": binding.RT_RESERVE_BACKWARD}.get(kind, 0))
    s = dict(case=case, ctx=ctx)
    sets = [r.layer(d) for _ in range(layers)]
    s["weights"], s["structs"] = [w for w, _ in sets], [st for _, st in sets]
    empty = lambda *shape, dtype=td: torch.empty(shape, dtype=dtype, device=DEVICE)  # noqa: E731
    if kind == "decode":
        s["x"], s["y"] = r.normal(B, d), empty(B, d)
        s["K"], s["V"] = r.cache(n, B, d)
        return s
    if kind in ("generate", "stack"):
        s["table"], s["head"], s["g_final"] = r.normal(VOCAB, d), r.normal(VOCAB, d, std=0.02), r.normal(d, std=0.1, mean=1.0)
        s["ids"] = torch.randint(0, VOCAB, (B, n), generator=r.g, device=DEVICE, dtype=torch.int32)
        s["logits"] = empty(B, VOCAB, dtype=torch.float32)
    if kind == "generate":
        s["rows"] = empty(layers + 1, B, 1, d)
        caches = [r.cache(n, B, d) for _ in range(layers)]
        s["K"], s["V"] = [k for k, _ in caches], [v for _, v in caches]
        return s
    if kind == "stack":
        s["x"] = empty(B, n, d)
        s["y"] = [empty(B, n, d) for _ in range(layers)]
        s["K"] = [empty(n, B, H, 64) for _ in range(layers)]
        s["V"] = [empty(n, B, H, 64) for _ in range(layers)]
        return s
    s["x"], s["y"] = r.normal(B, n, d), empty(B, n, d)
    s["K"], s["V"] = empty(n, B, H, 64), empty(n, B, H, 64)
    if kind == "backward" or case.get("source") == "z":
        s["z"] = empty(B, n, d)
        ctx.rt_layer_prefill(s["structs"][0], s["x"], s["z"], s["K"], s["V"])   # the forward pass of the training step
    if kind == "backward":
        s["gy"], s["gK"], s["gV"] = r.normal(B, n, d), None, None
        s["dx"] = empty(B, n, d, dtype=torch.float32)
        s["grads"] = {k: torch.empty(w.shape, dtype=torch.float32, device=DEVICE) for k, w in s["weights"][0].items()}
        del s["y"], s["K"], s["V"]
    return s


def run(s):
    case, ctx, w = s["case"], s["ctx"], s["structs"]
    kind = case["kind"]
    if kind == "decode":
        t = case["t"]
        ctx.rt_decode_step(w[0], s["x"], t, s["y"], s["K"], s["V"])
        return s["y"], s["K"], s["V"], s["K"][t], s["V"][t]   # the whole caches, and beside them the row that is new
    if kind == "generate":
        t, rows = case["t"], s["rows"]
        ctx.rt_embed_rows(s["table"], s["ids"], t, rows[0])
        for l in range(case["layers"]):
            ctx.rt_decode_step(w[l], rows[l, :, 0], t, rows[l + 1, :, 0], s["K"][l], s["V"][l])
        ctx.rt_lm_head(s["head"], s["g_final"], rows[-1], case["d"], case["B"], s["logits"])
        return s["logits"], rows, s["K"], s["V"]
    if kind == "prefill":
        ctx.rt_layer_prefill(w[0], s["x"], s["y"], s["K"], s["V"])
        return s["y"], s["K"], s["V"]
    if kind == "stack":
        ctx.rt_embed_rows(s["table"], s["ids"], 0, s["x"])
        ctx.rt_stack_prefill(w, s["x"], s["y"], s["K"], s["V"])
        last = s["y"][-1]
        ctx.rt_lm_head(s["head"], s["g_final"], last[:, -1], last.stride(0), case["B"], s["logits"])
        return s["logits"], s["y"], s["K"], s["V"]
    if kind == "parallel":
        if case["source"] == "x":
            ctx.rt_transformer_layer(w[0], s["x"], s["y"], s["K"], s["V"])
        else:
            ctx.rt_layer_recompute(w[0], s["x"], s["z"], s["y"], s["K"], s["V"])
        return s["y"], s["K"], s["V"]
    ctx.rt_layer_backward(w[0], s["x"], s["z"], s["gy"], s["gK"], s["gV"], s["dx"], s["grads"])
    return s["dx"], s["grads"]


def work(case):
    """Inputs read once and outputs written once; the products and the causal attention of the definition."""
    kind, B, d, layers = case["kind"], case["B"], case["d"], case.get("layers", 1)
    E = 2 if case["dtype"] == "bf16" else 4
    matrices = 12 * d * d                       # Wq, Wk, Wv, Wo, W1, W2 at a hidden width of 4 d
    per_token = 2.0 * (matrices + 2 * d * d)    # Wk and Wv serve the temporary and the persistent pair
    readout = 2.0 * B * VOCAB * d
    if kind in ("decode", "generate"):
        by = layers * ((matrices + 2.0 * case["t"] * B * d + 4.0 * B * d) * E)
        fl = layers * B * (per_token + 4.0 * d * (case["t"] + 1))
        return {"bytes": by + (VOCAB * d * E + 4.0 * B * VOCAB if kind == "generate" else 0.0),
                "flops": fl + (readout if kind == "generate" else 0.0)}
    N = case["N"]
    rows = float(B) * N
    attention = 2.0 * rows * (N + 1) * d
    if kind == "stack":
        return {"bytes": layers * (matrices + 3.0 * rows * d) * E + rows * d * E + VOCAB * d * E + 4.0 * B * VOCAB,
                "flops": layers * (rows * per_token + attention) + readout}
    if kind == "backward":   # the recomputed forward, then each product twice (its input's gradient, its matrix's)
        return {"bytes": (matrices + 3.0 * rows * d) * E + 4.0 * (matrices + rows * d),
                "flops": 3.0 * rows * per_token + 3.5 * attention}
    if kind == "parallel" and case["source"] == "x":
        return {"bytes": (matrices + 4.0 * rows * d) * E, "flops": rows * 2.0 * matrices + attention}
    return {"bytes": (matrices + (5.0 if kind == "parallel" else 4.0) * rows * d) * E, "flops": rows * per_token + attention}


def tolerance(case):
    """fp32: four times the distance from the same layer in 64 bits (forward 4.4e-7, gradients 1.3e-6 of the norm).
    bf16: the layer evaluated with its sums in another order and other vectors rounded on the way (one launch or several
    per position, matrix cores or not) differs by 0.1 - 0.5 % of the norm for one layer with scaled logits and for the
    gradients, 0.7 % with unscaled logits, 1.0 % behind twelve layers, and by 0.07 of a value at most."""
    if case["dtype"] == "f32":
        return {"rel": 6e-6 if case["kind"] == "backward" else 2e-6, "max": 1e-4}
    return {"rel": 2e-2, "max": 0.3}
