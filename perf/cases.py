"""Cases on which this framework's speed is measured: the work that a GRPO training loop over long videos has it do,
through the public entry points of `paper_2507_07966_amd`.

A case names what one pass does ("do"), the shape of the call and the rollout lengths:
  prefill   prefix_attn_forward + prefix_attn_lse on a workspace of the caller
  static    prefix_attn_forward_static (forward and LSE on the library's own workspace)
  backward  prefix_attn_backward; the forward's output and LSE are in hand, as a training stack keeps them per layer
  train     prefix_attn_forward + prefix_attn_lse + prefix_attn_backward
  shard     what one device of a prefix-key-sharded group computes: its shard's partial, then the merge of all shards'
            partials (those of the other devices are in hand, as after the exchange)
  logprob   token_logprob_forward against an LM head
Rollout g of a call has `lens_lo` .. `lens_hi` tokens of its own (prompt and response), drawn from `lens_seed`.
Inputs are N(0, 1) (a hidden state after its final norm; queries and keys after their norm and rotary embedding),
rounded to the case's data type; upstream gradients likewise; LM-head rows N(0, 0.02^2); the token ids are uniform.
"""
import math

import numpy as np
import torch

import paper_2507_07966_amd as pa

TORCH_DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def _attention(name, do, dtype, heads, head_dim, prefix, rollouts, lens_lo, lens_hi, lens_seed=0, shards=0):
    case = {"do": do, "dtype": dtype, "q_heads": heads[0], "kv_heads": heads[1], "head_dim": head_dim,
            "prefix": prefix, "rollouts": rollouts, "lens_lo": lens_lo, "lens_hi": lens_hi, "lens_seed": lens_seed}
    if shards:
        case["shards"] = shards
    return dict(case, name=name) if name else case


def _logprob(name, tokens, hidden, vocab):
    case = {"do": "logprob", "dtype": "bf16", "tokens": tokens, "hidden": hidden, "vocab": vocab}
    return dict(case, name=name) if name else case


LAYER = (28, 4)      # query and key/value heads of the 7B-class decoder layer that the repository's workloads use


def listed():
    return [
        # The smallest call: one head of a 16-frame clip in fp32, the configuration of exact checks.
        _attention("tiny_prefill_f32", "prefill", "f32", (1, 1), 64, 256, 2, 96, 96),
        # A full-precision training step of a small layer: what a user runs to check gradients and to debug a run.
        _attention("small_train_f32", "train", "f32", (8, 2), 128, 1000, 4, 70, 300, lens_seed=1),
        # One question over a short clip, prefilled without any allocation (serving loops, graph capture): latency.
        _attention("question_static", "static", "bf16", LAYER, 128, 1024, 1, 128, 128),
        # A training step of one layer on a 64-frame clip: the ordinary short-video batch.
        _attention("clip_train", "train", "bf16", LAYER, 128, 4096, 8, 1152, 1152),
        # A 512-frame video, 8 rollouts: the repository's headline workload, forward and backward.
        _attention("video_prefill", "prefill", "bf16", LAYER, 128, 32768, 8, 2304, 2304),
        _attention("video_backward", "backward", "bf16", LAYER, 128, 32768, 8, 2304, 2304),
        # The longest video (8,192 frames) with 16 ragged rollouts: the largest forward call.
        _attention("longest_prefill", "prefill", "bf16", LAYER, 128, 524288, 16, 768, 4608, lens_seed=2),
        # The video tokens' own causal attention, computed once per layer for all rollouts: no prefix, one sequence.
        _attention("prefix_self_train", "train", "bf16", LAYER, 128, 0, 1, 32768, 32768),
        # A smaller model's layer (head dimension 64), nothing a multiple of a tile, lengths far apart.
        _attention("ragged_train_d64", "train", "bf16", (14, 2), 64, 5377, 5, 37, 1901, lens_seed=3),
        # Sequence parallelism over 8 devices: one device's 4,096 prefix keys and the merge of the eight partials.
        _attention("shard_of_eight", "shard", "bf16", LAYER, 128, 4096, 8, 2304, 2304, shards=8),
        # Probabilities of all response tokens of a question under one model, and of a few hundred (one rollout).
        _logprob("responses_logprob", 16384, 3584, 152064),
        _logprob("rollout_logprob", 333, 3584, 152064),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# The dearest pass among the listed ones is longest_prefill; a drawn case stays below this many operations, and one in
# fp32 far below it (its operations cost more than the data type alone explains).
MOST_FLOPS = 3e14


def draw(rng):
    """One more case of the same ranges."""
    while True:
        do = rng.choice(("prefill", "prefill", "static", "backward", "backward", "train", "train", "shard", "logprob", "logprob"))
        if do == "logprob":
            case = _logprob(None, _log_uniform(rng, 64, 16384), 64 * rng.randint(14, 56), rng.randint(32000, 152064))
            if work(case)["flops"] <= MOST_FLOPS:
                return case
            continue
        dtype = "f32" if do in ("prefill", "backward", "train") and rng.random() < 0.25 else "bf16"
        heads = rng.choice(((28, 4), (14, 2), (12, 2), (16, 8), (8, 2), (4, 4), (1, 1) if dtype == "f32" else (16, 2)))
        head_dim = rng.choice((64, 128, 128))
        rollouts = rng.choice((1, 2, 4, 5, 8, 16))
        if do == "static":
            rollouts, prefix = rng.choice((1, 2, 4)), _log_uniform(rng, 256, 8192)
            lo = _log_uniform(rng, 16, 200)
            hi = _log_uniform(rng, lo, 400)
        elif dtype == "f32":
            prefix, lo = _log_uniform(rng, 64, 4096), _log_uniform(rng, 16, 400)
            hi = _log_uniform(rng, lo, 600)
        elif rng.random() < 0.2 and do != "shard":   # one causal sequence, no prefix
            rollouts, prefix = 1, 0
            lo = hi = _log_uniform(rng, 512, 40000)
        else:
            prefix = _log_uniform(rng, 512, 524288 if do == "prefill" else 65536)
            lo = _log_uniform(rng, 32, 2304)
            hi = _log_uniform(rng, lo, 4608)
        case = _attention(None, do, dtype, heads, head_dim, prefix, rollouts, lo, hi, rng.randint(0, 1 << 20),
                          shards=rng.choice((2, 4, 8)) if do == "shard" else 0)
        most = {"prefill": 1.0, "static": 1.0, "shard": 0.1}.get(do, 0.2) * (0.0005 if dtype == "f32" else 1.0)
        if do == "static" and not _fits_static(case):
            continue
        if work(case)["flops"] <= most * MOST_FLOPS:
            return case


def _lens(case):
    return np.random.default_rng(case["lens_seed"]).integers(case["lens_lo"], case["lens_hi"] + 1, size=case["rollouts"]).astype(np.int32)


def _plan(case, device=0):
    return pa.prefix_attn_plan(case["q_heads"], case["kv_heads"], case["head_dim"], case["prefix"], _lens(case),
                               1.0 / math.sqrt(case["head_dim"]), dtype=case["dtype"], device=device)


def _fits_static(case):
    """Whether the call surely fits the library's own workspace: up to 17 fp32 partial results of every query row (short
    calls split the prefix over the chip) and a copy of the prefix values."""
    rows = int(_lens(case).sum()) * case["q_heads"] * case["head_dim"] * 4
    return 17 * rows + 2 * case["prefix"] * case["kv_heads"] * case["head_dim"] * 2 < pa.STATIC_SCRATCH_BYTES


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))

    def normal(*shape, dtype=TORCH_DTYPE[case["dtype"]], std=1.0):
        flat = torch.empty(math.prod(shape), dtype=dtype, device="cuda")
        step = 1 << 26
        for i in range(0, flat.numel(), step):   # in pieces: the fp32 values before rounding need not all be held
            part = flat[i:i + step]
            part.copy_(torch.randn(part.shape, generator=gen, dtype=torch.float32, device="cuda") * std)
        return flat.view(shape)

    def empty(*shape, dtype=TORCH_DTYPE[case["dtype"]]):
        return torch.empty(shape, dtype=dtype, device="cuda")

    if case["do"] == "logprob":
        n, d, vocab = case["tokens"], case["hidden"], case["vocab"]
        return {"case": case, "hidden": normal(n, d), "lm_head": normal(vocab, d, std=0.02),
                "targets": torch.randint(0, vocab, (n,), generator=gen, dtype=torch.int32, device="cuda"),
                "logprob": empty(n, dtype=torch.float32), "lse": empty(n, dtype=torch.float32),
                "workspace": empty(pa.token_logprob_workspace(n, d, vocab), dtype=torch.uint8)}
    hq, hkv, dim, prefix = case["q_heads"], case["kv_heads"], case["head_dim"], case["prefix"]
    plan = _plan(case)
    tokens = plan.total_tokens
    inputs = [normal(tokens, hq, dim), normal(prefix, hkv, dim) if prefix else None,
              normal(prefix, hkv, dim) if prefix else None, normal(tokens, hkv, dim), normal(tokens, hkv, dim)]
    state = {"case": case, "plan": plan, "inputs": inputs, "out": empty(tokens, hq, dim),
             "lse": empty(hq, tokens, dtype=torch.float32)}
    if case["do"] != "static":
        state["workspace"] = empty(max(16, plan.workspace_bytes), dtype=torch.uint8)
    if case["do"] == "shard":
        # the partials of the other devices: normalised outputs of many keys and their log-sum-exp
        n = case["shards"]
        size = math.sqrt(1.0 / max(1, prefix))
        state["o"] = [empty(tokens, hq, dim, dtype=torch.float32)]
        state["o"] += [normal(tokens, hq, dim, dtype=torch.float32, std=size) for _ in range(n - 1)]
        state["l"] = [empty(tokens, hq, dtype=torch.float32)]
        state["l"] += [normal(tokens, hq, dtype=torch.float32, std=0.1) + (math.log(prefix) + 0.5) for _ in range(n - 1)]
    if case["do"] in ("backward", "train"):
        state["d_out"] = normal(tokens, hq, dim)
        state["grads"] = [None if x is None else torch.empty_like(x) for x in inputs]
        state["backward_workspace"] = empty(max(16, plan.backward_workspace_bytes), dtype=torch.uint8)
    if case["do"] == "backward":
        pa.prefix_attn_forward(plan, *inputs, state["out"], state["workspace"])
        pa.prefix_attn_lse(plan, state["workspace"], state["lse"])
        torch.cuda.synchronize()
        del state["workspace"]
    return state


def run(state):
    do = state["case"]["do"]
    if do == "logprob":
        pa.token_logprob_forward(state["hidden"], state["lm_head"], state["targets"], 1.0, state["logprob"], state["lse"],
                                 state["workspace"])
        return state["logprob"], state["lse"]
    plan, out, lse = state["plan"], state["out"], state["lse"]
    if do == "static":
        pa.prefix_attn_forward_static(plan, *state["inputs"], out, lse)
        return out, lse
    if do == "shard":
        pa.prefix_attn_forward_partial(plan, *state["inputs"], True, state["o"][0], state["l"][0], state["workspace"])
        pa.prefix_attn_merge_partials(plan, state["o"], state["l"], out, lse)
        return state["o"][0], state["l"][0], out, lse
    if do in ("prefill", "train"):
        pa.prefix_attn_forward(plan, *state["inputs"], out, state["workspace"])
        pa.prefix_attn_lse(plan, state["workspace"], lse)
        if do == "prefill":
            return out, lse
    pa.prefix_attn_backward(plan, *state["inputs"], out, state["d_out"], lse, *state["grads"], state["backward_workspace"])
    return (out, lse, *state["grads"]) if do == "train" else tuple(state["grads"])


def work(case):
    """What one pass cannot do without: every input read once, every output written once, and the products over the
    visible (query row, key) pairs: 4 D operations each forward, 10 D backward."""
    if case["do"] == "logprob":
        n, d, vocab = case["tokens"], case["hidden"], case["vocab"]
        return {"bytes": 2 * d * (n + vocab) + 12 * n, "flops": 2 * n * d * vocab}
    lens = _lens(case).astype(np.int64)
    tokens, prefix, hq, hkv, dim = int(lens.sum()), case["prefix"], case["q_heads"], case["kv_heads"], case["head_dim"]
    size = 2 if case["dtype"] == "bf16" else 4
    rows, keys, lse = tokens * hq * dim, 2 * (prefix + tokens) * hkv * dim, 4 * tokens * hq
    pairs = hq * int((lens * prefix + lens * (lens + 1) // 2).sum())
    forward = {"bytes": size * (2 * rows + keys) + lse, "flops": 4 * dim * pairs}
    # q, out, d_out, k, v and the LSE in; dq, dk, dv out
    backward = {"bytes": size * (4 * rows + 2 * keys) + lse, "flops": 10 * dim * pairs}
    if case["do"] == "shard":   # this device's partial is written, all partials are read, the result is written
        n = case["shards"]
        return {"bytes": size * (2 * rows + keys) + (n + 1) * (4 * rows + lse) + lse, "flops": 4 * dim * pairs + 2 * n * rows}
    if case["do"] == "backward":
        return backward
    if case["do"] == "train":
        return {k: forward[k] + backward[k] for k in forward}
    return forward


def tolerance(case):
    """About four times the largest error seen against the definition evaluated in float64 (over cases of every kind)."""
    if case["do"] == "logprob":
        return {"rel": 5e-7}     # seen 6.6e-8: exact bf16 products, fp32 sums, the result rounded to fp32
    if case["dtype"] == "f32":
        return {"rel": 5e-6}     # seen 1.2e-6 (the gradients of prefix keys, summed over all rollouts): fp32 throughout
    return {"rel": 1e-2}         # seen 2.4e-3: probabilities and results rounded to bf16, sums in fp32
