"""The work whose speed is followed from change to change: what a program that uses this library
has it do, through the public entry points, over the range of sizes it meets.

  rollout   one generation job: rollout_prefill, then rollout_decode_step until every sample has
            ended.  Prompts are ragged, response lengths long-tailed, so the live batch shrinks.
  turns     a multi-turn job: the same, with rollout_extend between two stretches of decoding.
  logprobs  rollout_logprobs, the teacher-forced pass over packed sequences.
  sample    rollout_sample / rollout_sample_static, the sampler over given logits.
  loss      rollout_policy_loss, the objective over packed log-probs.

The jobs' tokens are given (forced), as when known responses are replayed: a drawn token may flip
with the last bit of a logit, and everything after it would be another sample.  Every step still
makes the full pass over the vocabulary that its log-prob needs; the draw itself is the sampler
cases' work.  What the jobs return is the log-prob of every token.

Shapes are those of the benchmark's configurations; the mixture of experts is cut to 12 of its 48
equal layers so that it is quick to set up.  Weights are random, N(0, 0.02), the logits projection
wider so that log-probs spread as a trained model's do.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2506_06122_amd as R


def _shape(layers, hidden, heads, kv_heads, head_dim, ffn, vocab, dtype="bf16", experts=0, top_k=0, expert_ffn=0,
           theta=1e6):
    return SimpleNamespace(n_layers=layers, hidden=hidden, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=head_dim,
                           ffn_dim=ffn, vocab=vocab, dtype=dtype, n_experts=experts, top_k=top_k,
                           expert_ffn_dim=expert_ffn, rms_eps=1e-6, rope_theta=theta)


MODELS = {
    "tiny-fp32": _shape(2, 256, 4, 2, 64, 688, 1024, dtype="fp32", theta=1e4),
    "1.5b": _shape(28, 1536, 12, 2, 128, 8960, 151936),
    "7b": _shape(28, 3584, 28, 4, 128, 18944, 152064),
    "30b-a3b-12-layers": _shape(12, 2048, 32, 4, 128, 0, 151936, experts=128, top_k=8, expert_ffn=768),
}


# ---------------------------------------------------------------------------------------- cases
def _rollout(model, prompts, samples, prompt_min, prompt_max, new_mean, new_max, top_p=1.0):
    return dict(kind="rollout", model=model, prompts=prompts, samples=samples, prompt_min=prompt_min,
                prompt_max=prompt_max, new_mean=new_mean, new_max=new_max, top_p=top_p)


def _turns(model, prompts, samples, prompt_min, prompt_max, turn_tokens, append_min, append_max):
    return dict(kind="turns", model=model, prompts=prompts, samples=samples, prompt_min=prompt_min,
                prompt_max=prompt_max, turn_tokens=turn_tokens, append_min=append_min, append_max=append_max)


def _logprobs(model, seqs, len_min, len_max):
    return dict(kind="logprobs", model=model, seqs=seqs, len_min=len_min, len_max=len_max)


def _sample(rows, vocab, top_p, static):
    return dict(kind="sample", rows=rows, vocab=vocab, top_p=top_p, static=static)


def _loss(seqs, len_min, len_max, kl):
    return dict(kind="loss", seqs=seqs, len_min=len_min, len_max=len_max, kl=kl)


def listed():
    named = {
        # the smallest job: single precision, the path that takes any shape; launches and host work are all of it
        "tiny_fp32_job": _rollout("tiny-fp32", 4, 2, 32, 32, 1000, 32, top_p=0.9),
        # one request's time to first token
        "first_token_1.5b": _rollout("1.5b", 1, 1, 187, 187, 1000, 1),
        # the long tail of a batch: a few samples left, every step a walk over the weights
        "tail_1.5b": _rollout("1.5b", 2, 3, 64, 512, 1000, 32),
        # an ordinary batch, from 256 live samples down to a handful
        "batch_1.5b": _rollout("1.5b", 32, 8, 64, 512, 24, 64),
        # few samples with long contexts: cached keys and values outweigh the weights
        "long_context_1.5b": _rollout("1.5b", 2, 8, 2500, 3500, 1000, 24),
        # an ordinary batch of the larger dense model
        "batch_7b": _rollout("7b", 8, 8, 128, 512, 24, 40),
        # an ordinary batch of the mixture of experts
        "batch_moe": _rollout("30b-a3b-12-layers", 8, 16, 128, 512, 16, 32),
        # an agent's job: answer, read what the environment says, answer again
        "turns_1.5b": _turns("1.5b", 8, 8, 64, 256, 16, 40, 130),
        # scoring long sequences with the larger dense model: the largest matrix products
        "logprobs_7b": _logprobs("7b", 4, 512, 5500),
        # scoring a handful of short answers
        "logprobs_short_1.5b": _logprobs("1.5b", 17, 11, 190),
        # nucleus sampling over a batch's logits
        "sample_top_p": _sample(64, 151936, 0.9, False),
        # one optimizer step's objective: 512 sequences of up to 8192 tokens
        "loss_512": _loss(512, 512, 8192, True),
    }
    return [dict(name=k, **v) for k, v in named.items()]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["rollout", "turns", "logprobs", "sample", "loss"], [45, 10, 20, 13, 12])[0]
    if kind == "rollout":
        model = rng.choices(["1.5b", "7b", "30b-a3b-12-layers", "tiny-fp32"], [50, 18, 18, 14])[0]
        # rows of one prefill and live samples: what keeps a drawn job below the largest listed case
        max_rows, max_live, max_new = {"1.5b": (9000, 256, 64), "7b": (2500, 96, 32), "30b-a3b-12-layers": (3000, 256, 32),
                                       "tiny-fp32": (500, 16, 48)}[model]
        prompts = _log(rng, 1, min(32, max_live))
        samples = _log(rng, 1, max(1, min(16, max_live // prompts)))
        top = _log(rng, 16, min(4000, max_rows // prompts))
        low = max(1, int(top * rng.uniform(0.15, 1.0)))
        new = _log(rng, 1, max_new)
        return _rollout(model, prompts, samples, low, top, rng.choice([max(1, new // 2), 1000]), new,
                        rng.choice([1.0, 0.9]))
    if kind == "turns":
        prompts = _log(rng, 1, 12)
        samples = _log(rng, 1, 8)
        top = _log(rng, 16, 400)
        app = _log(rng, 2, min(200, 8000 // (prompts * samples)))
        return _turns("1.5b", prompts, samples, max(1, top // 3), top, _log(rng, 2, 20), max(1, app // 3), app)
    if kind == "logprobs":
        model = rng.choices(["1.5b", "7b", "30b-a3b-12-layers"], [50, 30, 20])[0]
        rows = _log(rng, 60, {"1.5b": 16000, "7b": 9000, "30b-a3b-12-layers": 9000}[model])
        top = min(8000, _log(rng, 8, rows))
        return _logprobs(model, max(1, rows // top), max(1, int(top * rng.uniform(0.1, 1.0))), top)
    if kind == "sample":
        return _sample(_log(rng, 1, 256), rng.choice([1024, 32001, 151936, 152064]), rng.choice([1.0, 0.9, 0.95]),
                       rng.random() < 0.5)
    top = _log(rng, 16, 8192)
    return _loss(_log(rng, 1, 512), max(1, int(top * rng.uniform(0.06, 1.0))), top, rng.random() < 0.5)


# ---------------------------------------------------------------------------------------- sizes
def _spread(n, lo, hi):
    """n ragged lengths over [lo, hi], the same for every seed."""
    return [lo + int((hi - lo + 1) * ((0.5 + 0.6180339887498949 * i) % 1.0)) for i in range(n)]


def _prompt_lens(c):
    return _spread(c["prompts"], c["prompt_min"], c["prompt_max"])


def _response_lens(c):
    """Geometric law's quantiles in a scattered order, capped: a few long responses set the job's length."""
    n = c["prompts"] * c["samples"]
    u = [(0.37 + 0.6180339887498949 * i) % 1.0 for i in range(n)]
    lens = [min(c["new_max"], 1 + int(-c["new_mean"] * math.log1p(-x))) for x in u]
    lens[n // 2] = c["new_max"]
    return lens


# ---------------------------------------------------------------------------------------- inputs
def _weights(shape, gen):
    dt = torch.bfloat16 if shape.dtype == "bf16" else torch.float32

    def matrix(*dims, std=0.02):
        return torch.empty(dims, dtype=dt, device="cuda").normal_(0.0, std, generator=gen)

    def gain(n):
        return torch.empty(n, dtype=torch.float32, device="cuda").normal_(1.0, 0.1, generator=gen).to(dt)

    d, qd, kd = shape.hidden, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim
    w = {"embed": matrix(shape.vocab, d), "final_norm": gain(d), "lm_head": matrix(shape.vocab, d, std=0.05)}
    for i in range(shape.n_layers):
        p = f"layers.{i}."
        w.update({p + "norm1": gain(d), p + "wq": matrix(qd, d), p + "wk": matrix(kd, d), p + "wv": matrix(kd, d),
                  p + "wo": matrix(d, qd), p + "norm2": gain(d)})
        if shape.n_experts:
            e, fe = shape.n_experts, shape.expert_ffn_dim
            w.update({p + "router": matrix(e, d), p + "experts.w_gate": matrix(e, fe, d),
                      p + "experts.w_up": matrix(e, fe, d), p + "experts.w_down": matrix(e, d, fe)})
        else:
            f = shape.ffn_dim
            w.update({p + "w_gate": matrix(f, d), p + "w_up": matrix(f, d), p + "w_down": matrix(d, f)})
    return w


def _engine(model, seed, positions, live, context, batch_rows):
    """A context with room for `positions` cached tokens and one page's rounding per sample."""
    shape = MODELS[model]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kv_per_token = 2 * shape.n_layers * shape.n_kv_heads * shape.head_dim * (2 if shape.dtype == "bf16" else 4)
    return R.Rollout(shape, _weights(shape, gen), kv_pool_bytes=(positions + 96 * live + 4096) * kv_per_token,
                     page_tokens=32, max_live_samples=live, max_context=context + 32, max_batch_tokens=batch_rows,
                     seed=seed)


def _offsets(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


def prepare(case, seed):
    c, rng = case, np.random.default_rng(seed)
    kind = c["kind"]
    if kind in ("rollout", "turns"):
        shape, plens = MODELS[c["model"]], _prompt_lens(c)
        n_live = c["prompts"] * c["samples"]
        offs = _offsets(plens)
        s = {"kind": kind, "n": c["samples"], "offsets": offs,
             "prompts": rng.integers(0, shape.vocab, int(offs[-1])).astype(np.int32)}
        if kind == "rollout":
            lens = np.array(_response_lens(c), np.int32)
            more = 0
        else:
            lens = np.full(n_live, 2 * c["turn_tokens"], np.int32)
            more = c["append_max"]
            aoffs = _offsets(_spread(n_live, c["append_min"], c["append_max"]))
            s.update(turn=c["turn_tokens"], append_offsets=aoffs,
                     append=rng.integers(0, shape.vocab, int(aoffs[-1])).astype(np.int32))
        s["max_new"] = lens
        s["top_p"] = c.get("top_p", 1.0)
        # tokens of step t for the samples that live at it, in id order
        s["forced"] = [rng.integers(0, shape.vocab, int((lens > t).sum())).astype(np.int32) for t in range(int(lens.max()))]
        positions = int(sum(plens)) + int(lens.sum()) + more * n_live
        s["eng"] = _engine(c["model"], seed, positions, n_live, max(plens) + int(lens.max()) + more,
                           16384 if shape.dtype == "bf16" else 1024)
        return s
    if kind == "logprobs":
        shape, lens = MODELS[c["model"]], _spread(c["seqs"], c["len_min"], c["len_max"])
        cu = _offsets(lens)
        return {"kind": kind, "cu": cu, "tokens": rng.integers(0, shape.vocab, int(cu[-1])).astype(np.int32),
                "eng": _engine(c["model"], seed, 16384, 8, 8192, 16384)}
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if kind == "sample":
        rows = c["rows"]
        s = {"kind": kind, "static": c["static"], "top_p": c["top_p"],
             "logits": torch.empty(rows, c["vocab"], device="cuda").normal_(0.0, 2.5, generator=gen)}
        uni = rng.integers(0, 1 << 32, rows, dtype=np.uint64).astype(np.uint32)
        if c["static"]:
            s.update(uniforms=torch.from_numpy(uni.view(np.int32)).cuda(),
                     tokens=torch.empty(rows, dtype=torch.int32, device="cuda"),
                     logprobs=torch.empty(rows, dtype=torch.float32, device="cuda"),
                     sums=torch.empty(rows, dtype=torch.int64, device="cuda"))
        else:
            s["uniforms"] = uni
        return s
    lens = _spread(c["seqs"], c["len_min"], c["len_max"])
    cu = _offsets(lens)
    total = int(cu[-1])
    old = torch.rand(2, total, device="cuda", generator=gen).clamp_min_(1e-7).log_().sum(0)

    def near(std):
        return old + torch.empty(total, device="cuda").normal_(0.0, std, generator=gen)

    mask = np.ones(total, np.uint8)  # the first tokens of a sequence are its prompt
    for a, n, f in zip(cu[:-1], lens, rng.uniform(0.02, 0.6, len(lens))):
        mask[a:a + int(f * n)] = 0
    return {"kind": kind, "cu": cu, "old": old, "new": near(0.1), "ref": near(0.2) if c["kl"] else None,
            "kl": 0.05 if c["kl"] else 0.0, "mask": torch.from_numpy(mask).cuda(),
            "rewards": rng.choice([0.0, 1.0, -1.0], len(lens)).astype(np.float32)}


# ---------------------------------------------------------------------------------------- one pass
def _decode(eng, forced, out):
    for tokens in forced:
        out.append(eng.rollout_decode_step(forced_tokens=tokens)[2])


def run(state):
    s = state
    kind = s["kind"]
    if kind in ("rollout", "turns"):
        eng, forced = s["eng"], s["forced"]
        ids, _, lps, _ = eng.rollout_prefill(s["prompts"], s["offsets"], s["n"], s["max_new"], top_p=s["top_p"],
                                             forced_first=forced[0])
        out = [lps]
        if kind == "rollout":
            _decode(eng, forced[1:], out)
        else:
            k = s["turn"]
            _decode(eng, forced[1:k], out)
            out.append(eng.rollout_extend(ids, s["append"], s["append_offsets"], forced_next=forced[k])[1])
            _decode(eng, forced[k + 1:], out)
        return np.concatenate(out)
    if kind == "logprobs":
        return s["eng"].rollout_logprobs(s["tokens"], s["cu"], temperature=1.0)
    if kind == "sample":
        if not s["static"]:
            return list(R.rollout_sample(s["logits"], 1.0, s["top_p"], s["uniforms"]))
        R.rollout_sample_static(s["logits"], 1.0, s["top_p"], s["uniforms"], s["tokens"], s["logprobs"],
                                weight_sums=s["sums"])
        return [s["tokens"], s["logprobs"], s["sums"]]
    return list(R.rollout_policy_loss(s["cu"], s["new"], s["old"], s["ref"], s["mask"], s["rewards"], kl_coef=s["kl"]))


# ---------------------------------------------------------------------------------------- what it takes
def _forward(shape, rows, logit_rows, attended, cached_read):
    """bytes and flops of one forward pass: weights once, keys and values read and written once."""
    d, qd, kd = shape.hidden, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim
    size = 2 if shape.dtype == "bf16" else 4
    dense = d * (qd + 2 * kd) + qd * d
    if shape.n_experts:
        per_expert = 3 * d * shape.expert_ffn_dim
        touched = shape.n_experts * (1.0 - (1.0 - shape.top_k / shape.n_experts) ** rows)
        active = dense + shape.n_experts * d + shape.top_k * per_expert
        read = dense + shape.n_experts * d + touched * per_expert
    else:
        active = read = dense + 3 * d * shape.ffn_dim
    flops = shape.n_layers * (2.0 * active * rows + 4.0 * qd * attended) + 2.0 * shape.vocab * d * logit_rows
    moved = size * (shape.n_layers * (read + 2.0 * kd * (cached_read + rows)) + shape.vocab * d + d * rows)
    return moved, flops


def work(case):
    c = case
    kind = c["kind"]
    if kind == "sample":
        return {"bytes": 4.0 * c["rows"] * c["vocab"], "flops": 20.0 * c["rows"] * c["vocab"]}
    if kind == "loss":
        total = sum(_spread(c["seqs"], c["len_min"], c["len_max"]))
        return {"bytes": (4.0 * (4 + c["kl"]) + 1.0) * total, "flops": 15.0 * total}
    shape = MODELS[c["model"]]
    parts = []
    if kind == "logprobs":
        lens = _spread(c["seqs"], c["len_min"], c["len_max"])
        rows = sum(lens)
        parts.append(_forward(shape, rows, rows, sum(n * (n + 1) / 2 for n in lens), 0))
    else:
        plens = _prompt_lens(c)
        n = c["samples"]
        total = sum(plens)
        parts.append(_forward(shape, total, len(plens), sum(p * (p + 1) / 2 for p in plens), 0))
        lens = _response_lens(c) if kind == "rollout" else [2 * c["turn_tokens"]] * (len(plens) * n)
        app = _spread(len(lens), c["append_min"], c["append_max"]) if kind == "turns" else [0] * len(lens)
        for t in range(1, max(lens)):
            live = [i for i, x in enumerate(lens) if x > t]
            turn = kind == "turns" and t == c["turn_tokens"]
            late = kind == "turns" and t > c["turn_tokens"]
            own = [t - 1 + (app[i] if late else 0) for i in live]            # cached positions behind the prompt
            prefix = sum(plens[p] for p in {i // n for i in live})           # a prompt's positions once for its samples
            new = [app[i] + 1 if turn else 1 for i in live]
            attended = sum(k * (plens[i // n] + o) + k * (k + 1) / 2 for i, o, k in zip(live, own, new))
            parts.append(_forward(shape, sum(new), len(live), attended, prefix + sum(own)))
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    kind = case["kind"]
    if kind == "sample":
        return {"rel": 1e-6}   # ids and weight sums are whole numbers; a log-prob is one 32-bit rounding of a double
    if kind == "loss":
        return {"rel": 1e-5}
    if case["model"] == "tiny-fp32":
        return {"rel": 1e-5}
    # 16-bit keys and values, activations of about 17 bits, 28 layers deep: a few 1e-3 of a nat on log-probs of 12
    return {"rel": 2e-3, "max": 1e-2}
