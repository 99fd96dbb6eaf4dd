"""The work a user of this framework has it do, as cases that can be timed and checked.

Every case goes through the engine's public calls (paper_2308_01320_amd.binding.Engine, the C ABI of include/he.h) on
synthetic weights and token ids drawn on the GPU from the seed.  Layer, head and vocabulary sizes are those of
synth.CONFIGS; layer counts are cut so that a 64-bit reference is affordable (a layer costs the same wherever it stands).
A case is a dict:

  kind     "generate"  he_generate: the whole job, prompt pass plus steps decode steps replayed by the engine
           "decode"    he_reset, he_prefill(_ragged), then steps times he_decode_step on given token ids (a serving loop, or
                       forced decoding: the ids fed back do not depend on rounding, so every step can be compared)
           "prompt"    he_reset, he_prefill with its logits: time to the first token
           "score"     he_score over batch x prompt tokens
           "update"    he_refresh_weights(_lora) after a training update, then a short prompt pass on the new weights
  dtype    "bf16" (the tuned path) or "f32";  fp8: layer matrices held as 8-bit codes
  layers, hidden, heads, ffn, vocab;  batch, prompt (tokens per sequence), steps, ragged (prompts of different lengths),
  gumbel (Gumbel-max sampling, else greedy), rank (adapters folded in by "update", 0: none)
"""
import math

import torch

from paper_2308_01320_amd import binding, synth

# ------------------------------------------------------------------ the cases


def _shape(name):
    d = synth.CONFIGS[name]
    return {"dtype": d.dtype, "hidden": d.hidden, "heads": d.n_heads, "ffn": d.ffn, "vocab": d.vocab}


def _case(kind, layers, batch, prompt, steps=0, ragged=False, gumbel=False, fp8=False, rank=0, **shape):
    return {"kind": kind, "layers": layers, "batch": batch, "prompt": prompt, "steps": steps, "ragged": ragged,
            "gumbel": gumbel, "fp8": fp8, "rank": rank, **shape}


def listed():
    s, m, h = _shape("opt-1.3b"), _shape("opt-6.7b"), _shape("opt-13b")
    return [
        # the tiny configuration in full, float32: the smallest job there is; launches and their gaps are all of it
        dict(_case("generate", 2, 4, 32, 16, **_shape("tiny")), name="generate_tiny_f32"),
        # a whole generation call of the smallest actor at full depth, short prompts and answers
        dict(_case("generate", 24, 16, 48, 16, **s), name="generate_1.3b_b16"),
        # one user, one sequence, some context behind it: the latency of a token
        dict(_case("decode", 12, 1, 500, 32, **s), name="decode_1.3b_b1"),
        # an odd small batch of prompts of different lengths, as a serving loop holds it
        dict(_case("decode", 4, 7, 200, 48, ragged=True, **m), name="decode_6.7b_b7_ragged"),
        # the headline workload: experience generation of the 13B-shaped actor, batch 32, prompts of 256, sampled
        dict(_case("decode", 4, 32, 256, 128, gumbel=True, **h), name="decode_13b_b32"),
        # the same actor with 8-bit layer matrices
        dict(_case("decode", 4, 32, 128, 64, gumbel=True, fp8=True, **h), name="decode_13b_b32_fp8"),
        # a batch above the weight-streaming kernels' 64 rows
        dict(_case("decode", 2, 96, 64, 32, gumbel=True, **h), name="decode_13b_b96"),
        # the first token of a single prompt of odd length
        dict(_case("prompt", 8, 1, 250, **m), name="prompt_6.7b_b1"),
        # the headline workload's prompt pass
        dict(_case("prompt", 4, 32, 256, **h), name="prompt_13b_b32"),
        # long prompts: attention is a good part of the pass
        dict(_case("prompt", 3, 2, 1999, **h), name="prompt_13b_long"),
        # the scoring pass that follows generation: prompt plus answer of every sequence
        dict(_case("score", 6, 32, 512, **s), name="score_1.3b"),
        # the hand-over from training: adapters folded into new weights, then the first prompts on them
        dict(_case("update", 3, 8, 16, rank=16, **m), name="update_6.7b_lora"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# (hidden, heads): the configurations' layers, and narrower ones of the kinds the tests use (head dimensions 64 and 128)
_WIDTHS = [(128, 2), (256, 2), (512, 8), (1024, 16), (2048, 32), (4096, 32), (5120, 40), (9216, 72)]


def _draw(rng):
    kind = rng.choice(("generate", "decode", "decode", "decode", "prompt", "prompt", "prompt", "score", "update"))
    if kind == "generate" and rng.random() < 0.6:  # float32, any small model
        hidden, heads = rng.choice(((128, 4), (192, 3), (256, 4), (512, 8), (1024, 8)))
        return _case(kind, rng.randint(1, 4), _log_int(rng, 1, 16), _log_int(rng, 1, 96), _log_int(rng, 2, 32),
                     gumbel=rng.random() < 0.5, dtype="f32", hidden=hidden, heads=heads, ffn=64 * rng.randint(1, hidden // 16),
                     vocab=_log_int(rng, 100, 4000))
    hidden, heads = rng.choice(_WIDTHS[3:] if rng.random() < 0.75 else _WIDTHS[:4])
    shape = dict(dtype="bf16", hidden=hidden, heads=heads, ffn=4 * hidden if rng.random() < 0.8 else 64 * rng.randint(hidden // 64, hidden // 16),
                 vocab=50272 if rng.random() < 0.6 else _log_int(rng, 300, 50272))
    layers = rng.randint(1, 3)
    if kind == "generate":  # greedy answers short enough that a thin margin in one of them does not decide the comparison
        return _case(kind, layers, rng.randint(12, 64), _log_int(rng, 8, 256), rng.randint(8, 16), **shape)
    if kind == "decode":
        return _case(kind, layers, _log_int(rng, 1, 128), _log_int(rng, 1, 1024), _log_int(rng, 8, 96), ragged=rng.random() < 0.4,
                     gumbel=rng.random() < 0.5, fp8=rng.random() < 0.25, **shape)
    if kind == "prompt":
        return _case(kind, layers, _log_int(rng, 1, 64), _log_int(rng, 2, 2000), ragged=rng.random() < 0.4, fp8=rng.random() < 0.15, **shape)
    if kind == "score":
        return _case(kind, layers, _log_int(rng, 1, 48), _log_int(rng, 2, 1024), **shape)
    return _case(kind, layers, _log_int(rng, 1, 16), _log_int(rng, 1, 32), rank=rng.choice((0, 8, 16, 64, rng.randint(1, 40))), **shape)


def draw(rng):
    most = [work(c) for c in listed()]
    bytes_, flops = max(w["bytes"] for w in most), max(w["flops"] for w in most)
    while True:
        c = _draw(rng)
        w = work(c)
        rows = c["batch"] * (c["prompt"] + c["steps"])
        if w["bytes"] <= bytes_ / 3 and w["flops"] <= flops / 2 and rows <= 20000:
            return c


# ------------------------------------------------------------------ inputs

_STREAM = None


def _stream():
    """The stream a program keeps for its engines (the engine captures its decode step on it)."""
    global _STREAM
    if _STREAM is None:
        _STREAM = torch.cuda.Stream()
    return _STREAM


def _inputs(case, seed, device):
    """Weights as synth.device_weights draws them (random initialisation of an OPT-style decoder) and token ids."""
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    H, F, V, B, S = case["hidden"], case["ffn"], case["vocab"], case["batch"], case["prompt"]

    def normal(*shape, mean=0.0):
        return torch.randn(shape, generator=g, device=device).mul_(0.02).add_(mean).to(dt)

    w = {"tok_emb": normal(V, H), "pos_emb": normal(S + case["steps"] + 1, H), "layers": []}
    for _ in range(case["layers"]):
        w["layers"].append({
            "ln1_g": normal(H, mean=1.0), "ln1_b": normal(H), "wqkv": normal(3 * H, H), "bqkv": normal(3 * H),
            "wo": normal(H, H), "bo": normal(H), "ln2_g": normal(H, mean=1.0), "ln2_b": normal(H),
            "w1": normal(F, H), "b1": normal(F), "w2": normal(H, F), "b2": normal(H)})
    w["lnf_g"], w["lnf_b"] = normal(H, mean=1.0), normal(H)
    w["lm_head"] = w["tok_emb"]

    def ids(*shape):
        return torch.randint(0, V, shape, generator=g, device=device, dtype=torch.int32)

    tokens = {"prompt": ids(B, S), "forced": ids(max(1, case["steps"]), B),
              "lens": torch.randint((S + 1) // 2, S + 1, (B,), generator=g, device=device, dtype=torch.int32)}
    if not case["ragged"]:
        tokens["lens"].fill_(S)
    adapters = []
    if case["rank"]:
        for lw in w["layers"]:
            adapters.append({k: (normal(case["rank"], lw[k].shape[1]), normal(lw[k].shape[0], case["rank"]))
                             for k in ("wqkv", "wo", "w1", "w2")})
    return w, tokens, adapters


_LORA_SCALE = 0.5


def prepare(case, seed):
    w, tokens, adapters = _inputs(case, seed, "cuda")
    S, steps = case["prompt"], case["steps"]
    cfg = binding.he_config(case["layers"], case["hidden"], case["heads"], case["ffn"], case["vocab"], S + steps + 1, 0, 1e-5,
                            binding.HE_BF16 if case["dtype"] == "bf16" else binding.HE_F32, case["batch"], S + steps, 0,
                            _stream().cuda_stream, 0, 0, 1 if case["fp8"] else 0)
    return {"case": case, "engine": binding.Engine(cfg, w), "tokens": tokens, "adapters": adapters,
            "sampling": binding.sampling("gumbel" if case["gumbel"] else "greedy", 1.0, seed)}


# ------------------------------------------------------------------ one pass


def _prefill(state, want_logits):
    e, t, s = state["engine"], state["tokens"], state["sampling"]
    e.he_reset()
    if state["case"]["ragged"]:
        return e.he_prefill_ragged(t["prompt"], t["lens"], s, want_logits)
    return e.he_prefill(t["prompt"], s, want_logits)


def _returns_ids(case):
    # Token ids are compared where one of them decided by a thin margin is a small share of all: in float32, and over the
    # thousands of draws of a sampled run.  Greedy 16-bit runs return the log-probability of the arg-max, which a tie
    # does not move.
    if case["kind"] == "generate":
        return case["dtype"] == "f32"
    return case["gumbel"] and case["batch"] * (case["steps"] + 1) >= 2000


def run(state):
    case, e, t, s = state["case"], state["engine"], state["tokens"], state["sampling"]
    with torch.cuda.stream(_stream()):
        if case["kind"] == "generate":
            ids, lp = e.he_generate(t["prompt"], case["steps"], s)
            return {"ids": ids, "logprobs": lp} if _returns_ids(case) else {"logprobs": lp}
        if case["kind"] == "score":
            return {"logprobs": e.he_score(t["prompt"])}
        if case["kind"] == "update":
            if case["rank"]:
                e.he_refresh_weights_lora(state["adapters"], case["rank"], _LORA_SCALE)
            else:
                e.he_refresh_weights()
        if case["kind"] != "decode":
            _, lp, logits = _prefill(state, True)
            return {"logprobs": lp, "logits": logits}
        first = _prefill(state, False)
        ids, lps, logits = [first[0]], [first[1]], None
        for i in range(case["steps"]):
            nid, lp, logits = e.he_decode_step(t["forced"][i], s, i == case["steps"] - 1)
            ids.append(nid)
            lps.append(lp)
        out = {"logprobs": torch.stack(lps), "logits": logits}
        if _returns_ids(case):
            out["ids"] = torch.stack(ids)
        return out


# ------------------------------------------------------------------ what a pass cannot do without


def work(case):
    H, F, V, L, B, S, n = (case[k] for k in ("hidden", "ffn", "vocab", "layers", "batch", "prompt", "steps"))
    el = 4 if case["dtype"] == "f32" else 2
    params = 4 * H * H + 2 * H * F
    layer = params * (1 if case["fp8"] else el) + (9 * H + F) * el  # a layer's weights, read once per pass over them
    head = V * H * el
    kvrow = 2 * H * el  # a position's key and value in one layer
    mean = 0.75 if case["ragged"] else 1.0  # mean share of the prompt rows that hold tokens
    rows = B * S * mean

    def attn(r, t):  # r queries over t keys each: multiply-adds of scores and values
        return 4.0 * r * t * H

    score = case["kind"] == "score"
    nbytes = L * layer + head + B * S * 4 + L * rows * kvrow * (1 if score else 2)
    # the scoring pass needs every row of every layer; a prompt pass, of all but the last row of a sequence, only the
    # last layer's key and value
    full = L if score else L - 1
    flops = full * (2.0 * rows * params + attn(rows, S * mean / 2)) + 2.0 * (rows if score else B) * V * H
    if not score:
        flops += 4.0 * rows * H * H + 2.0 * B * (params - 2 * H * H) + attn(B, S * mean)
    nbytes += rows * 4 if score else B * 8 + (B * V * 4 if case["kind"] != "generate" else 0)
    later = n - 1 if case["kind"] == "generate" else n
    for i in range(later):
        T = S * mean + i + 1
        nbytes += L * (layer + B * (T + 1) * kvrow) + head + B * 12
        flops += L * (2.0 * B * params + attn(B, T)) + 2.0 * B * V * H
    if case["kind"] == "update":
        r = case["rank"]
        nbytes += L * (params * 4 + r * 2 * (9 * H + 2 * F + H)) + 2 * head  # the caller's matrices in, the engine's out
        flops += L * 2.0 * r * params
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # Measured: 16-bit logits are 5e-4 to 8e-4 off the 64-bit ones (rounding of activations and cache), a sequence's
    # log-probabilities, which are large against their differences, 4e-5 to 2e-4; float32 log-probabilities 1e-7.
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-5, "differ": 0.0}
    if case["kind"] == "generate":
        # free running: where a greedy margin is thinner than the rounding the rest of that answer is another one
        return {"rel": 0.03, "max": 0.9}
    if case["gumbel"] and case["kind"] == "decode":
        # a draw decided by a thin margin has another token's log-probability
        return {"rel": 0.02, "max": 0.9, "differ": 0.01}
    if case["kind"] == "score":
        return {"rel": 4e-4, "max": 4e-3}
    return {"rel": 4e-3, "max": 3e-2}


# ------------------------------------------------------------------ the same in 64 bits


def _e4m3_rows(w):
    """Row n as E4M3 values times 2^e, e the smallest integer with max|row| 2^-e <= 448 (the definition of the 8-bit form)."""
    top = w.abs().amax(dim=1, keepdim=True).clamp_min(1e-30)
    e = torch.ceil(torch.log2(top / 448.0))
    e = torch.where(top * torch.exp2(-(e - 1)) <= 448.0, e - 1, e)
    e = torch.where(top * torch.exp2(-e) > 448.0, e + 1, e)
    return (w * torch.exp2(-e)).float().to(torch.float8_e4m3fn).double() * torch.exp2(e)


def _norm(x, g, b):
    mu = x.mean(-1, keepdim=True)
    var = (x - mu).square().mean(-1, keepdim=True)
    return (x - mu) / torch.sqrt(var + 1e-5) * g.double() + b.double()


def _hidden(case, w, adapters, tokens):
    """Final-LayerNorm outputs [B, T, H] of tokens [B, T] at positions 0 .. T-1, causal, float64."""
    nh = case["heads"]
    B, T = tokens.shape
    H = case["hidden"]
    d = H // nh
    x = w["tok_emb"].double()[tokens.long()] + w["pos_emb"].double()[:T]
    mask = torch.full((T, T), -math.inf, device=x.device, dtype=torch.float64).triu(1)
    chunk = max(1, min(B, int(2e9 // (8 * nh * T * T)) or 1))
    for l, lw in enumerate(w["layers"]):
        def mat(k):
            m = lw[k].double()
            if adapters:
                a, b = adapters[l][k]
                m = (m + _LORA_SCALE * (b.double() @ a.double())).float().to(torch.bfloat16).double()
            return _e4m3_rows(m) if case["fp8"] else m

        qkv = _norm(x, lw["ln1_g"], lw["ln1_b"]) @ mat("wqkv").t() + lw["bqkv"].double()
        att = torch.empty_like(x)
        for b0 in range(0, B, chunk):
            q, k, v = (p.reshape(-1, T, nh, d).transpose(1, 2).contiguous() for p in qkv[b0:b0 + chunk].split(H, dim=-1))
            sc = torch.matmul(q, k.transpose(2, 3).contiguous()).mul_(d ** -0.5).add_(mask)
            att[b0:b0 + chunk] = torch.matmul(torch.softmax(sc, -1), v).transpose(1, 2).reshape(-1, T, H)
            del sc
        x = x + att @ mat("wo").t() + lw["bo"].double()
        h = torch.relu(_norm(x, lw["ln2_g"], lw["ln2_b"]) @ mat("w1").t() + lw["b1"].double())
        x = x + h @ mat("w2").t() + lw["b2"].double()
    return _norm(x, w["lnf_g"], w["lnf_b"])


def exact(case, seed):
    if case["kind"] == "generate" and case["dtype"] != "f32":
        return None  # free running: later tokens follow earlier ones
    device = "cuda" if torch.cuda.is_available() else "cpu"
    w, t, adapters = _inputs(case, seed, device)
    B, S, n = case["batch"], case["prompt"], case["steps"]
    head = w["lm_head"].double().t()
    if case["kind"] == "generate":
        if case["gumbel"]:
            return None
        seq, lps, ids = t["prompt"], [], []
        for _ in range(n):
            z = _hidden(case, w, adapters, seq)[:, -1] @ head
            top, nid = z.max(dim=1)
            lps.append(top - torch.logsumexp(z, 1))
            ids.append(nid.to(torch.int32))
            seq = torch.cat([seq, ids[-1][:, None]], dim=1)
        return {"ids": torch.stack(ids, 1), "logprobs": torch.stack(lps, 1)}
    if case["kind"] == "score":
        x = _hidden(case, w, adapters, t["prompt"])
        out = torch.empty(B, S - 1, device=device, dtype=torch.float64)
        for b in range(B):
            z = x[b, :-1] @ head
            out[b] = z.gather(1, t["prompt"][b, 1:, None].long())[:, 0] - torch.logsumexp(z, 1)
        return {"logprobs": out}
    # every sequence's own tokens from position 0 on, then the tokens fed to the decode steps
    rows = torch.zeros(B, S + n, device=device, dtype=torch.int32)
    lens = t["lens"].tolist()
    for b, m in enumerate(lens):
        rows[b, :m] = t["prompt"][b, S - m:]
        if n:
            rows[b, m:m + n] = t["forced"][:n, b]
    x = _hidden(case, w, adapters, rows)
    first = t["lens"].long() - 1
    at = torch.arange(B, device=device)
    lps = []
    for i in range(n + 1):
        z = x[at, first + i] @ head
        lps.append(z.max(dim=1).values - torch.logsumexp(z, 1))
    if case["kind"] == "decode":
        return {"logprobs": None if case["gumbel"] else torch.stack(lps), "logits": z, **({"ids": None} if _returns_ids(case) else {})}
    return {"logprobs": lps[0], "logits": z}
