"""GPU parity of the prompt and scoring passes of few rows and of wide decode steps (the deep-ring GEMM), the LM head of many
rows and the decode attention of few, each against the oracle.  The narrow shapes all take 64-row tiles: rows at the edges
of those and of the 32-row blocks, columns that end inside a 256-column tile, k ranges of different lengths.
test_passes_on_every_tile reaches the other tiles, by what the planner says."""
import functools

import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

BF16_TOL, MARGIN = 2e-2, 1e-2


@pytest.mark.parametrize("B,S", [(1, 33), (1, 64), (1, 65), (2, 64), (3, 43), (1, 191), (4, 48), (1, 193), (5, 51), (3, 86), (9, 64)])
@pytest.mark.parametrize("H,nh,F", [(320, 5, 1344), (1024, 8, 2112)])
def test_prompt_rows_at_tile_edges(H, nh, F, B, S):
    d = synth.ModelDims("x", 2, H, nh, F, 300, 256, B, S, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, 2, "greedy", 1.0, seed=3)
    eng = util.make_engine(d, w)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], 2, binding.sampling("greedy", 1.0, 3))
    eng.he_destroy()
    util.compare(got, want, BF16_TOL, MARGIN)


@functools.lru_cache(maxsize=1)
def _layers_4480():
    d = synth.ModelDims("x", 2, 4480, 35, 8960, 300, 1024, 1, 2, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    return d, util.weights_f64(w), binding.upload_weights(w, "bf16")


# rows B S of the prompt pass (70 and more sequences: B rows of the pass ahead of the last token, and of the wide step); tile rows x
# tile columns / k ranges of the GEMMs it is there for.  65, 129, 193, 257, 385, 577, 769 and 1793 rows: one row in the last tile
# of at least one of them, or one 32-row block and a row; 128, 192, 256, 384: full tiles; 127, 191, 255, 383: a row short.
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("B,S,plan", [
    (5, 13, {"qkv": (128, 256, 4), "fc1": (128, 256, 7), "fc2": (128, 256, 14)}),
    (1, 127, {"qkv": (128, 256, 4), "out_proj": (64, 256, 7)}),
    (4, 32, {"qkv": (128, 256, 4), "out_proj": (64, 256, 7)}),
    (3, 43, {"qkv": (192, 256, 4), "fc1": (192, 256, 5), "fc2": (128, 256, 7)}),
    (1, 191, {"qkv": (192, 256, 4), "fc1": (128, 256, 3)}),
    (4, 48, {"qkv": (192, 256, 4), "fc1": (128, 256, 3)}),
    (1, 193, {"qkv": (128, 256, 2), "out_proj": (128, 256, 7)}),
    (5, 51, {"qkv": (128, 256, 2), "fc1": (128, 256, 3), "fc2": (128, 256, 7)}),
    (1, 257, {"qkv": (192, 256, 2), "out_proj": (128, 256, 4), "fc1": (192, 256, 3), "fc2": (192, 256, 7)}),
    (1, 383, {"qkv": (192, 256, 2), "fc2": (192, 256, 7)}),
    (6, 64, {"qkv": (192, 256, 2), "fc2": (192, 256, 7)}),
    (7, 55, {"qkv": (128, 256, 1), "out_proj": (128, 256, 3), "fc2": (192, 256, 4)}),
    (1, 577, {"qkv": (192, 256, 1), "fc1": (128, 256, 1), "fc2": (192, 256, 3)}),
    (1, 769, {"qkv": (256, 256, 1), "fc2": (128, 256, 2)}),
    (12, 75, {"qkv": (256, 256, 1), "fc1": (192, 256, 1), "fc2": (256, 256, 3)}),
    (11, 163, {"qkv": (256, 256, 1), "fc1": (256, 320, 1), "fc2": (256, 320, 2)}),
    (80, 2, {"qkv": (128, 256, 4), "fc1": (128, 256, 7), "fc2": (128, 256, 14)}),
    (129, 2, {"qkv": (192, 256, 4), "fc1": (192, 256, 5), "fc2": (128, 256, 7)}),
])
def test_passes_on_every_tile(B, S, plan, ragged):
    """Prompt pass and a decode step on its keys and values, the first, the last and a middle sequence against the oracle's run
    of it alone; lengths that differ send a left-padded batch through QKV's finishing kernel as well."""
    import torch
    base, w64, w_dev = _layers_4480()
    cfg = binding.make_config(base, max_batch=B, max_seq_len=S + 1)
    rows = B * S if B <= 64 else B
    for g, want in plan.items():
        a = binding.he_plan_pass_gemm(cfg, rows, g)
        assert (a.tile_rows, a.tile_cols, a.ksplit) == want, g
    rng = np.random.default_rng(17 * B + S)
    prompts = rng.integers(0, base.vocab, (B, S)).astype(np.int32)
    lens = rng.integers(1, S + 1, B).astype(np.int32) if ragged else np.full(B, S, np.int32)
    if ragged:
        lens[0], lens[-1] = S, 1 if B > 1 else S - 37
    some = sorted({0, B // 2, B - 1})
    want = {b: O.generate(w64, prompts[b:b + 1, S - lens[b]:], 2, base.n_heads, mode="greedy", eps=base.ln_eps) for b in some}
    feed = np.zeros(B, np.int32)
    for b in some:
        feed[b] = want[b]["ids"][0, 0]
    eng = binding.Engine(cfg, w_dev)
    p, samp = torch.from_numpy(prompts).cuda(), binding.sampling("greedy")
    first = eng.he_prefill_ragged(p, torch.from_numpy(lens).cuda(), samp, True) if ragged else eng.he_prefill(p, samp, True)
    second = eng.he_decode_step(torch.from_numpy(feed).cuda(), samp, True)
    torch.cuda.synchronize()
    got = [first[2].cpu().numpy(), second[2].cpu().numpy()]
    eng.he_destroy()
    for b in some:
        for n in range(2):
            assert float(np.abs(got[n][b] - want[b]["logits"][n, 0]).max()) <= BF16_TOL, (b, n)


@pytest.mark.parametrize("B", [65, 96, 129, 200])
def test_wide_decode_rows(B):
    d = synth.ModelDims("x", 2, 1024, 8, 4096, 300, 64, B, 3, 3, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, 3, "greedy", 1.0, seed=3)
    eng = util.make_engine(d, w)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], 3, binding.sampling("greedy", 1.0, 3))
    eng.he_destroy()
    util.compare(got, want, BF16_TOL, MARGIN)


@pytest.mark.parametrize("B,T", [(1, 17), (1, 64), (2, 33), (3, 64)])
def test_score_few_rows(B, T):
    import torch
    d = synth.ModelDims("x", 1, 256, 4, 512, 1111, 128, B, T, 1, "bf16", "greedy")
    w = synth.make_weights(d, seed=3)
    ids = synth.make_prompts(d, seed=4, batch=B, prompt_len=T)
    eng = util.make_engine(d, w, max_batch=B, max_seq_len=T)
    got = eng.he_score(torch.from_numpy(ids).cuda())
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    eng.he_destroy()
    want = O.score(util.weights_f64(w), ids, d.n_heads, eps=d.ln_eps, pos_offset=d.pos_offset)
    assert float(np.abs(got - want).max()) <= BF16_TOL


@pytest.mark.parametrize("B,S,max_seq,H,nh", [(1, 30, 40, 256, 4), (1, 200, 260, 256, 2), (2, 500, 1100, 128, 2), (9, 33, 300, 2048, 32),
                                              (9, 33, 130, 2048, 16), (3, 1, 600, 64, 1)])
def test_decode_attention_wavefront_counts(B, S, max_seq, H, nh):
    """Few (row, head) pairs: caches below and above one round of keys, both head dimensions."""
    d = synth.ModelDims("x", 1, H, nh, 2 * H, 300, 1200, B, S, 4, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, 4, "greedy", 1.0, seed=3)
    eng = util.make_engine(d, w, max_seq_len=max_seq)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], 4, binding.sampling("greedy", 1.0, 3))
    eng.he_destroy()
    util.compare(got, want, BF16_TOL, MARGIN)


@functools.lru_cache(maxsize=1)
def _lm_weights(V, H):
    return synth.make_weights(synth.ModelDims("x", 1, H, H // 64, 2 * H, V, 64, 1, 2, 3, "bf16", "gumbel"), seed=5)


# The streamed form (slices of 32 rows, the noise formed between the load rounds): one slice or several, vocabularies that end
# inside a 32-wide tile, a k range too short for a load round.  The tiled form (the noise behind the product): rows at the
# edges of its 64-, 128- and 192-row tiles, a vocabulary that ends inside a 256-wide tile.
@pytest.mark.parametrize("V,H,B,tile", [(V, H, B, 32) for V, H in ((31, 64), (257, 128), (2500, 512), (9000, 64))
                                        for B in (1, 17, 32, 33, 65, 100, 130)] +
                         [(50272, 512, B, t) for B, t in ((33, 64), (63, 64), (64, 64), (65, 128), (127, 128), (128, 128), (129, 192),
                                                          (191, 192), (192, 192), (193, 128))])
def test_lm_head_sampled_rows_and_vocabularies(V, H, B, tile):
    d = synth.ModelDims("x", 1, H, H // 64, 2 * H, V, 64, B, 2, 3, "bf16", "gumbel")
    assert binding.he_plan_pass_gemm(binding.make_config(d), B, "lm_head").tile_rows == tile
    w = _lm_weights(V, H)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, 3, "gumbel", 0.9, seed=3)
    eng = util.make_engine(d, w)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], 3, binding.sampling("gumbel", 0.9, 3))
    eng.he_destroy()
    util.compare(got, want, BF16_TOL, MARGIN)


def test_prompt_attention_large_queries():
    """A query component near the end of the half range (49152, against a key component of 2^-13): the two half terms of the
    prompt attention hold it."""
    d = synth.ModelDims("x", 2, 128, 2, 256, 300, 64, 2, 40, 1, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    lw = w["layers"][0]
    for h in range(2):
        q, k = 64 * h, 128 + 64 * h
        lw["wqkv"][k] = 0.0
        lw["bqkv"][k] = 2.0 ** -13
        lw["bqkv"][q] = 8 * 49152.0
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, 1, "greedy", 1.0, seed=3)
    eng = util.make_engine(d, w)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], 1, binding.sampling("greedy", 1.0, 3))
    eng.he_destroy()
    util.compare(got, want, BF16_TOL, MARGIN)


@pytest.mark.parametrize("B", [4, 40, 70])
def test_lm_head_nan_slice_reaches_the_logprob(B):
    """A stretch of the vocabulary whose logits are all NaN: the soft-max over the whole vocabulary is NaN, the chosen token
    the best of the others."""
    import torch
    d = synth.ModelDims("x", 1, 128, 2, 256, 2000, 64, B, 3, 2, "bf16", "greedy")
    w = binding.upload_weights(synth.make_weights(d, seed=5, tied=False), "bf16")
    w["lm_head"][512:1024] = float("nan")
    eng = binding.Engine(binding.make_config(d), w)
    p = torch.from_numpy(synth.make_prompts(d, seed=6)).cuda()
    s = binding.sampling("greedy")
    for ids, lp, lg in (eng.he_prefill(p, s, True), eng.he_decode_step(p[:, 0].contiguous(), s, True)):
        torch.cuda.synchronize()
        assert torch.isnan(lg[:, 512:1024]).all() and torch.isfinite(lg[:, :512]).all() and torch.isfinite(lg[:, 1024:]).all()
        assert torch.isnan(lp).all()
        assert torch.equal(ids.long(), torch.nan_to_num(lg, nan=-1e30).argmax(1))
    eng.he_destroy()


@pytest.mark.parametrize("dtype,impl", [("f32", 0), ("bf16", 1), ("bf16", 0)])
def test_logits_of_nothing_but_nan(dtype, impl):
    """No token is the best of such a row: NaN log-probabilities, and the id that stands for none is looked up nowhere -- the
    following step clamps it like any id outside the vocabulary."""
    import torch
    d = synth.ModelDims("x", 1, 128, 2, 256, 2000, 64, 3, 3, 4, dtype, "greedy")
    w = binding.upload_weights(synth.make_weights(d, seed=5, tied=False), dtype)
    w["lm_head"][:] = float("nan")
    eng = binding.Engine(binding.make_config(d, impl=impl), w)
    ids, lp = eng.he_generate(torch.from_numpy(synth.make_prompts(d, seed=6)).cuda(), d.gen_len, binding.sampling("greedy"))
    torch.cuda.synchronize()
    assert torch.isnan(lp).all() and not ((ids >= 0) & (ids < d.vocab)).any()
    eng.he_destroy()


@pytest.mark.parametrize("B,S,H,nh", [(1, 32, 128, 2), (3, 129, 192, 3), (2, 257, 256, 2), (5, 400, 640, 5)])
def test_prompt_attention_blocks_and_pairs(B, S, H, nh):
    """Query blocks of 128 with remainders, (sequence, head) pairs that do not divide over the eight XCDs, both head dimensions,
    lengths that differ (rows of padding, blocks of nothing but padding)."""
    import torch
    d = synth.ModelDims("x", 2, H, nh, 2 * H, 300, 512, B, S, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    lens = np.array([max(1, (S * (b + 1)) // B - (b % 2)) for b in range(B)], np.int32)
    eng = util.make_engine(d, w)
    _, lp, lg = eng.he_prefill_ragged(torch.from_numpy(prompts).cuda(), torch.from_numpy(lens).cuda(), binding.sampling("greedy"), True)
    torch.cuda.synchronize()
    got = lg.cpu().numpy()
    eng.he_destroy()
    w64 = util.weights_f64(w)
    for b in range(B):
        one = util.oracle_run(d, w64, prompts[b:b + 1, S - lens[b]:], 1, "greedy")
        assert float(np.abs(got[b] - one["logits"][0, 0]).max()) <= BF16_TOL, b
