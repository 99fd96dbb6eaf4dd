"""GPU parity: the HIP engine, called through the C ABI, against the CPU oracle
on the same seeded inputs.  Tolerances: logits / log-probs max-abs 1e-4 on the
f32 path and 2e-2 on the bf16 path; token ids bit-exact wherever the oracle's
top-2 margin of the arg-maxed score exceeds 1e-2, one of the oracle's two best
elsewhere.  The oracle is the unrounded definition in both cases: float64
arithmetic on the configuration's weights (bf16 values on the bf16 path)."""
import numpy as np
import pytest
from ctypes import byref as C_byref

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

F32_TOL, BF16_TOL, MARGIN = 1e-4, 2e-2, 1e-2


def test_rng_words_bit_exact():
    for seed, b, n, v0, cnt in [(0, 0, 0, 0, 1000), (42, 31, 255, 50000, 272), ((1 << 63) + 12345, 7, 3, 0, 4097)]:
        got = binding.he_rng_words(seed, b, n, v0, cnt).cpu().numpy().view(np.uint32)
        want = O.random_u32(seed, b, n, np.arange(v0, v0 + cnt, dtype=np.uint32))
        assert np.array_equal(got, want)


@pytest.mark.parametrize("mode", ["greedy", "gumbel"])
def test_tiny_f32_teacher_forced(mode):
    d = synth.CONFIGS["tiny"]
    w = synth.make_weights(d, seed=0)
    prompts = synth.make_prompts(d, seed=1234)
    want = util.oracle_run(d, w, prompts, d.gen_len, mode, 1.0, seed=42)
    eng = util.make_engine(d, w)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], d.gen_len, binding.sampling(mode, 1.0, 42))
    rep = util.compare(got, want, F32_TOL, MARGIN)
    print(mode, rep)
    assert rep["sure_frac"] > 0.5  # the bit-exact id check is not vacuous
    eng.he_destroy()


def test_tiny_f32_generate_matches_oracle_free_running():
    import torch
    d = synth.CONFIGS["tiny"]
    w = synth.make_weights(d, seed=0)
    prompts = synth.make_prompts(d, seed=1234)
    eng = util.make_engine(d, w)
    for mode in ("greedy", "gumbel"):
        want = util.oracle_run(d, w, prompts, d.gen_len, mode, 1.0, seed=7)
        ids, lp = eng.he_generate(torch.from_numpy(prompts).cuda(), d.gen_len, binding.sampling(mode, 1.0, 7))
        torch.cuda.synchronize()
        ids, lp = ids.cpu().numpy(), lp.cpu().numpy()
        # free running: rows agree up to (not including) the first low-margin step
        for b in range(d.batch):
            unsure = np.nonzero(want["margins"][b] <= MARGIN)[0]
            k = int(unsure[0]) if len(unsure) else d.gen_len
            assert np.array_equal(ids[b, :k], want["ids"][b, :k])
            assert k == 0 or np.abs(lp[b, :k] - want["logprobs"][b, :k]).max() <= F32_TOL
    eng.he_destroy()


@pytest.mark.parametrize("L,H,nh,F,V,B,S,G,tied", [
    (1, 64, 2, 128, 100, 1, 1, 3, True),      # single-token prompt, batch 1
    (2, 192, 3, 320, 777, 3, 37, 5, False),   # ragged everything, head_dim 64, untied head
    (0, 128, 1, 128, 300, 2, 5, 2, True),     # no layers: embedding -> final LN -> head
    (1, 256, 2, 512, 1000, 5, 70, 3, True),   # head_dim 128, rows beyond one tile
])
def test_f32_shapes(L, H, nh, F, V, B, S, G, tied):
    d = synth.ModelDims("x", L, H, nh, F, V, 128, B, S, G, "f32", "gumbel")
    w = synth.make_weights(d, seed=5, tied=tied)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, w, prompts, G, "gumbel", 0.8, seed=3)
    eng = util.make_engine(d, w)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], G, binding.sampling("gumbel", 0.8, 3))
    print(util.compare(got, want, F32_TOL, MARGIN))
    eng.he_destroy()


def test_capacity_and_state_errors():
    import torch
    d = synth.CONFIGS["tiny"].sliced(n_layers=1)
    w = synth.make_weights(d, seed=0)
    eng = util.make_engine(d, w, max_batch=2, max_seq_len=8)
    s = binding.sampling()
    ids8 = torch.zeros(2, 8, dtype=torch.int32, device="cuda")
    with pytest.raises(binding.HeError) as ei:
        eng.he_decode_step(ids8[:, 0].contiguous(), s)
    assert ei.value.status == 6  # decode before prefill
    with pytest.raises(binding.HeError) as ei:
        eng.he_prefill(torch.zeros(3, 4, dtype=torch.int32, device="cuda"), s)
    assert ei.value.status == 3  # batch above capacity
    with pytest.raises(binding.HeError) as ei:
        eng.he_prefill(torch.zeros(2, 9, dtype=torch.int32, device="cuda"), s)
    assert ei.value.status == 3
    eng.he_prefill(ids8, s)
    assert eng.cache_len() == 8
    with pytest.raises(binding.HeError) as ei:
        eng.he_decode_step(ids8[:, 0].contiguous(), s)
    assert ei.value.status == 3  # cache full
    with pytest.raises(binding.HeError) as ei:
        eng.he_prefill(ids8, s)
    assert ei.value.status == 6  # cache not empty
    with pytest.raises(binding.HeError) as ei:
        eng.he_generate(ids8[:, :4].contiguous(), 6, s)
    assert ei.value.status == 3  # 4 + 6 - 1 > 8
    out, _ = eng.he_generate(ids8[:, :4].contiguous(), 5, s)  # exactly fits; engine usable after errors
    torch.cuda.synchronize()
    assert out.shape == (2, 5) and eng.cache_len() == 8
    # out-of-range token ids are clamped, never read out of bounds
    big = torch.full((2, 4), 10 ** 6, dtype=torch.int32, device="cuda")
    a, _ = eng.he_generate(big, 2, s)
    b, _ = eng.he_generate(torch.full((2, 4), d.vocab - 1, dtype=torch.int32, device="cuda"), 2, s)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    eng.he_destroy()


# ------------------------------------------------------------------ bf16 path

def _bf16_case(d, tied, G, mode, temp, impl, seed=3, half_cache_diagnostic=False):
    w = synth.make_weights(d, seed=5, tied=tied)
    prompts = synth.make_prompts(d, seed=6)
    w64 = util.weights_f64(w)
    want = util.oracle_run(d, w64, prompts, G, mode, temp, seed=seed)
    eng = util.make_engine(d, w, impl=impl)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], G, binding.sampling(mode, temp, seed))
    rep = util.compare(got, want, BF16_TOL, MARGIN)
    if half_cache_diagnostic:  # how much of the distance is the half-precision KV cache: the oracle with that one rounding
        diag = util.oracle_run(d, w64, prompts, G, mode, temp, seed=seed, kv_dtype="f16")
        rep["logit_err_vs_half_cache_oracle"] = float(np.abs(got["logits"] - diag["logits"]).max())
    eng.he_destroy()
    return rep


@pytest.mark.parametrize("impl", [0, 1])
@pytest.mark.parametrize("L,H,nh,F,V,B,S,G,tied", [
    (2, 256, 4, 512, 1000, 3, 37, 5, False),   # head_dim 64, ragged rows, prompt pass on the tiled GEMM
    (2, 256, 2, 576, 1111, 5, 70, 4, True),    # head_dim 128, vocab not a multiple of 32, >2 row tiles
    (1, 128, 2, 128, 300, 1, 1, 4, True),      # single-token prompt, batch 1: skinny path only
    (0, 128, 1, 128, 300, 2, 5, 2, True),      # no layers
    (1, 192, 3, 320, 513, 40, 3, 3, True),     # decode batch above one 32-row tile
])
def test_bf16_shapes(impl, L, H, nh, F, V, B, S, G, tied):
    d = synth.ModelDims("x", L, H, nh, F, V, 128, B, S, G, "bf16", "gumbel")
    rep = _bf16_case(d, tied, G, "gumbel", 0.9, impl)
    print(impl, rep)
    assert rep["id_match"] > 0.9


@pytest.mark.parametrize("name,L,B,S,G", [
    ("opt-1.3b", 2, 32, 20, 4),   # full decode batch
    ("opt-13b", 2, 4, 131, 3),    # prompt rows span several 128-row tiles plus a ragged tail
    ("opt-13b", 1, 32, 9, 3),     # full decode batch of the headline workload
    ("opt-13b", 1, 5, 221, 2),    # 1100 prompt rows: QKV and FC1 tiles two to a CU, ragged last tile
    ("opt-6.7b", 2, 16, 64, 3),
    ("opt-13b", 1, 64, 5, 3),     # 33..64 sequences: two 32-row slices per workgroup of the weight-streaming GEMMs
    ("opt-13b", 1, 40, 4, 3),     # ... with a ragged second slice
    ("opt-13b", 1, 16, 4, 2),     # at most 16 sequences: only the first 16-row half of the activation panel is multiplied
    ("opt-13b", 1, 17, 4, 2),     # ... one more: both halves
    ("opt-13b", 1, 48, 3, 2),     # at most 48: three of the two slices' four halves
    ("opt-13b", 1, 49, 3, 2),     # ... one more: all four
    ("opt-13b", 1, 96, 5, 3),     # more than 64 sequences: the decode step on k-split prompt-pass tiles
])
def test_bf16_real_layer_shapes(name, L, B, S, G):
    """Layer-truncated models at the real GEMM / head / vocabulary shapes of the benchmark configs."""
    base = synth.CONFIGS[name]
    d = base.sliced(n_layers=L, batch=B, prompt_len=S, gen_len=G, max_positions=256)
    rep = _bf16_case(d, True, G, base.sampling, 1.0, 0, seed=42, half_cache_diagnostic=(B == 32 and name == "opt-13b"))
    print(name, L, B, S, G, rep)
    # measured against the unrounded definition: 13B / 6.7B layer shapes 3e-3 .. 6e-3, 1.3B 2e-3; half of the stated
    # tolerance is kept as a regression bound so that a loss of precision shows before the tolerance is reached
    assert rep["logit_err"] <= 1e-2
    assert rep["id_match"] > 0.9


def test_generate_graph_replay_matches_step_by_step():
    """he_generate on a stream of its own replays captured decode steps (runs of eight steps per graph launch, single
    steps for the remainder: 44 steps here are five runs and four single steps); on the NULL stream it launches step
    by step.  Same kernels, so ids and log-probs must be bit-identical -- on every one of several calls, with other
    work and synchronisations in between."""
    import torch
    d = synth.ModelDims("x", 2, 256, 4, 512, 1000, 128, 5, 9, 45, "bf16", "gumbel")
    w = synth.make_weights(d, seed=5)
    prompts = torch.from_numpy(synth.make_prompts(d, seed=6)).cuda()
    samp = binding.sampling("gumbel", 1.0, 11)
    ref_eng = util.make_engine(d, w)
    ref_ids, ref_lp = ref_eng.he_generate(prompts, d.gen_len, samp)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    w_dev = binding.upload_weights(w, d.dtype)
    eng = binding.Engine(binding.make_config(d, stream=stream.cuda_stream), w_dev)
    for rep in range(4):
        with torch.cuda.stream(stream):
            ids, lp = eng.he_generate(prompts, d.gen_len, samp)
        stream.synchronize()
        assert torch.equal(ids, ref_ids) and torch.equal(lp, ref_lp), rep
        junk = torch.randn(1 << 16, device="cuda").sum().item()  # eager work between replays
        assert junk == junk
    # a different batch size and length re-captures
    with torch.cuda.stream(stream):
        ids2, lp2 = eng.he_generate(prompts[:3].contiguous(), 7, samp)
    stream.synchronize()
    r2, l2 = ref_eng.he_generate(prompts[:3].contiguous(), 7, samp)
    torch.cuda.synchronize()
    assert torch.equal(ids2, r2) and torch.equal(lp2, l2)
    # f32 path through the same mechanism
    d32 = synth.CONFIGS["tiny"]
    w32 = synth.make_weights(d32, seed=0)
    p32 = torch.from_numpy(synth.make_prompts(d32, seed=1234)).cuda()
    e_null = util.make_engine(d32, w32)
    a, al = e_null.he_generate(p32, d32.gen_len, binding.sampling("greedy"))
    torch.cuda.synchronize()
    e_str = binding.Engine(binding.make_config(d32, stream=stream.cuda_stream), binding.upload_weights(w32, "f32"))
    for rep in range(3):
        with torch.cuda.stream(stream):
            b, bl = e_str.he_generate(p32, d32.gen_len, binding.sampling("greedy"))
        stream.synchronize()
        assert torch.equal(a, b) and torch.equal(al, bl)
    for e in (ref_eng, eng, e_null, e_str):
        e.he_destroy()


def test_reset_clears_every_arrival_counter():
    """Counters that a failed launch left behind -- of the k-split hand-off and of the kernel that ends a step -- are gone
    after he_reset, and the next generation is the one of an untouched engine."""
    import torch
    d = synth.ModelDims("x", 2, 1024, 8, 4096, 1000, 64, 5, 9, 6, "bf16", "gumbel")
    eng = util.make_engine(d, synth.make_weights(d, seed=5))
    p = torch.from_numpy(synth.make_prompts(d, seed=6)).cuda()
    s = binding.sampling("gumbel", 1.0, 11)
    ids0, lp0 = eng.he_generate(p, d.gen_len, s)
    assert eng.he_arrival_counters_nonzero() == 0
    eng.he_arrival_counters_set(0x5A5A)
    assert eng.he_arrival_counters_nonzero() > 1
    eng.he_reset()
    assert eng.he_arrival_counters_nonzero() == 0
    ids1, lp1 = eng.he_generate(p, d.gen_len, s)
    torch.cuda.synchronize()
    assert torch.equal(ids0, ids1) and torch.equal(lp0, lp1)
    assert eng.he_arrival_counters_nonzero() == 0
    eng.he_destroy()


def test_timing_hook_counts_launches():
    import torch
    d = synth.ModelDims("x", 3, 256, 4, 512, 1000, 128, 4, 6, 4, "bf16", "greedy")
    eng = util.make_engine(d, synth.make_weights(d, seed=5))
    p = torch.from_numpy(synth.make_prompts(d, seed=6)).cuda()
    s = binding.sampling()
    ids0, lp0 = eng.he_generate(p, 4, s)
    eng.he_timing_enable(True)
    ids1, lp1 = eng.he_generate(p, 4, s)
    t = eng.he_timing_read()
    eng.he_timing_enable(False)
    assert torch.equal(ids0, ids1) and torch.equal(lp0, lp1)
    # 3 decode steps x 3 layers, plus the last prompt token's share of the last layer (attention, out-projection, FC1,
    # FC2 on the decode kernels; its QKV projection runs with the other prompt rows) and its LM head; "layernorm"
    # counts the decode steps' embedding kernel (their LayerNorms are folded into the GEMMs)
    assert t["fc1"][1] == 10 and t["fc2"][1] == 10 and t["attention"][1] == 10 and t["qkv"][1] == 9
    assert t["lm_head"][1] == 4 and t["layernorm"][1] == 3
    assert all(ms > 0 for ms, n in t.values() if n)
    eng.he_destroy()


@pytest.mark.parametrize("B,S,G", [(1, 2, 1), (2, 1, 1), (3, 33, 2), (64, 4, 2)])
def test_bf16_edge_batches_and_lengths(B, S, G):
    """G = 1 (prompt pass only), a prompt of exactly one 32-query tile plus one, a decode batch of two
    full 32-row slices."""
    d = synth.ModelDims("x", 2, 128, 2, 256, 500, 64, B, S, G, "bf16", "greedy")
    rep = _bf16_case(d, True, G, "greedy", 1.0, 0)
    print(rep)


def test_bf16_long_cache_and_generate_to_capacity():
    """A cache of 2048 positions filled to the last slot: he_generate up to S + G - 1 == max_seq_len,
    checked against the oracle on one sequence at the last steps."""
    import torch
    d = synth.ModelDims("x", 1, 128, 2, 256, 300, 2048, 2, 2000, 49, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    eng = util.make_engine(d, w, max_batch=2, max_seq_len=2048)
    ids, lp = eng.he_generate(torch.from_numpy(prompts).cuda(), d.gen_len, binding.sampling("greedy"))
    torch.cuda.synchronize()
    assert eng.cache_len() == 2048
    with pytest.raises(binding.HeError) as ei:
        eng.he_decode_step(ids[:, -1].contiguous(), binding.sampling("greedy"))
    assert ei.value.status == 3
    want = O.generate(util.weights_f64(w), prompts, d.gen_len, d.n_heads, forced_ids=ids.cpu().numpy())
    sure = want["margins"] > MARGIN
    got = ids.cpu().numpy()
    assert np.array_equal(got[sure], want["ids"][sure])
    same = got == want["ids"]
    assert (same | (got == want["second"])).all()
    assert np.abs(lp.cpu().numpy()[same] - want["logprobs"][same]).max() <= BF16_TOL
    eng.he_destroy()


def test_refresh_weights_picks_up_in_place_update():
    """The training half overwrites the actor's weights in place between generation phases; after
    he_refresh_weights the engine must generate from the new values."""
    import torch
    d = synth.ModelDims("x", 2, 128, 2, 256, 300, 64, 3, 6, 4, "bf16", "greedy")
    w1 = synth.make_weights(d, seed=1)
    w2 = synth.make_weights(d, seed=2)
    p = torch.from_numpy(synth.make_prompts(d, seed=3)).cuda()
    s = binding.sampling("greedy")
    e1 = util.make_engine(d, w1)
    e2 = util.make_engine(d, w2)
    a1, l1 = e1.he_generate(p, 4, s)
    a2, l2 = e2.he_generate(p, 4, s)
    torch.cuda.synchronize()
    assert not torch.equal(l1, l2)
    # overwrite engine 1's borrowed tensors with model 2's values, in place
    dev2 = binding.upload_weights(w2, "bf16")
    for k in ("tok_emb", "pos_emb", "lnf_g", "lnf_b"):
        e1.weights[k].copy_(dev2[k])
    for lw, lw2 in zip(e1.weights["layers"], dev2["layers"]):
        for k in lw:
            lw[k].copy_(lw2[k])
    e1.he_refresh_weights()
    b1, m1 = e1.he_generate(p, 4, s)
    torch.cuda.synchronize()
    assert torch.equal(b1, a2) and torch.equal(m1, l2)
    e1.he_destroy(); e2.he_destroy()


def test_bf16_opt66b_layer_shape():
    """The largest configuration's layer shape (hidden 9216, 72 heads, ffn 36864), one layer."""
    base = synth.CONFIGS["opt-66b"]
    d = base.sliced(n_layers=1, batch=8, prompt_len=40, gen_len=3, max_positions=64)
    rep = _bf16_case(d, True, 3, "greedy", 1.0, 0, seed=1)
    print(rep)


def test_pretiled_weights_give_identical_results():
    """he_config.weights_tiled = 1: the caller tiles the GEMM matrices with he_tile_matrix and the engine
    keeps no copies; ids and log-probs must be bit-identical to the default mode."""
    import torch
    d = synth.ModelDims("x", 2, 256, 2, 576, 1111, 64, 5, 40, 6, "bf16", "gumbel")
    w = synth.make_weights(d, seed=5, tied=True)
    p = torch.from_numpy(synth.make_prompts(d, seed=6)).cuda()
    s = binding.sampling("gumbel", 1.0, 3)
    e0 = util.make_engine(d, w)
    a, al = e0.he_generate(p, d.gen_len, s)
    dev = binding.tile_weights_in_place(binding.upload_weights(w, "bf16"))
    cfg = binding.make_config(d, weights_tiled=1)
    assert binding.lib().he_workspace_bytes(C_byref(cfg)) < binding.lib().he_workspace_bytes(C_byref(e0.cfg))
    e1 = binding.Engine(cfg, dev)
    b, bl = e1.he_generate(p, d.gen_len, s)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(al, bl)
    e0.he_destroy(); e1.he_destroy()


@pytest.mark.parametrize("L,H,nh,F,V,B,S,G", [
    (2, 96, 3, 77, 101, 3, 5, 3),       # odd ffn and vocabulary: element-wise loads and stores
    (1, 136, 17, 24, 64, 1, 1, 2),      # head dimension 8, one row
    (2, 200, 1, 300, 333, 17, 4, 3),    # head dimension 200, a second 16-row tile, a k range that ends inside a step
    (1, 256, 4, 1024, 900, 5, 13, 2),   # 65 prompt rows: one more than the few-row kernel takes
    (1, 512, 8, 2048, 500, 9, 29, 2),   # 64 x 64 tiles with row and column remainders
])
def test_f32_gemm_variants(L, H, nh, F, V, B, S, G):
    d = synth.ModelDims("x", L, H, nh, F, V, 128, B, S, G, "f32", "greedy")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, G, "greedy", 1.0, seed=3)
    eng = util.make_engine(d, w)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], G, binding.sampling("greedy", 1.0, 3))
    eng.he_destroy()
    util.compare(got, want, 1e-5, 1e-4)  # logits of order one: a few hundred float roundings
