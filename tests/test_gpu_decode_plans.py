"""GPU parity of the weight-streaming decode GEMMs at the edges of their plans, against the oracle: one unit of 16 weight rows per
workgroup with one k range and with several, k steps that do not divide over the wavefronts (fewer than one round each, whole
rounds and a remainder), row counts at the edges of the 16-row halves and 32-row slices, 16- and 8-bit weights, sequences of
different lengths."""
import functools

import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

BF16_TOL, MARGIN = 2e-2, 1e-2


@functools.lru_cache(maxsize=1)
def _model(H, nh, F, B, fp8):
    d = synth.ModelDims("x", 2, H, nh, F, 300, 64, B, 5, 3, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    ref = w
    if fp8:
        ref = dict(w, layers=[{k: (O.quantize_e4m3_rows(v)[0] if k in ("wqkv", "wo", "w1", "w2") else v) for k, v in lw.items()}
                              for lw in w["layers"]])
    return d, w, util.weights_f64(ref)


# 320: 10 steps of 32 (5 of 64) over eight wavefronts; 1344 = 42 (21); 1088 = 34 (17); 2240 = 70 (35); 128: 4 (2)
@pytest.mark.parametrize("fp8", [0, 1])
@pytest.mark.parametrize("B", [1, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("H,nh,F", [(128, 2, 192), (320, 5, 1344), (1088, 17, 2240)])
def test_decode_steps_at_plan_edges(H, nh, F, B, fp8):
    d, w, ref = _model(H, nh, F, B, fp8)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, ref, prompts, 3, "greedy")
    eng = binding.Engine(binding.make_config(d, weights_fp8=fp8), binding.upload_weights(w, "bf16"))
    got = util.engine_teacher_forced(eng, prompts, want["ids"], 3, binding.sampling("greedy"))
    assert eng.he_arrival_counters_nonzero() == 0
    eng.he_destroy()
    util.compare(got, want, BF16_TOL, MARGIN)


def test_one_unit_plans_are_the_ones_reached():
    cap = 2 * 8 * 64 * 4096
    assert binding.he_plan_decode_gemm(16, 1088, 1088, True, cap, 256) == (16, 1, 1)
    assert binding.he_plan_decode_gemm(48, 1088, 1088, True, cap, 256) == (16, 1, 1)
    assert binding.he_plan_decode_gemm(1, 4096, 4096, True, cap, 256) == (16, 1, 1)
    assert binding.he_plan_decode_gemm(16, 2048, 8192, True, cap, 256) == (16, 1, 2)


@pytest.mark.parametrize("B,ragged", [(1, False), (13, True), (32, False), (40, True)])
def test_decode_steps_of_one_unit_and_several_ranges(B, ragged):
    """2048 x 8192: FC2 in k ranges of two or more workgroups; sequences of different lengths look their cache rows up."""
    import torch
    d = synth.ModelDims("x", 1, 2048, 32, 8192, 200, 64, B, 4, 3, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    ref = util.weights_f64(w)
    prompts = synth.make_prompts(d, seed=6)
    lens = (1 + np.arange(B) % 4).astype(np.int32) if ragged else np.full(B, 4, np.int32)
    eng = util.make_engine(d, w)
    s = binding.sampling("greedy")
    eng.he_reset()
    feeds = np.random.default_rng(3).integers(0, 200, (2, B)).astype(np.int32)
    _, _, logits = eng.he_prefill_ragged(torch.from_numpy(prompts).cuda(), torch.from_numpy(lens).cuda(), s, want_logits=True)
    got = [logits.cpu().numpy()]
    for f in feeds:
        got.append(eng.he_decode_step(torch.from_numpy(f).cuda(), s, want_logits=True)[2].cpu().numpy())
    assert eng.he_arrival_counters_nonzero() == 0
    eng.he_destroy()
    for b in range(0, B, max(1, B // 5)):
        seq = np.concatenate([prompts[b, 4 - lens[b]:], feeds[:, b]])[None]
        z = O.forward_full(ref, seq, d.n_heads, eps=d.ln_eps, pos_offset=d.pos_offset)[0]
        for n in range(3):
            assert float(np.abs(got[n][b] - z[lens[b] - 1 + n]).max()) <= BF16_TOL, (b, n)
