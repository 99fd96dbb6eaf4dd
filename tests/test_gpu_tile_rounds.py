"""Prompt passes whose GEMMs have more 256-row tiles than workgroups, each workgroup taking several: slots that hold no tile, a last round
that not every workgroup has, and k ranges behind whole tiles; the LayerNorms' two forms (of 96 MB of residual on, and below).  Against the
oracle."""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


# (room for partial sums grows with max_batch: none to spare in a full batch, so no k ranges)
@pytest.mark.parametrize("H,nh,F,max_batch,B,S,ragged,split", [
    (1280, 20, 5120, 56, 56, 253, True, None), (1536, 24, 6144, 53, 53, 253, False, None),
    (3072, 24, 3072, 64, 32, 253, False, 2048), (2048, 16, 2048, 100, 47, 253, True, 0),
])
def test_rounds_of_tiles(H, nh, F, max_batch, B, S, ragged, split):
    import torch
    d = synth.ModelDims("x", 1, H, nh, F, 300, S + 2, 1, 2, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=11)
    cfg = binding.make_config(d, max_batch=max_batch, max_seq_len=S + 1)
    plans = {g: binding.he_plan_pass_gemm(cfg, B * S, g) for g in binding.PASS_GEMMS[:4]}
    for g, n in (("qkv", 3 * H), ("fc1", F)):
        p = plans[g]
        assert p.tile_rows == 256 and p.workgroup_cols >= 256 and -(-n // p.workgroup_cols) * -(-B * S // 256) > 256
    assert split is None or all(plans[g].ksplit == 2 and plans[g].split_col == split for g in ("out_proj", "fc2"))
    rng = np.random.default_rng(B)
    prompts = rng.integers(0, d.vocab, (B, S)).astype(np.int32)
    lens = rng.integers(1, S + 1, B).astype(np.int32) if ragged else np.full(B, S, np.int32)
    feed = rng.integers(0, d.vocab, B).astype(np.int32)
    eng = binding.Engine(cfg, binding.upload_weights(w, "bf16"))
    p, samp = torch.from_numpy(prompts).cuda(), binding.sampling("greedy")
    first = eng.he_prefill_ragged(p, torch.from_numpy(lens).cuda(), samp, True) if ragged else eng.he_prefill(p, samp, True)
    second = eng.he_decode_step(torch.from_numpy(feed).cuda(), samp, True)
    got = [first[2].cpu().numpy(), second[2].cpu().numpy()]
    eng.he_destroy()
    w64 = util.weights_f64(w)
    for b in sorted({0, B // 2, B - 1}):
        z = O.forward_full(w64, np.append(prompts[b, S - lens[b]:], feed[b])[None], nh, eps=d.ln_eps)[0]
        for n in range(2):
            assert float(np.abs(got[n][b] - z[lens[b] - 1 + n]).max()) <= 2e-2, (b, n)  # (the other bfloat16 passes' bound)
