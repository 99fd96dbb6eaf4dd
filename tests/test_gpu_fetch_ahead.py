"""Decode steps whose attention launch fetches the out-projection's weights as well: few and odd numbers of heads, rows and 16-row units, k ranges,
8-bit weights; against the oracle.  (Which lines they are: tests/test_fetch_ahead_cpu.py.)"""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("H,nh,B", [(128, 1, 1), (192, 3, 3), (1088, 17, 2), (2048, 32, 5), (2048, 32, 16), (2560, 20, 1), (512, 8, 48)])
def test_decode_steps(H, nh, B, fp8):
    import torch
    d = synth.ModelDims("x", 2, H, nh, 512, 300, 40, 1, 2, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=21)
    w_dev = binding.upload_weights(w, "bf16")
    rng = np.random.default_rng(B)
    prompts = rng.integers(0, d.vocab, (B, 9)).astype(np.int32)
    feed = rng.integers(0, d.vocab, (2, B)).astype(np.int32)
    cfg = binding.make_config(d, max_batch=B, max_seq_len=16, weights_fp8=int(fp8))
    eng = binding.Engine(cfg, w_dev)
    samp = binding.sampling("greedy")
    eng.he_prefill(torch.from_numpy(prompts).cuda(), samp, True)
    got = [eng.he_decode_step(torch.from_numpy(f).cuda(), samp, True)[2].cpu().numpy() for f in feed]
    eng.he_destroy()
    assert len(binding.he_plan_fetch_ahead(cfg, B)) > 0
    if fp8:  # against the model that the codes stand for
        w = dict(w, layers=[dict(lw, **{m: O.quantize_e4m3_rows(lw[m])[0].astype(np.float32) for m in ("wqkv", "wo", "w1", "w2")}) for lw in w["layers"]])
    for b in sorted({0, B // 2, B - 1}):
        z = O.forward_full(util.weights_f64(w), np.concatenate([prompts[b], feed[:, b]])[None], nh, eps=d.ln_eps)[0]
        for n in range(2):
            assert float(np.abs(got[n][b] - z[9 + n]).max()) <= 2e-2, (b, n)  # (the other bfloat16 passes' bound)
