"""GPU parity of the folded LayerNorm's vectors W gamma and W beta (through the decode steps that use them) against the oracle: matrices
of few and of many tiles of 32 rows, an odd number of them, a last one partly filled, and fewer blocks of k than wavefronts."""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2


# 16384 rows: 512 tiles, the fewest that are taken two to a workgroup; 16416: 513, the last workgroup with one; 64 wide: four blocks of k
@pytest.mark.parametrize("H,F,vocab", [(128, 256, 16352), (128, 256, 16384), (128, 256, 16385), (128, 256, 16447), (64, 16448, 333),
                                       (192, 16384, 16416), (576, 1152, 16417)])
@pytest.mark.parametrize("B", [1, 9])
def test_decode_step_with_folded_layernorm(H, F, vocab, B):
    import torch
    base = synth.ModelDims("x", 2, H, H // 64, F, vocab, 64, 1, 2, 2, "bf16", "greedy")
    w = synth.make_weights(base, seed=13)
    w64 = util.weights_f64(w)
    eng = binding.Engine(binding.make_config(base, max_batch=B, max_seq_len=8), binding.upload_weights(w, "bf16"))
    rng = np.random.default_rng(B + vocab)
    prompts = rng.integers(0, vocab, (B, 5)).astype(np.int32)
    feed = rng.integers(0, vocab, B).astype(np.int32)
    samp = binding.sampling("greedy")
    eng.he_prefill(torch.from_numpy(prompts).cuda(), samp, True)
    got = eng.he_decode_step(torch.from_numpy(feed).cuda(), samp, True)[2].cpu().numpy()
    eng.he_destroy()
    for b in sorted({0, B - 1}):
        z = O.forward_full(w64, np.append(prompts[b], feed[b])[None], H // 64, eps=base.ln_eps)[0]
        assert float(np.abs(got[b] - z[5]).max()) <= BF16_TOL, b
