"""GPU parity of decode attention at the edges of its one-pass form, against the oracle: two, four and eight wavefronts to a (row, head) and
the two-pass form with four and eight, on both sides of the rule's lines (pairs per CU, size of the cache), with one key, one short of a round of keys, a
whole round and one more, and sequences of different lengths."""
import functools

import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

# Six binary16 roundings lie between a token and its logits (the inputs of the five GEMMs, and the cache), 2^-11 each of values that make up logits
# of at most 1.2: 3.5e-3.  A key left out or counted twice moves them by 5e-3 (257 keys) to 0.6 (two).
TOL = 3.5e-3


@functools.lru_cache(maxsize=2)
def _model(H, nh):
    d = synth.ModelDims("x", 1, H, nh, 2 * H, 300, 320, 1, 2, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=11)
    return d, util.weights_f64(w), binding.upload_weights(w, "bf16")


# (B, S, cache): attention over S, S + 1 and S + 2 keys.  A round is 16 keys a wavefront with heads of 128, 32 with heads of 64.  On
# 256 CUs two heads make 2, 4, 6 (at most eight wavefronts), 260 or 512 (four), 514 pairs (two, or two passes above a cache of 160 with
# heads of 128, of 256 with heads of 64); 512 pairs with a long cache two passes of eight wavefronts, 2050 one pass of four
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("H,nh,B,S,cache", [
    (256, 2, 1, 1, 20), (256, 2, 1, 30, 32), (256, 2, 2, 31, 33), (256, 2, 3, 62, 64), (256, 2, 1, 63, 65), (256, 2, 2, 127, 200),
    (256, 2, 1, 255, 260), (256, 2, 130, 63, 100), (256, 2, 256, 31, 40), (256, 2, 257, 31, 40), (256, 2, 257, 63, 160),
    (256, 2, 257, 63, 161), (256, 2, 256, 1, 520), (256, 2, 256, 127, 520), (256, 2, 256, 255, 520), (256, 2, 1025, 63, 128),
    (128, 2, 1, 1, 8), (128, 2, 1, 62, 64), (128, 2, 2, 126, 128), (128, 2, 3, 127, 129), (128, 2, 1, 255, 258), (128, 2, 130, 127, 200),
    (128, 2, 257, 63, 256), (128, 2, 257, 63, 257), (128, 2, 256, 255, 1030), (128, 2, 1025, 127, 256),
])
def test_decode_attention_at_its_edges(H, nh, B, S, cache, ragged):
    import torch
    base, w64, w_dev = _model(H, nh)
    rng = np.random.default_rng(17 * B + S)
    prompts = rng.integers(0, base.vocab, (B, S)).astype(np.int32)
    feeds = rng.integers(0, base.vocab, (2, B)).astype(np.int32)
    lens = rng.integers(1, S + 1, B).astype(np.int32) if ragged else np.full(B, S, np.int32)
    eng = binding.Engine(binding.make_config(base, max_batch=B, max_seq_len=cache), w_dev)
    p, samp = torch.from_numpy(prompts).cuda(), binding.sampling("greedy")
    first = eng.he_prefill_ragged(p, torch.from_numpy(lens).cuda(), samp, True) if ragged else eng.he_prefill(p, samp, True)
    got = [first[2].cpu().numpy()]
    for f in feeds:
        got.append(eng.he_decode_step(torch.from_numpy(f).cuda(), samp, True)[2].cpu().numpy())
    eng.he_destroy()
    for b in sorted({0, B // 2, B - 1}):
        seq = np.concatenate([prompts[b, S - lens[b]:], feeds[:, b]])[None]
        z = O.forward_full(w64, seq, nh, eps=base.ln_eps)[0]
        for n in range(3):
            assert float(np.abs(got[n][b] - z[lens[b] - 1 + n]).max()) <= TOL, (b, n)
