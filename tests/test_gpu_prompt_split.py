"""GPU parity of prompt attention with few (sequence, head) pairs, four wavefronts to a block of 32 queries, against the oracle: lengths
at the edges of its blocks of queries and tiles of keys, lengths that differ, and the sizes on both sides of the rule."""
import functools

import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2


@functools.lru_cache(maxsize=1)
def _model(H, nh):
    d = synth.ModelDims("x", 2, H, nh, 4 * H, 300, 1024, 1, 2, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=9)
    return d, util.weights_f64(w), binding.upload_weights(w, "bf16")


# 64 rows: the kernel of 128 queries to a workgroup; 65 .. 160: one to five tiles of keys (fewer than the wavefronts, as many, one more); 500 x 32
# and 161 x 64 pairs: more workgroups than CUs; 65 x 128 and more pairs: 128 queries again, 97 x 128: not with heads of 64
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("H,nh,B,S", [
    (512, 4, 1, 64), (512, 4, 1, 65), (512, 4, 2, 96), (512, 4, 3, 97), (512, 4, 1, 128), (512, 4, 1, 129), (512, 4, 5, 160), (512, 4, 2, 500),
    (512, 4, 32, 65), (512, 4, 36, 65), (512, 4, 8, 500), (512, 4, 12, 96),
    (512, 8, 1, 65), (512, 8, 3, 97), (512, 8, 1, 129), (512, 8, 2, 161), (512, 8, 1, 700), (512, 8, 16, 70), (512, 8, 18, 70), (512, 8, 8, 161), (512, 8, 16, 97),
])
def test_prompt_pass_of_few_pairs(H, nh, B, S, ragged):
    """Prompt pass and a decode step over the cache it left, the first, a middle and the last sequence against the oracle's run of it
    alone; sequences of one token among the ragged ones (blocks of nothing but padding rows)."""
    import torch
    base, w64, w_dev = _model(H, nh)
    rng = np.random.default_rng(31 * B + S)
    prompts = rng.integers(0, base.vocab, (B, S)).astype(np.int32)
    lens = np.full(B, S, np.int32)
    if ragged:
        lens = rng.integers(1, S + 1, B).astype(np.int32)
        lens[B // 2] = 1
    feed = rng.integers(0, base.vocab, B).astype(np.int32)
    eng = binding.Engine(binding.make_config(base, max_batch=B, max_seq_len=S + 1), w_dev)
    p, samp = torch.from_numpy(prompts).cuda(), binding.sampling("greedy")
    first = eng.he_prefill_ragged(p, torch.from_numpy(lens).cuda(), samp, True) if ragged else eng.he_prefill(p, samp, True)
    second = eng.he_decode_step(torch.from_numpy(feed).cuda(), samp, True)
    got = [first[2].cpu().numpy(), second[2].cpu().numpy()]
    scores = eng.he_score(p).cpu().numpy() if not ragged else None
    eng.he_destroy()
    for b in sorted({0, B // 2, B - 1}):
        seq = np.append(prompts[b, S - lens[b]:], feed[b])[None]
        z = O.forward_full(w64, seq, nh, eps=base.ln_eps)[0]
        for n in range(2):
            assert float(np.abs(got[n][b] - z[lens[b] - 1 + n]).max()) <= BF16_TOL, (b, n)
        if scores is not None:
            want = O.log_softmax(z[:S - 1])[np.arange(S - 1), prompts[b, 1:]]
            assert float(np.abs(scores[b] - want).max()) <= BF16_TOL, b
