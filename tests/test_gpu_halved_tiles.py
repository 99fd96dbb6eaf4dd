"""GPU parity of prompt passes, wide decode steps and few-row scoring on halved tiles (two workgroups to 256 columns of a deep-ring
GEMM) against the oracle: rows at the edges of tiles of 64, 128, 192 and 256 rows, whole sums and k ranges, lengths that differ."""
import functools

import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2


@functools.lru_cache(maxsize=1)
def _model(H, nh, F):
    d = synth.ModelDims("x", 2, H, nh, F, 300, 1024, 1, 2, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=5)
    return d, util.weights_f64(w), binding.upload_weights(w, "bf16")


# rows of QKV's halved tiles by the rows of the pass (else 64); batches above 64: rows of the wide step as well
QKV_ROWS = {1500: 128, 750: 128, 897: 128, 1495: 192, 2001: 256, 2112: 256}
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("H,nh,F,B,S", [
    (512, 8, 1536, 1, 2), (512, 8, 1536, 1, 63), (512, 8, 1536, 2, 64), (512, 4, 1536, 7, 37), (512, 8, 1536, 30, 50),
    (1024, 8, 4096, 1, 33), (1024, 8, 4096, 1, 64), (1024, 8, 4096, 5, 13), (1024, 8, 4096, 1, 129), (1024, 8, 4096, 3, 64),
    (1024, 16, 4096, 5, 150), (1024, 8, 4096, 39, 23), (1024, 8, 4096, 13, 115), (1024, 8, 4096, 23, 87), (1024, 8, 4096, 33, 64),
    (1024, 8, 4096, 65, 2), (1024, 8, 4096, 129, 3), (1024, 8, 4096, 200, 2),
])
def test_passes_on_halved_tiles(H, nh, F, B, S, ragged):
    """Prompt pass and a decode step, the first, a middle and the last sequence against the oracle's run of it alone."""
    import torch
    base, w64, w_dev = _model(H, nh, F)
    cfg = binding.make_config(base, max_batch=B, max_seq_len=S + 1)
    rows = B * S if B <= 64 else B * (S - 1)
    for r in {rows, B if B > 64 else rows}:
        plans = {g: binding.he_plan_pass_gemm(cfg, r, g) for g in binding.PASS_GEMMS[:4]}
        assert all(a.workgroup_cols == 128 for g, a in plans.items() if (r, g) != (2112, "fc1"))
        assert plans["qkv"].tile_rows == QKV_ROWS.get(r, 64)
        assert r > 1024 or plans["fc2"].ksplit > 1  # (k ranges among them)
    rng = np.random.default_rng(17 * B + S)
    prompts = rng.integers(0, base.vocab, (B, S)).astype(np.int32)
    lens = rng.integers(1, S + 1, B).astype(np.int32) if ragged else np.full(B, S, np.int32)
    feed = rng.integers(0, base.vocab, B).astype(np.int32)
    eng = binding.Engine(cfg, w_dev)
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
