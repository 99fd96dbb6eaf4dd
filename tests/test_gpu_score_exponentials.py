"""The scoring pass's soft-max to the accuracy of single exponentials: a model without layers whose logits are exact in float32 -- one entry at 0, the
next token, the others x below it, another x for every position -- against the same sum of terms that are off by an ulp at most, added up in the order
that a lane and its neighbour have them.  (Terms from an argument that was rounded in units of log2 are off by up to five ulps here, which 127 additions
in the same direction make 5e-6 of the result.)"""
import numpy as np
import pytest

from paper_2308_01320_amd import binding, synth

pytestmark = pytest.mark.gpu


def test_terms_of_the_partial_sums():
    import torch
    H, V, T = 64, 128, 512
    d = synth.ModelDims("x", 0, H, 1, 64, V, T, 1, T, 1, "bf16", "greedy")
    w = synth.make_weights(d, seed=1)
    # columns in pairs of opposite signs: rows of mean 0 and variance 1, which the LayerNorm leaves as they are (their rounding to 16 bits included)
    bits = np.arange(T)[:, None] >> np.arange(H // 2) & 1
    signs = np.where(bits == 1, -1.0, 1.0)
    signs[:, 31] = 1.0
    w["tok_emb"] = np.zeros((V, H), np.float32)
    w["pos_emb"] = np.concatenate([signs, -signs], 1).astype(np.float32)
    w["lnf_g"], w["lnf_b"] = np.ones(H, np.float32), np.zeros(H, np.float32)
    step = synth.round_to_bf16(np.array([0.0711, 0.0362, 0.0183, 0.0094, 0.0047, 0.0023, 0.0012, 0.0006, 0.0003]))
    head = np.zeros((V, H), np.float32)
    head[1:, :9], head[1:, 31] = -step, -5.75
    w["lm_head"] = head
    x = 5.75 + (signs[:, :9] * step).sum(1)  # 5.6 .. 5.9
    assert np.array_equal(x, x.astype(np.float32)) and x.min() * np.log2(np.e) > 8
    eng = binding.Engine(binding.make_config(d), binding.upload_weights(w, "bf16"))
    got = eng.he_score(torch.zeros(1, T, dtype=torch.int32, device="cuda")).cpu().numpy()[0].astype(np.float64)
    eng.he_destroy()
    x = x[:T - 1]
    errs = []
    for ulps in (-1, 0, 1):  # of the term rounded once
        term = (np.exp(-x).astype(np.float32).view(np.int32) + np.int32(ulps)).view(np.float32)
        halves = np.zeros((2, T - 1), np.float32)
        for n in range(V):
            halves[n >> 2 & 1] += term if n else np.float32(1)
        errs.append(np.abs(got + np.log((halves[0] + halves[1]).astype(np.float64))))
    off = np.min(errs, axis=0) > 2.0 ** -24  # two ulps of the logarithm, which is 0.25 to 0.5
    assert not off.any(), (int(off.sum()), float(np.min(errs, axis=0).max()))
