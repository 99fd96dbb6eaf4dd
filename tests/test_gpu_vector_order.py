"""GPU check of the folded LayerNorm's vectors to the last bit: of a model without layers whose embeddings are zeros the logits ARE W beta, in the
stated order -- eight shares of k, the halves of their blocks of 16 columns apart, k ascending, then the shares in turn -- which numpy follows in
float32 (the products of halves and bfloat16 values are exact).  The caller's weights row by row or tiled, fewer blocks than shares, shares of
different lengths, a last tile of rows partly filled."""
import numpy as np
import pytest

from paper_2308_01320_amd import binding, synth

pytestmark = pytest.mark.gpu


def _in_order(w, beta):
    blocks = w.shape[1] // 16
    w, beta = w.astype(np.float16).astype(np.float32).reshape(len(w), blocks, 2, 8), beta.reshape(blocks, 2, 8)
    total = np.zeros(len(w), np.float32)
    for share in range(8):
        halves = np.zeros((len(w), 2), np.float32)
        for kb in range(share * blocks // 8, (share + 1) * blocks // 8):
            for x in range(8):
                halves += w[:, kb, :, x] * beta[kb, :, x]
        total += halves[:, 0] + halves[:, 1]
    return total


@pytest.mark.parametrize("tiled", [0, 1])
@pytest.mark.parametrize("H,V", [(64, 40), (192, 333), (576, 1000), (1024, 96), (2112, 65), (5120, 300)])
def test_vectors_to_the_last_bit(H, V, tiled):
    import torch
    d = synth.ModelDims("x", 0, H, H // 64, 64, V, 8, 2, 1, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=H)
    w["tok_emb"], w["pos_emb"] = np.zeros_like(w["tok_emb"]), np.zeros_like(w["pos_emb"])
    w["lm_head"] = synth.round_to_bf16(np.random.default_rng(V).normal(0, 0.05, (V, H)))
    w["lnf_b"] = synth.round_to_bf16(np.random.default_rng(H).normal(0, 1, H))
    dev = binding.upload_weights(w, "bf16")
    if tiled:
        dev = binding.tile_weights_in_place(dev)
    eng = binding.Engine(binding.make_config(d, max_batch=2, max_seq_len=8, weights_tiled=tiled), dev)
    ids = torch.zeros(2, 1, dtype=torch.int32, device="cuda")
    got = eng.he_prefill(ids, binding.sampling("greedy"), True)[2].cpu().numpy()
    eng.he_destroy()
    want = _in_order(w["lm_head"], w["lnf_b"])
    assert np.array_equal(got, np.stack([want, want]))
