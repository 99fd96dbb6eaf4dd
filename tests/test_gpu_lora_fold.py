"""Refreshes with adapters on every way that B's rows come (16 bytes, single values, through LDS in one go and in several; aligned and not), of
matrices whose vectors W gamma and W beta are formed on the way: bit for bit an engine built on the oracle's merged weights."""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth

pytestmark = pytest.mark.gpu

MATS = ("wqkv", "wo", "w1", "w2")


@pytest.mark.parametrize("H,F", [(64, 192), (576, 1152), (1088, 640)])
@pytest.mark.parametrize("rank,shift", [(1, 0), (8, 0), (8, 1), (9, 0), (17, 0), (40, 0), (40, 1), (70, 0)])
def test_refresh_equals_merged_weights(H, F, rank, shift):
    import torch
    d = synth.ModelDims("x", 1, H, H // 64, F, 200, 16, 3, 6, 2, "bf16", "greedy")
    w = synth.make_weights(d, seed=3)
    rng, scale = np.random.default_rng(rank), 0.75
    bf = synth.round_to_bf16
    ads = {m: (bf(rng.normal(0, 0.05, (rank, w["layers"][0][m].shape[1]))), bf(rng.normal(0, 0.05, (w["layers"][0][m].shape[0], rank)))) for m in MATS}
    merged = dict(w, layers=[dict(w["layers"][0], **{m: O.merge_lora(w["layers"][0][m], a, b, scale).astype(np.float32) for m, (a, b) in ads.items()})])

    def on_device(x, off=0):  # `off` values behind an allocation's start
        room = torch.zeros(x.size + off, dtype=torch.bfloat16, device="cuda")
        room[off:].copy_(torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda().reshape(-1))
        return room[off:].view(x.shape)

    def logits(eng):
        s = binding.sampling("greedy")
        first = eng.he_prefill(torch.from_numpy(synth.make_prompts(d, seed=5)).cuda(), s, True)[2]
        return first, eng.he_decode_step(torch.tensor([1, 2, 3], dtype=torch.int32, device="cuda"), s, True)[2]

    eng = binding.Engine(binding.make_config(d), binding.upload_weights(w, "bf16"))
    eng.he_refresh_weights_lora([{m: (on_device(a), on_device(b, shift)) for m, (a, b) in ads.items()}], rank, scale)
    plain = binding.Engine(binding.make_config(d), binding.upload_weights(merged, "bf16"))
    got, want = logits(eng), logits(plain)
    torch.cuda.synchronize()
    eng.he_destroy(), plain.he_destroy()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
