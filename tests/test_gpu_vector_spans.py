"""GPU parity of the folded LayerNorm's vectors W gamma and W beta of a vocabulary of many rows, the last tile of 32 partly filled, from the caller's
rows and from tiles: every logit of a decode step."""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiled", [0, 1])
def test_vectors_of_many_rows(tiled):
    import torch
    H, V = 576, 73901
    base = synth.ModelDims("x", 1, H, 9, 64, V, 8, 1, 2, 2, "bf16", "greedy")
    w = synth.make_weights(base, seed=13)
    cfg = binding.make_config(base, max_batch=1, max_seq_len=8, weights_tiled=tiled)
    dev = binding.upload_weights(w, "bf16")
    if tiled:
        dev = binding.tile_weights_in_place(dev)
    eng = binding.Engine(cfg, dev)
    ids = np.array([[5, 70000, 73900, 17]], np.int32)
    s = binding.sampling("greedy")
    eng.he_prefill(torch.from_numpy(ids[:, :3].copy()).cuda(), s, True)
    got = eng.he_decode_step(torch.from_numpy(ids[:, 3].copy()).cuda(), s, True)[2].cpu().numpy()[0]
    eng.he_destroy()
    want = O.forward_full(util.weights_f64(w), ids, 9, eps=base.ln_eps)[0][3]
    assert float(np.abs(got - want).max()) <= 2e-2
