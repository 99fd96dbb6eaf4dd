"""GPU parity of the folded LayerNorm's vectors W gamma and W beta where their partial sums (one per 512 columns and row) do not fit the
engine's scratch at once: a vocabulary of more rows than that, formed in two goes, and the vectors of rows at both sides of the cut."""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiled", [0, 1])
def test_vectors_formed_in_two_goes(tiled):
    import torch
    H, V, cut = 576, 73901, 73728  # two partial sums to a row; 512 H floats of scratch hold them for 73728 rows
    base = synth.ModelDims("x", 1, H, 9, 64, V, 8, 1, 2, 2, "bf16", "greedy")
    w = synth.make_weights(base, seed=13)
    cfg = binding.make_config(base, max_batch=1, max_seq_len=8, weights_tiled=tiled)
    assert binding.he_plan_pass_gemm(cfg, 1, "qkv").scratch_reserved // 4 // 32 * 32 == cut
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
    assert float(np.abs(got[cut - 64:cut + 64] - want[cut - 64:cut + 64]).max()) <= 2e-2
