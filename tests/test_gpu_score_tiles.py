"""The scoring head's two kernels and the ring kernel below them: rows and vocabularies that end inside a tile, each against the oracle,
and a sequence alone (ring kernel) against the same in a batch, to the bit."""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,V,rows", [(3, 700, 14000, 256), (2, 1027, 14001, 256), (3, 700, 15013, 128)])
def test_score_head_tiles(B, T, V, rows):
    import torch
    d = synth.ModelDims("x", 0, 1024, 8, 64, V, T, B, T, 1, "bf16", "greedy")
    w = synth.make_weights(d, seed=3)
    cfg = binding.make_config(d, max_batch=B, max_seq_len=T)
    assert binding.he_plan_pass_gemm(cfg, B * T, "lm_head", scoring=True).tile_rows == rows
    assert binding.he_plan_pass_gemm(cfg, T, "lm_head", scoring=True).tile_rows == 128
    ids = synth.make_prompts(d, seed=4, batch=B, prompt_len=T)
    ids[:, 1::97] = V - 1  # the last entry, among the targets
    eng = binding.Engine(cfg, binding.upload_weights(w, "bf16"))
    got = eng.he_score(torch.from_numpy(ids).cuda()).cpu().numpy()
    alone = eng.he_score(torch.from_numpy(ids[1:2].copy()).cuda()).cpu().numpy()
    eng.he_destroy()
    assert np.array_equal(got[1], alone[0])
    want = O.score(util.weights_f64(w), ids, d.n_heads, eps=d.ln_eps, pos_offset=d.pos_offset)
    assert float(np.abs(got - want).max()) <= 4e-3  # (16-bit logits of order one)
