"""Prompt passes on the ring kernel whose weights one row of tiles reads, and several do, on 128 and 256 columns, copied through the caches and
(matrices of 96 MB and more) past them, against the oracle."""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,nh,F", [(768, 12, 3072), (1024, 16, 4096)])
@pytest.mark.parametrize("S", [33, 64, 65, 127, 129, 257])
def test_one_row_of_tiles_and_more(H, nh, F, S):
    import torch
    d = synth.ModelDims("x", 1, H, nh, F, 300, S + 1, 1, S, 1, "bf16", "greedy")
    w = synth.make_weights(d, seed=13)
    eng = binding.Engine(binding.make_config(d), binding.upload_weights(w, "bf16"))
    ids = np.random.default_rng(S).integers(0, d.vocab, (1, S)).astype(np.int32)
    scores = eng.he_score(torch.from_numpy(ids).cuda()).cpu().numpy()
    last = eng.he_prefill(torch.from_numpy(ids).cuda(), binding.sampling("greedy"), True)[2].cpu().numpy()
    eng.he_destroy()
    z = O.forward_full(util.weights_f64(w), ids, nh, eps=d.ln_eps)[0]
    want = O.log_softmax(z[:S - 1])[np.arange(S - 1), ids[0, 1:]]
    assert float(np.abs(last[0] - z[S - 1]).max()) <= 2e-2  # (the other bfloat16 passes' bound)
    assert float(np.abs(scores[0] - want).max()) <= 2e-2


@pytest.mark.parametrize("S", [193, 256])
def test_k_ranges_of_up_to_256_rows(S):
    import torch
    d = synth.ModelDims("x", 1, 4096, 32, 16384, 300, S + 1, 1, S, 1, "bf16", "greedy")
    w = synth.make_weights(d, seed=17)
    cfg = binding.make_config(d)
    p = binding.he_plan_pass_gemm(cfg, S, "fc2")
    assert (p.tile_rows, p.workgroup_cols, p.ksplit) == (128, 128, 4)
    eng = binding.Engine(cfg, binding.upload_weights(w, "bf16"))
    ids = np.random.default_rng(S).integers(0, d.vocab, (1, S)).astype(np.int32)
    last = eng.he_prefill(torch.from_numpy(ids).cuda(), binding.sampling("greedy"), True)[2].cpu().numpy()
    eng.he_destroy()
    z = O.forward_full(util.weights_f64(w), ids, d.n_heads, eps=d.ln_eps)[0]
    assert float(np.abs(last[0] - z[S - 1]).max()) <= 2e-2


@pytest.fixture(scope="module")
def wide():
    d = synth.ModelDims("x", 2, 4096, 32, 16384, 300, 500, 1, 500, 1, "bf16", "greedy")
    w = synth.make_weights(d, seed=19)
    return d, binding.upload_weights(w, "bf16"), util.weights_f64(w)


@pytest.mark.parametrize("S,tile_rows,streamed", [  # of QKV
    (64, 64, ("qkv", "fc1", "fc2")), (96, 128, ("qkv", "fc1", "fc2")), (128, 64, ("qkv", "fc1", "fc2")), (170, 192, ("qkv", "fc2")), (193, 128, ()),
    (240, 128, ("qkv", "fc1")), (384, 192, ("qkv", "fc1")), (500, 256, ("qkv", "fc1")),
])
def test_matrices_past_the_caches(wide, S, tile_rows, streamed):
    import torch
    d, dev, w64 = wide
    cfg = binding.make_config(d, max_batch=1, max_seq_len=S)
    assert binding.he_plan_pass_gemm(cfg, S, "qkv").tile_rows == tile_rows
    assert tuple(g for g in binding.PASS_GEMMS[:4] if binding.he_plan_weight_copies(cfg, S, g)) == streamed
    eng = binding.Engine(cfg, dev)
    ids = np.random.default_rng(S).integers(0, d.vocab, (1, S)).astype(np.int32)
    scores = eng.he_score(torch.from_numpy(ids).cuda()).cpu().numpy()
    eng.he_reset()
    last = eng.he_prefill(torch.from_numpy(ids).cuda(), binding.sampling("greedy"), True)[2].cpu().numpy()
    eng.he_destroy()
    z = O.forward_full(w64, ids, d.n_heads, eps=d.ln_eps)[0]
    want = O.log_softmax(z[:S - 1])[np.arange(S - 1), ids[0, 1:]]
    assert float(np.abs(last[0] - z[S - 1]).max()) <= 2e-2  # (the other bfloat16 passes' bound)
    assert float(np.abs(scores[0] - want).max()) <= 2e-2
