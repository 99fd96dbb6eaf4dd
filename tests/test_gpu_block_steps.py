"""GPU parity of the float path's decode steps in blocks (a launch per attention block and per FFN block) against the oracle: widths, heads,
FFN slices, rows and vocabularies at the edges of what a block takes, caches longer than one round of keys, sequences of different lengths
that end, and models just outside, whose steps are launches of one matrix each."""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,H,nh,F,V,B,S,G", [
    (1, 16, 2, 32, 5, 1, 1, 3),          # the smallest block: heads of 8, one FFN slice, fewer ids than a workgroup takes
    (2, 256, 4, 1024, 1024, 4, 32, 4),   # every limit but the rows'
    (3, 256, 8, 1024, 333, 16, 5, 3),    # eight heads, 32 slices, sixteen rows; ids past the last whole quad
    (2, 224, 4, 448, 90, 7, 63, 4),      # heads of 56: the cache grows across a round of 64 keys
    (1, 192, 3, 704, 1000, 9, 130, 3),   # ... a third round; two threads to a quad of rows no longer
    (2, 48, 1, 128, 64, 3, 126, 5),
    (1, 320, 8, 1024, 300, 3, 9, -3),    # outside (negative here): too wide,
    (1, 256, 2, 512, 300, 3, 9, -3),     # heads too large,
    (1, 128, 4, 512, 300, 17, 4, -3),    # too many rows,
    (1, 128, 4, 528, 300, 2, 4, -3),     # no whole slices
])
def test_steps_in_blocks(L, H, nh, F, V, B, S, G):
    import torch
    blocks, G = G > 0, abs(G)
    d = synth.ModelDims("x", L, H, nh, F, V, 256, B, S, G, "f32", "greedy")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, G, "greedy", 1.0, seed=3)
    eng = util.make_engine(d, w)
    assert (binding.he_plan_plain_gemm(binding.make_config(d), B, 1, "fc1") == "blocks") == blocks
    got = util.engine_teacher_forced(eng, prompts, want["ids"], G, binding.sampling("greedy", 1.0, 3))
    ids, lp = eng.he_generate(torch.from_numpy(prompts).cuda(), G, binding.sampling("greedy"))
    torch.cuda.synchronize()
    eng.he_destroy()
    util.compare(got, want, 1e-5, 1e-4)  # logits of order one: a few hundred float roundings
    # the replayed steps of he_generate, running freely: as far as no margin is thin
    ids, lp = ids.cpu().numpy(), lp.cpu().numpy()
    compared = 0
    for b in range(B):
        unsure = np.nonzero(want["margins"][b] <= 1e-4)[0]
        k = int(unsure[0]) if len(unsure) else G
        assert np.array_equal(ids[b, :k], want["ids"][b, :k])
        assert k == 0 or np.abs(lp[b, :k] - want["logprobs"][b, :k]).max() <= 1e-5
        compared += k - (k > 0)
    assert compared >= B * (G - 1) / 2  # (steps behind the prompt pass)


def test_ragged_steps_in_blocks_and_ended_sequences():
    import torch
    d = synth.ModelDims("x", 2, 128, 4, 256, 50, 64, 6, 7, 24, "f32", "gumbel")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    lens = np.array([7, 1, 3, 7, 2, 5], np.int32)
    own = [prompts[b, 7 - n:] for b, n in enumerate(lens)]
    want = O.generate_ragged(util.weights_f64(w), own, 24, d.n_heads, mode="gumbel", temperature=1.0, seed=3, eos_id=11, pad_id=0,
                             eps=d.ln_eps)
    eng = util.make_engine(d, w)
    assert binding.he_plan_plain_gemm(binding.make_config(d), 6, 1, "fc1") == "blocks"
    ids, lp, n = eng.he_generate_ragged(torch.from_numpy(prompts).cuda(), torch.from_numpy(lens).cuda(), 24, binding.sampling("gumbel", 1.0, 3), 11, 0)
    torch.cuda.synchronize()
    eng.he_destroy()
    assert np.array_equal(ids.cpu().numpy(), want["ids"]) and np.abs(lp.cpu().numpy() - want["logprobs"]).max() <= 1e-4


def test_unaligned_tables_take_the_plain_steps():
    import torch
    d = synth.ModelDims("x", 1, 64, 2, 128, 40, 64, 3, 5, 3, "f32", "greedy")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, 3, "greedy", 1.0, seed=3)
    dev = binding.upload_weights(w, "f32")
    room = torch.zeros(dev["lnf_g"].numel() + 4, device="cuda")
    shifted = room[1:1 + dev["lnf_g"].numel()]
    shifted.copy_(dev["lnf_g"])
    eng = binding.Engine(binding.make_config(d), dict(dev, lnf_g=shifted))
    got = util.engine_teacher_forced(eng, prompts, want["ids"], 3, binding.sampling("greedy", 1.0, 3))
    eng.he_destroy()
    util.compare(got, want, 1e-5, 1e-4)
