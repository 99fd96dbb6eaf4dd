"""A prompt pass and decode steps captured into a caller's HIP graph: every replay computes what the same calls compute
eagerly, whatever the replay before it left in the engine's device-side state."""
import numpy as np
import pytest

from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

REPLAYS = 3


# (a cache and a position table for all replays laid end to end: a pass that does not begin at the start computes something
# else, inside its buffers)
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("dtype,H,nh,B,S", [("f32", 128, 4, 3, 5), ("bf16", 256, 4, 3, 40), ("bf16", 128, 2, 5, 1),
                                            ("bf16", 128, 2, 4, 9), ("bf16", 256, 2, 70, 3)])
def test_captured_prompt_pass_replays_from_the_start(dtype, H, nh, B, S, ragged):
    import torch
    n = REPLAYS * (S + 1)
    d = synth.ModelDims("x", 2, H, nh, 2 * H, 500, n, B, S, n - S, dtype, "gumbel")
    w = synth.make_weights(d, seed=5)
    samp = binding.sampling("gumbel", 0.9, 11)
    stream = torch.cuda.Stream()
    ref = util.make_engine(d, w)
    eng = binding.Engine(binding.make_config(d, stream=stream.cuda_stream), binding.upload_weights(w, dtype))
    ids = [torch.from_numpy(synth.make_prompts(d, seed=6 + r)).cuda() for r in range(REPLAYS)]
    lens = [torch.from_numpy(np.random.default_rng(r).integers(1, S + 1, B).astype(np.int32)).cuda() for r in range(REPLAYS)]
    feed = [torch.from_numpy(np.random.default_rng(9 + r).integers(0, d.vocab, B).astype(np.int32)).cuda() for r in range(REPLAYS)]

    def calls(e, p, l, f):
        e.he_reset()
        return work(e, p, l, f)

    def work(e, p, l, f):
        first = e.he_prefill_ragged(p, l, samp, True) if ragged else e.he_prefill(p, samp, True)
        return (*first, *e.he_decode_step(f, samp, True))

    p_in, l_in, f_in = ids[0].clone(), lens[0].clone(), feed[0].clone()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        calls(eng, p_in, l_in, f_in)  # (kernels are loaded before the capture)
        eng.he_reset()
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        out = work(eng, p_in, l_in, f_in)
    for r in range(REPLAYS):
        p_in.copy_(ids[r]), l_in.copy_(lens[r]), f_in.copy_(feed[r])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in out]
        want = calls(ref, ids[r], lens[r], feed[r])
        torch.cuda.synchronize()
        for g, x in zip(got, want):
            assert torch.equal(g, x), r
    ref.he_destroy()
    eng.he_destroy()
