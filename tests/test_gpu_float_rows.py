"""GPU parity of the float path's few-row kernels against the oracle: head dimensions that fill 16 lanes once, twice and four times or
leave some idle, caches of less and more than a round of keys, rows at the edges of the 16-row tile, widths beyond what a
wavefront keeps of a row in registers, an inner width that is no multiple of four, vocabularies beyond the sampler's registers."""
import pytest

from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

F32_TOL, MARGIN = 1e-4, 1e-4  # the float path's bound on logits


@pytest.mark.parametrize("mode", ["greedy", "gumbel"])
@pytest.mark.parametrize("H,nh,F,V,B,S", [
    (72, 9, 30, 100, 1, 1),      # heads of 8; inner width 30
    (64, 1, 64, 257, 15, 3),
    (144, 2, 100, 2049, 16, 2),  # heads of 72
    (256, 2, 510, 2048, 17, 4),  # heads of 128
    (400, 2, 64, 300, 3, 70),    # heads of 200, two rounds of keys and more
    (512, 2, 128, 5000, 2, 20),  # heads of 256
    (1280, 10, 192, 300, 5, 2),  # rows wider than 1024
    (256, 4, 1024, 1000, 4, 129),
])
def test_float_rows(H, nh, F, V, B, S, mode):
    d = synth.ModelDims("x", 2, H, nh, F, V, 256, B, S, 4, "f32", mode)
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, 4, mode, 0.8, seed=3)
    eng = util.make_engine(d, w)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], 4, binding.sampling(mode, 0.8, 3))
    eng.he_destroy()
    util.compare(got, want, F32_TOL, MARGIN)
