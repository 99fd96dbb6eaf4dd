"""GPU parity of the plain path's passes of 65 to 256 rows, whose small matrices (at most 2^20 weights, 2^27 multiply-adds) go through the few-row kernel: the
last row count it takes and the first it does not, a matrix of exactly that size, one above it between others below (its LayerNorm a
launch of its own), and a width without whole quads."""
import pytest

from paper_2308_01320_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,H,nh,F,V,B,S,G", [
    (1, 128, 4, 512, 300, 4, 64, 2),    # 256 rows
    (1, 128, 4, 512, 300, 1, 257, 2),   # one more
    (1, 512, 8, 2048, 100, 1, 65, 2),   # 512 x 2048: the largest such matrix
    (2, 512, 8, 2112, 100, 5, 14, 2),   # FC1 and FC2 above it, the others not
    (2, 64, 2, 77, 50, 15, 17, 2),      # element-wise loads, 255 rows
])
def test_small_matrices_up_to_256_rows(L, H, nh, F, V, B, S, G):
    d = synth.ModelDims("x", L, H, nh, F, V, 512, B, S, G, "f32", "greedy")
    w = synth.make_weights(d, seed=5)
    prompts = synth.make_prompts(d, seed=6)
    want = util.oracle_run(d, util.weights_f64(w), prompts, G, "greedy", 1.0, seed=3)
    eng = util.make_engine(d, w)
    got = util.engine_teacher_forced(eng, prompts, want["ids"], G, binding.sampling("greedy", 1.0, 3))
    eng.he_destroy()
    util.compare(got, want, 1e-5, 1e-4)  # logits of order one: a few hundred float roundings
