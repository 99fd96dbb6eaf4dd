"""Bit-exact GPU parity of the adapter merge against the oracle: ranks around the groups that B's values are loaded in, B aligned to 16
bytes and not, rows and columns that leave wavefronts partly filled."""
import numpy as np
import pytest

from oracle import opt_oracle as O
from paper_2308_01320_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(33, 48), (130, 160), (64, 1024)])
@pytest.mark.parametrize("rank", [1, 2, 3, 4, 5, 7, 8, 9, 12, 16, 24, 64])
@pytest.mark.parametrize("shift", [0, 1, 4])
def test_merge_at_every_rank_and_alignment(rows, cols, rank, shift):
    import torch
    rng = np.random.default_rng(rows + rank)
    bf = synth.round_to_bf16
    W, A, B = bf(rng.normal(0, 0.05, (rows, cols))), bf(rng.normal(0, 0.05, (rank, cols))), bf(rng.normal(0, 0.05, (rows, rank)))
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda().to(torch.bfloat16).contiguous()
    room = torch.zeros(rows * rank + 8, dtype=torch.bfloat16, device="cuda")
    b = room[shift:shift + rows * rank].view(rows, rank)  # values from the start of an allocation: 0, 2 and 8 bytes off a multiple of 16
    b.copy_(dev(B))
    got = binding.he_tile_matrix_lora(dev(W), dev(A), b, 0.75)
    want = binding.he_tile_matrix(dev(O.merge_lora(W, A, B, 0.75)))
    torch.cuda.synchronize()
    assert int((got != want).sum()) == 0
