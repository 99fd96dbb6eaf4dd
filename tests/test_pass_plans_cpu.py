"""The k ranges of the products of 193 to 256 rows: their number is the order of the sums, by which activations round, so it is part of what a pass
returns and not only of how fast it is (host logic, no GPU)."""
import dataclasses

import pytest

from paper_2308_01320_amd import binding, synth


@pytest.mark.parametrize("H,rows,ranges", [  # QKV, out-projection, FC1, FC2
    (4096, (193, 200), (1, 4, 1, 4)), (4096, (224, 256), (1, 2, 1, 4)), (5120, (193, 200), (1, 3, 3, 6)), (6144, (200,), (3, 5, 1, 5)),
    (6144, (224, 256), (3, 2, 1, 5)), (7168, (193, 250), (3, 2, 1, 9)), (7168, (256,), (3, 2, 1, 4)), (9216, (193, 200), (2, 3, 1, 7)),
    (9216, (224, 256), (1, 3, 1, 7)),
])
def test_k_ranges(H, rows, ranges):
    for m in rows:
        d = dataclasses.replace(synth.CONFIGS["opt-13b"], hidden=H, n_heads=H // 128, ffn=4 * H)
        cfg = binding.make_config(d, max_batch=1, max_seq_len=256)
        assert tuple(binding.he_plan_pass_gemm(cfg, m, g).ksplit for g in binding.PASS_GEMMS[:4]) == ranges, m
