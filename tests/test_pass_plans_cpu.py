"""Plans of the few-row tiles (host logic, no GPU): the k ranges of the products of 193 to 256 rows, whose number is the order of the sums, by which
activations round, so part of what a pass returns and not only of how fast it is; and which launches copy their weights past the caches."""
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


def _plan(H, rows, which, scoring=False):
    d = dataclasses.replace(synth.CONFIGS["opt-13b"], hidden=H, n_heads=H // 64, ffn=4 * H)
    cfg = binding.make_config(d, max_batch=1, max_seq_len=rows)
    p = binding.he_plan_pass_gemm(cfg, rows, which, scoring=scoring)
    return (p.tile_rows, p.workgroup_cols, p.ksplit), binding.he_plan_weight_copies(cfg, rows, which, scoring)


@pytest.mark.parametrize("H,rows,which,plan,streamed", [
    (5120, 96, "fc1", (128, 128, 1), True), (4096, 96, "qkv", (128, 128, 2), True),         # one row of tiles; k ranges of 101 MB
    (3584, 64, "qkv", (64, 128, 3), False), (5120, 64, "out_proj", (64, 128, 5), False),    # of 77, 52
    (3072, 140, "fc2", (192, 128, 10), False), (768, 64, "fc1", (64, 128, 1), False),       # of 75; 5 MB
    (4096, 128, "qkv", (64, 128, 1), True), (3584, 120, "fc1", (64, 128, 1), True),         # two of 64 rows, 101 and 103 MB
    (2048, 256, "fc1", (64, 128, 1), False), (2560, 130, "qkv", (64, 128, 1), False),       # 34, 39 MB
    (3584, 160, "fc1", (128, 128, 1), False), (4096, 239, "qkv", (128, 128, 1), False),     # a last row of tiles a quarter full, 111 of 128 rows
    (4096, 240, "qkv", (128, 128, 1), True), (4096, 250, "fc1", (128, 128, 1), True),
    (3584, 240, "qkv", (128, 128, 1), False), (2048, 512, "fc1", (128, 128, 1), False),     # 77, 34 MB
    (4096, 256, "fc2", (128, 128, 4), False), (1024, 100, "fc2", None, False),              # k ranges
    (4096, 4096, "fc1", (256, 256, 1), False),                                              # the big tiles
])
def test_weight_copies(H, rows, which, plan, streamed):
    got = _plan(H, rows, which)
    assert (plan is None or got[0] == plan) and got[1] == streamed, got
