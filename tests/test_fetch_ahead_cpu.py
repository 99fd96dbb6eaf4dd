"""What a decode step's attention launch fetches of the out-projection's weights, against the plan and the weights' layout (host logic, no GPU):
every line of the matrix once, by the workgroup that reads it -- its column group's units, its k range --, in both layouts."""
import numpy as np
import pytest

from paper_2308_01320_amd import binding, synth


def _cfg(H, B, fp8):
    d = synth.ModelDims("x", 1, H, H // 64, 4 * H, 100, 64, B, 8, 1, "bf16", "greedy")
    return binding.make_config(d, max_batch=B, max_seq_len=16, weights_fp8=int(fp8))


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("H", [64, 192, 512, 1088, 2048, 2560])
@pytest.mark.parametrize("B", [1, 16, 17, 48, 64])
def test_lines_of_every_workgroup(H, B, fp8):
    cfg = _cfg(H, B, fp8)
    account = binding.he_decode_scratch_account(cfg, B, 0)
    shares = binding.he_plan_fetch_ahead(cfg, B)
    groups = account.stat_pairs // 32 // ((B + 31) // 32)  # column groups
    assert len(shares) == groups * account.ksplit
    units = -(-H // 16 // groups)
    assert -(-H // 16 // units) == groups
    lines_of_step, step_k = 8, 64 if fp8 else 32  # a step of k of a unit of 16 rows
    # the rows and k steps that a line belongs to, from the layout: codes in units [row / 16][k / 64] of 1 KB; halves in blocks [row / 32][k / 16] of 1 KB,
    # a row's eight values of either half of a block 16 bytes at 16 (row % 32) + 512 half
    line = np.arange(H * H * (1 if fp8 else 2) // 128)
    if fp8:
        unit, step = line // 8 // (H // 64), line // 8 % (H // 64)
    else:
        block, at = line * 128 // 1024, line * 128 % 1024
        unit, step = block // (H // 16) * 2 + at % 512 // 256, block % (H // 16) // 2
    seen = np.zeros(len(line), int)
    for g in range(groups):
        end = 0
        for ks in range(account.ksplit):
            own = np.array(shares[g * account.ksplit + ks], int)
            first, last = end, end + len(own) // (lines_of_step * units)
            end = last
            wanted = (unit >= g * units) & (unit < (g + 1) * units) & (step >= first) & (step < last)
            assert np.array_equal(np.unique(own), np.flatnonzero(wanted)), (g, ks)
            assert abs((last - first) * account.ksplit - H // step_k) <= 8 * account.ksplit  # (eight wavefronts at most, one step more each)
            seen[np.unique(own)] += 1
        assert end == H // step_k
    assert (seen == 1).all()


def test_large_matrices_are_left_alone():
    assert binding.he_plan_fetch_ahead(_cfg(4096, 7, False), 7) == []  # 32 MiB
    assert len(binding.he_plan_fetch_ahead(_cfg(4096, 7, True), 7)) > 0
    assert binding.he_plan_fetch_ahead(_cfg(5120, 7, True), 7) == []
    with pytest.raises(binding.HeError):
        binding.he_plan_fetch_ahead(_cfg(512, 65, False), 65)
