"""Which kernel computes a product of a float model, and whether a decode step goes in blocks: both sides of each line (host logic, no GPU)."""
import pytest

from paper_2308_01320_amd import binding, synth


def _cfg(H, nh, F, V=1000, dtype="f32", L=2, max_batch=32, max_seq=512, impl=0):
    d = synth.ModelDims("x", L, H, nh, F, V, max_seq, max_batch, max_seq, 1, dtype, "greedy")
    return binding.make_config(d, max_batch=max_batch, max_seq_len=max_seq, impl=impl)


@pytest.mark.parametrize("H,nh,F,rows,few", [
    (256, 4, 1024, 256, ("qkv", "out_proj", "fc1", "fc2")),
    (256, 4, 1024, 257, ()),
    (512, 8, 2048, 64, ("qkv", "out_proj", "fc1", "fc2")),
    (512, 8, 2048, 128, ("qkv", "out_proj", "fc1", "fc2")),  # 2^20 weights: up to 2^27 multiply-adds
    (512, 8, 2048, 129, ("qkv", "out_proj")),
    (512, 8, 2048, 256, ("out_proj",)),
    (512, 8, 2112, 65, ("qkv", "out_proj")),
    (768, 12, 768, 256, ()),
    (1024, 16, 1024, 65, ("out_proj", "fc1", "fc2")),
    (1024, 16, 1024, 256, ()),
    (1024, 16, 4096, 192, ()),
])
def test_few_rows(H, nh, F, rows, few):
    for cfg in (_cfg(H, nh, F), _cfg(H, nh, F, dtype="bf16", impl=1)):
        forms = {g: binding.he_plan_plain_gemm(cfg, 1, rows, g) for g in binding.PASS_GEMMS[:4]}
        assert tuple(g for g in forms if forms[g] == "few rows") == few
        assert binding.he_plan_plain_gemm(cfg, 1, rows, "lm_head") == "few rows"  # one row


def test_large_products_take_tiles():
    cfg = _cfg(1024, 16, 4096)
    assert binding.he_plan_plain_gemm(cfg, 1, 65, "fc1") == "32 x 32"
    assert binding.he_plan_plain_gemm(cfg, 1, 256, "fc1") == "64 x 64"


@pytest.mark.parametrize("kw,B,blocks", [
    (dict(H=256, nh=4, F=1024), 16, True), (dict(H=256, nh=4, F=1024), 17, False), (dict(H=256, nh=8, F=32), 1, True),
    (dict(H=16, nh=2, F=32), 1, True), (dict(H=72, nh=9, F=32), 1, False), (dict(H=128, nh=16, F=32), 1, False),
    (dict(H=272, nh=34, F=32), 1, False), (dict(H=256, nh=2, F=32), 1, False), (dict(H=256, nh=4, F=1056), 1, False),
    (dict(H=256, nh=4, F=48), 1, False), (dict(H=256, nh=4, F=1024, L=0), 1, False),
    (dict(H=256, nh=4, F=1024, dtype="bf16", impl=1), 1, False),
    (dict(H=256, nh=8, F=1024, max_batch=1, max_seq=8), 1, True),    # no more room for partial sums than they need ...
    (dict(H=256, nh=8, F=1024, max_batch=1, max_seq=7), 1, False),   # ... and less
])
def test_steps_in_blocks(kw, B, blocks):
    cfg = _cfg(**kw)
    for g in binding.PASS_GEMMS:
        assert (binding.he_plan_plain_gemm(cfg, B, 1, g) == "blocks") == blocks
        if cfg.max_seq_len > 1:
            assert binding.he_plan_plain_gemm(cfg, B, 2, g) != "blocks"


def test_refused():
    cfg = _cfg(256, 4, 1024)
    for B, S in ((0, 1), (33, 1), (1, 0), (1, 513)):
        with pytest.raises(binding.HeError):
            binding.he_plan_plain_gemm(cfg, B, S, "qkv")
    with pytest.raises(binding.HeError):
        binding.he_plan_plain_gemm(_cfg(256, 4, 1024, dtype="bf16"), 1, 1, "qkv")  # the tuned path
