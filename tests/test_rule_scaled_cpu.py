"""The built-in rule for bf16 and e4m3 (host only, no GPU): which form each kind of problem takes."""
import pytest


@pytest.mark.parametrize("dt,shape,form", [
    ("bf16", (512, 4096, 4096), (64, 64, 0)),        # few whole tiles: direct, one launch
    ("bf16", (300, 300, 128), (64, 64, 0)),          # shallow K
    ("bf16", (300, 300, 700), (128, 128, 1)),        # partial direct tiles lose with K
    ("bf16", (2048, 4096, 4096), (128, 128, 1)),     # 128 tiles of 256 x 256 would fill half the CUs
    ("bf16", (3000, 3000, 3000), (256, 256, 1)),     # one round of 256 x 256 against two of 128 x 128
    ("bf16", (16384, 16384, 16384), (256, 256, 1)),
    ("bf16", (2657, 512, 7104), (256, 256, 1)),      # stream-K
    ("fp8", (512, 4096, 2048), (64, 128, 0)),
    ("fp8", (128, 4096, 8192), (64, 128, 0)),        # narrow
    ("fp8", (1000, 1000, 8000), (128, 128, 1)),
    ("fp8", (16384, 16384, 16384), (256, 256, 1)),
])
def test_scaled_rule(dt, shape, form):
    from paper_1804_10694_amd import tgemm as tg
    tg.set_policy("default")
    i = tg.schedule_info(tg.select_schedule(*shape, dt)[0])
    assert (i["BM"], i["BN"], int(i["vec"] == 0)) == form
