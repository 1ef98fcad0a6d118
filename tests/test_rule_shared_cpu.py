"""Where the built-in rule shares the last round of tiles out (stream-K), host only."""
import pytest


@pytest.fixture(scope="module")
def tg():
    from paper_1804_10694_amd import tgemm
    tgemm.set_policy("default")
    yield tgemm


@pytest.mark.parametrize("dtype,shape,shared", [
    ("x3", (4096, 4096, 4096), False),     # 256 tiles of 256 x 256: no last round
    ("x3", (4096, 4352, 2000), True),      # 272
    ("x3", (4096, 4352, 1999), False),     # too shallow
    ("x3", (4096, 5632, 4000), True),      # 352: 96 in the last round
    ("x3", (4095, 5889, 4000), False),     # 384: 128
    ("x3", (2560, 2560, 2000), True),      # 100, and 400 of 128 x 128
    ("x3", (2049, 2561, 4096), True),      # 9 x 11 = 99, above the deep-K range
    ("x3", (2560, 2817, 2000), False),     # 120
    ("x3", (1800, 1793, 2000), True),      # 8 x 8 = 64
    ("x3", (1790, 1793, 2000), False),     # 7 x 8 = 56
    ("f32", (6608, 1249, 4037), False),    # f32 shares the last round as quarters of tiles
])
def test_shared_rule(tg, dtype, shape, shared):
    assert tg.schedule_info(tg.select_schedule(*shape, dtype)[0])["split"] == int(shared)
