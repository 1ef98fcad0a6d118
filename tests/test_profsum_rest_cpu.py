"""Profile summaries: launches of 128 x 128 in-place tiles with quarters go to the path whose
shape has that grid."""
from paper_1804_10694_amd import profsum

REST = "tg::inplace_rest_kernel(tg::GemmArgs, int)"


def test_rest_launches_are_told_apart_by_shape():
    path = {"grid_threads": 0, "schedule_key": "sched:0:64x64x16", "inplace": True}
    bench = {"paths": {"f32_4097x3001x2053": dict(path), "x3_4097x3001x2053": dict(path),
                       "f32_3706x4759x2398": dict(path, grid_threads=1)}}
    first, second = 256 * (792 + 3 * 24), 256 * (1102 + 3 * 78)
    assert profsum.rest_grid("f32_4097x3001x2053") == first
    calls = [({"name": REST, "grid": g}, []) for g in (first, second, second, 256 * 300)]
    got = profsum.match(calls, bench)
    assert {k: len(v[1]) for k, v in got.items()} == {"f32_4097x3001x2053": 1, "f32_3706x4759x2398": 2}
