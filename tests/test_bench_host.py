"""Host-side check of the benchmark's class rates (no GPU needed)."""
import bench


def test_attention_is_charged_with_the_merge_of_its_key_splits():
    prof = {"attention": (10, 0.07, 10), "attention_merge": (10, 0.04, 10), "gemm_o": (10, 0.2, 10)}
    got = bench.with_merge(prof)
    assert got["attention"] == (10, 0.07 + 0.04, 10)
    assert {k: v for k, v in got.items() if k != "attention"} == \
        {k: v for k, v in prof.items() if k != "attention"}
    assert prof["attention"] == (10, 0.07, 10)
    whole = {"attention": (3, 0.1, 3)}
    assert bench.with_merge(whole) == whole and bench.with_merge({}) == {}
