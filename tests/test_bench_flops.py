"""Operations that the benchmark counts for a gravity launch: each unordered
pair once where the pairwise kernel runs, so never more than the time allows
at the vector peak because of pairs that are only credited."""
import pytest


def test_executed_flops():
    import bench
    n = 2097152
    assert bench.executed_flops("fp32c", n)[0] == 31 * 0.5 * n * n
    assert bench.executed_flops("fp64", n)[0] == 39 * 0.5 * n * n
    for form, variant, per in (("fp32c", 1, 21), ("fp64", 4, 29), ("fp64", 1, 29)):
        if form == "fp64":
            assert bench.executed_flops(form, n, variant)[0] == per * float(n) * n
        assert bench.executed_flops(form, 12287, 0 if form == "fp32c" else variant)[0] == per * 12287.0 ** 2
    r = bench.alu_roofline("fp32c", n, 0, 0.983)
    assert r["frac"] == pytest.approx(31 * 0.5 * n * n / 0.983 / 157.3e12)
    assert r["credited"]["rate"] == pytest.approx(22.0 * n * n / 0.983e12)
