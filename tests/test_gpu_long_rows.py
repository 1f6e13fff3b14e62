"""Plan-free calls on rows of every class side by side: long rows as the outliers of their workgroup and as its normal case,
at the ends of the stretches in which the first workgroups look for them, for every run length."""
import numpy as np
import pytest

from workloads import csr_from_row_lengths, integer_valued

from gpu_util import DeviceProblem, check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [4100, 9000, 17000, 140000])  # runs of 1, 2 and 4 rows, and stretches of 128 rows
@pytest.mark.parametrize("n", [1, 20, 128, 300])
def test_long_rows(m, n):
    rng = np.random.default_rng(m + n)
    lens = rng.integers(0, 4, size=m)
    lens[[0, 63, 64, m - 1]] = [257, 256, 700, 2100]
    lens[rng.integers(0, m, size=20)] = 300
    if m < 100000:
        lens[1024:1024 + 40] = 260  # more long rows than a quarter of any workgroup's
        lens[2048:2048 + 4] = [258, 2049, 2048, 33]
    p = csr_from_row_lengths(lens, 500, n, seed=m, duplicates=True)
    for q, exact in ((p, False), (integer_valued(p, seed=n), True)):
        d = DeviceProblem(q)
        check_against_oracle(q, d.run_natural(), d.ldc, exact=exact, label=f"m={m} n={n}")


@pytest.mark.parametrize("m,n", [(600, 256), (2048, 64), (9000, 36)])
def test_rows_beyond_the_long_limit_are_the_normal_case(m, n):
    """Every wavefront takes its own rows then; a stretch of short rows beside them, and one of a few long rows, stay as they were."""
    rng = np.random.default_rng(m)
    lens = rng.integers(2049, 2500, size=m) if m < 5000 else rng.integers(0, 30, size=m)
    lens[m // 3:m // 3 + 100] = rng.integers(0, 40, size=100)
    lens[m // 2:m // 2 + 40] = 2100
    p = csr_from_row_lengths(lens, 3000, n, seed=n, duplicates=False)
    d = DeviceProblem(p)
    check_against_oracle(p, d.run_natural(), d.ldc, label=f"long rows m={m} n={n}")
