"""Plan-free calls on rows of every class side by side: long rows as the outliers of the matrix and as its normal case, in
clusters, at regular distances and first of all, for every run length and way of dealing them to workgroups."""
import numpy as np
import pytest
import torch

from workloads import csr_from_row_lengths, integer_valued, with_padding

from gpu_util import DeviceProblem, check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [4100, 9000, 17000, 140000])  # runs of 1, 2 and 4 rows
@pytest.mark.parametrize("n", [1, 20, 128, 300])
def test_long_rows(m, n):
    rng = np.random.default_rng(m + n)
    lens = rng.integers(0, 4, size=m)
    lens[[0, 63, 64, m - 1]] = [257, 256, 700, 2100]
    lens[rng.integers(0, m, size=20)] = 300
    if m < 100000:
        lens[1024:1024 + 40] = 260  # long rows only in some workgroups
        lens[2048:2048 + 4] = [258, 2049, 2048, 33]
    p = csr_from_row_lengths(lens, 500, n, seed=m, duplicates=True)
    for q, exact in ((p, False), (integer_valued(p, seed=n), True)):
        d = DeviceProblem(q)
        check_against_oracle(q, d.run_natural(), d.ldc, exact=exact, label=f"m={m} n={n}")


@pytest.mark.parametrize("m,n", [(600, 256), (2048, 64), (9000, 36)])
def test_rows_beyond_the_long_limit_are_the_normal_case(m, n):
    """Every wavefront takes its own rows then; short rows beside them, and a cluster of a few long rows among short ones."""
    rng = np.random.default_rng(m)
    lens = rng.integers(2049, 2500, size=m) if m < 5000 else rng.integers(0, 30, size=m)
    lens[m // 3:m // 3 + 100] = rng.integers(0, 40, size=100)
    lens[m // 2:m // 2 + 40] = 2100
    p = csr_from_row_lengths(lens, 3000, n, seed=n, duplicates=False)
    d = DeviceProblem(p)
    check_against_oracle(p, d.run_natural(), d.ldc, label=f"long rows m={m} n={n}")


# every number of workgroups that look for long rows, and groups of four rows; rows of 400 entries are long
# beside rows of 2, rows of 1000 are not beside a mean of 254 or more
@pytest.mark.parametrize("m,n", [(2050, 32), (8190, 64), (32768, 20), (33000, 36), (524287, 4), (524288, 4), (600001, 3)])
def test_long_rows_at_a_distance_in_a_cluster_and_first(m, n):
    base = np.random.default_rng(m).integers(0, 4, size=m)
    for where, longs in (("every 64th", np.arange(0, m, max(64, m // 500))), ("cluster", np.arange(m // 2, m // 2 + 150)),
                         ("first", np.arange(300)), ("last", np.arange(m - 3, m))):
        lens = base.copy()
        lens[longs] = 400
        p = integer_valued(csr_from_row_lengths(lens, 500, n, seed=m, duplicates=True), seed=n)
        d = DeviceProblem(p)
        check_against_oracle(p, d.run_natural(), d.ldc, exact=True, label=f"{where} m={m} n={n}")


@pytest.mark.parametrize("every", [3, 4, 5])
def test_long_rows_on_either_side_of_four_times_the_mean(every):
    lens = np.full(4104, 2)
    lens[::every] = 1000
    p = integer_valued(csr_from_row_lengths(lens, 1500, 64, seed=every, duplicates=True), seed=1)
    d = DeviceProblem(p)
    check_against_oracle(p, d.run_natural(), d.ldc, exact=True, label=f"every {every}")


@pytest.mark.parametrize("m,n", [(9000, 128), (5000, 192), (199999, 128), (200001, 128), (6000, 32)])
def test_long_rows_with_column_slices_on_either_side_of_the_scouts_rule(m, n):
    lens = np.random.default_rng(m).integers(0, 4, size=m)
    lens[::max(64, m // 100)] = 700
    lens[5] = 5000
    p = integer_valued(csr_from_row_lengths(lens, 17000, n, seed=m, duplicates=True), seed=n)
    d = DeviceProblem(p)
    check_against_oracle(p, d.run_natural(), d.ldc, exact=True, label=f"m={m} n={n}")


@pytest.mark.parametrize("m,k,n", [(1500, 17000, 128), (700, 11000, 192)])  # shapes with 64-column slices, groups of 16 lanes either way
@pytest.mark.parametrize("ldb,ldc,shift", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 3, 0), (4, 4, 0), (0, 0, 1), (2, 0, 3)])
def test_few_rows_with_operands_of_any_alignment(m, k, n, ldb, ldc, shift):
    """Padded rows of B or C, or a B that starts `shift` floats into its array, take the loads and stores for any alignment."""
    lens = np.random.default_rng(m).integers(0, 40, size=m)
    lens[[1, m // 2, m - 1]] = [300, 2100, 700]
    p = integer_valued(with_padding(csr_from_row_lengths(lens, k, n, seed=m, duplicates=True), n + ldb), seed=n)
    d = DeviceProblem(p, ldc=n + ldc)
    if shift:
        moved = torch.empty(d.Bfull.numel() + shift, device=d.dev)[shift:].view_as(d.Bfull)
        moved.copy_(d.Bfull)
        d.Bfull = moved
    check_against_oracle(p, d.run_natural(), d.ldc, exact=True, label=f"m={m} n={n} +{ldb} +{ldc} at {shift}")
