"""Plan-free SpMM on few rows: the workgroup-per-row kernel at the edges of its chunks, tiles and range of row counts."""
import numpy as np
import pytest

from workloads import csr_from_row_lengths, integer_valued, with_padding

from gpu_util import DeviceProblem, check_against_oracle

pytestmark = pytest.mark.gpu


# 2 and 16 rows: 16 wavefronts per row; 300 rows: 4; 2048 x 1 tile and 1024 x 2 tiles are the last of the range, the
# next two run as runs of rows with narrow tiles.  Lengths: one chunk of 128 entries more or less, and the 4 or 16
# chunks that the wavefronts of a workgroup take at once.
@pytest.mark.parametrize("m,n", [(2, 1), (2, 2), (2, 3), (16, 36), (16, 100), (300, 33), (300, 128), (2048, 32), (1024, 64),
                                 (2049, 32), (1030, 128), (1030, 270)])
def test_few_rows(m, n):
    edge = np.array([0, 1, 127, 128, 129, 511, 512, 513, 2047, 2048, 2049, 3000])
    rng = np.random.default_rng(m * 1000 + n)
    lens = edge[rng.integers(0, len(edge), size=m)] if m <= 300 else rng.integers(0, 150, size=m)
    p = csr_from_row_lengths(lens, 3000, n, seed=m + n)
    for q, exact in ((p, False), (with_padding(p, n + 3), False), (integer_valued(p, seed=n), True)):
        d = DeviceProblem(q, ldc=n + 1 if exact else n)
        check_against_oracle(q, d.run_natural(), d.ldc, exact=exact, label=f"m={m} n={n} ldb={q.ldb}")
