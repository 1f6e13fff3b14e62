"""One and two columns: rows of every length a window's wavefront may meet, and means on either side of the rule."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2405_16883_amd as sp
from workloads import csr_from_row_lengths, integer_valued, with_padding

from gpu_util import DeviceProblem, check_against_oracle, tuning

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4])
@pytest.mark.parametrize("spec", [None, "bn=16", "bn=256", "bn=256,alpha=1", "ch=512"])
@pytest.mark.parametrize("many", [0, 7, 40])  # of the longer lengths: none, among short rows, most rows (mean above 32)
def test_rows_of_every_length(n, spec, many):
    rng = np.random.default_rng(many)
    m = 700
    lens = rng.integers(0, 12, size=m)
    edges = [31, 32, 33, 63, 64, 65, 128, 255, 256, 257, 300, 700]
    at = rng.permutation(m)[:many * len(edges)]
    lens[at] = np.resize(edges, at.size)
    lens[[0, m - 1]] = [256, 257] if many else [32, 31]
    p = csr_from_row_lengths(lens, 900, n, seed=many, duplicates=True)
    with tuning(spec):
        for q, exact, pad in ((p, False, 0), (with_padding(p, n + 3), False, 1), (integer_valued(p, seed=n), True, 0)):
            d = DeviceProblem(q, ldc=n + pad)
            plan = d.make_plan()
            plain = d.run_planned(plan)
            check_against_oracle(q, plain, d.ldc, exact=exact, label=f"n={n} {spec} {many}")
            bias = torch.arange(1, n + 1, dtype=torch.float32, device=d.dev) - 2
            sp.scorch_spmm_csr_planned_epilogue(plan, d.rowptr, d.colidx, d.vals, d._B_arg(), bias, sp.ACT_RELU, d._C_arg())
            torch.cuda.synchronize()
            if exact:
                assert np.array_equal(d.Cfull.cpu().numpy()[:, :n], np.maximum(plain[:, :n] + bias.cpu().numpy(), 0))
            plan.destroy()


@pytest.mark.parametrize("lens", [[0] * 130, [1] * 64 + [0] * 64 + [256], [257], [256], [0, 300, 0], [255, 256, 255, 256] + [0] * 60])
def test_few_rows(lens):
    p = integer_valued(csr_from_row_lengths(lens, 400, 1, seed=1), seed=2)
    d = DeviceProblem(p)
    plan = d.make_plan()
    check_against_oracle(p, d.run_planned(plan), d.ldc, exact=True, label=str(lens[:4]))
    plan.destroy()


@pytest.mark.parametrize("n", [1, 2])
@pytest.mark.parametrize("ch", [64, 128, 255])
def test_rows_beyond_a_smaller_ch_are_summed_by_one_workgroup_in_its_order(n, ch):
    """Rows of more than `ch` entries belong to the workgroups of long rows: an entry per lane of four wavefronts, the lanes in pairs,
    then pairs of pairs, then the wavefronts.  If a window stored such a row as well, its bits would depend on who is last."""
    lens = np.random.default_rng(ch).integers(0, 20, size=900)
    lens[::30] = np.resize([ch + 1, 200, 256], lens[::30].size)
    long_rows = np.flatnonzero(lens > ch)
    p = csr_from_row_lengths(lens, 700, n, seed=ch, duplicates=True)
    assert p.nnz <= 32 * p.m
    d = DeviceProblem(p)
    with tuning(f"bn=256,ch={ch}"):
        plan = d.make_plan()
    want = np.zeros((long_rows.size, n), dtype=np.float32)
    for i, r in enumerate(long_rows):
        e = slice(p.rowptr[r], p.rowptr[r + 1])
        prod = np.zeros((256, n), dtype=np.float32)
        prod[:lens[r]] = p.vals[e, None] * p.B[p.colidx[e], :n]
        waves = prod.reshape(4, 64, n)
        for off in (1, 2, 4, 8, 16, 32):
            waves = waves + waves[:, np.arange(64) ^ off]
        want[i] = ((waves[0, 0] + waves[1, 0]) + waves[2, 0]) + waves[3, 0]
    for _ in range(4):
        got = d.run_planned(plan)
        check_against_oracle(p, got, d.ldc, label=f"n={n} ch={ch}")
        assert np.array_equal(got[long_rows], want)
    plan.destroy()


@pytest.mark.parametrize("n", [1, 2])
@pytest.mark.parametrize("length,at", [(65, 0), (100, 30), (128, 63), (256, 191)])
def test_rows_of_more_than_64_entries_are_summed_by_fused_multiply_adds(n, length, at):
    """Entries 64 apart are one lane's.  The first is -(1 + 2^-11), the second (1 + 2^-12)^2 = 1 + 2^-11 + 2^-24, the others add nothing:
    2^-24 is left, unless the second product was rounded to 24 bits on the way."""
    lens = np.random.default_rng(length).integers(0, 20, size=500)
    rows = np.arange(3, 500, 50)
    lens[rows] = length
    p = csr_from_row_lengths(lens, 700, n, seed=length, duplicates=True)
    vals, col, B = p.vals.copy(), p.colidx.copy(), p.B.copy()
    B[0, :n], B[1, :n] = 1, 1 + 2.0 ** -12
    for r in rows:
        e = p.rowptr[r]
        vals[e:e + length] = 0
        first = e + min(at, length - 65)
        vals[first], col[first] = -(1 + 2.0 ** -11), 0
        vals[first + 64], col[first + 64] = 1 + 2.0 ** -12, 1
    q = dataclasses.replace(p, vals=vals, colidx=col, B=B)
    d = DeviceProblem(q)
    with tuning("bn=256"):
        plan = d.make_plan()
    got = d.run_planned(plan)
    check_against_oracle(q, got, d.ldc, label=f"n={n} length={length}")
    assert (got[rows, :n] == 2.0 ** -24).all()
    plan.destroy()


@pytest.mark.parametrize("n", [1, 2])
@pytest.mark.parametrize("spec", ["bn=256", "bn=128", "bn=64"])
@pytest.mark.parametrize("medium", [0, 3, 4, 40])  # of 1024 rows: on either side of one in 256
def test_windows_that_walk_whole_rows_or_short_ones_only(n, spec, medium):
    lens = np.random.default_rng(medium).integers(0, 32, size=1024)
    lens[np.arange(medium) * 25] = np.resize([33, 64, 200, 256], medium)
    p = csr_from_row_lengths(lens, 900, n, seed=medium, duplicates=True)
    for q, exact in ((p, False), (integer_valued(p, seed=n), True)):
        d = DeviceProblem(q)
        with tuning(spec):
            plan = d.make_plan()
        assert plan.info().n_wave_rows == medium
        check_against_oracle(q, d.run_planned(plan), d.ldc, exact=exact, label=f"n={n} {spec} {medium}")
        plan.destroy()
