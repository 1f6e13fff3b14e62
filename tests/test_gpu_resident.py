"""The resident kernel (narrow B kept in LDS in chunks) against the oracle: one chunk and several, the last of one row,
every padded width, rows of no, one and many windows of a chunk, rows whose columns are not increasing, and other columns
at the call than at the plan."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2405_16883_amd as sp
from workloads import csr_from_row_lengths, integer_valued, with_padding

from gpu_util import DeviceProblem, check_against_oracle, tuning

pytestmark = pytest.mark.gpu


def chunk_rows(n):
    w = 4
    while w < n:
        w *= 2
    return 158 * 256 // w


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 15, 16, 20, 32, 33, 64])
@pytest.mark.parametrize("extra", [-1, 0, 1, 700])  # columns beyond one chunk
@pytest.mark.parametrize("m", [1, 40, 300])
def test_resident(m, extra, n):
    k = chunk_rows(n) + extra
    rng = np.random.default_rng(m * 100 + n)
    lens = rng.integers(0, 400, size=m)  # up to six windows of 64 in a chunk
    lens[rng.integers(0, m)] = min(k, 1100)
    lens[-1] = 64
    p = csr_from_row_lengths(lens, k, n, seed=m + n)
    with tuning("res=1"):
        for q, exact, pad in ((p, False, 0), (with_padding(p, n + 3), False, 2), (integer_valued(p, seed=n), True, 0)):
            d = DeviceProblem(q, ldc=n + pad)
            plan = d.make_plan()
            assert plan.info().mode == 3
            check_against_oracle(q, d.run_planned(plan), d.ldc, exact=exact, label=f"m={m} k={k} n={n} ldb={q.ldb}")
            plan.destroy()


@pytest.mark.parametrize("k", [500, 6000])
def test_resident_epilogue_is_the_plain_result_plus_bias_and_relu(k):
    p = integer_valued(csr_from_row_lengths([30] * 50, k, 20, seed=k), seed=1)
    with tuning("res=1"):
        d = DeviceProblem(p)
        plan = d.make_plan()
        plain = d.run_planned(plan)
        bias = torch.arange(-10, 10, dtype=torch.float32, device=d.dev)
        sp.scorch_spmm_csr_planned_epilogue(plan, d.rowptr, d.colidx, d.vals, d._B_arg(), bias, sp.ACT_RELU, d._C_arg())
        torch.cuda.synchronize()
        assert np.array_equal(d.Cfull.cpu().numpy(), np.maximum(plain + bias.cpu().numpy(), 0))
        plan.destroy()


def test_resident_is_left_to_rows_of_increasing_columns_and_chosen_for_a_dense_weight():
    with tuning("res=1"):
        for sorted_cols, duplicates in ((False, False), (True, True)):
            p = csr_from_row_lengths([40] * 60, 50, 16, seed=3, sorted_cols=sorted_cols, duplicates=duplicates)
            d = DeviceProblem(p)
            plan = d.make_plan()
            assert plan.info().mode != 3
            check_against_oracle(p, d.run_planned(plan), d.ldc, label="not increasing")
            plan.destroy()
    p = csr_from_row_lengths([1000] * 4096, 4096, 16, seed=4)
    d = DeviceProblem(p)
    plan = d.make_plan()
    assert plan.info().mode == 3
    check_against_oracle(p, d.run_planned(plan), d.ldc, label="chosen")
    plan.destroy()


@pytest.mark.parametrize("m,n", [(40, 16), (2500, 5)])
def test_a_plan_serves_other_columns_of_the_same_row_pointers(m, n):
    """A plan is bound to the row pointers; the columns are the call's own (increasing, as the planner saw them)."""
    k = 2 * chunk_rows(n) + 50
    lens = np.random.default_rng(m).integers(0, 300, size=m)
    p, q = (csr_from_row_lengths(lens, k, n, seed=s, duplicates=False) for s in (1, 2))
    assert np.array_equal(p.rowptr, q.rowptr) and not np.array_equal(p.colidx, q.colidx)
    with tuning("res=1"):
        d, e = DeviceProblem(p), DeviceProblem(integer_valued(q, seed=3))
        plan = d.make_plan()
        assert plan.info().mode == 3
        check_against_oracle(e.p, e.run_planned(plan), e.ldc, exact=True, label="other columns")
        check_against_oracle(p, d.run_planned(plan), d.ldc, label="the planner's columns")
        plan.destroy()


@pytest.mark.parametrize("n", [3, 8, 15, 20, 64])  # every padded width
@pytest.mark.parametrize("m", [40, 2500])
def test_a_plan_serves_columns_in_any_order_and_repeated(m, n):
    """The columns of the call need not be increasing either: entries in any chunk's place, repeated ones, a row left as it
    was planned beside them, and rows of B that no entry names are never added (here they are not numbers)."""
    k = 2 * chunk_rows(n) + 50
    lens = np.random.default_rng(m).integers(0, 300, size=m)
    lens[3] = 0
    p = csr_from_row_lengths(lens, k, n, seed=1, duplicates=False)
    q = integer_valued(csr_from_row_lengths(lens, k - 2, n, seed=2, sorted_cols=False, duplicates=True), seed=3)
    cols = q.colidx + 1  # columns 0 and k - 1 are named by no entry
    some = p.rowptr[m // 2]  # wavefronts meet both kinds of rows
    cols[:some] = np.clip(p.colidx[:some], 1, k - 2)
    B = np.full((k, n), np.nan, dtype=np.float32)
    B[1:k - 1] = q.B
    q = dataclasses.replace(q, k=k, colidx=cols, B=B)
    with tuning("res=1"):
        plan = DeviceProblem(p).make_plan()
        assert plan.info().mode == 3
        for r in (q, with_padding(q, n + 3)):
            e = DeviceProblem(r)
            check_against_oracle(r, e.run_planned(plan), e.ldc, exact=True, label=f"any order m={m} n={n} ldb={r.ldb}")
        plan.destroy()


@pytest.mark.parametrize("m,k,share,n", [(4096, 16384, 0.1, 64), (4096, 16384, 0.1, 33), (16384, 16384, 0.1, 40), (1040, 8192, 0.2, 64)])
def test_the_one_shot_call_gives_the_planned_bits_when_its_scratch_holds_the_partial_rows_of_some_rows_only(m, k, share, n):
    """The partial rows take turns there.  Columns that are not increasing leave both calls to the gather kernels."""
    dev = torch.device("cuda")
    per_row = int(share * k)
    g = torch.Generator(device=dev).manual_seed(n)
    rows = min(m, 512)  # row lengths and columns of 512 rows, over and over
    lens = torch.randint(per_row // 2, per_row * 3 // 2, (rows,), generator=g, device=dev)
    keep = torch.rand((rows, k), generator=g, device=dev).argsort(dim=1).argsort(dim=1) < lens[:, None]
    cols = keep.nonzero()[:, 1].int().repeat((m + rows - 1) // rows)
    lens = lens.repeat((m + rows - 1) // rows)[:m]
    rowptr = torch.zeros(m + 1, dtype=torch.int32, device=dev)
    rowptr[1:] = lens.cumsum(0)
    nnz = int(rowptr[-1])
    cols = cols[:nnz].contiguous()
    vals, B = torch.rand(nnz, generator=g, device=dev) - 0.5, torch.randn((k, n), generator=g, device=dev)
    swapped = cols.clone()
    swapped[[5, 6]] = cols[[6, 5]]  # the first row is out of order
    for c, mode in ((cols, 3), (swapped, None)):
        planned, static = torch.empty((m, n), device=dev), torch.empty((m, n), device=dev)
        plan = sp.scorch_spmm_plan(m, k, n, rowptr, nnz, colidx=c)
        assert (plan.info().mode == 3) == (mode == 3)
        sp.scorch_spmm_csr_planned(plan, rowptr, c, vals, B, planned)
        for _ in range(2):  # the second finds what the first left
            static.fill_(float("nan"))
            sp.scorch_spmm_csr_static(m, k, n, rowptr, c, vals, B, static)
            assert torch.equal(static, planned)
        plan.destroy()
    # against double precision, from the same operands, on rows of the first and the last turn
    for r in (0, m // 2 + 1, m - 1):
        a, b = int(rowptr[r]), int(rowptr[r + 1])
        terms = vals[a:b].double()[:, None] * B[swapped[a:b].long()].double()
        assert bool(((planned[r] - terms.sum(0)).abs() <= 1e-5 * terms.abs().sum(0)).all())


@pytest.mark.parametrize("m,k,n", [(512, 16384, 16), (250, 3000, 60), (4096, 5200, 32), (17, 10113, 4), (300, 2529, 16)])
def test_resident_with_more_chunks_than_b_needs(m, k, n):
    """Chunks are even, and may be more than the fewest so that the workgroups come out in whole rounds."""
    p = csr_from_row_lengths([300] * m, k, n, seed=m)
    with tuning("res=1"):
        for q, exact in ((p, False), (integer_valued(p, seed=n), True)):
            d = DeviceProblem(q)
            plan = d.make_plan()
            assert plan.info().mode == 3
            check_against_oracle(q, d.run_planned(plan), d.ldc, exact=exact, label=f"m={m} k={k} n={n}")
            plan.destroy()


@pytest.mark.parametrize("m,k,n,length,more", [(4096, 16384, 16, 1638, 1), (1024, 9000, 33, 1800, 1), (1152, 7000, 64, 2500, 2)])
def test_resident_with_room_for_the_fewest_chunks_only(m, k, n, length, more):
    """More chunks than B needs take a larger table of row pointers and more partial rows; a workspace without room for them will do."""
    p = integer_valued(csr_from_row_lengths([length] * m, k, n, seed=m, duplicates=False), seed=n)
    d = DeviceProblem(p)
    full = sp.scorch_spmm_plan_workspace_bytes(m, k, n, p.nnz)
    width = 16 if n == 16 else 64
    least = full - more * (m * 4 + m * width * 4)  # m: a multiple of 64, so that every section ends on 256 bytes
    for size in (full, full - 1, least):
        ws = torch.full((full + 4096,), 77, dtype=torch.uint8, device=d.dev)
        plan = sp.scorch_spmm_plan(m, k, n, d.rowptr, p.nnz, colidx=d.colidx, workspace=ws[:size])
        assert plan.info().mode == 3 and plan.info().workspace_bytes_used == (full if size == full else least)
        check_against_oracle(p, d.run_planned(plan), d.ldc, exact=True, label=f"m={m} {size}")
        assert bool((ws[size:] == 77).all())
        plan.destroy()
    with pytest.raises(sp.ScorchError):
        sp.scorch_spmm_plan(m, k, n, d.rowptr, p.nnz, colidx=d.colidx, workspace=ws[:least - 1])
