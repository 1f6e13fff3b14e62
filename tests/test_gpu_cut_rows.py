"""Long rows cut by columns, a range of columns per accelerator die: every class of rows, all lane mappings, rows whose
columns are in no order or bunched, other columns at the call than at the plan, the one-shot call, and the sampled product."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2405_16883_amd as sp
from oracle import sddmm_csr_oracle
from workloads import csr_from_row_lengths, integer_valued, with_padding

from gpu_util import ATOL, RTOL_T, DeviceProblem, check_against_oracle, tuning

pytestmark = pytest.mark.gpu


def problem(n, seed=0, duplicates=False, k=9000, m=7000):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 30, size=m)
    lens[rng.permutation(m)[:260]] = np.repeat([63, 64, 65, 127, 128, 200, 255, 256, 300, 511, 512, 1023, 1024], 20)
    lens[[0, 7, m - 1]] = [2047, 2048, 5000]
    return csr_from_row_lengths(lens, k, n, seed=seed, duplicates=duplicates)


@pytest.mark.parametrize("n", [17, 20, 47, 64, 100, 128, 130, 300, 600])
@pytest.mark.parametrize("finest", [0, 2, 4])
def test_cut_rows(n, finest):
    p = problem(n, seed=n)
    for q, exact, pad in ((p, False, 0), (with_padding(p, n + 3), False, 2), (integer_valued(p, seed=n), True, 0)):
        d = DeviceProblem(q, ldc=n + pad)
        with tuning(f"cut=1,cutj={finest}"):
            plan = d.make_plan()
        got = d.run_planned(plan)
        check_against_oracle(q, got, d.ldc, exact=exact, label=f"n={n} finest={finest} ldb={q.ldb}")
        with tuning("cut=0"):
            whole = d.make_plan()
        if not exact:  # another order of summation: the rows really are cut
            assert not np.array_equal(d.run_planned(whole), got)
        plan.destroy()
        whole.destroy()


@pytest.mark.parametrize("spec", ["sliced=64", "sliced=32,pack=0", "hot=512", "ch=64,bch=64", "bn=16", "lw=64"])
def test_cut_rows_beside_every_other_path(spec):
    p = integer_valued(problem(128, seed=3), seed=4)
    with tuning("cut=1," + spec):
        d = DeviceProblem(p)
        plan = d.make_plan()
        plain = d.run_planned(plan)
        check_against_oracle(p, plain, d.ldc, exact=True, label=spec)
        bias = torch.arange(-64, 64, dtype=torch.float32, device=d.dev)
        sp.scorch_spmm_csr_planned_epilogue(plan, d.rowptr, d.colidx, d.vals, d._B_arg(), bias, sp.ACT_RELU, d._C_arg())
        torch.cuda.synchronize()
        assert np.array_equal(d.Cfull.cpu().numpy(), np.maximum(plain + bias.cpu().numpy(), 0))
        plan.destroy()


@pytest.mark.parametrize("kind", ["any order", "bunched", "one column"])
def test_cut_rows_of_any_columns_and_the_one_shot_call(kind):
    """Bunched columns leave most pieces empty and some as long as a row: then no row is cut."""
    p = problem(64, seed=5, duplicates=True)
    rng = np.random.default_rng(1)
    col = p.colidx.copy()
    if kind == "any order":
        col = rng.integers(0, p.k, size=p.nnz).astype(np.int32)
    elif kind == "bunched":
        col = (col // 300).astype(np.int32)
    else:
        col[:] = 17
    q = dataclasses.replace(p, colidx=col)
    with tuning("cut=1,res=0"):
        d = DeviceProblem(q)
        plan = d.make_plan()
        got = d.run_planned(plan)
        check_against_oracle(q, got, d.ldc, label=kind)
        d.reset_C()
        sp.scorch_spmm_csr_static(q.m, q.k, q.n, d.rowptr, d.colidx, d.vals, d._B_arg(), d._C_arg())
        torch.cuda.synchronize()
        assert np.array_equal(d.Cfull.cpu().numpy(), got)
        # a plan is bound to the row pointers: other columns at the call
        e = DeviceProblem(p)
        check_against_oracle(p, e.run_planned(plan), e.ldc, label=kind + ", others at the call")
        plan.destroy()


@pytest.mark.parametrize("n", [1001, 1002])
def test_cut_rows_by_the_planners_own_choice_and_in_graphs(n):
    """A matrix large enough for it, skewed rows: planned and replayed calls agree to the bit; the one-shot call does not serve it."""
    rng = np.random.default_rng(n)
    lens = np.minimum(6000, (36.0 / rng.random(24000) ** 0.7).astype(np.int64))
    p = csr_from_row_lengths(lens, 24000, n, seed=n)
    assert p.nnz >= 1 << 20
    d = DeviceProblem(p)
    plan = d.make_plan()
    got = d.run_planned(plan)
    check_against_oracle(p, got, d.ldc, rows=np.argsort(lens)[-100:], label="longest rows")
    check_against_oracle(p, got, d.ldc, rows=rng.integers(0, p.m, size=200), label="any rows")
    with tuning("cut=0"):
        whole = d.make_plan()
    assert whole.info().workspace_bytes_used > sp.STATIC_SCRATCH_BYTES
    assert not np.array_equal(d.run_planned(whole), got)
    whole.destroy()
    with pytest.raises(sp.ScorchError):
        sp.scorch_spmm_csr_static(p.m, p.k, p.n, d.rowptr, d.colidx, d.vals, d._B_arg(), d._C_arg())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp.scorch_spmm_csr_planned(plan, d.rowptr, d.colidx, d.vals, d._B_arg(), d._C_arg())
    for _ in range(3):
        d.reset_C()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(d.Cfull.cpu().numpy(), got)
    plan.destroy()


def test_a_workspace_without_room_for_the_pieces_leaves_the_rows_whole():
    rng = np.random.default_rng(7)
    n = 1001
    lens = np.minimum(6000, (36.0 / rng.random(24000) ** 0.7).astype(np.int64))
    p = csr_from_row_lengths(lens, 24000, n, seed=7)
    d = DeviceProblem(p)
    with tuning("cut=0"):
        least = sp.scorch_spmm_plan_workspace_bytes(p.m, p.k, n, p.nnz)
        plan = d.make_plan()
    whole = d.run_planned(plan)
    plan.destroy()
    full = sp.scorch_spmm_plan_workspace_bytes(p.m, p.k, n, p.nnz)
    assert full > least
    for size in (least, least + 1000, full - 1, full):
        ws = torch.empty(full + 4096, dtype=torch.uint8, device=d.dev)
        ws[size:] = 77
        plan = sp.scorch_spmm_plan(p.m, p.k, n, d.rowptr, p.nnz, colidx=d.colidx, workspace=ws[:size])
        assert plan.info().workspace_bytes_used == (full if size == full else least)
        assert np.array_equal(d.run_planned(plan), whole) == (size < full)
        assert bool((ws[size:] == 77).all())
        plan.destroy()
    with pytest.raises(sp.ScorchError):
        sp.scorch_spmm_plan(p.m, p.k, n, d.rowptr, p.nnz, colidx=d.colidx, workspace=torch.empty(least - 1, dtype=torch.uint8, device=d.dev))


@pytest.mark.parametrize("m", [1, 64, 400])
def test_cut_where_no_or_every_row_is_long(m):
    for length in (0, 63, 64, 3000):
        p = integer_valued(csr_from_row_lengths([length] * m, 4000, 36, seed=m), seed=2)
        with tuning("cut=1,res=0"):
            d = DeviceProblem(p)
            plan = d.make_plan()
            check_against_oracle(p, d.run_planned(plan), d.ldc, exact=True, label=f"m={m} length={length}")
            plan.destroy()


@pytest.mark.parametrize("dcols", [3, 20, 100, 128, 300])
def test_sampled_product_of_cut_rows_keeps_its_bits(dcols):
    p = problem(64, seed=6)
    rng = np.random.default_rng(dcols)
    Bm = rng.standard_normal((p.m, dcols)).astype(np.float32)
    Ct = rng.standard_normal((p.k, dcols)).astype(np.float32)
    d = DeviceProblem(p)
    out = {}
    for spec in ("cut=1,cutj=2,sdblk=0", "cut=0,sdblk=0"):
        with tuning(spec):
            plan = d.make_plan()
        o = torch.full((p.nnz,), -7.0, device=d.dev)
        sp.scorch_sddmm_csr_planned(plan, dcols, d.rowptr, d.colidx, d.vals, torch.from_numpy(Bm).to(d.dev), torch.from_numpy(Ct).to(d.dev), o)
        out[spec] = o.cpu().numpy()
        plan.destroy()
    a, b = out.values()
    assert np.array_equal(a, b)
    ref, T = sddmm_csr_oracle(p.m, dcols, p.rowptr, p.colidx, p.vals, Bm, Ct)
    assert (np.abs(a - ref) <= RTOL_T * T + ATOL).all()
