"""Plan lists against the plan oracle, bit for bit, at the edges of the planning kernels' tiles of 256 rows, of the
workgroups that count the rows before their own (up to 8), and of windows that reach past a tile; workspaces that are too small."""
import numpy as np
import pytest
import torch

import paper_2405_16883_amd as sp

from oracle.plan import plan_oracle
from workloads import csr_from_row_lengths

from gpu_util import DeviceProblem, read_plan_arrays, tuning

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 255, 256, 257, 320, 2047, 2048, 2049, 5000])
@pytest.mark.parametrize("tune", [None, "bn=256,alpha=4,lw=8,ch=40,bch=64", "bn=16,alpha=1,lw=0,ch=32,bch=48", "bn=48,alpha=3"])
def test_lists_at_tile_edges(m, tune):
    rng = np.random.default_rng(m)
    lens = rng.integers(0, 3, size=m)  # nearly empty rows: 64 rows per window
    lens[rng.integers(0, m, size=m // 20 + 1)] = rng.integers(30, 300, size=m // 20 + 1)
    lens[-1] = 700
    with tuning(tune):
        p = csr_from_row_lengths(lens, 900, 8, seed=m)
        plan = DeviceProblem(p).make_plan()
        info, got = read_plan_arrays(plan)
        want = plan_oracle(p.rowptr, info.BN, info.ALPHA, info.LW, info.CH, info.BCH)
        assert info.nnz == p.nnz and info.n_short_rows == int(want["n_short"])
        for key in ("win_row_start", "win_stage", "wave_rows", "wave_span", "items", "split"):
            assert np.array_equal(got[key], want[key]), key
        plan.destroy()


@pytest.mark.parametrize("m", [300, 2049, 100000, 600000])  # without a count per workgroup and with one, up to 20 KB of them
def test_a_workspace_that_is_too_small_is_refused_and_left_alone(m):
    dev = torch.device("cuda")
    rowptr = torch.arange(0, 3 * m + 1, 3, dtype=torch.int32, device=dev)
    need = sp.scorch_spmm_plan_workspace_bytes(m, m, 64, 3 * m)
    for size in (256, need // 2, need - 1):
        whole = torch.full((need + 256,), 90, dtype=torch.uint8, device=dev)
        with pytest.raises(sp.ScorchError, match=f"workspace of {size} bytes is smaller than the {need} needed"):
            sp.scorch_spmm_plan(m, m, 64, rowptr, 3 * m, workspace=whole[:size])
        assert bool((whole == 90).all())
    sp.scorch_spmm_plan(m, m, 64, rowptr, 3 * m, workspace=torch.empty(need, dtype=torch.uint8, device=dev)).destroy()


@pytest.mark.parametrize("m", [4, 300, 5000, 600000])
def test_row_pointers_that_decrease_are_refused(m):
    """A plan of them would lack windows, which an execution would then read."""
    dev = torch.device("cuda")
    for at in (1, m // 2, m - 1):
        rowptr = torch.arange(0, 5 * m + 1, 5, dtype=torch.int32, device=dev)
        rowptr[at] += 7
        with pytest.raises(sp.ScorchError, match="rowptr decreases") as e:
            sp.scorch_spmm_plan(m, 100, 8, rowptr, 5 * m)
        assert e.value.status == sp.binding.SCORCH_ERR_INVALID_ARG


def test_a_refused_one_shot_call_leaves_nothing_on_the_stream():
    dev = torch.device("cuda")
    m, per_row = 1_000_000, 40
    assert sp.scorch_spmm_plan_workspace_bytes(m, 4, 64, per_row * m) > sp.STATIC_SCRATCH_BYTES
    rowptr = torch.arange(0, per_row * m + 1, per_row, dtype=torch.int32, device=dev)
    cols, vals = torch.zeros(per_row * m, dtype=torch.int32, device=dev), torch.zeros(per_row * m, device=dev)
    B, C = torch.zeros((4, 64), device=dev), torch.full((m, 64), 7.0, device=dev)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with pytest.raises(sp.ScorchError) as e:
        sp.scorch_spmm_csr_static(m, 4, 64, rowptr, cols, vals, B, C, stream=s)
    assert e.value.status == sp.binding.SCORCH_ERR_UNSUPPORTED and s.query()
    with pytest.raises(sp.ScorchError) as e:
        sp.scorch_spmm_csr_static(m // 100, 4, 64, rowptr, cols[:0], vals, B, C, stream=s)
    assert e.value.status == sp.binding.SCORCH_ERR_INVALID_ARG and s.query()
    torch.cuda.synchronize()
    assert bool((C == 7.0).all())
