"""What a plan takes, by the sizes alone (no GPU needed): the workspace says whether rows may be cut by columns, since their pieces
stand in it."""
import random

import pytest

import paper_2405_16883_amd as sp


def size(monkeypatch, m, k, n, nnz, tune=None):
    monkeypatch.delenv("SCORCH_SPMM_TUNE", raising=False)
    if tune:
        monkeypatch.setenv("SCORCH_SPMM_TUNE", tune)
    return sp.scorch_spmm_plan_workspace_bytes(m, k, n, nnz)


SHAPES = [(169343, 169343, 128, 2489000), (169343, 169343, 100, 2489000), (100000, 100000, 100, 5000000), (400000, 400000, 33, 4800000),
          (60000, 60000, 256, 3000000), (4000, 8000, 333, 1600000), (1024, 16384, 201, 8388608), (10000, 40000, 61, 12000000),
          (2000, 20000, 150, 4000000), (2000, 4000, 777, 2400000)]


def drawn(count):
    rng = random.Random(5)
    for _ in range(count):
        m, k, n = int(10 ** rng.uniform(2.5, 6.5)), int(10 ** rng.uniform(2.5, 6.5)), int(10 ** rng.uniform(1.5, 3.2))
        yield m, k, n, min(m * k, int(10 ** rng.uniform(6, 8.5)))


def test_no_rows_are_cut_where_the_one_shot_call_serves(monkeypatch):
    """It analyses at every call, which costs more than the cut gives, and has the planned call's bits."""
    served = cut = 0
    for m, k, n, nnz in [*SHAPES, *drawn(2000)]:
        whole = size(monkeypatch, m, k, n, nnz, "cut=0")
        if whole <= sp.STATIC_SCRATCH_BYTES:
            served += 1
            assert size(monkeypatch, m, k, n, nnz) == whole, (m, k, n, nnz)
        else:
            cut += size(monkeypatch, m, k, n, nnz) > whole
    assert served > 100 and cut > 100


def test_the_pieces_take_no_more_than_half_of_b_and_c_unless_rows_are_long(monkeypatch):
    for m, k, n, nnz in [(2449029, 2449029, 100, 122200000), (1000000, 1000000, 100, 100000000), (1000000, 1000000, 256, 25000000), *drawn(2000)]:
        whole, full = size(monkeypatch, m, k, n, nnz, "cut=0"), size(monkeypatch, m, k, n, nnz)
        stride, pieces = (n + 3) // 4 * 4, (m + k) // 2 if nnz < 320 * m else nnz // 16
        assert full - whole <= pieces * (stride * 4 + 8 + 1) + 100000, (m, k, n, nnz)


@pytest.mark.parametrize("m,k,n,nnz", [(14126, 34665, 36, 76700000), (8763, 23237, 51, 85000000), (26500, 16390, 22, 148600000),
                                       (20534, 28154, 64, 52700000), (4096, 16384, 16, 6710886)])
def test_narrow_b_is_kept_in_lds_with_fewer_chunks_where_more_do_not_fit(monkeypatch, m, k, n, nnz):
    """The table of row pointers per chunk of B stands in the workspace, and the one-shot call has to run in its scratch too."""
    assert size(monkeypatch, m, k, n, nnz) > size(monkeypatch, m, k, n, nnz, "res=0")


@pytest.mark.parametrize("tune", ["cold=1", "cold=3", "fix=1", "u=4", "nt=0"])
def test_experiments_with_the_gather_kernels_find_whole_rows(monkeypatch, tune):
    shape = 2449029, 2449029, 100, 122200000
    assert size(monkeypatch, *shape) > size(monkeypatch, *shape, "cut=0")
    assert size(monkeypatch, *shape, tune) == size(monkeypatch, *shape, tune + ",cut=0")
