"""scorch_dense_layer against float64: edges of the 16-column and 16-row tiles, parts of W, strided operands, few rows.

Tolerance: a sum of k rounded products of float32 numbers in any order is within (k + 2) 2^-24 of sum |x w| + |bias|."""
import pytest
import torch

import paper_2405_16883_amd as sp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("m,k,n,pad", [(1, 1, 1, 0), (15, 16, 16, 0), (17, 17, 15, 1), (1000, 128, 128, 0), (40000, 47, 129, 3),
                                       (33000, 144, 256, 4), (70001, 100, 47, 0), (270000, 3, 40, 0), (16385, 31, 144, 1)])
@pytest.mark.parametrize("relu,with_bias", [(True, True), (False, False)])
def test_dense_layer_matches_float64(m, k, n, pad, relu, with_bias):
    g = torch.Generator(device=DEV).manual_seed(m + 7 * k + n)
    X = torch.randn((m, k + pad), generator=g, device=DEV)[:, :k]
    W = torch.randn((k, n + pad), generator=g, device=DEV)[:, :n]
    b = torch.randn(n, generator=g, device=DEV) if with_bias else None
    whole = torch.full((m + 1, n + pad), float("nan"), device=DEV)
    Y = whole[:m, :n]
    sp.scorch_dense_layer(X, W, b, sp.ACT_RELU if relu else sp.ACT_IDENTITY, Y)
    ref, T = X.double() @ W.double(), X.double().abs() @ W.double().abs()
    if with_bias:
        ref, T = ref + b.double(), T + b.double().abs()
    if relu:
        ref = ref.clamp(min=0)
    assert bool(((Y.double() - ref).abs() <= (k + 2) * 2.0 ** -24 * T).all())
    assert bool(whole[m:].isnan().all()) and bool(whole[:, n:].isnan().all()), "written outside Y"


@pytest.mark.parametrize("m,k,n,pad", [(291683, 25, 208, 0), (291683, 25, 205, 3), (1000003, 16, 53, 0), (475007, 47, 100, 1)])
def test_wide_results_beyond_the_memory_side_cache(m, k, n, pad):
    """Two row tiles per wavefront although one has fewer rounds."""
    test_dense_layer_matches_float64(m, k, n, pad, True, True)


def test_dense_layer_keeps_nan_and_refuses_wide_x():
    X = torch.zeros((4, 8), device=DEV)
    X[1, 2] = float("nan")
    Y = torch.empty((4, 5), device=DEV)
    sp.scorch_dense_layer(X, torch.ones((8, 5), device=DEV), None, sp.ACT_RELU, Y)
    assert bool(Y[1].isnan().all()) and bool((Y[[0, 2, 3]] == 0).all())
    k = sp.DENSE_LAYER_K_MAX + 1
    with pytest.raises(sp.ScorchError):
        sp.scorch_dense_layer(torch.zeros((4, k), device=DEV), torch.zeros((k, 5), device=DEV), None, sp.ACT_RELU, Y)


@pytest.mark.parametrize("k", [1, 8, 9, 16, 24, 33, 64])
def test_dense_layer_adds_up_the_even_then_the_odd_columns_of_eight(k):
    """The order of the sums, which the dense library shares: each a fused multiply-add, here in float64 rounded to float32."""
    m, n = 100, 20
    g = torch.Generator(device=DEV).manual_seed(k)
    X, W = torch.randn((m, k), generator=g, device=DEV), torch.randn((k, n), generator=g, device=DEV)
    Y = torch.empty((m, n), device=DEV)
    sp.scorch_dense_layer(X, W, None, sp.ACT_IDENTITY, Y)
    acc = torch.zeros((m, n), device=DEV)
    for c in [b + 2 * q + s for b in range(0, k, 8) for s in range(2) for q in range(4) if b + 2 * q + s < k]:
        acc = (acc.double() + X[:, c:c + 1].double() * W[c:c + 1].double()).float()
    # rounded twice (the sum to 53 bits first) only where 29 bits below the last one read 10...0: one sum in 2^28
    assert torch.equal(acc, Y)
