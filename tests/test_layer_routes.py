"""Which torch states leave the dense product of a layer to torch; needs no GPU."""
import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2405_16883_amd import gcn


def test_modes_and_transforms_are_seen():
    class Watch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    assert gcn._unwatched()
    with Watch():
        assert not gcn._unwatched()
    with torch.autograd.forward_ad.dual_level():
        assert not gcn._unwatched()
    assert torch.vmap(lambda x: x * float(gcn._unwatched()))(torch.ones(2)).sum() == 0
    assert gcn._unwatched()


@pytest.mark.parametrize("owner,name", [(torch._C, "_len_torch_dispatch_stack"), (torch._C, "_len_torch_function_stack"),
                                        (torch._C._functorch, "peek_interpreter_stack"), (torch.autograd.forward_ad, "_current_level")])
def test_a_torch_without_one_of_these_names_keeps_the_product(monkeypatch, owner, name):
    monkeypatch.delattr(owner, name)
    assert not gcn._unwatched()


@pytest.mark.parametrize("m,k,n", [(45000, 128, 128), (62973, 128, 128), (80867, 144, 128), (97551, 128, 128), (97551, 128, 64), (86084, 144, 64),
                                   (46000, 144, 96), (131072, 144, 144), (21754, 144, 144), (229376, 128, 128), (214772, 144, 128), (100000, 128, 40 * 2), (20000, 40, 40)])
def test_products_that_the_library_makes_faster_stay_there(m, k, n):
    assert not gcn._native_first(m, k, n)


@pytest.mark.parametrize("m,k,n", [(169343, 128, 128), (20000, 64, 64), (62973, 112, 112), (97551, 128, 47), (1000000, 128, 128), (2000, 144, 128)])
def test_products_that_the_own_kernel_makes_faster(m, k, n):
    assert gcn._native_first(m, k, n)
