"""Tensors that torch will not give a pointer for are Python errors in every entry point of the extension, never the end of
the process.  Fake GPU tensors stand in for real ones, so no GPU is needed; each case is a process of its own."""
import os
import subprocess
import sys

import pytest

import paper_2405_16883_amd as sp

SETUP = """
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
import paper_2405_16883_amd as sp
native = sp.binding._load_native()
with FakeTensorMode():
    d = torch.zeros(2, 2, device="cuda")
    sparse = torch.sparse_coo_tensor(torch.zeros(2, 1, dtype=torch.int64, device="cuda"), torch.zeros(1, device="cuda"), (2, 2))
    isparse = torch.sparse_coo_tensor(torch.zeros(1, 1, dtype=torch.int64, device="cuda"),
                                      torch.zeros(1, dtype=torch.int32, device="cuda"), (2,))
"""

CALLS = {  # one tensor that has no memory; what comes before it is absent
    "spmm_csr": "native.spmm_csr(2, 2, 2, None, None, {x}, {b}, d, None)",
    "spmm_csr_static": "native.spmm_csr_static(2, 2, 2, None, None, {x}, {b}, d, None)",
    "spmm_csr_planned": "native.spmm_csr_planned(0, None, None, {x}, {b}, d, None)",
    "spmm_csr_planned_epilogue": "native.spmm_csr_planned_epilogue(0, None, None, {x}, {b}, None, 0, d, None)",
    "sddmm_csr": "native.sddmm_csr(2, 2, 2, None, None, {x}, {b}, d, None, None)",
    "sddmm_csr_planned": "native.sddmm_csr_planned(0, 2, None, None, {x}, {b}, d, None, None)",
    "dense_layer": "native.dense_layer({b}, d, {x}, 0, d, None)",
    "coo_to_csr_rowptr": "native.coo_to_csr_rowptr(2, isparse, None, None, None)",
}


def run(body):
    if not os.path.exists(sp.LIB_PATH):
        pytest.skip("library not built")
    res = subprocess.run([sys.executable, "-c", SETUP + body], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True,
                         cwd=sp.__path__[0] + "/..")
    assert res.returncode == 0, f"exit status {res.returncode}\n{res.stderr[-2000:]}"
    return res.stdout.split()


@pytest.mark.parametrize("name", sorted(CALLS))
def test_a_tensor_without_memory_is_a_python_error(name):
    body = ""
    for x, b in (("None", "sparse"), ("sparse", "d")):
        call = CALLS[name].format(x=x, b=b)
        body += f"try:\n    {call}\nexcept Exception as e:\n    print(type(e).__name__)\n"
    assert run(body) == ["RuntimeError"] * 2


def test_a_tensor_inside_vmap_is_a_python_error():
    assert run("""
with FakeTensorMode():
    B = torch.zeros(3, 2, 2, device="cuda")
    try:
        torch.vmap(lambda b: native.spmm_csr(2, 2, 2, None, None, None, b, d, None))(B)
    except RuntimeError:
        print("raised")
""") == ["raised"]
