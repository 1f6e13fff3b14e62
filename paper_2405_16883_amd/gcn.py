"""One graph-convolution layer  H' = act(A_hat H W + b)  on top of the C ABI (paper, Section 5.1).

The neighbourhood aggregation runs in scorch_spmm_csr_planned_epilogue.  The dense product is one call of scorch_dense_layer
where that applies (see _native_product) and is the faster one, otherwise the dense library's (torch.mm), to which the paper
leaves dense work.  The order of the two products is chosen by width: the aggregation costs 2*nnz*n flops and gathers n floats per
stored entry, so it is done at the narrower of the two feature widths:

    n_out <= n_in :  H' = act(A_hat (H W) + b)      dense product first, epilogue fused into the aggregation
    n_out >  n_in :  H' = act((A_hat H) W + b)      aggregation first, epilogue fused into the dense product

Orchestration only: no sparse arithmetic happens in this file.
"""
from __future__ import annotations

from typing import Dict, Optional

import torch

from . import binding as _b


def _plain(t: torch.Tensor) -> bool:
    """A float32 GPU tensor that is nothing else besides (no subclass, no gradient to record)."""
    return (type(t) in (torch.Tensor, torch.nn.Parameter) and t.is_cuda and t.dtype == torch.float32 and t.layout == torch.strided
            and not t.is_neg() and not (t.requires_grad and torch.is_grad_enabled()))


def _native_product(X: torch.Tensor, W: torch.Tensor, bias: Optional[torch.Tensor]) -> bool:
    """Whether X W (+ bias) goes to scorch_dense_layer: rows that are contiguous, as many columns of X as the kernel takes, and
    nobody but the caller watching the operation (gradients, transforms, autocast and dispatch modes need torch's own)."""
    if not (_plain(X) and _plain(W) and (bias is None or _plain(bias))):
        return False
    m, k = X.shape
    if W.dim() != 2 or not 0 < k <= _b.DENSE_LAYER_K_MAX or W.device != X.device or X.device.index != torch.cuda.current_device():
        return False
    n = W.shape[1]
    if m == 0 or n == 0 or X.stride(1) != 1 or W.stride(1) != 1 or not (k <= X.stride(0) < 1 << 31 and n <= W.stride(0) < 1 << 31):
        return False
    if bias is not None and (bias.device != X.device or bias.dim() != 1 or bias.shape[0] != n or bias.stride(0) != 1):
        return False
    return _unwatched()


def _native_first(m: int, k: int, n: int) -> bool:
    """Whether the dense product alone, m x k times k x n with n <= k, is better made by scorch_dense_layer.  With k in multiples of 16 it
    adds up in the dense library's usual order (the same bits as torch.mm on nearly all shapes tried).  Drawn from sweeps of 45 to 67 row
    counts from 2000 to 2.4 M for 33 pairs of widths, time own / library: 0.1 to 1.0 for k <= 112 or n <= 48.  Wider, the library's time jumps
    by half from one row count to the next and back (tiles of several heights that do or do not come out in whole rounds over the chip), and
    the own kernel is behind at its best ones: 128 -> 128 45 000 rows 1.21, 62 000 1.08, 80 000 1.04, 97 551 1.19, 131 072 1.01, 214 772 1.04, 229 376 1.03
    (but 52 000 0.70, 86 000 0.72); 128 -> 64 97 551 1.11; 144 -> 96 46 000 1.06; 144 -> 144 21 754 1.04.  So only where no row count
    was behind: below 40 000 rows 0.4 to 1.0, 133 000 to 210 000 0.6 to 1.0 (169 343, 128 -> 128 0.83), from 232 000 on 0.6 to 1.0, twice 1.02."""
    return k % 16 == 0 and (k <= 112 or n <= 48 or (m < 40000 and n <= 128) or 133000 <= m < 210000 or m >= 232000)


def _unwatched() -> bool:
    try:
        return not (torch._C._len_torch_dispatch_stack() or torch._C._len_torch_function_stack()
                    or torch._C._functorch.peek_interpreter_stack() is not None or torch.is_autocast_enabled("cuda")
                    or torch.autograd.forward_ad._current_level >= 0)
    except AttributeError:  # a torch that keeps these elsewhere: its own operations are right in any case
        return False


class GcnLayer:
    """Holds the normalised adjacency (CSR, device tensors) and one plan per feature width it has been used with."""

    def __init__(self, m: int, rowptr: torch.Tensor, colidx: torch.Tensor, vals: torch.Tensor, nnz: int):
        self.m, self.nnz = int(m), int(nnz)
        self.rowptr, self.colidx, self.vals = rowptr, colidx, vals
        self._plans: Dict[int, _b.SpmmPlan] = {}

    def _plan(self, n: int) -> _b.SpmmPlan:
        if n not in self._plans:
            self._plans[n] = _b.scorch_spmm_plan(self.m, self.m, n, self.rowptr, self.nnz, colidx=self.colidx)
        return self._plans[n]

    @staticmethod
    def aggregates_first(n_in: int, n_out: int) -> bool:
        return n_out > n_in

    def forward(self, H: torch.Tensor, W: torch.Tensor, bias: Optional[torch.Tensor] = None, relu: bool = True,
                stream: Optional[torch.cuda.Stream] = None) -> torch.Tensor:
        """All of it runs on ``stream`` (default: the current one): what it reads has to be there, as for any call on a stream."""
        n_in, n_out = int(W.shape[0]), int(W.shape[1])
        if H.shape != (self.m, n_in):
            raise ValueError(f"H must be {self.m} x {n_in}")
        if stream is not None:
            self._plan(min(n_in, n_out))  # on the current stream, as the adjacency
            with torch.cuda.stream(stream):
                return self.forward(H, W, bias, relu)
        act = _b.ACT_RELU if relu else _b.ACT_IDENTITY
        if not self.aggregates_first(n_in, n_out):
            if _native_first(self.m, n_in, n_out) and _native_product(H, W, None):
                Z = torch.empty((self.m, n_out), dtype=torch.float32, device=H.device)
                _b.scorch_dense_layer(H, W, None, _b.ACT_IDENTITY, Z)
            else:
                Z = torch.mm(H, W)
            out = torch.empty((self.m, n_out), dtype=torch.float32, device=H.device)
            _b.scorch_spmm_csr_planned_epilogue(self._plan(n_out), self.rowptr, self.colidx, self.vals, Z, bias, act, out)
            return out
        Y = torch.empty((self.m, n_in), dtype=torch.float32, device=H.device)
        _b.scorch_spmm_csr_planned(self._plan(n_in), self.rowptr, self.colidx, self.vals, H, Y)
        # With an activation the dense library makes one more pass over the result (addmm adds the bias inside the product,
        # relu_ runs on what it wrote): one kernel for all three takes 0.15 to 0.85 of the time.  Without one, the product alone
        # takes 0.17 to 1.35 of the library's time, more than all of it on 20 000 to 60 000 rows, so that case stays there.
        if relu and _native_product(Y, W, bias):
            out = torch.empty((self.m, n_out), dtype=torch.float32, device=H.device)
            _b.scorch_dense_layer(Y, W, bias, act, out)
            return out
        out = torch.mm(Y, W) if bias is None else torch.addmm(bias, Y, W)
        return torch.relu_(out) if relu else out

    def close(self) -> None:
        for p in self._plans.values():
            p.destroy()
        self._plans.clear()
