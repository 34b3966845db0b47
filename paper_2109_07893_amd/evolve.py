"""Caller-side plumbing for EvolveGCN's weights (Section "EvolveGCN"): the GCN weight of timestep t comes from the
one before through an LSTM, W_t = LSTM(W_{t-1}).  Reading (the section gives only that line; this is the variant
it names, EGCN-O): the weight matrix is the LSTM's hidden state AND its input, its F rows are the batch, and a cell
state C of the same shape is carried along,

    a_t = W_{t-1} U_x + W_{t-1} U_h + b,    (W_t, C_t) = cell(a_t, C_{t-1})          W_0 given, C_0 = 0.

The matrices are F x F', so the recurrence over all timesteps is one launch (dgnn_evolve_weights) and its adjoint two
(dgnn_evolve_weights_backward).  fp32, F' 16 or 32.  Buffers and calls only."""
from __future__ import annotations

from typing import List

import torch

from . import binding as B


class EvolvingWeights:
    def __init__(self, w0: torch.Tensor, u_x: torch.Tensor, u_h: torch.Tensor, bias: torch.Tensor, T: int):
        f, f2 = w0.shape
        assert w0.dtype == torch.float32 and tuple(u_x.shape) == (f2, 4 * f2) and tuple(u_h.shape) == (f2, 4 * f2)
        dev = w0.device
        self.w0, self.u_x, self.u_h, self.bias, self.T = w0, u_x, u_h, bias, T
        self.w = torch.empty((T, f, f2), device=dev)              # W_1 .. W_T
        self.c = torch.zeros((T + 1, f, f2), device=dev)          # C_0 = 0, C_t
        self.du_x = torch.zeros((f2, 4 * f2), device=dev)
        self.du_h = torch.zeros((f2, 4 * f2), device=dev)
        self.db = torch.zeros(4 * f2, device=dev)
        self.dw0 = torch.empty((f, f2), device=dev)
        self.ws = torch.empty(B.evolve_weights_backward_workspace(f, f2), dtype=torch.uint8, device=dev)
        self.frames = [self.w[t] for t in range(T)]

    def forward(self) -> List[torch.Tensor]:
        """W_1 .. W_T (views of one buffer)."""
        B.evolve_weights(self.w0, self.u_x, self.u_h, self.bias, self.w, self.c)
        return list(self.frames)

    def backward(self, dw_t: List[torch.Tensor]) -> None:
        """dw_t[t-1] = dL/dW_t (fp32, from the GCN steps).  Leaves dL/dU_x, dL/dU_h, dL/db and dL/dW_0."""
        B.evolve_weights_backward(self.w0, self.u_x, self.u_h, self.bias, self.w, self.c, dw_t, self.dw0, self.du_x, self.du_h, self.db, self.ws)
