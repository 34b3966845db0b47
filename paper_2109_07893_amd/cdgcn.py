"""Caller-side plumbing for the CD-GCN layer over a block of timesteps, forward and backward (Section "CD-GCN"): per snapshot
the GCN operation with skip connection, then one LSTM step per vertex,

    Y0 = A~_t X_t           dgnn_spmm_batch            Y1 = Y0 W      dgnn_feature_transform
    Y  = relu(Y0 o Y1)      dgnn_concat_relu           (both in one pass where the widths allow: dgnn_transform_concat_relu)
    a  = Y W_x + h W_h + b,  (h, c) <- LSTM cell       dgnn_lstm_series over several timesteps where it has the widths, else
                            two dgnn_feature_transform and dgnn_lstm_cell per timestep

Only the LSTM ties timesteps together: snapshots are rebuilt as a series and the GCN operations of several timesteps enqueued
together while they are small (batch.py).  Buffers and call order only; the arithmetic is in the HIP kernels."""
from __future__ import annotations

from typing import Optional

import torch

from . import binding as B
from .batch import GATHERED_DINV_ROWS, Frames, SpmmTable, TransformTable, pointers, upstream_frames
from .pipeline import BlockInputs, BlockRunner

# Bytes of gate gradients (N x 4 hidden per timestep) that one call of the adjoint leaves for the weight gradients behind it.
GATE_BYTES = 1 << 30


class CdgcnLayer(BlockRunner):
    """Reuses the runner's snapshot slots and rebuilds; `hidden` is the LSTM state width (4 * hidden and
    blk.f + f_out must be feature widths the dense transform takes)."""

    two_stream_safe = False       # the layer's own pass is run(); its buffers do not alternate with t

    def __init__(self, blk: BlockInputs, w: torch.Tensor, w_x: torch.Tensor, w_h: torch.Tensor,
                 bias: Optional[torch.Tensor], hidden: int, fused: bool = True):
        super().__init__(blk, keep_all_z=False)
        if self.series:
            self._widen()
        self.fused = fused            # one-kernel LSTM (and Y) where the library has the widths
        n, f, m = blk.n, blk.f, self.together
        f_out = w.shape[1]
        dt, dev = blk.x[0].dtype, self.dev
        self.w, self.w_x, self.w_h, self.bias, self.hidden, self.f_out = w, w_x, w_h, bias, hidden, f_out
        assert tuple(w_x.shape) == (f + f_out, 4 * hidden) and tuple(w_h.shape) == (hidden, 4 * hidden)
        # the right-hand D^(-1/2) of A~: gathered with the rows of X, or, where the factors no longer fit beside them in the
        # caches, put into the rows by a pass of its own; bf16 rows always the latter, so that one size rounds as the next
        self.prescale = dt == torch.bfloat16 or n > GATHERED_DINV_ROWS
        self.xs = torch.empty((m, n, f), dtype=dt, device=dev) if self.prescale else None
        self.y0_batch = torch.empty((m, n, f), dtype=dt, device=dev)
        self.y_batch = torch.empty((m, n, f + f_out), dtype=dt, device=dev)
        self.y0, self.y = self.y0_batch[0], self.y_batch[0]                     # of the timestep that form_y is asked for
        self.lstm_fused = fused and B.lstm_step_supported(self.y_batch, hidden)
        self.y1 = self.gx = self.gh = None
        if not (fused and B.transform_concat_relu_supported(self.y0_batch[0], f_out)):
            self.y1 = torch.empty((m, n, f_out), dtype=dt, device=dev)
        if not self.lstm_fused:
            self.gx = torch.empty((n, 4 * hidden), dtype=dt, device=dev)
            self.gh = torch.empty((n, 4 * hidden), dtype=dt, device=dev)
        self.c = torch.zeros((n, hidden), dtype=dt, device=dev)
        self.h_all = torch.empty((blk.T, n, hidden), dtype=dt, device=dev)      # h_t for every timestep
        self.h0 = torch.zeros((n, hidden), dtype=dt, device=dev)                # h_0 = c_0 = 0
        self._aggregations = self._aggregation_tables([self.y0_batch[t % m] for t in range(blk.T)])

    def _aggregation_tables(self, y0):
        blk = self.blk
        order = [self.slot_of(t) for t in range(1, blk.T + 1)]
        scaled, b = TransformTable(blk.T), SpmmTable(blk.T)
        dinv = pointers([self.dinv[k] for k in order])
        b.column(b.ROWPTR, pointers([self.rowptr[k] for k in order]))
        b.column(b.COLIDX, pointers([self.colidx[k] for k in order]))
        b.column(b.DINV, dinv)
        b.column(b.Z, pointers(y0))
        self.x_frames = Frames((blk.n, blk.f), blk.x[0].dtype, "x")
        if self.prescale:
            xs = pointers([self.xs[t % self.together] for t in range(blk.T)])
            scaled.column(scaled.SCALE, dinv)
            scaled.column(scaled.H, xs)
            b.column(b.H, xs)
        self.ws_batch = torch.empty(SpmmTable.workspace(self.together, self.cap, blk.f), dtype=torch.uint8, device=self.dev)
        return scaled, b

    def _overrides(self, name: str) -> bool:
        return getattr(type(self), name) is not getattr(CdgcnLayer, name)

    def _series_pays(self) -> bool:
        return super()._series_pays() and not (self._overrides("step") or self._overrides("form_y"))     # ... is asked for every timestep

    def rebuild_all(self) -> None:
        """Every snapshot of the block (where the block is small enough to be rebuilt in one go)."""
        blk, one = self.blk, self.slot_of(1)
        with self._stage("delta_rebuild"):
            self._tables.series.rebuild(blk.n, self.rowptr[one], self.colidx[one], blk.nnz[0], blk.deltas[:blk.T - 1], self.cap,
                                        torch.cuda.current_stream(self.dev).cuda_stream, blk.nnz[1:blk.T])

    def _bind(self) -> None:
        scaled, b = self._aggregations
        x = self.x_frames.addresses(self.blk.x[: self.blk.T])
        b.refresh(b.NNZ, self.blk.nnz[: self.blk.T], self.blk.T)
        if self.prescale:
            scaled.refresh(scaled.X, x, self.blk.T)
        else:
            b.refresh(b.H, x, self.blk.T)

    def gcn_steps(self, t: int, k: int, y0: torch.Tensor, y: torch.Tensor) -> None:
        """Y0 (where the tables say; y0 is that place) and Y of timesteps t .. t + k - 1 (0-based), their snapshots resident."""
        blk = self.blk
        n, f, dt = blk.n, blk.f, B._dtype_code(y)
        stream = torch.cuda.current_stream(self.dev).cuda_stream
        scaled, b = self._aggregations
        if self.prescale:
            with self._stage("row_scale"):
                B.feature_transform_batch(k, scaled.at(t), n, f, f, 0, dt, stream)
        with self._stage("spmm"):
            b.run(n, t, k, f, dt, B.DGNN_H_PRESCALED if self.prescale else 0, self.ws_batch, stream)
        if self._overrides("form_y"):
            self.y0, self.y = y0[0], y[0]
            self.form_y()
        else:
            self._form(k, y0, y)

    def form_y(self) -> None:
        """Y = relu(Y0 o Y0 W) of one timestep from self.y0 into self.y."""
        self._form(1, self.y0, self.y)

    def _form(self, k: int, y0: torch.Tensor, y: torch.Tensor) -> None:
        rows = k * self.blk.n
        y0, y = y0.view(rows, self.blk.f), y.view(rows, self.blk.f + self.f_out)
        if self.y1 is None:
            with self._stage("transform_concat_relu"):
                B.transform_concat_relu(y0, self.w, y)
            return
        y1 = self.y1[:k].view(rows, self.f_out)
        with self._stage("feature_transform"):
            B.feature_transform(y0, self.w, y1)
        with self._stage("concat_relu"):
            B.concat_relu(y0, y1, y)

    def lstm_steps(self, t: int, k: int, y: torch.Tensor, c0: torch.Tensor, c: torch.Tensor) -> None:
        """h of timesteps t .. t + k - 1 from Y [k, n, f + f_out]; c [n, hidden] (the last state) or [k, n, hidden] (every one)."""
        h_prev = self.h0 if t == 0 else self.h_all[t - 1]
        if self.lstm_fused:
            with self._stage("lstm_step"):
                B.lstm_series(y, h_prev, self.w_x, self.w_h, self.bias, c0, c, self.h_all[t:t + k])
            return
        for j in range(k):
            h_prev = self.h0 if t + j == 0 else self.h_all[t + j - 1]
            c_to = c[j] if c.dim() == 3 else c
            with self._stage("feature_transform"):
                B.feature_transform(y[j], self.w_x, self.gx)
                B.feature_transform(h_prev, self.w_h, self.gh)
            with self._stage("lstm_cell"):
                B.lstm_cell(self.gx, self.gh, self.bias, c0, c_to, self.h_all[t + j])
            c0 = c_to

    def _gcn_of_one(self, t: int, y0: torch.Tensor, y: torch.Tensor) -> None:
        """Y0 and Y of timestep t (1-based) recomputed into the first place of the batch buffers."""
        scaled, b = self._aggregations
        kept = b.words[t - 1, b.Z]
        b.words[t - 1, b.Z] = y0.data_ptr()
        self.gcn_steps(t - 1, 1, y0, y)
        b.words[t - 1, b.Z] = kept

    def step(self, t: int) -> None:
        """Timestep t (1-based) alone, its snapshot resident: h_t from h_{t-1}, the state c in place."""
        self._bind()
        y0, y = self.y0_batch[:1], self.y_batch[:1]
        self._gcn_of_one(t, y0, y)
        self.lstm_steps(t - 1, 1, y, self.c, self.c)

    def run(self) -> torch.Tensor:
        """The whole block from the initial state (h, c) = 0; returns h_t for t = 1..T."""
        blk, m = self.blk, self.together
        if self._overrides("step"):
            self.c.zero_()
            for t in range(1, blk.T + 1):
                if t >= 2:
                    self.rebuild(t, blk.deltas[t - 2])
                self.step(t)
            return self.h_all
        self._bind()
        if self.series:
            self.rebuild_all()
        for t in range(0, blk.T, m):
            k = min(m, blk.T - t)
            if t > 0 and not self.series:
                self.rebuild(t + 1, blk.deltas[t - 1])
            self.gcn_steps(t, k, self.y0_batch[:k], self.y_batch[:k])
            self.lstm_steps(t, k, self.y_batch[:k], self.h0 if t == 0 else self.c, self.c)
        return self.h_all


class CdgcnTrainer(CdgcnLayer):
    """Forward and backward over one block for the CD-GCN layer (Section "CD-GCN", trained as in Section "Gradient
    Checkpoint": the forward pass keeps only the LSTM states (h_t, c_t) of every timestep, and Y0 and Y where they are asked
    for; the backward pass walks the timesteps in reverse, recomputing what was not kept):

        a stretch of timesteps, last stretch first:
            (da, dY1, dh, dc) <- adjoint of the LSTM and of Y's ReLU               dgnn_lstm_series_backward
            dW_x += Y^T da, dW_h += h_{t-1}^T da, db += colsum(da)                 dgnn_lstm_weight_grad
            dW += Y0^T dY1                                                         dgnn_weight_grad
        where the adjoint has no kernel for the widths, or dL/dX is wanted, timestep by timestep:
            (da, dc_{t-1}) <- LSTM cell backward of (G_t + dh_t, dc_t)             dgnn_lstm_step_backward or dgnn_lstm_cell_backward
            dW_x, dW_h, db as above                                                dgnn_weight_grad, dgnn_bias_grad
            dY = da W_x^T, dh_{t-1} = da W_h^T                                     dgnn_input_grad
            dY1 = (dY where Y > 0)[:, F:], dW += Y0^T dY1                          dgnn_concat_relu_backward, dgnn_weight_grad

    Gradients with respect to the layer's parameters (fp32): dw, dw_x, dw_h, db.  The input features are leaves."""

    def __init__(self, blk: BlockInputs, w, w_x, w_h, bias, hidden: int, fused: bool = True, keep_activations: bool = False,
                 want_dx: bool = False, transposed_first=None, transposed_deltas=None):
        super().__init__(blk, w, w_x, w_h, bias, hidden, fused)
        # want_dx: also dL/dX_t = A~_t^T (dY0 + dY1 W^T), for a layer that lies below (the paper stacks two of these
        # layers).  For a directed workload that takes the transposed snapshots, a second chain rebuilt from the
        # difference lists sorted by (col, row), handed in as (rowptr, colidx) of A_1^T and one list tuple per step.
        self.want_dx = want_dx
        self.at = None
        n, f, T, m = blk.n, blk.f, blk.T, self.together
        f_out = w.shape[1]
        dt, dev = blk.x[0].dtype, self.dev
        if want_dx:
            from .training import _Chain
            self.dx = torch.empty((T, n, f), dtype=dt, device=dev)
            self.d0 = torch.empty((n, f), dtype=dt, device=dev)
            self.tmp = torch.empty((n, f), dtype=dt, device=dev)
            if transposed_first is not None:
                self.at = _Chain(n, self.cap, dev, transposed_first[0], transposed_first[1], with_dinv=False)
                self.t_deltas = transposed_deltas
        # With keep_activations the forward pass also keeps Y0 and Y of every timestep (N x (2F + F') per step: 6.4 GB
        # at c5's size, a matter of course in 288 GB) and the backward pass neither recomputes the GCN operation
        # nor needs the snapshots again; without, only the LSTM states are kept, as gradient checkpointing has it.
        # Where the batch buffers hold the whole block they are still there without being asked for.
        self.keep = keep_activations or m >= T
        if m >= T:
            self.y0_all, self.y_all = self.y0_batch, self.y_batch
        elif self.keep:
            self.y0_all = torch.empty((T, n, f), dtype=dt, device=dev)
            self.y_all = torch.empty((T, n, f + f_out), dtype=dt, device=dev)
        if self.keep:
            self._aggregations = self._aggregation_tables(list(self.y0_all))
        self.c_all = torch.zeros((T + 1, n, hidden), dtype=dt, device=dev)     # c_0 = 0, c_t after step t
        self.dw = torch.zeros((f, f_out), dtype=torch.float32, device=dev)
        self.dw_x = torch.zeros((f + f_out, 4 * hidden), dtype=torch.float32, device=dev)
        self.dw_h = torch.zeros((hidden, 4 * hidden), dtype=torch.float32, device=dev)
        self.db = torch.zeros(4 * hidden, dtype=torch.float32, device=dev)
        # the adjoint of several timesteps at once: Y1 must be as wide as the state
        self.back_fused = self.lstm_fused and not want_dx and f_out == hidden and B.lstm_series_backward_supported(self.y_batch, hidden)
        if self.back_fused:
            frame = n * 4 * hidden * self.y_batch.element_size()
            self.back_steps = max(1, min(T if self.keep else m, GATE_BYTES // frame))
            self.da = torch.empty((self.back_steps, n, 4 * hidden), dtype=dt, device=dev)
            self.dy1 = torch.empty((self.back_steps, n, f_out), dtype=dt, device=dev)
            self.dh = torch.empty((n, hidden), dtype=torch.float32, device=dev)
            self.dc = torch.empty((n, hidden), dtype=torch.float32, device=dev)
            need = max(B.lstm_weight_grad_workspace(f + f_out, hidden), B.weight_grad_workspace(f, f_out))
        else:
            self.da = torch.empty((n, 4 * hidden), dtype=dt, device=dev)
            self.dy = torch.empty((n, f + f_out), dtype=dt, device=dev)
            self.dy1 = torch.empty((n, f_out), dtype=dt, device=dev)
            self.dh = torch.empty((n, hidden), dtype=dt, device=dev)
            self.dc = torch.empty((n, hidden), dtype=dt, device=dev)
            if self.gx is None and not B.lstm_step_backward_supported(self.y_batch, hidden):
                self.gx = torch.empty((n, 4 * hidden), dtype=dt, device=dev)
                self.gh = torch.empty((n, 4 * hidden), dtype=dt, device=dev)
            need = max(B.weight_grad_workspace(f + f_out, 4 * hidden), B.weight_grad_workspace(hidden, 4 * hidden),
                       B.weight_grad_workspace(f, f_out))
            self.ws_bias = torch.empty(B.bias_grad_workspace(4 * hidden), dtype=torch.uint8, device=dev)
        self.ws_wgrad = torch.empty(need, dtype=torch.uint8, device=dev)

    def _activations(self, t: int, k: int):
        """Y0 and Y of timesteps t .. t + k - 1 (0-based) as they lie when gcn_steps has formed them."""
        return (self.y0_all[t:t + k], self.y_all[t:t + k]) if self.keep else (self.y0_batch[:k], self.y_batch[:k])

    def forward(self) -> torch.Tensor:
        blk, m = self.blk, self.together
        # Where Y of all timesteps is kept, one LSTM over them, whose state then stays on chip between the steps (2^18 vertices, 64 + 32
        # columns fp32, four timesteps: a launch each 1341 us a training step, one for all 1247).  A subclass that has a part of a
        # timestep's work in its own hands meets the states of the timesteps before, and is asked for them in turn.
        whole = self.keep and self.lstm_fused and not any(map(self._overrides, ("gcn_steps", "form_y", "lstm_steps")))
        self._bind()
        if self.series:
            self.rebuild_all()
        for t in range(0, blk.T, m):
            k = min(m, blk.T - t)
            if t > 0 and not self.series:
                self.rebuild(t + 1, blk.deltas[t - 1])
            if self.at is not None:
                for j in range(max(t, 1), t + k):
                    self._rebuild_transposed(j, j + 1, blk.nnz[j - 1], reverse=False)
            y0, y = self._activations(t, k)
            self.gcn_steps(t, k, y0, y)
            if not whole:
                self.lstm_steps(t, k, y, self.c_all[t], self.c_all[t + 1:t + 1 + k])
        if whole:
            self.lstm_steps(0, blk.T, self._activations(0, blk.T)[1], self.c_all[0], self.c_all[1:1 + blk.T])
        return self.h_all

    def _rebuild_transposed(self, src_t: int, dst_t: int, nnz_src: int, reverse: bool) -> None:
        ar, ac, dr, dc = self.t_deltas[max(src_t, dst_t) - 2]
        if reverse:
            ar, ac, dr, dc = dr, dc, ar, ac
        a = self.at
        s, d = a.slot_of(src_t), a.slot_of(dst_t)
        with self._stage("delta_rebuild"):
            B.delta_rebuild(a.rowptr[s], a.colidx[s], nnz_src, ar, ac, int(ar.numel()), dr, dc, int(dr.numel()),
                            a.rowptr[d], a.colidx[d], None, self.ws_rebuild)

    def _rebuild_backwards(self, t: int) -> None:
        """A_{t-1} from A_t: the two lists exchanged (A_1 was kept; a series is resident anyway)."""
        blk = self.blk
        if t < 3 or self.series or (self.keep and not self.want_dx):
            return
        ar, ac, dr, dc = blk.deltas[t - 2]
        src, dst = self.slot_of(t), self.slot_of(t - 1)
        with self._stage("delta_rebuild"):
            B.delta_rebuild(self.rowptr[src], self.colidx[src], blk.nnz[t - 1], dr, dc, int(dr.numel()), ar, ac,
                            int(ar.numel()), self.rowptr[dst], self.colidx[dst], self.dinv[dst], self.ws_rebuild)

    def backward(self, g_h: torch.Tensor) -> None:
        """g_h [T, n, hidden] = dL/dh_t.  Must follow forward() (A_T resident)."""
        g_h = upstream_frames(g_h, self.blk.T, self.blk.n, self.hidden, self.h_all.dtype)
        if self.back_fused:
            self._backward_stretches(g_h)
        else:
            self._backward_steps(g_h)

    def _backward_stretches(self, g_h: torch.Tensor) -> None:
        blk, steps = self.blk, self.back_steps
        T, n = blk.T, blk.n
        last = (T - 1) // steps * steps
        for t in range(last, -1, -steps):
            k = min(steps, T - t)
            y0, y = self._activations(t, k)
            if not self.keep:
                self.gcn_steps(t, k, y0, y)
            h_prev = self.h0 if t == 0 else self.h_all[t - 1]
            h, da, dy1 = self.h_all[t:t + k], self.da[:k], self.dy1[:k]
            with self._stage("lstm_step_backward"):
                B.lstm_series_backward(y, h_prev, h, self.w_x, self.w_h, self.bias, self.c_all[t], self.c_all[t + 1:t + 1 + k], g_h[t:t + k], da,
                                       dy1, self.dh, self.dc, carried=t != last)
            with self._stage("weight_grad"):
                B.lstm_weight_grad(y, h_prev, h, da, self.dw_x, self.dw_h, self.db, self.ws_wgrad, accumulate=t != last)
                B.weight_grad(y0.view(k * n, blk.f), dy1.view(k * n, self.f_out), self.dw, self.ws_wgrad, accumulate=t != last)
            self._rebuild_backwards(t + 1)

    def _backward_steps(self, g_h: torch.Tensor) -> None:
        blk = self.blk
        T = blk.T
        first = True
        for t in range(T, 0, -1):
            y0, y = self._activations(t - 1, 1)
            if not self.keep:
                self._gcn_of_one(t, y0, y)
            y0, y = y0[0], y[0]
            h_prev = self.h0 if t == 1 else self.h_all[t - 2]
            carried = (None, None) if t == T else (self.dh, self.dc)
            if self.fused and B.lstm_step_backward_supported(y, self.hidden):
                with self._stage("lstm_step_backward"):
                    B.lstm_step_backward(y, h_prev, self.w_x, self.w_h, self.bias, self.c_all[t - 1], g_h[t - 1],
                                         carried[0], carried[1], self.da, self.dc)
            else:
                with self._stage("feature_transform"):
                    B.feature_transform(y, self.w_x, self.gx)
                    B.feature_transform(h_prev, self.w_h, self.gh)
                with self._stage("lstm_cell_backward"):
                    B.lstm_cell_backward(self.gx, self.gh, self.bias, self.c_all[t - 1], g_h[t - 1], carried[0], carried[1],
                                         self.da, self.dc)
            with self._stage("weight_grad"):
                B.weight_grad(y, self.da, self.dw_x, self.ws_wgrad, accumulate=not first)
                B.weight_grad(h_prev, self.da, self.dw_h, self.ws_wgrad, accumulate=not first)
            with self._stage("bias_grad"):
                B.bias_grad(self.da, self.db, self.ws_bias, accumulate=not first)
            with self._stage("input_grad"):
                B.input_grad(self.da, self.w_x, self.dy)
                if t >= 2:
                    B.input_grad(self.da, self.w_h, self.dh)
            with self._stage("concat_relu_backward"):
                B.concat_relu_backward(self.dy, y, self.d0 if self.want_dx else None, self.dy1, blk.f)
            with self._stage("weight_grad"):
                B.weight_grad(y0, self.dy1, self.dw, self.ws_wgrad, accumulate=not first)
            if self.want_dx:
                with self._stage("input_grad"):
                    B.input_grad(self.dy1, self.w, self.tmp)
                    B.add(self.d0, self.tmp, self.d0)                           # dY0: its own block and the path through Y1
                with self._stage("spmm_transposed"):
                    slot = self.slot_of(t)
                    rp, ci = (self.rowptr[slot], self.colidx[slot]) if self.at is None else (
                        self.at.rowptr[self.at.slot_of(t)], self.at.colidx[self.at.slot_of(t)])
                    src = self.d0
                    if self.prescale:
                        scaled, src = TransformTable(1), self.tmp
                        scaled.words[0] = (self.d0.data_ptr(), 0, self.dinv[slot].data_ptr(), src.data_ptr())
                        B.feature_transform_batch(1, scaled.at(), blk.n, blk.f, blk.f, 0, B._dtype_code(src),
                                                  torch.cuda.current_stream(self.dev).cuda_stream)
                    B.spmm(rp, ci, blk.nnz[t - 1], self.dinv[slot], src, self.dx[t - 1], self.ws_spmm,
                           flags=B.DGNN_H_PRESCALED if self.prescale else 0)
                if t >= 3 and self.at is not None:
                    self._rebuild_transposed(t, t - 1, blk.nnz[t - 1], reverse=True)
            first = False
            self._rebuild_backwards(t)
