"""Caller-side plumbing for a training step over one GPU's block of timesteps (Section "Gradient
Checkpoint": a block is run forward, keeping its activations, and gradients then travel through it in
the reverse direction).  Like pipeline.py this owns buffers and the order of library calls only:

    forward    A_2 .. A_T (dgnn_delta_rebuild_series, or dgnn_delta_rebuild per step on large snapshots), then per timestep
                   first layer    P = A~_t X,  Z = relu(P W)                     both kept (fp32)
                   other layers   H = Z_below W,  Z = relu(A~_t H)               Z kept
               then Y = Z x_1 M
    backward   G = G_Y x_1 M^T (dgnn_mproduct_backward_block), then per timestep, last layer to first:
                   other layers   G_P = dinv * (Z > 0 ? G : 0)                   dgnn_relu_backward; for the top layer together with
                                                                                 G (dgnn_mproduct_relu_backward_block)
                                  G_H = A~_t^T G_P                               dgnn_spmm on the transposed snapshot
                                  dW += Z_below^T G_H,  G = G_H W^T              dgnn_weight_grad, dgnn_input_grad
                   first layer    dW += P^T (Z > 0 ? G : 0)                      dgnn_weight_grad_batch

The first layer's weight gradient is X^T A~^T G_P = (A~ X)^T G_P: with A~ X kept from the forward pass it needs no aggregation
and no transposed snapshot, which leaves a one-layer step with half the gathers.  Where dL/dX is wanted (a layer lies below)
the aggregation is needed anyway, and the first layer is treated like the others; so it is where frames are stored in bf16 or
A~ X of the block would take more than AGGREGATED_BYTES (see first_layer_keeps_aggregated).

For a directed workload the transposed snapshots, where needed, are a second dynamic graph, rebuilt the same way from the
difference lists sorted by (col, row).  Timesteps are enqueued together while their frames are small (batch.py).  Nothing here
computes: every step runs in the HIP kernels.
"""
from __future__ import annotations

import contextlib
import weakref
from dataclasses import replace
from typing import List, Optional, Tuple

import torch

from . import binding as B
from .batch import GATHERED_DINV_ROWS, SERIES_ENTRIES, Frames, SeriesTable, SmoothTable, SpmmTable, TransformTable, WeightGradTable, pointers, series_pays, snapshots_fit, steps_together, upstream_frames
from .pipeline import BlockInputs, BlockRunner


class _Chain:
    """CSR slots for a series of snapshots walked forwards or backwards by rebuilds: by default two alternating slots
    plus a kept first snapshot; with `slots` given, one slot per timestep, so that every snapshot of the block stays
    resident and nothing has to be rebuilt on the way back."""

    def __init__(self, n, cap, dev, rowptr1, colidx1, with_dinv: bool, slots: Optional[int] = None):
        self.per_step = slots is not None
        count = slots if self.per_step else 3
        self.rowptr = [torch.empty(n + 1, dtype=torch.int32, device=dev) for _ in range(count)]
        self.colidx = [torch.empty(cap, dtype=torch.int32, device=dev) for _ in range(count)]
        self.dinv_all = torch.empty((count, n), dtype=torch.float32, device=dev) if with_dinv else None
        self.dinv = [self.dinv_all[k] if with_dinv else None for k in range(count)]
        self.load_first(rowptr1, colidx1)

    def load_first(self, rowptr1, colidx1) -> None:
        """The block's first snapshot, which arrives whole, goes into its slot."""
        k = self.slot_of(1)
        self.rowptr[k].copy_(rowptr1)
        self.colidx[k][: colidx1.numel()].copy_(colidx1)
        if self.dinv[k] is not None:
            B.csr_dinv(self.rowptr[k], self.dinv[k])

    def slot_of(self, t: int) -> int:
        if self.per_step:
            return t - 1
        return 2 if t == 1 else t % 2

    def slots_of(self, T: int) -> List[int]:
        return [self.slot_of(t) for t in range(1, T + 1)]


def _stage_of(trainer):
    """trainer._stage for the stack that it owns, which does not own it in turn: a trainer that is let go gives its memory back
    at once and not when the garbage collector comes by."""
    owner = weakref.ref(trainer)
    return lambda name: owner()._stage(name)


class GcnStack:
    """The GCN layers of a training step over T snapshots, forward and backward, from tables of the snapshots' arrays (a
    value per stored entry where `vals` is given); T frames of activations are kept.  What differs between the trainers is
    where the snapshots come from."""

    def __init__(self, blk: BlockInputs, cap: int, rowptr, colidx, dinv, vals=None, transposed=None, want_dx: bool = False,
                 stage=None, together: Optional[int] = None):
        dev, dt = blk.rowptr1.device, blk.x[0].dtype
        n, f, T, L = blk.n, blk.f, blk.T, blk.layers
        self.n, self.f, self.L, self.T_max, self.dev, self.dt = n, f, L, T, dev, B._dtype_code(blk.x[0])
        self.stage, self.want_dx, self.weighted = stage, want_dx, vals is not None
        self.together = m = together or steps_together(n * f * blk.x[0].element_size(), T)
        self.z = torch.empty((L, T, n, f), dtype=dt, device=dev)
        # A~_t X_t, from which the first layer's weight gradient follows without an aggregation
        keep_p0 = first_layer_keeps_aggregated(blk, want_dx, self.weighted)
        self.p0 = torch.empty((T, n, f), dtype=dt, device=dev) if keep_p0 else None
        # rows of X are scaled by dinv in a pass of their own, or dinv is gathered with them (see GATHERED_DINV_ROWS)
        self.prescale = keep_p0 and n > GATHERED_DINV_ROWS
        aggregated = L - 1 if keep_p0 else L                                             # layers that need A~^T going back
        self.needs_transposed = aggregated > 0
        buffers = aggregated > 0 or self.prescale
        self.h = torch.empty((m, n, f), dtype=dt, device=dev) if buffers else None       # H going forward, G_H going back
        self.gp = torch.empty((m, n, f), dtype=dt, device=dev) if aggregated > 0 else None
        self.g_mid = torch.empty((m, n, f), dtype=dt, device=dev) if L > 1 else None
        self.dx = torch.empty((T, n, f), dtype=dt, device=dev) if want_dx else None
        self.ws_spmm = torch.empty(SpmmTable.workspace(m, cap, f), dtype=torch.uint8, device=dev)
        self.ws_wgrad = torch.empty(B.weight_grad_workspace(f, f), dtype=torch.uint8, device=dev)
        self.x, self.w = Frames((n, f), dt, "x"), [Frames((f, f), dt, "w") for _ in range(L)]

        h = pointers([self.h[t % m] for t in range(T)]) if buffers else None
        z = [pointers(self.z[layer]) for layer in range(L)]
        p0 = pointers(self.p0) if self.p0 is not None else None
        snapshot = (pointers(rowptr), pointers(colidx), pointers(dinv), pointers(vals) if vals is not None else 0)

        def spmm_table(arrays, src, dst):
            b = SpmmTable(T)
            for k, col in enumerate(arrays):
                b.column(k, col)
            b.column(b.H, src)
            b.column(b.Z, dst)
            return b
        self.transform, self.spmm = [], []
        self.scaled = None
        for layer in range(L):
            a = TransformTable(T)
            if layer == 0 and self.p0 is not None:
                if self.prescale:
                    self.scaled = TransformTable(T)
                    self.scaled.column(a.SCALE, snapshot[2])
                    self.scaled.column(a.H, h)
                a.column(a.X, p0)
                a.column(a.H, z[0])
                self.spmm.append(spmm_table(snapshot, h if self.prescale else 0, p0))
            else:
                if layer > 0:
                    a.column(a.X, z[layer - 1])
                a.column(a.SCALE, snapshot[2])
                a.column(a.H, h)
                self.spmm.append(spmm_table(snapshot, h, z[layer]))
            self.transform.append(a)
        self.spmm_t = self.spmm_top = None
        if aggregated > 0:
            rp_t, ci_t, val_t = transposed if transposed is not None else (rowptr, colidx, vals)
            arrays = (pointers(rp_t), pointers(ci_t), snapshot[2], pointers(val_t) if val_t is not None else 0)
            self.spmm_t = spmm_table(arrays, pointers([self.gp[t % m] for t in range(T)]), h)
            # the top layer's, where its G_P is formed with the M-transform's adjoint; the frames are named going back
            self.spmm_top = spmm_table(arrays, 0, h) if blk.window else None
            self.input = TransformTable(T)                  # with one weight per timestep: G_H W_t^T
            self.input.column(TransformTable.X, h)
        self.wgrad = WeightGradTable(T)

    def bind(self, blk: BlockInputs, nnz) -> None:
        """The frames, weights and entry counts of the coming pass."""
        T = blk.T
        for b in self.spmm + [b for b in (self.spmm_t, self.spmm_top) if b is not None]:
            b.refresh(b.NNZ, nnz[:T], T)
        x = self.x.addresses(blk.x[:T])
        if self.p0 is None:
            self.transform[0].refresh(TransformTable.X, x, T)
        elif self.prescale:
            self.scaled.refresh(TransformTable.X, x, T)
        else:
            self.spmm[0].refresh(SpmmTable.H, x, T)
        for layer in range(self.L):
            w = self.w[layer].addresses([w[layer] for w in blk.w_t[:T]] if blk.w_t is not None else [blk.w[layer]])
            self.transform[layer].refresh(TransformTable.W, w, T)

    def forward(self, t: int, k: int, stream) -> None:
        """All layers of timesteps t .. t + k - 1 (0-based), their snapshots resident."""
        n, f, dt = self.n, self.f, self.dt
        for layer in range(self.L):
            first = layer == 0 and self.p0 is not None
            if first and self.prescale:
                with self.stage("feature_transform"):
                    B.feature_transform_batch(k, self.scaled.at(t), n, f, f, 0, dt, stream)
            if not first:
                with self.stage("feature_transform"):
                    B.feature_transform_batch(k, self.transform[layer].at(t), n, f, f, 0, dt, stream)
            flags = (0 if first else B.DGNN_RELU) | (0 if first and not self.prescale else B.DGNN_H_PRESCALED)
            with self.stage("spmm_weighted" if self.weighted else "spmm"):
                self.spmm[layer].run(n, t, k, f, dt, flags, self.ws_spmm, stream)
            if first:
                with self.stage("feature_transform"):
                    B.feature_transform_batch(k, self.transform[0].at(t), n, f, f, B.DGNN_RELU, dt, stream)

    def steps_back(self, dw_t, T: int) -> int:
        """Timesteps that backward takes at a time: with one layer, one weight and nothing to aggregate the rows of all of them
        in one product."""
        whole = not self.needs_transposed and dw_t is None and T * self.n < (1 << 31) - 65536
        return T if whole else self.together

    def _weight_grad(self, blk, t, k, layer, x, g, masked, dw, dw_t, accumulate, stream) -> None:
        n, f, dt, a = self.n, self.f, self.dt, self.wgrad
        with self.stage("weight_grad"):
            if dw_t is None:                       # one weight for all timesteps: one product over all their rows
                a.words[0] = (x.data_ptr(), g.data_ptr(), self.z[layer, t].data_ptr() if masked else 0, dw[layer].data_ptr())
                B.weight_grad_batch(1, a.at(), k * n, f, f, accumulate, dt, self.ws_wgrad, stream)
            else:
                step = n * f * x.element_size()
                for j in range(k):
                    a.words[j] = (x.data_ptr() + j * step if x.dim() == 3 else 0, g.data_ptr() + j * step,
                                  self.z[layer, t + j].data_ptr() if masked else 0, dw_t[t + j][layer].data_ptr())
                B.weight_grad_batch(k, a.at(), n, f, f, False, dt, self.ws_wgrad, stream)

    def masks_ahead(self, blk: BlockInputs, per_step: bool) -> bool:
        """Whether the M-transform's adjoint forms the top layer's G_P: the block of this pass has one, that layer's gradient goes
        through an aggregation, and the normalisations of all timesteps are there."""
        return bool(blk.window) and self.spmm_top is not None and per_step

    def backward(self, blk: BlockInputs, t: int, k: int, g_top: torch.Tensor, dinv: torch.Tensor, dw, dw_t, accumulate: bool, stream,
                 masked: bool = False) -> None:
        """Gradients of timesteps t .. t + k - 1; g_top [k, n, f] = dL/dZ of the last layer (masked: its G_P), dinv [k, n]."""
        n, f, dt = self.n, self.f, self.dt
        flat = (k * n, f)
        g = g_top
        for layer in range(self.L - 1, -1, -1):
            if layer == 0 and self.p0 is not None:
                self._weight_grad(blk, t, k, 0, self.p0[t:t + k], g, True, dw, dw_t, accumulate, stream)
                return
            table = self.spmm_t
            if masked and layer == self.L - 1:
                table = self.spmm_top
                table.column(table.H, pointers(g), slice(t, t + k))
            else:
                with self.stage("relu_backward"):
                    B.relu_backward(g.view(flat), self.z[layer, t:t + k].view(flat), self.gp[:k].view(flat), row_scale=dinv.view(-1))
            with self.stage("spmm_weighted_transposed" if self.weighted else "spmm_transposed"):
                table.run(n, t, k, f, dt, B.DGNN_H_PRESCALED, self.ws_spmm, stream)
            if layer > 0:
                self._weight_grad(blk, t, k, layer, self.z[layer - 1, t:t + k], self.h, False, dw, dw_t, accumulate, stream)
            elif dw_t is not None:
                # A call per timestep, each spread over the whole device: side by side in one launch the sums of a wavefront are k times
                # as long (12 x 60 K x 128, error against 64 bits: fp32 2.0e-7 / 6.8e-7, bf16 0.7e-7 / 2.2e-7)
                for j in range(k - 1, -1, -1):
                    with self.stage("weight_grad"):
                        B.weight_grad(blk.x[t + j], self.h[j], dw_t[t + j][0], self.ws_wgrad)
            else:                                  # the frames of X are tensors of their own, added up from the last one on
                B._need(dw[0], torch.float32, "dw")
                if dw[0].shape != (f, f):
                    raise ValueError("shape mismatch in weight_grad")
                a, h, down = self.wgrad, self.h, range(k - 1, -1, -1)
                a.words[:k, a.X] = self.x.addresses([blk.x[t + j] for j in down])
                a.words[:k, a.G] = pointers([h[j] for j in down])
                a.words[:k, a.Z] = 0
                a.words[:k, a.DW] = B._ptr(dw[0])
                with self.stage("weight_grad"):
                    B.weight_grad_batch(k, a.at(), n, f, f, accumulate, dt, self.ws_wgrad, stream)
            if layer == 0 and not self.want_dx:
                return
            dst = self.g_mid[:k] if layer > 0 else self.dx[t:t + k]
            with self.stage("input_grad"):
                if blk.w_t is None:
                    B.input_grad(self.h[:k].view(flat), blk.w[layer], dst.view(flat))
                else:
                    rows = slice(t, t + k)
                    self.input.column(TransformTable.W, self.transform[layer].words[rows, TransformTable.W], rows)
                    self.input.column(TransformTable.H, pointers(dst), rows)
                    B.feature_transform_batch(k, self.input.at(t), n, f, f, B.DGNN_W_TRANSPOSED, dt, stream)
            g = dst


class BlockTrainer:
    """Forward and backward over one block; gradients of the layer weights (fp32) come out in `dw`."""

    def __init__(self, blk: BlockInputs, directed: bool,
                 transposed_first: Optional[Tuple[torch.Tensor, torch.Tensor]] = None,
                 transposed_deltas: Optional[List[Tuple[torch.Tensor, ...]]] = None, want_dx: bool = False,
                 cap: Optional[int] = None, max_list: Optional[int] = None, keep_snapshots: bool = False):
        self.blk = blk
        dev = blk.rowptr1.device
        self.dev = dev
        n, f, T, L = blk.n, blk.f, blk.T, blk.layers
        dt = blk.x[0].dtype
        cap = max(max(blk.nnz), cap or 0)          # room for the densest snapshot this trainer will ever hold
        self.cap, self.T_max = cap, T
        self.t0 = 0                     # timesteps of the series before this block
        self.z_before = None            # last w-1 frames of the top layer's Z before this block
        self.directed = directed
        # keep_snapshots: every A_t (and A_t^T) of the block stays resident (T index arrays instead of three), so the
        # backward pass rebuilds nothing; without, the snapshots are rebuilt in reverse, as gradient checkpointing
        # has it.  4 nnz bytes per snapshot and chain: 9.6 GB for c5's eight, a matter of course in 288 GB.
        self.series = cap <= SERIES_ENTRIES and series_pays(T, cap) and snapshots_fit(T, n, cap)     # all snapshots in one go: they are resident then in any case
        self.keep_snapshots = keep_snapshots or self.series
        slots = T if self.keep_snapshots else None
        self.a = _Chain(n, cap, dev, blk.rowptr1, blk.colidx1, with_dinv=True, slots=slots)
        self.at = None
        if directed and needs_transposed(blk, want_dx):
            assert transposed_first is not None and transposed_deltas is not None
            self.at = _Chain(n, cap, dev, transposed_first[0], transposed_first[1], with_dinv=False, slots=slots)
            self.t_deltas = transposed_deltas
        self.timer = None
        arrays = [[side[k] for k in self.a.slots_of(T)] for side in (self.a.rowptr, self.a.colidx, self.a.dinv)]
        back = None if self.at is None else ([self.at.rowptr[k] for k in self.at.slots_of(T)], [self.at.colidx[k] for k in self.at.slots_of(T)], None)
        self.stack = GcnStack(blk, cap, *arrays, transposed=back, want_dx=want_dx, stage=_stage_of(self), together=None if self.series else 1)
        self.z, self.dx = self.stack.z, self.stack.dx                     # activations of the block
        self.y = torch.empty((T, n, f), dtype=dt, device=dev) if blk.window else None
        # dL/dZ of the last layer, if g_y must be kept, and wherever it is; where a pass masks ahead (GcnStack.masks_ahead) it is not
        # formed on its own, and G_P is what there is
        self.g = self.g_top = self.g_p = None
        self.dw = [torch.zeros((f, f), dtype=torch.float32, device=dev) for _ in range(L)]
        # with one weight per timestep (Section "EvolveGCN") every timestep has a gradient of its own
        self.dw_t = ([[torch.zeros((f, f), dtype=torch.float32, device=dev) for _ in range(L)] for _ in range(T)]
                     if blk.w_t is not None else None)
        max_list = max([int(d[0].numel()) for d in blk.deltas] + [int(d[2].numel()) for d in blk.deltas] + [1, max_list or 0])
        self.ws_rebuild = torch.empty(B.delta_rebuild_workspace(n, cap, max_list, max_list), dtype=torch.uint8, device=dev)
        self.tables = None
        if self.series:
            def table(chain):          # one step more than the block has: the next block's first snapshot (see forward)
                return SeriesTable(chain.rowptr[1:] + chain.rowptr[:1], chain.colidx[1:] + chain.colidx[:1], chain.dinv[1:] + chain.dinv[:1])
            self.tables = [(self.a, table(self.a))] + ([(self.at, table(self.at))] if self.at is not None else [])
            for (_, tb), (_, lists, _) in zip(self.tables, self._chains()):
                tb.prepare(lists, blk.nnz[0], dev)

    def rebind(self, blk: BlockInputs, t0: int = 0, z_before: Optional[torch.Tensor] = None,
               transposed_first=None, transposed_deltas=None) -> None:
        """Point the same buffers at another block of the same series (not longer, not denser than the first)."""
        assert blk.T <= self.T_max and max(blk.nnz) <= self.cap and blk.n == self.blk.n and blk.f == self.blk.f
        self.blk, self.t0, self.z_before = blk, t0, z_before
        self.a.load_first(blk.rowptr1, blk.colidx1)
        if self.at is not None:
            self.at.load_first(*transposed_first)
            self.t_deltas = transposed_deltas

    def _stage(self, name):
        return self.timer.stage(name) if self.timer is not None else contextlib.nullcontext()

    def _rebuild(self, chain: _Chain, lists, nnz_src: int, src_t: int, dst_t: int, reverse: bool) -> None:
        ar, ac, dr, dc = lists
        if reverse:
            ar, ac, dr, dc = dr, dc, ar, ac
        s, d = chain.slot_of(src_t), chain.slot_of(dst_t)
        with self._stage("delta_rebuild"):
            B.delta_rebuild(chain.rowptr[s], chain.colidx[s], nnz_src, ar, ac, int(ar.numel()), dr, dc, int(dr.numel()),
                            chain.rowptr[d], chain.colidx[d], chain.dinv[d], self.ws_rebuild)

    def _chains(self, after=None):
        """(chain, difference lists of the block's steps, what follows: (lists, rowptr, colidx) or None)."""
        steps = self.blk.T - 1
        out = [(self.a, self.blk.deltas[:steps], after[0] if after is not None else None)]
        if self.at is not None:
            out.append((self.at, self.t_deltas[:steps], after[1] if after is not None else None))
        return out

    # ------------------------------------------------------------------ forward, keeping activations
    def forward(self, after=None, mix: bool = True) -> torch.Tensor:
        """`after`: the snapshot behind the block is wanted too, [(lists, rowptr, colidx)] for A and, where a transposed
        chain is kept, for A^T.  Without `mix` the pass ends with the top layer's frames, which is all that backward() takes."""
        blk, stack = self.blk, self.stack
        stream = torch.cuda.current_stream(self.dev).cuda_stream
        if self.series:
            for (chain, table), (_, lists, extra) in zip(self.tables, self._chains(after)):
                steps = len(lists)
                if extra is not None:                      # behind a block of full length only: the table's last row
                    assert steps == self.T_max - 1
                    lists = list(lists) + [extra[0]]
                    table.column(6, extra[1].data_ptr(), steps)
                    table.column(7, extra[2].data_ptr(), steps)
                    table.column(8, 0, steps)
                if lists:
                    with self._stage("delta_rebuild"):
                        table.rebuild(blk.n, chain.rowptr[0], chain.colidx[0], blk.nnz[0], lists, self.cap, stream, blk.nnz[1:])
        stack.bind(blk, blk.nnz)
        m = stack.together
        for t in range(0, blk.T, m):
            if not self.series and t > 0:
                for chain, lists, _ in self._chains():
                    self._rebuild(chain, lists[t - 1], blk.nnz[t - 1], t, t + 1, reverse=False)
            stack.forward(t, min(m, blk.T - t), stream)
        if not self.series and after is not None:
            for chain, _, (lists, rowptr, colidx) in self._chains(after):
                slot = chain.slot_of(blk.T)
                ar, ac, dr, dc = lists
                with self._stage("delta_rebuild"):
                    B.delta_rebuild(chain.rowptr[slot], chain.colidx[slot], blk.nnz[-1], ar, ac, int(ar.numel()), dr, dc, int(dr.numel()),
                                    rowptr, colidx, None, self.ws_rebuild)
        top = self.z[blk.layers - 1, : blk.T]
        if blk.window and mix:
            with self._stage("mproduct"):
                B.mproduct_block(top, self.y[: blk.T], blk.window, self.t0, z_before=self.z_before)
            return self.y[: blk.T]
        return top

    # ------------------------------------------------------------------ backward
    def backward(self, g_y: torch.Tensor, overwrite: bool = False, g_after: Optional[torch.Tensor] = None,
                 accumulate: bool = False) -> None:
        """g_y [T, n, f] = dL/dY.  Must follow forward() (A_T and, where needed, A_T^T are resident).
        With overwrite the adjoint of the M-transform is taken in place, on g_y itself; g_after = upstream
        gradient of the (up to w-1) timesteps after this block; accumulate adds to dw instead of replacing it."""
        blk, stack = self.blk, self.stack
        T = blk.T
        g_y = upstream_frames(g_y, T, blk.n, blk.f, self.z.dtype, blk.window)
        stream = torch.cuda.current_stream(self.dev).cuda_stream
        masked = not overwrite and stack.masks_ahead(blk, self.a.per_step)
        if masked:
            if self.g_p is None:
                self.g_p = torch.empty((self.T_max,) + tuple(g_y.shape[1:]), dtype=g_y.dtype, device=g_y.device)
            g_top = self.g_p[:T]
            with self._stage("mproduct_relu_backward"):
                B.mproduct_relu_backward_block(g_y, self.z[blk.layers - 1, :T], self.a.dinv_all[:T], g_top, blk.window, self.t0, g_after=g_after)
        elif blk.window:
            if overwrite:
                g_top = g_y
            else:
                if self.g is None:
                    self.g = torch.empty((self.T_max,) + tuple(g_y.shape[1:]), dtype=g_y.dtype, device=g_y.device)
                g_top = self.g[:T]
            with self._stage("mproduct_backward"):
                B.mproduct_backward_block(g_y, g_top, blk.window, self.t0, g_after=g_after)
        else:
            g_top = g_y
        self.g_top = None if masked else g_top
        m = stack.steps_back(self.dw_t, T)
        last = (T - 1) // m * m
        for t in range(last, -1, -m):
            k = min(m, T - t)
            slot = self.a.slot_of(t + 1)
            stack.backward(blk, t, k, g_top[t:t + k], self.a.dinv_all[slot:slot + k] if self.a.per_step else self.a.dinv_all[slot:slot + 1],
                           self.dw, self.dw_t, accumulate or t != last, stream, masked)
            if stack.needs_transposed and t >= 2 and not self.keep_snapshots:   # A_{t-1} from A_t: the lists exchanged (A_1 was kept)
                for chain, lists, _ in self._chains():
                    self._rebuild(chain, lists[t - 1], blk.nnz[t], t + 1, t, reverse=True)


    @property
    def h(self) -> torch.Tensor:
        """The first layer's G_H = A~_1^T G_P of the block's first timestep, the last one that backward() takes.  Where the step
        aggregates this gradient itself it is still in the buffer; where it does not (see above) this inspection does."""
        if self.stack.p0 is None:
            return self.stack.h[0]
        blk, slot = self.blk, self.a.slot_of(1)
        assert self.g_top is not None, "after backward()"
        g = self.g_top[0] if blk.layers == 1 else self.stack.g_mid[0]       # dL/dZ of the first layer and timestep
        rowptr, colidx, dinv = self.a.rowptr[slot], self.a.colidx[slot], self.a.dinv[slot]
        if self.directed:
            rowptr, colidx = B.csr_transpose(rowptr, colidx, blk.nnz[0])
        g_p, g_h = torch.empty_like(g), torch.empty_like(g)
        B.relu_backward(g, self.z[0, 0], g_p, row_scale=dinv)
        ws = torch.empty(B.spmm_workspace(blk.n, blk.nnz[0], blk.f), dtype=torch.uint8, device=self.dev)
        B.spmm(rowptr, colidx, blk.nnz[0], dinv, g_p, g_h, ws, flags=B.DGNN_H_PRESCALED)
        return g_h


# Bytes of A~ X over the timesteps of a block up to which it is kept.  It comes on top of what the step holds in any case (X, Z of
# every layer, Y and the gradients, layers + 4 tensors of the same size at most); a block that fills the device's 288 GB without
# it is to fit as well, and aggregates again on the way back.
AGGREGATED_BYTES = 16 << 30


def first_layer_keeps_aggregated(blk: BlockInputs, want_dx: bool = False, weighted: bool = False) -> bool:
    """Whether the first layer is evaluated as relu((A~ X) W) with A~ X kept, so that its weight gradient needs no aggregation.
    Only in fp32: a bf16 A~ X is rounded once per row before the product and the ReLU see it, where the roundings of X W average
    out over a row's neighbours (features that are all positive, 16 neighbours: dW 1.6 to 3.2 times as far from 64 bits).  In fp32
    both forms are at the rounding of the type: Z 1.1e-7 to 2.2e-7 either way with N(0, 1) features, 1.0e-7 to 2.2e-7 against
    0.8e-7 to 1.7e-7 with positive ones; dW 0.6e-7 to 0.9e-7 against 0.5e-7 to 1.0e-7, where no ReLU's mask differs.
    And not with values and further layers above, where the transposed snapshots are resident anyway."""
    fits = blk.T * blk.n * blk.f * 4 <= AGGREGATED_BYTES
    return blk.x[0].dtype == torch.float32 and fits and not want_dx and not (weighted and blk.layers > 1)


def needs_transposed(blk: BlockInputs, want_dx: bool = False, weighted: bool = False) -> bool:
    """Whether gradients travel through an aggregation at all."""
    return blk.layers > 1 or not first_layer_keeps_aggregated(blk, want_dx, weighted)


def capture_training_step(tr: "BlockTrainer", g_y: torch.Tensor) -> "torch.cuda.CUDAGraph":
    """One training step (forward keeping activations, then backward for the upstream gradient g_y) recorded as a HIP
    graph: every library call on the way only enqueues kernels, so the step is capturable, and replaying it costs one
    launch instead of one per kernel, which is what bounds small workloads.  The step is run once eagerly first, so
    that one-time host-side set-up inside the library is not part of the recording.  Replays read g_y and the block's
    inputs where they lie and leave the gradients in tr.dw."""
    tr.forward()
    tr.backward(g_y)
    torch.cuda.synchronize(tr.dev)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tr.forward()
        tr.backward(g_y)
    return graph


def transposed_inputs(blk: BlockInputs):
    """(rowptr, colidx) of A_1^T and the difference lists of the transposed series (dgnn_csr_transpose,
    dgnn_coo_transpose: input formatting, once per block)."""
    n = blk.n
    first = B.csr_transpose(blk.rowptr1, blk.colidx1, blk.nnz[0])
    return first, [B.coo_transpose(n, ar, ac) + B.coo_transpose(n, dr, dc) for ar, ac, dr, dc in blk.deltas]


def make_smoothed_trainer(wl, blk: BlockInputs, life: int) -> "SmoothedTrainer":
    directed = wl.graph != "er"
    if not directed or not needs_transposed(blk, weighted=True):
        return SmoothedTrainer(blk, life, directed)
    first, deltas = transposed_inputs(blk)
    return SmoothedTrainer(blk, life, True, transposed_first=first, transposed_deltas=deltas)


def make_trainer(wl, blk: BlockInputs, want_dx: bool = False, keep_snapshots: bool = False) -> BlockTrainer:
    """Trainer for a block; for a directed workload the transposed first snapshot and lists are prepared here."""
    directed = wl.graph != "er"
    if not directed or not needs_transposed(blk, want_dx):
        return BlockTrainer(blk, directed, want_dx=want_dx, keep_snapshots=keep_snapshots)
    first, t_deltas = transposed_inputs(blk)
    return BlockTrainer(blk, True, transposed_first=first, transposed_deltas=t_deltas, want_dx=want_dx,
                        keep_snapshots=keep_snapshots)


class CheckpointedTrainer:
    """The paper's gradient checkpointing over a series of T timesteps cut into blocks (Section "Gradient
    Checkpoint"): a forward pass block by block that keeps only what the next block needs (the last w - 1 frames
    of Z; here also each block's first snapshot, which the paper sends whole), then, from the last block to the
    first, a rerun of the block's forward pass followed by its backward pass.  Activations of one block at a
    time are resident."""

    def __init__(self, wl, series: BlockInputs, bsize: int):
        self.series, self.bsize = series, bsize
        self.directed = wl.graph != "er"
        T = series.T
        self.bounds = [(a, min(a + bsize, T)) for a in range(0, T, bsize)]
        dev = series.rowptr1.device
        # first snapshot of every block: block 0 has it, the others are filled in by the forward pass
        self.first = [(series.rowptr1, series.colidx1)] + [
            (torch.empty_like(series.rowptr1), torch.empty(max(series.nnz), dtype=torch.int32, device=dev))
            for a, _ in self.bounds[1:]]
        self.t_first, self.t_deltas = None, None
        if self.directed and needs_transposed(replace(series, T=self.bounds[0][1])):
            (rp_t, tc), self.t_deltas = transposed_inputs(series)
            self.t_first = [(rp_t, tc)] + [(torch.empty_like(rp_t), torch.empty(max(series.nnz), dtype=torch.int32, device=dev))
                                           for a, _ in self.bounds[1:]]
        self.pi: List[Optional[torch.Tensor]] = [None] * len(self.bounds)   # frames handed to block b
        self.resident: Optional[int] = None                                 # the block whose activations the trainer holds
        longest_list = max([int(d[0].numel()) for d in series.deltas] + [int(d[2].numel()) for d in series.deltas] + [1])
        self.trainer = BlockTrainer(self._block(0), self.directed,       # block 0 is as long as any
                                    transposed_first=self.t_first[0] if self.t_first is not None else None,
                                    transposed_deltas=self._t_deltas(*self.bounds[0]),
                                    cap=max(series.nnz), max_list=longest_list)
        self.dw = self.trainer.dw

    def _block(self, b: int) -> BlockInputs:
        s = self.series
        a, e = self.bounds[b]
        nnz = list(s.nnz[a:e])
        blk = BlockInputs(n=s.n, T=e - a, f=s.f, layers=s.layers, window=s.window, rowptr1=self.first[b][0],
                          colidx1=self.first[b][1][: nnz[0]], deltas=s.deltas[a:e - 1], x=s.x[a:e], w=s.w,
                          w_t=s.w_t[a:e] if s.w_t is not None else None, nnz=nnz)
        return blk

    def _t_deltas(self, a: int, e: int):
        return self.t_deltas[a:e - 1] if self.t_deltas is not None else None

    def _bind(self, b: int) -> None:
        a, e = self.bounds[b]
        t_first = None if self.t_first is None else (self.t_first[b][0], self.t_first[b][1][: self.series.nnz[a]])
        self.trainer.rebind(self._block(b), t0=a, z_before=self.pi[b], transposed_first=t_first, transposed_deltas=self._t_deltas(a, e))

    def forward(self, on_block=None) -> None:
        """Block by block; on_block(b, a, e, y) sees the block's output frames before they are overwritten."""
        s, tr = self.series, self.trainer
        w1 = max(s.window - 1, 0)
        for b, (a, e) in enumerate(self.bounds):
            self._bind(b)
            after = None
            if b + 1 < len(self.bounds):          # the next block's first snapshot (the paper sends it whole; here it is one more rebuild)
                after = [(s.deltas[e - 1],) + self.first[b + 1]]
                if self.t_first is not None:
                    after.append((self.t_deltas[e - 1],) + self.t_first[b + 1])
            y = tr.forward(after)
            if on_block is not None:
                on_block(b, a, e, y)
            if b + 1 < len(self.bounds) and w1:
                top = tr.z[s.layers - 1, : e - a]
                keep = min(w1, e)                       # frames of the series so far that the window reaches
                own = top[max(e - a - keep, 0):]
                if own.shape[0] < keep:                 # a block shorter than the window: older frames come along
                    own = torch.cat([self.pi[b][-(keep - own.shape[0]):], own])
                self.pi[b + 1] = own.clone()
        self.resident = len(self.bounds) - 1

    def backward(self, g_y: torch.Tensor) -> None:
        """g_y [T, n, f] for the whole series.  Must follow forward()."""
        s, tr = self.series, self.trainer
        w1 = max(s.window - 1, 0)
        last = len(self.bounds) - 1
        for b in range(last, -1, -1):
            a, e = self.bounds[b]
            if self.resident != b:                      # the last block's activations are still there from the forward pass
                self._bind(b)
                # the rerun: of the M-transform's frames nothing goes back (24 x 60 K x 128 bf16 in blocks of 12: 68 us of 2300)
                tr.forward(mix=False)
            self.resident = None
            after = g_y[e:min(e + w1, s.T)] if (w1 and e < s.T) else None
            tr.backward(g_y[a:e], g_after=after, accumulate=b != last)


class _Ring:
    """`slots` CSR slots used in turn by the raw snapshots A_1, A_2, ...: A_{t-life} is still resident when A_t is."""

    def __init__(self, n, cap, dev, slots: int, with_dinv: bool):
        self.slots = slots
        self.rowptr = [torch.empty(n + 1, dtype=torch.int32, device=dev) for _ in range(slots)]
        self.colidx = [torch.empty(cap, dtype=torch.int32, device=dev) for _ in range(slots)]
        self.dinv = [torch.empty(n, dtype=torch.float32, device=dev) if with_dinv else None for _ in range(slots)]

    def slot_of(self, t: int) -> int:
        return t % self.slots

    def load_first(self, rowptr1, colidx1) -> None:
        s = self.slot_of(1)
        self.rowptr[s].copy_(rowptr1)
        self.colidx[s][: colidx1.numel()].copy_(colidx1)

    def snapshot(self, t: int, nnz: int):
        s = self.slot_of(t)
        return self.rowptr[s], self.colidx[s], nnz


class SmoothedTrainer:
    """A training step on SMOOTHED snapshots (Section "Smoothening the Input Graphs": the graphs TM-GCN and EvolveGCN
    are trained on), with the smoothing done on the device: every S_t and its normalisation by dgnn_smooth_series, or, for
    series longer than one such call takes, the raw A_t by dgnn_delta_rebuild, S_t = S_{t-1} + A_t - A_{t-life} by
    dgnn_csr_combine and its normalisation by dgnn_csr_weighted_dinv.  The layers are those of BlockTrainer with the counts as
    values.  Every S_t stays resident (index and value arrays of all T smoothed snapshots: 21 GB at c5's size; and as many
    again for the transposed ones, where a directed workload has more than one layer), so the backward pass needs no graph
    work at all.  Buffers and call order only."""

    def __init__(self, blk: BlockInputs, life: int, directed: bool,
                 transposed_first: Optional[Tuple[torch.Tensor, torch.Tensor]] = None,
                 transposed_deltas: Optional[List[Tuple[torch.Tensor, ...]]] = None, diag_value: float = 1.0):
        self.blk, self.life, self.directed = blk, life, directed
        # edge-life smoothing acts on A; Eqn (1) then adds the self loop once: the stored diagonal stays 1 (0.0 here
        # leaves the summed diagonal min(life, t), which is the M-transform of the adjacency tensor instead)
        self.diag_value = diag_value
        dev = blk.rowptr1.device
        self.dev = dev
        n, f, T, L = blk.n, blk.f, blk.T, blk.layers
        dt = blk.x[0].dtype
        cap = max(blk.nnz)
        max_del = max([int(d[2].numel()) for d in blk.deltas] + [0])
        max_list = max([int(d[0].numel()) for d in blk.deltas] + [max_del, 1])
        self.cap_s = cap + life * max_del                  # the window's union: A_t and what the window's steps deleted
        self.series = T - 1 <= B.DGNN_SERIES_STEPS and life <= 32 and blk.nnz[0] > 0
        transposed = directed and needs_transposed(blk, weighted=True)
        if transposed:
            assert transposed_first is not None and transposed_deltas is not None
        self.t_first, self.t_deltas = transposed_first, transposed_deltas
        ones = torch.ones(cap, dtype=torch.float32, device=dev)              # S_1 = A_1, every entry counted once

        def smoothed():                                    # S_1's arrays are filled anew for every pass, as A_1 may lie elsewhere then
            return [(torch.empty(n + 1, dtype=torch.int32, device=dev), torch.empty(cap, dtype=torch.int32, device=dev), ones)] + [
                (torch.empty(n + 1, dtype=torch.int32, device=dev), torch.empty(self.cap_s, dtype=torch.int32, device=dev),
                 torch.empty(self.cap_s, dtype=torch.float32, device=dev)) for _ in range(T - 1)]
        self.s = smoothed()
        self.st = smoothed() if transposed else self.s
        # what the calls that take S_t are told about its size: an upper bound (the count is its last row pointer)
        self.s_nnz = [blk.nnz[0]] + [self.cap_s] * (T - 1)
        self.dinv_s = torch.empty((T, n), dtype=torch.float32, device=dev)
        self.timer = None
        arrays = [[s[k] for s in self.s] for k in range(3)]
        back = [[s[k] for s in self.st] for k in range(3)] if transposed else None
        self.stack = GcnStack(blk, max(self.cap_s, blk.nnz[0]), arrays[0], arrays[1], self.dinv_s, vals=arrays[2], transposed=back, stage=_stage_of(self))
        self.z = self.stack.z
        self.y = torch.empty((T, n, f), dtype=dt, device=dev) if blk.window else None
        self.g = self.g_p = None                           # dL/dZ of the last layer, or G_P where a pass masks ahead
        self.dw = [torch.zeros((f, f), dtype=torch.float32, device=dev) for _ in range(L)]
        # with one weight per timestep (Section "EvolveGCN") every timestep has a gradient of its own
        self.dw_t = ([[torch.zeros((f, f), dtype=torch.float32, device=dev) for _ in range(L)] for _ in range(T)]
                     if blk.w_t is not None else None)
        self.status = torch.zeros(T + 1, dtype=torch.int32, device=dev)     # per timestep: whether S_t fitted its arrays
        if self.series:
            self.table = SmoothTable(self.s[1:], list(self.dinv_s[1:]))
            self.table_t = SmoothTable(self.st[1:], None) if transposed else None
            self.ws_smooth = torch.empty(B.smooth_series_workspace(blk.nnz[0], sum(int(d[0].numel()) for d in blk.deltas), T - 1), dtype=torch.uint8, device=dev)
        else:
            self.raw = _Ring(n, cap, dev, life + 1, with_dinv=False)
            self.raw_t = _Ring(n, cap, dev, life + 1, with_dinv=False) if transposed else None
            self.ws_rebuild = torch.empty(B.delta_rebuild_workspace(n, cap, max_list, max_list), dtype=torch.uint8, device=dev)
            self.ws_combine = torch.empty(B.csr_combine_workspace(self.cap_s), dtype=torch.uint8, device=dev)
            self.ws_dinv = torch.empty(B.csr_weighted_dinv_workspace(self.cap_s), dtype=torch.uint8, device=dev)

    def _stage(self, name):
        return self.timer.stage(name) if self.timer is not None else contextlib.nullcontext()

    def _advance(self, ring: _Ring, lists, t: int) -> None:
        ar, ac, dr, dc = lists
        s, d = ring.slot_of(t - 1), ring.slot_of(t)
        with self._stage("delta_rebuild"):
            B.delta_rebuild(ring.rowptr[s], ring.colidx[s], self.blk.nnz[t - 2], ar, ac, int(ar.numel()), dr, dc, int(dr.numel()),
                            ring.rowptr[d], ring.colidx[d], None, self.ws_rebuild)

    def _smooth(self, ring: _Ring, store, t: int) -> None:
        """store[t-1] <- S_t (t >= 2) from store[t-2], A_t and A_{t-life}."""
        blk = self.blk
        prev = store[t - 2] + (self.s_nnz[t - 2],)
        a_out = ring.snapshot(t - self.life, blk.nnz[t - self.life - 1]) if t - self.life >= 1 else None
        with self._stage("csr_combine"):
            B.csr_combine(prev, ring.snapshot(t, blk.nnz[t - 1]), 1.0, a_out, -1.0, store[t - 1], self.ws_combine,
                          diag_value=self.diag_value, status=self.status[t:t + 1])

    def _snapshots(self, stream) -> None:
        """S_1 .. S_T (and their transposes, where needed) with their normalisation."""
        blk = self.blk
        self.s_nnz[0] = blk.nnz[0]
        firsts = [(self.s, blk.rowptr1, blk.colidx1)] + ([(self.st,) + tuple(self.t_first)] if self.st is not self.s else [])
        for store, rowptr1, colidx1 in firsts:
            rowptr, colidx, _ = store[0]
            rowptr.copy_(rowptr1)
            colidx[: blk.nnz[0]].copy_(colidx1[: blk.nnz[0]])
        with self._stage("csr_weighted_dinv"):
            B.csr_dinv(self.s[0][0], self.dinv_s[0])
        if self.series:
            for table, store, lists in ((self.table, self.s, blk.deltas), (self.table_t, self.st, self.t_deltas)):
                if table is not None and blk.T > 1:
                    size = B.smooth_series_workspace(blk.nnz[0], sum(table.lists(lists[:blk.T - 1])[::2]), blk.T - 1)
                    if self.ws_smooth.numel() < size:
                        self.ws_smooth = torch.empty(size, dtype=torch.uint8, device=self.dev)
                    with self._stage("smooth_series"):
                        B.smooth_series(blk.n, store[0][0], store[0][1], blk.nnz[0], blk.T - 1, table.at(), self.life, self.diag_value,
                                        self.cap_s, self.status[2:], self.ws_smooth, stream)
            return
        self.raw.load_first(blk.rowptr1, blk.colidx1)
        if self.raw_t is not None:
            self.raw_t.load_first(*self.t_first)
        for t in range(2, blk.T + 1):
            self._advance(self.raw, blk.deltas[t - 2], t)
            self._smooth(self.raw, self.s, t)
            if self.raw_t is not None:
                self._advance(self.raw_t, self.t_deltas[t - 2], t)
                self._smooth(self.raw_t, self.st, t)
            rp, _, val = self.s[t - 1]
            with self._stage("csr_weighted_dinv"):
                B.csr_weighted_dinv(rp, val, self.s_nnz[t - 1], self.dinv_s[t - 1], self.ws_dinv)

    def forward(self) -> torch.Tensor:
        blk, stack = self.blk, self.stack
        stream = torch.cuda.current_stream(self.dev).cuda_stream
        self._snapshots(stream)
        stack.bind(blk, self.s_nnz)
        for t in range(0, blk.T, stack.together):
            stack.forward(t, min(stack.together, blk.T - t), stream)
        top = self.z[blk.layers - 1]
        if blk.window:
            with self._stage("mproduct"):
                B.mproduct_block(top, self.y, blk.window, 0)
            return self.y
        return top

    def backward(self, g_y: torch.Tensor) -> None:
        """g_y [T, n, f] = dL/dY.  Must follow forward()."""
        blk, stack = self.blk, self.stack
        T = blk.T
        g_y = upstream_frames(g_y, T, blk.n, blk.f, self.z.dtype, blk.window)
        stream = torch.cuda.current_stream(self.dev).cuda_stream
        masked = g_y.shape[0] == T and stack.masks_ahead(blk, True)       # (frames behind the block count in the window)
        if masked:
            if self.g_p is None:
                self.g_p = torch.empty_like(g_y)
            with self._stage("mproduct_relu_backward"):
                B.mproduct_relu_backward_block(g_y, self.z[blk.layers - 1], self.dinv_s, self.g_p, blk.window, 0)
            g_top = self.g_p
        elif blk.window:
            if self.g is None:
                self.g = torch.empty_like(g_y)
            with self._stage("mproduct_backward"):
                B.mproduct_backward_block(g_y, self.g, blk.window, 0)
            g_top = self.g
        else:
            g_top = g_y
        m = stack.steps_back(self.dw_t, T)
        last = (T - 1) // m * m
        for t in range(last, -1, -m):
            k = min(m, T - t)
            stack.backward(blk, t, k, g_top[t:t + k], self.dinv_s[t:t + k], self.dw, self.dw_t, t != last, stream, masked)
