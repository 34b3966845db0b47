"""Tables for the library calls that take several timesteps at once (dgnn_delta_rebuild_series, dgnn_smooth_series,
dgnn_feature_transform_batch, dgnn_spmm_batch).  A table is a numpy array of 64-bit words laid out like the C structs of
include/dgnn.h: device pointers and counts; the drivers fill it once and refresh, per pass, the columns a caller may have
replaced (features, weights, difference lists)."""
from __future__ import annotations

import ctypes
from typing import List, Optional, Sequence

import numpy as np
import torch

from . import binding as B

# Timesteps whose GCN operation is enqueued together: as many as keep the rows of H that the aggregations gather within this
# many bytes (a quarter of the Infinity Cache).  Snapshots with larger frames fill the chip one at a time, and their H is
# still in the cache when it is gathered.
BATCH_BYTES = 64 << 20

# Stored entries up to which a block's snapshots are rebuilt as a series.  Its set-up takes 9 us per million entries, which
# the launches it saves, 13 us a step, make up for; per further step it is as fast as the step-by-step merge (per step, series /
# step by step: 11 thousand entries, 7 steps 2.0 / 13.8 us; 1.7 M, 15 steps 5.3 / 15.6 us; 17 M, 15 steps 48 / 54 us, 3 steps
# 85 / 62 us), and it keeps every snapshot in an array of its own.
SERIES_ENTRIES = 1 << 22

# Vertices up to which the aggregation of X gathers dinv with the rows instead of finding them scaled by a pass of their own.
# The pass costs per byte of X, the gather per entry, and far more once the factors (4 bytes per vertex, 1 MB here) leave an
# L2 of 4 MB to the rows no more: per aggregation of 128-byte rows, gather against pass, 2^16 vertices 8 / 6 us, 2^18
# 15 / 15, 2^19 37 / 27, 2^20 130 / 49; of 256-byte rows 2^18 17 / 24, 2^19 62 / 52, 2^20 200 / 98.
GATHERED_DINV_ROWS = 1 << 18


def steps_together(frame_bytes: int, T: int) -> int:
    return max(1, min(T, BATCH_BYTES // max(frame_bytes, 1)))


def pointers(tensors: Sequence[Optional[torch.Tensor]]) -> List[int]:
    return [0 if t is None else t.data_ptr() for t in tensors]


class Seen:
    """Whether a list of tensors (or tuples of them) holds the objects it held before; the checks of shape, type and layout
    that a call makes are only repeated when it does not."""

    def __init__(self):
        self.ids = None

    def same(self, objects) -> bool:
        ids = [id(o) for o in objects]
        if ids == self.ids:
            return True
        self.ids = ids
        return False


class Table:
    """`rows` structs of `words` 64-bit words each; addresses of the stretch [a, b) for a call."""

    def __init__(self, rows: int, words: int):
        self.words = np.zeros((max(rows, 1), words), dtype=np.int64)
        self.base, self.stride = self.words.ctypes.data, words * 8

    def at(self, row: int = 0) -> int:
        return self.base + row * self.stride

    def column(self, k: int, values, rows: slice = slice(None)) -> None:
        self.words[rows, k] = values


class StepsTable(Table):
    """What the two series calls have in common: the difference lists of a step, add_row, add_col, del_row, del_col, n_add,
    n_del, before the arrays it leads to."""

    def __init__(self, rows: int, words: int):
        super().__init__(rows, words)
        self.seen, self.kept = Seen(), None

    def lists(self, deltas) -> None:
        """The difference lists of the steps, (add_row, add_col, del_row, del_col) each."""
        if self.seen.same(deltas):
            return
        self.kept = list(deltas)                     # the objects compared by identity must stay alive
        for k, d in enumerate(deltas):
            for t in d:
                B._need(t, torch.int32, "difference list")
                assert t.is_contiguous()
            self.words[k, :6] = [t.data_ptr() if t.numel() else 0 for t in d] + [d[0].numel(), d[2].numel()]


class SeriesTable(StepsTable):
    """dgnn_series_step: the lists, then rowptr, colidx, dinv."""

    def __init__(self, rowptr, colidx, dinv):
        super().__init__(len(rowptr), 9)
        for k, tensors in ((6, rowptr), (7, colidx), (8, dinv)):
            if tensors:
                self.column(k, pointers(tensors))
        self.ws = None

    def prepare(self, lists, nnz: int, dev) -> None:
        """The difference lists of the coming calls, behind a first snapshot of nnz entries."""
        if not self.seen.same(lists) or self.ws is None:
            self.seen.ids = None
            self.lists(lists)
            size = B.delta_rebuild_series_workspace(nnz, len(lists), self.at())
            if self.ws is None or self.ws.numel() < size:
                self.ws = torch.empty(size, dtype=torch.uint8, device=dev)

    def rebuild(self, n: int, rowptr, colidx, nnz: int, lists, cap: int, stream) -> None:
        """All snapshots behind (rowptr, colidx) with its nnz entries."""
        self.prepare(lists, nnz, rowptr.device)
        B.delta_rebuild_series(n, rowptr, colidx, nnz, len(lists), self.at(), cap, self.ws, stream)


class SmoothTable(StepsTable):
    """dgnn_smooth_step: the lists, then rowptr, colidx, val, dinv."""

    def __init__(self, snapshots, dinv):
        super().__init__(len(snapshots), 10)
        for k in range(3):
            if len(snapshots):
                self.column(6 + k, pointers([s[k] for s in snapshots]))
        if len(snapshots) and dinv is not None:
            self.column(9, pointers(dinv))


class TransformTable(Table):
    """dgnn_transform_item: x, w, row_scale, h."""
    X, W, SCALE, H = range(4)

    def __init__(self, rows: int):
        super().__init__(rows, 4)


class SpmmTable(Table):
    """dgnn_spmm_item: rowptr, colidx, dinv, val, h, z, nnz."""
    ROWPTR, COLIDX, DINV, VAL, H, Z, NNZ = range(7)

    def __init__(self, rows: int):
        super().__init__(rows, 7)


class WeightGradTable(Table):
    """dgnn_weight_grad_item: x, g, z, dw."""
    X, G, Z, DW = range(4)

    def __init__(self, rows: int):
        super().__init__(rows, 4)


class Frames:
    """Checks of a list of per-timestep tensors, made when the list's objects change, and their addresses."""

    def __init__(self, shape, dtype, name: str):
        self.shape, self.dtype, self.name = tuple(shape), dtype, name
        self.seen, self.kept = Seen(), None

    def addresses(self, tensors) -> List[int]:
        if not self.seen.same(tensors):
            self.kept = list(tensors)
            for t in tensors:
                if tuple(t.shape) != self.shape or t.dtype != self.dtype or not t.is_contiguous():
                    raise ValueError(f"{self.name}: expected contiguous {self.dtype} tensors of shape {self.shape}")
        return [t.data_ptr() for t in tensors]
