"""Tables for the library calls that take several timesteps at once (dgnn_delta_rebuild_series, dgnn_smooth_series,
dgnn_feature_transform_batch, dgnn_spmm_batch).  A table is a numpy array of 64-bit words laid out like the C structs of
include/dgnn.h: device pointers and counts; the drivers fill it once and refresh, per pass, the columns a caller may have
replaced (features, weights, difference lists)."""
from __future__ import annotations

from typing import List, Optional, Sequence

import numpy as np
import torch

from . import binding as B

# Timesteps whose GCN operation is enqueued together: as many as keep the rows of H that the aggregations gather within this many
# bytes.  An aggregation deals whole frames to the XCDs, each of which then gathers out of one frame at a time, so eight frames or
# more are worth having, and every launch pair has a start and an end of its own; whether all of H stays in the Infinity Cache
# (256 MB) matters less.  Whole passes in us for 64 / 256 / 512 / 1024 MB, uniform graphs: two layers forward, 100 K vertices x 64 fp32,
# 2330 / 2118 / 2062 / 2064; trained, 50 K, 1984 / 1676 / 1675 / 1675; 100 K x 128 bf16 forward 3379 / 2976 / 2947 / 2950; CD-GCN in bf16,
# 200 K x 64, 944 / 860 / 858 / 859; R-MAT: two layers forward, 2^16 x 64 fp32, 1242 / 1119 / 1113 / 1113, 2^17 2494 / 2227 / 2218 / 2212;
# trained, 2^16, 2519 / 2250 / 2249 / 2241; 2^17 x 128 bf16 forward 2572 / 2332 / 2307 / 2284; CD-GCN in bf16, 2^17 x 64, 1073 / 1050 / 1043 /
# 1054.  The price is memory: a driver holds up to four buffers of a batch's frames (H, the masked gradient, and with several layers
# a layer's output and its gradient), 2 GB at most, beside the scratch of 32 aggregations (SpmmTable.workspace).
BATCH_BYTES = 512 << 20

# Stored entries up to which a block's snapshots are rebuilt as a series, and how many of them a step must make up for.  The
# set-up takes 9 us per million entries; a step saves one rebuild's launches and the products and aggregations of its timestep
# a launch of their own, less the more entries there are.  Whole passes (32 columns), series / step by step in us: uniform graph, one
# step 1.4 M entries 79 / 88, 2.0 M 115 / 110, 2.8 M 162 / 149, 4.0 M 228 / 210; two steps 2.8 M 220 / 231, 4.0 M 316 / 326; nine steps
# 4.0 M 915 / 1085; R-MAT, one step 1.4 M 73 / 85, 2.0 M 102 / 106, 2.7 M 115 / 116, 3.9 M 171 / 162; two steps 3.9 M 229 / 255; nine 662 / 894.
# Above 2^22 the chip is full with one timestep, and what a long series still gains gets less (15 steps, uniform 5.6 M 2134 / 2416, 8 M
# 3079 / 3382, 17 M 6749 / 7010), a short one loses (3 steps of 17 M 1834 / 1799): such blocks keep the step-by-step order, and its
# three slots instead of a snapshot per timestep.
SERIES_ENTRIES = 1 << 22
SERIES_ENTRIES_PER_STEP = 1 << 21

# ... and the bytes its snapshots may take together.  A series of many dense snapshots on few vertices holds far more in them than
# in its features (10 000 steps of 4 M entries: 160 GB, where the step-by-step rebuild needs three slots), so a long one is
# rebuilt step by step again; 33 snapshots of 4 M entries and 2^20 vertices take 0.8 GB.
SERIES_BYTES = 16 << 30

# Vertices up to which the aggregation of X gathers dinv with the rows instead of finding them scaled by a pass of their own.
# The pass costs per byte of X and a launch, the gather per entry, and far more once the factors (4 bytes per vertex, 1 MB here)
# leave an L2 of 4 MB to the rows no more.  Uniform graphs, timesteps together as batch.py has them, gather / pass in us per
# aggregation, 16 entries per row:
#                  2^14          2^15          2^16          2^17          2^18          2^19          2^20 vertices
#   64-byte rows   2.9 / 2.4     6.1 / 5.0    13.0 / 9.8    28.7 / 25.0   87.3 / 75.7    194 / 171     466 / 355
#   128            3.7 / 3.5     7.5 / 6.5    15.6 / 14.9   35.7 / 37.8   96.0 / 99.6    213 / 202     490 / 400
#   256            5.9 / 6.2    14.2 / 12.2   31.9 / 29.7   73.3 / 78.8    185 / 199     400 / 387     863 / 765
#   512           11.2 / 11.6   29.9 / 25.4   65.1 / 61.3    146 / 160     358 / 383     793 / 766    1722 / 1509
# and 4 entries per row, 128-byte rows, 2^14 1.5 / 2.2, 2^16 6.4 / 8.1, 2^18 30.5 / 38.5, 2^19 69.7 / 79.7, 2^20 168 / 171.  Rows of 64 bytes and
# graphs of 2^15 - 2^16 with many entries per row are the exceptions, for which the rule takes neither a width nor a degree.
GATHERED_DINV_ROWS = 1 << 18


def steps_together(frame_bytes: int, T: int) -> int:
    return max(1, min(T, BATCH_BYTES // max(frame_bytes, 1)))


def series_pays(T: int, cap: int) -> bool:
    return cap <= max(T - 1, 1) * SERIES_ENTRIES_PER_STEP


def snapshots_fit(T: int, n: int, cap: int) -> bool:
    return T * (4 * cap + 8 * n) <= SERIES_BYTES


def pointers(tensors: Sequence[Optional[torch.Tensor]]) -> List[int]:
    return [0 if t is None else t.data_ptr() for t in tensors]


_numel, _data_ptr, _is_contiguous = torch.Tensor.numel, torch.Tensor.data_ptr, torch.Tensor.is_contiguous


class Table:
    """`rows` structs of `words` 64-bit words each; addresses of the stretch [a, b) for a call."""

    def __init__(self, rows: int, words: int):
        self.words = np.zeros((max(rows, 1), words), dtype=np.int64)
        self.base, self.stride = self.words.ctypes.data, words * 8
        self.bound = {}

    def at(self, row: int = 0) -> int:
        return self.base + row * self.stride

    def column(self, k: int, values, rows: slice = slice(None)) -> None:
        self.words[rows, k] = values

    def refresh(self, k: int, values: List[int], rows: int) -> None:
        """The first `rows` entries of a column that is bound anew for every pass (one value: for all of them); written where
        they are not what the last pass wrote."""
        if self.bound.get(k) != (rows, values):
            self.words[:rows, k] = values
            self.bound[k] = (rows, list(values))


class StepsTable(Table):
    """What the two series calls have in common: the difference lists of a step, add_row, add_col, del_row, del_col, n_add,
    n_del, before the arrays it leads to."""

    entered = None                                   # the rows as they stand

    def lists(self, deltas) -> List[int]:
        """The difference lists of the steps, (add_row, add_col, del_row, del_col) each, checked and entered anew for every
        call; returns the counts (n_add, n_del of every step)."""
        flat = [t for d in deltas for t in d]
        if not all(map(_is_contiguous, flat)):
            raise AssertionError("dgnn takes contiguous tensors")
        for t in flat:
            if t.dtype is not torch.int32:
                B._need(t, torch.int32, "difference list")
        count, at = list(map(_numel, flat)), list(map(_data_ptr, flat))
        adds, dels = count[0::4], count[2::4]
        if count[1::4] != adds or count[3::4] != dels:
            assert all(c >= r for c, r in zip(count[1::4] + count[3::4], adds + dels)), "a difference list has fewer columns than rows"
        if 0 in count:                               # an empty list has no address
            at = [p if count[k & ~1] else 0 for k, p in enumerate(at)]
        rows = [at, adds, dels]
        if flat and rows != self.entered:
            steps = len(adds)
            self.words[:steps, :4] = np.array(at, dtype=np.int64).reshape(steps, 4)
            self.words[:steps, 4] = adds
            self.words[:steps, 5] = dels
            self.entered = rows
        return [c for pair in zip(adds, dels) for c in pair]


class SeriesTable(StepsTable):
    """dgnn_series_step: the lists, then rowptr, colidx, dinv."""

    def __init__(self, rowptr, colidx, dinv):
        super().__init__(len(rowptr), 9)
        for k, tensors in ((6, rowptr), (7, colidx), (8, dinv)):
            if tensors:
                self.column(k, pointers(tensors))
        self.ws, self.sized_for = None, None

    def prepare(self, lists, nnz: int, dev) -> List[int]:
        """The difference lists of the coming call, behind a first snapshot of nnz entries; returns their counts."""
        counts = self.lists(lists)
        if self.sized_for != (nnz, counts):          # what the workspace depends on
            size = B.delta_rebuild_series_workspace(nnz, len(lists), self.at())
            if self.ws is None or self.ws.numel() < size:
                self.ws = torch.empty(size, dtype=torch.uint8, device=dev)
            self.sized_for = (nnz, counts)
        return counts

    def rebuild(self, n: int, rowptr, colidx, nnz: int, lists, cap: int, stream, leads_to=()) -> None:
        """All snapshots behind (rowptr, colidx) with its nnz entries; leads_to: how many entries the caller will take those
        behind the first steps to have."""
        counts = self.prepare(lists, nnz, rowptr.device)
        have = nnz
        for k, want in enumerate(leads_to):
            have += counts[2 * k] - counts[2 * k + 1]
            assert have == want, "difference lists and entry counts disagree"
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
    LAUNCH = 32                                      # aggregations that the library enqueues together

    def __init__(self, rows: int):
        super().__init__(rows, 7)

    @staticmethod
    def workspace(together: int, cap: int, f: int) -> int:
        """Bytes of scratch for run(): it follows the entries, not the frames (2048 vertices, 4 M entries, 128 columns: 1 MB a frame,
        34 MB an aggregation), so no more than one launch has it at a time."""
        return B.spmm_batch_workspace(min(together, SpmmTable.LAUNCH), cap, f)

    def run(self, n: int, row: int, count: int, f: int, dt: int, flags: int, ws: torch.Tensor, stream) -> None:
        """The aggregations of rows row .. row + count - 1, a launch's worth after the other on the same scratch."""
        for k in range(0, count, self.LAUNCH):
            B.spmm_batch(n, min(self.LAUNCH, count - k), self.at(row + k), f, dt, flags, ws, stream)


class WeightGradTable(Table):
    """dgnn_weight_grad_item: x, g, z, dw."""
    X, G, Z, DW = range(4)

    def __init__(self, rows: int):
        super().__init__(rows, 4)


class Frames:
    """Addresses of a list of per-timestep tensors, after the checks that a call on each of them would make."""

    def __init__(self, shape, dtype, name: str):
        self.shape, self.dtype, self.name = torch.Size(shape), dtype, name

    def addresses(self, tensors) -> List[int]:
        shape, dtype = self.shape, self.dtype
        for t in tensors:
            if t.shape != shape or t.dtype is not dtype or not t.is_contiguous():
                raise ValueError(f"{self.name}: expected contiguous {dtype} tensors of shape {tuple(shape)}")
        return list(map(_data_ptr, tensors))


def upstream_frames(g, T: int, n: int, f: int, dtype, window: int = 0) -> torch.Tensor:
    """The gradients [T, n, f] handed to a backward pass, whose rows go to the kernels by address.  Without a window, which
    takes them whole in any case, frames of their own (a list, or a tensor that is strided over the timesteps) are brought
    together."""
    if not isinstance(g, torch.Tensor):
        g = torch.stack([g[t] for t in range(T)])
    if g.dim() != 3 or g.shape[0] < T or g.shape[1] != n or g.shape[2] != f or g.dtype is not dtype or not g.is_cuda:
        raise ValueError(f"upstream gradients: expected a {dtype} device tensor of shape {(T, n, f)}")
    if not g.is_contiguous():
        assert not window and g[0].is_contiguous(), "dgnn takes contiguous tensors"
        g = g[:T].contiguous()
    return g
