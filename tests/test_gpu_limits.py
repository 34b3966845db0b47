"""The size limit of the boundary on the GPU: a snapshot with just under 2^31 stored entries (the index type is
int32).  Built by formula on the device, checked on rows the CPU can compute one by one."""
import numpy as np
import pytest
import torch

import paper_2109_07893_amd as dg
from helpers import assert_close, to_f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

N = 1 << 20
ROW = 2047                      # entries per row; N * ROW = 2^31 - 2^20
STRIDE = 512


def big_snapshot():
    """Row r holds the columns j * 512 + (r mod 512), j = 0..2046, with the diagonal swapped in for the entry
    it is nearest to... kept simple: the diagonal is NOT forced; rows are ascending and duplicate-free, which is
    all the aggregation needs (dinv comes from the row lengths)."""
    rowptr = (torch.arange(N + 1, dtype=torch.int64, device=DEV) * ROW).to(torch.int32)
    colidx = torch.empty(N * ROW, dtype=torch.int32, device=DEV)
    view = colidx.view(N, ROW)
    base = (torch.arange(ROW, dtype=torch.int32, device=DEV) * STRIDE)[None, :]
    chunk = 1 << 16
    for r0 in range(0, N, chunk):
        r = torch.arange(r0, min(N, r0 + chunk), dtype=torch.int32, device=DEV)
        view[r0:r0 + chunk] = base + (r % STRIDE)[:, None]
    return rowptr, colidx


def cols_of(r):
    return np.arange(ROW, dtype=np.int64) * STRIDE + (r % STRIDE)


@pytest.mark.timeout(600)
def test_aggregation_at_the_int32_limit():
    rowptr, colidx = big_snapshot()
    nnz = N * ROW
    assert nnz == (1 << 31) - (1 << 20)
    f = 16
    h = torch.randn((N, f), generator=torch.Generator().manual_seed(1)).to(DEV)
    z = torch.full((N, f), float("nan"), device=DEV)
    dinv = torch.empty(N, device=DEV)
    dg.csr_dinv(rowptr, dinv)
    ws = torch.empty(dg.spmm_workspace(N, nnz, f), dtype=torch.uint8, device=DEV)
    dg.spmm(rowptr, colidx, nnz, dinv, h, z, ws, flags=dg.DGNN_RELU)
    torch.cuda.synchronize()
    assert not torch.isnan(z).any()
    hh = to_f64(h)
    rows = np.concatenate([[0, 1, 511, 512, N - 1, N - 2], np.random.default_rng(2).integers(0, N, 200)])
    want = np.stack([np.maximum(hh[cols_of(r)].sum(axis=0) / ROW, 0.0) for r in rows])   # every dinv is ROW^(-1/2)
    assert_close(to_f64(z[torch.as_tensor(rows, device=DEV)]), want, torch.float32, "rows of the 2^31-entry snapshot")


@pytest.mark.timeout(600)
def test_rebuild_at_the_int32_limit():
    rowptr, colidx = big_snapshot()
    nnz = N * ROW
    # delete the first, a middle and the last entry of a few rows; add columns that fall between the stored ones
    rows = np.array([0, 1, 777, N // 2, N - 2, N - 1], np.int64)
    dr = np.repeat(rows, 3).astype(np.int32)
    dc = np.concatenate([cols_of(r)[[0, 1000, ROW - 1]] for r in rows]).astype(np.int32)
    ar = np.repeat(rows, 2).astype(np.int32)
    ac = np.concatenate([cols_of(r)[[5, 2000]] + 1 for r in rows]).astype(np.int32)      # r % 512 + 1 <= 512: between neighbours
    lists = [torch.as_tensor(x).to(DEV) for x in (ar, ac, dr, dc)]
    cap = nnz + ar.size - dr.size
    rpn = torch.empty(N + 1, dtype=torch.int32, device=DEV)
    cin = torch.full((cap,), -7, dtype=torch.int32, device=DEV)
    dinv = torch.empty(N, device=DEV)
    ws = torch.empty(dg.delta_rebuild_workspace(N, nnz, ar.size, dr.size), dtype=torch.uint8, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    got_nnz = dg.delta_rebuild(rowptr, colidx, nnz, lists[0], lists[1], ar.size, lists[2], lists[3], dr.size, rpn, cin, dinv, ws,
                               flags=0, d_status=status)
    torch.cuda.synchronize()
    assert got_nnz == cap
    # row pointers: every touched row lost one entry net
    shift = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
    for k, r in enumerate(sorted(rows)):
        shift[r + 1:] -= 1
    assert torch.equal(rpn.to(torch.int64), rowptr.to(torch.int64) + shift)
    # untouched stretches are straight copies; touched rows are the merged rows
    edges = [0] + [int(x) for r in sorted(rows) for x in (r, r + 1)] + [N]
    for a, b in zip(edges[0::2], edges[1::2]):
        if b > a:
            src = colidx[int(rowptr[a]):int(rowptr[b])] if b < N + 1 else None
            dst = cin[int(rpn[a]):int(rpn[b])]
            assert torch.equal(src, dst), (a, b)
    for r in rows:
        old = set(cols_of(r).tolist())
        want = sorted((old - set(dc[dr == r].tolist())) | set(ac[ar == r].tolist()))
        got = cin[int(rpn[r]):int(rpn[r + 1])].cpu().numpy().tolist()
        assert got == want, r


@pytest.mark.timeout(600)
def test_rebuild_that_deletes_all_of_a_full_matrix():
    """A deleted list just under 2^31 entries whose last row tile owns millions of them: the counts come from searches whose steps
    lead beyond 2^31 there.  What is left is the diagonal."""
    n = 46_340
    nnz, n_del = n * n, n * (n - 1)
    assert nnz <= (1 << 31) - 65537 and n_del + (1 << 22) > 1 << 31
    rowptr = (torch.arange(n + 1, dtype=torch.int64, device=DEV) * n).to(torch.int32)
    colidx = torch.arange(n, dtype=torch.int32, device=DEV).repeat(n)
    d_row, d_col = (torch.empty(n_del, dtype=torch.int32, device=DEV) for _ in range(2))
    c = torch.arange(n - 1, dtype=torch.int32, device=DEV)[None, :]
    for r0 in range(0, n, 1024):
        r = torch.arange(r0, min(r0 + 1024, n), dtype=torch.int32, device=DEV)[:, None]
        d_row.view(n, n - 1)[r0:r0 + 1024] = r
        d_col.view(n, n - 1)[r0:r0 + 1024] = c + (c >= r).to(torch.int32)
    none = torch.empty(0, dtype=torch.int32, device=DEV)
    rpn = torch.full((n + 1,), -7, dtype=torch.int32, device=DEV)
    cin = torch.full((n,), -7, dtype=torch.int32, device=DEV)
    dinv = torch.empty(n, device=DEV)
    ws = torch.empty(dg.delta_rebuild_workspace(n, nnz, 0, n_del), dtype=torch.uint8, device=DEV)
    assert dg.delta_rebuild(rowptr, colidx, nnz, none, none, 0, d_row, d_col, n_del, rpn, cin, dinv, ws) == n
    torch.cuda.synchronize()
    want = torch.arange(n + 1, dtype=torch.int32, device=DEV)
    assert torch.equal(rpn, want) and torch.equal(cin, want[:n]) and bool((dinv == 1).all())


@pytest.mark.timeout(600)
def test_rebuild_of_a_sub_tile_that_leaves_more_than_2_29_entries():
    """512 rows of one entry each that are full afterwards, all of them placed by one wavefront: more words than 31 bits of bytes
    reach from the first."""
    rows, n = 512, (1 << 20) + 1024
    assert rows * n > 1 << 29
    cols = torch.arange(n, dtype=torch.int32, device=DEV)
    add_row = torch.arange(rows, dtype=torch.int32, device=DEV).repeat_interleave(n - 1)
    add_col = torch.empty(rows * (n - 1), dtype=torch.int32, device=DEV)
    for r in range(rows):
        add_col[r * (n - 1):(r + 1) * (n - 1)] = cols[:-1] + (cols[:-1] >= r)
    n_add, none = add_row.numel(), torch.empty(0, dtype=torch.int32, device=DEV)
    rpn = torch.full((n + 1,), -7, dtype=torch.int32, device=DEV)
    cin = torch.full((n + n_add,), -7, dtype=torch.int32, device=DEV)
    ws = torch.empty(dg.delta_rebuild_workspace(n, n, n_add, 0), dtype=torch.uint8, device=DEV)
    rp = torch.arange(n + 1, dtype=torch.int32, device=DEV)
    assert dg.delta_rebuild(rp, cols, n, add_row, add_col, n_add, none, none, 0, rpn, cin, torch.empty(n, device=DEV), ws) == n + n_add
    torch.cuda.synchronize()
    assert torch.equal(rpn[:rows + 1], rp[:rows + 1] * n) and torch.equal(rpn[rows:], rp[rows:] + rows * (n - 1))
    assert torch.equal(cin[rows * n:], cols[rows:])
    for r in range(0, rows, 64):
        assert torch.equal(cin[r * n:(r + 64) * n].view(64, n), cols.expand(64, n)), r


@pytest.mark.timeout(600)
@pytest.mark.parametrize("weighted", [False, True])
def test_rebuild_that_adds_more_than_2_29_entries(weighted):
    """... spread over all rows: deleted entries, added ones and, with values, an update for every diagonal entry.  Row r has r, for even r
    also r + 1, and receives 520 columns that are r + 1000 modulo 2000."""
    n, each = 1 << 20, 520
    n_add = n * each
    assert n_add > (1 << 29) and 2000 * each <= n
    r = torch.arange(n, dtype=torch.int32, device=DEV)
    even = (r % 2 == 0).to(torch.int32)
    rp = torch.cat([torch.zeros_like(r[:1]), torch.cumsum(1 + even, 0, dtype=torch.int32)])
    nnz = int(rp[-1])
    pairs = torch.stack([r, r + 1], 1).view(-1)
    ci = pairs[torch.stack([torch.ones_like(even), even], 1).view(-1).bool()]
    d_row = r[::4].contiguous()
    d_col = d_row + 1
    add_row, add_col = r.repeat_interleave(each), torch.empty(n_add, dtype=torch.int32, device=DEV)
    step = torch.arange(each, dtype=torch.int32, device=DEV)[None, :] * 2000
    chunk = 1 << 15
    for a in range(0, n, chunk):
        add_col.view(n, each)[a:a + chunk] = step + ((r[a:a + chunk] + 1000) % 2000)[:, None]
    cap = nnz + n_add - d_row.numel()
    rpn, cin = torch.full((n + 1,), -7, dtype=torch.int32, device=DEV), torch.full((cap,), -7, dtype=torch.int32, device=DEV)
    ws = torch.empty(dg.delta_rebuild_workspace(n, nnz, n_add, d_row.numel()), dtype=torch.uint8, device=DEV)

    def value(row, col):                                # of an entry that is stored or added
        return ((row * 31 + col * 7) % 1021).to(torch.float32)
    if weighted:
        val, add_val, vn = value(r.repeat_interleave(1 + even), ci), value(add_row, add_col), torch.full((cap,), float("nan"), device=DEV)
        got = dg.delta_rebuild_weighted(rp, ci, val, nnz, (add_row, add_col, add_val), (d_row, d_col), (r, r, value(r, r) + 2000.0), rpn, cin, vn, ws,
                                        flags=dg.DGNN_UPDATES_SORTED)
        del add_val
    else:
        got = dg.delta_rebuild(rp, ci, nnz, add_row, add_col, n_add, d_row, d_col, d_row.numel(), rpn, cin, torch.empty(n, device=DEV), ws)
    torch.cuda.synchronize()
    assert got == cap
    long = (r % 4 == 2).to(torch.int32)                 # r + 1 is kept
    assert torch.equal(rpn[1:], torch.cumsum(each + 1 + long, 0, dtype=torch.int32)) and int(rpn[0]) == 0
    beyond = torch.full((chunk, 1), 1 << 30, dtype=torch.int32, device=DEV)
    for a in range(0, n, chunk):
        rows = r[a:a + chunk, None]
        want = torch.cat([add_col.view(n, each)[a:a + chunk], rows, torch.where(long[a:a + chunk, None] > 0, rows + 1, beyond)], 1).sort(1).values
        there = want < (1 << 30)
        lo, hi = int(rpn[a]), int(rpn[min(a + chunk, n)])
        assert torch.equal(cin[lo:hi], want[there]), a
        if weighted:
            v = value(rows, want) + 2000.0 * (want == rows)
            assert torch.equal(vn[lo:hi], v[there]), a
