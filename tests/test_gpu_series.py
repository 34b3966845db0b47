"""The calls that take several timesteps at once against the calls that take one: snapshots rebuilt as a series bit for bit
those of step-by-step rebuilds, batched products and aggregations bit for bit the single ones."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import paper_2109_07893_amd as dg
from dtdg_synth import WORKLOADS, DynamicGraph
from dtdg_synth.blocks import make_block
from paper_2109_07893_amd import binding as B
from paper_2109_07893_amd.batch import SeriesTable, SmoothTable, SpmmTable, TransformTable, WeightGradTable, pointers
from paper_2109_07893_amd.pipeline import BlockRunner

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def graph(kind, n, deg, T, dels, adds, seed=11):
    return replace(WORKLOADS["c2" if kind == "er" else "c5"], name=kind, n=n, T=T, avg_deg=float(deg), n_draws=n * deg,
                   del_frac=dels, add_frac=adds, seed=seed)


# stretches of up to 1536 entries and what all steps add to them, launches of 31 steps
@pytest.mark.parametrize("kind,n,deg,T,dels,adds", [
    ("er", 7, 3, 5, 0.2, 0.2), ("er", 257, 4, 40, 0.1, 0.1), ("er", 1536, 1, 3, 0.0, 0.5), ("rmat", 1024, 20, 12, 0.05, 0.05),
    ("er", 300, 8, 6, 0.0, 0.5), ("er", 2000, 6, 10, 0.05, 0.4), ("er", 5000, 30, 5, 0.5, 0.9), ("er", 4001, 10, 5, 0.6, 0.0),
    ("rmat", 1 << 14, 16, 34, 0.03, 0.03), ("er", 30_000, 40, 3, 0.02, 0.02), ("rmat", 1 << 15, 40, 33, 0.01, 0.05)])
def test_series_equals_step_by_step(kind, n, deg, T, dels, adds):
    g = DynamicGraph(graph(kind, n, deg, T, dels, adds), device=DEV)
    rp, ci = g.csr()
    steps = [g.advance() for _ in range(T - 1)]
    nnz = [int(ci.numel())]
    for d in steps:
        nnz.append(nnz[-1] + d[0].numel() - d[2].numel())
    cap = max(nnz)
    got = ([torch.full((n + 1,), -7, dtype=torch.int32, device=DEV) for _ in steps],
           [torch.full((cap,), -7, dtype=torch.int32, device=DEV) for _ in steps], [torch.zeros(n, device=DEV) for _ in steps])
    table = SeriesTable(*got)
    table.rebuild(n, rp, ci, nnz[0], steps, cap, torch.cuda.current_stream().cuda_stream)
    longest = max(max(d[0].numel(), d[2].numel()) for d in steps) + 1
    ws = torch.empty(dg.delta_rebuild_workspace(n, cap, longest, longest), dtype=torch.uint8, device=DEV)
    for k, (ar, ac, dr, dc) in enumerate(steps):
        rp2, ci2, dinv2 = torch.empty_like(rp), torch.empty(cap, dtype=torch.int32, device=DEV), torch.empty(n, device=DEV)
        dg.delta_rebuild(rp, ci, nnz[k], ar, ac, ar.numel(), dr, dc, dr.numel(), rp2, ci2, dinv2, ws)
        assert torch.equal(rp2, got[0][k]) and torch.equal(ci2[: nnz[k + 1]], got[1][k][: nnz[k + 1]]), k
        assert bool((got[1][k][nnz[k + 1]:] == -7).all()) and torch.equal(dinv2, got[2][k]), k
        rp, ci = rp2, ci2


def toggled_series(n, places, T, dels, adds, seed):
    """A_1 (the diagonal and half of `places`, off-diagonal keys row * n + column) and difference lists that take entries out
    and put them back: of the absent places `adds` per step, of the present ones `dels`."""
    rng = np.random.default_rng(seed)
    present = rng.random(places.size) < 0.5 if adds < 1 else np.zeros(places.size, bool)
    def split(keys):
        keys = np.sort(keys)
        return [torch.from_numpy((k).astype(np.int32)).to(DEV) for k in (keys // n, keys % n)]
    first = np.sort(np.concatenate([np.arange(n, dtype=np.int64) * (n + 1), places[present]]))
    rp = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(first // n, minlength=n), out=rp[1:])
    steps = []
    for _ in range(T - 1):
        flip = rng.random(places.size) < np.where(present, dels, adds if adds < 1 else adds / places.size)
        steps.append(tuple(split(places[flip & ~present])) + tuple(split(places[flip & present])))
        present = present ^ flip
    return torch.from_numpy(rp).to(DEV), torch.from_numpy((first % n).astype(np.int32)).to(DEV), steps


# entries that come back while they are remembered; stretches of 1536 entries; a gap between two entries of A_1 into which more
# than the LDS holds is added, so that the keys have to be halved; the longest window and series
@pytest.mark.parametrize("n,rows,T,life,dels,adds,diag", [
    (1, 1, 3, 2, 0.0, 0.0, 1.0), (40, 40, 8, 3, 0.3, 0.3, 1.0), (40, 40, 32, 32, 0.2, 0.1, 1.0), (130, 130, 9, 1, 0.1, 0.1, 1.0),
    (300, 300, 6, 4, 0.02, 0.02, 0.0), (1537, 1, 5, 2, 0.1, 0.0, 0.5), (9000, 1, 6, 3, 0.1, 400, 1.0), (9000, 2, 5, 4, 0.3, 4000, 1.0),
    (5000, 3, 3, 2, 0.0, 900, 2.0), (2000, 70, 5, 5, 0.05, 0.05, 1.0)])
def test_smoothed_series_equals_step_by_step(n, rows, T, life, dels, adds, diag):
    where = np.arange(rows, dtype=np.int64) * max(1, n // rows)
    places = (where[:, None] * n + np.arange(n, dtype=np.int64)[None, :]).reshape(-1)
    places = places[places % (n + 1) != 0]
    rp, ci, steps = toggled_series(n, places, T, dels, adds, seed=n + T)
    nnz = [int(ci.numel())]
    for d in steps:
        nnz.append(nnz[-1] + d[0].numel() - d[2].numel())
    cap = max(nnz) + life * max(d[2].numel() for d in steps)
    def room():
        return torch.full((n + 1,), -7, dtype=torch.int32, device=DEV), torch.full((cap,), -7, dtype=torch.int32, device=DEV), torch.zeros(cap, device=DEV)
    got, dinv = [room() for _ in steps], torch.zeros(T - 1, n, device=DEV)
    status = torch.full((T - 1,), -1, dtype=torch.int32, device=DEV)
    table = SmoothTable(got, list(dinv))
    table.lists(steps)
    ws = torch.empty(B.smooth_series_workspace(nnz[0], sum(d[0].numel() for d in steps), T - 1), dtype=torch.uint8, device=DEV)
    B.smooth_series(n, rp, ci, nnz[0], T - 1, table.at(), life, diag, cap, status, ws, torch.cuda.current_stream().cuda_stream)
    assert int(status.abs().sum()) == 0
    longest = max(max(d[0].numel(), d[2].numel()) for d in steps) + 1
    ws = torch.empty(dg.delta_rebuild_workspace(n, max(nnz), longest, longest), dtype=torch.uint8, device=DEV)
    ws_c = torch.empty(dg.csr_combine_workspace(cap), dtype=torch.uint8, device=DEV)
    ws_d = torch.empty(dg.csr_weighted_dinv_workspace(cap), dtype=torch.uint8, device=DEV)
    raw, s = [(rp, ci, nnz[0])], (rp, ci, None, nnz[0])
    for k, (ar, ac, dr, dc) in enumerate(steps):
        rp2, ci2 = torch.empty_like(rp), torch.empty(max(nnz), dtype=torch.int32, device=DEV)
        dg.delta_rebuild(raw[-1][0], raw[-1][1], nnz[k], ar, ac, ar.numel(), dr, dc, dr.numel(), rp2, ci2, None, ws)
        raw.append((rp2, ci2, nnz[k + 1]))
        out, d = room(), torch.empty(n, device=DEV)
        dg.csr_combine(s, raw[-1], 1.0, raw[k + 1 - life] if k + 1 >= life else None, -1.0, out, ws_c, diag_value=diag)
        dg.csr_weighted_dinv(out[0], out[2], cap, d, ws_d)
        m = int(out[0][n])
        for a, b in zip(got[k], out):
            assert torch.equal(a[: n + 1 if a is got[k][0] else m], b[: n + 1 if a is got[k][0] else m]), k
        assert bool((got[k][1][m:] == -7).all()) and torch.equal(dinv[k], d), k
        s = out + (cap,)
    # arrays that are too small: said so, and nothing written behind them
    small = [(r, c[:max(1, int(r[n]) // 2)], v[:max(1, int(r[n]) // 2)]) for r, c, v in got]
    keep = [c[max(1, int(r[n]) // 2):].clone() for r, c, v in got]
    room_left = min(int(c.numel()) for _, c, _ in small)
    ws = torch.empty(B.smooth_series_workspace(nnz[0], sum(d[0].numel() for d in steps), T - 1), dtype=torch.uint8, device=DEV)
    B.smooth_series(n, rp, ci, nnz[0], T - 1, table.at(), life, diag, room_left, status, ws, torch.cuda.current_stream().cuda_stream)
    assert all(bool(x) == (int(r[n]) > room_left) for x, (r, _, _) in zip(status, got))
    assert all(torch.equal(c[max(1, int(r[n]) // 2):], k) for (r, c, v), k in zip(got, keep))


@pytest.mark.parametrize("dtype,f", [(torch.float32, 16), (torch.float32, 64), (torch.float32, 128), (torch.bfloat16, 32), (torch.bfloat16, 128)])
@pytest.mark.parametrize("count", [1, 3, 33])
def test_batched_products_and_aggregations_equal_single_ones(dtype, f, count):
    """33 items: one more than a launch takes.  Snapshots of different sizes, hub rows over many ranges among them."""
    torch.manual_seed(count)
    n, dt = 1 << 11, (B.DGNN_F32 if dtype == torch.float32 else B.DGNN_BF16)
    snaps = [DynamicGraph(graph("rmat", n, 4 + 12 * (k % 3), 2, 0, 0, seed=k), device=DEV).csr() for k in range(count)]
    x = [torch.randn(n, f, device=DEV).to(dtype) for _ in range(count)]
    w = [(torch.randn(f, f, device=DEV) / f ** 0.5).to(dtype) for _ in range(count)]
    dinv = [torch.empty(n, device=DEV) for _ in range(count)]
    for (rp, _), d in zip(snaps, dinv):
        dg.csr_dinv(rp, d)
    h, z, h1, z1 = (torch.zeros(count, n, f, dtype=dtype, device=DEV) for _ in range(4))
    nnz = [int(ci.numel()) for _, ci in snaps]
    a, b = TransformTable(count), SpmmTable(count)
    for k, col in ((a.X, x), (a.W, w), (a.SCALE, dinv), (a.H, list(h))):
        a.column(k, pointers(col))
    for k, col in ((b.ROWPTR, [s[0] for s in snaps]), (b.COLIDX, [s[1] for s in snaps]), (b.DINV, dinv), (b.H, list(h)), (b.Z, list(z))):
        b.column(k, pointers(col))
    b.column(b.NNZ, nnz)
    ws = torch.empty(B.spmm_batch_workspace(count, max(nnz), f), dtype=torch.uint8, device=DEV)
    stream = torch.cuda.current_stream().cuda_stream
    B.feature_transform_batch(count, a.at(), n, f, f, 0, dt, stream)
    B.spmm_batch(n, count, b.at(), f, dt, B.DGNN_RELU | B.DGNN_H_PRESCALED, ws, stream)
    ws1 = torch.empty(dg.spmm_workspace(n, max(nnz), f), dtype=torch.uint8, device=DEV)
    for k in range(count):
        dg.feature_transform(x[k], w[k], h1[k], row_scale=dinv[k])
        dg.spmm(snaps[k][0], snaps[k][1], nnz[k], dinv[k], h1[k], z1[k], ws1, flags=dg.DGNN_RELU | dg.DGNN_H_PRESCALED)
    assert torch.equal(h, h1) and torch.equal(z, z1)
    a.column(a.SCALE, 0)
    B.feature_transform_batch(count, a.at(), n, f, f, B.DGNN_RELU, dt, stream)
    dg.feature_transform(x[0], w[0], h1[0])
    assert torch.equal(h[0].float(), torch.relu(h1[0].float()))


@pytest.mark.parametrize("dtype,f", [(torch.float32, 32), (torch.float32, 128), (torch.bfloat16, 64)])
@pytest.mark.parametrize("count", [2, 33])
def test_batched_aggregations_with_values_equal_single_ones(dtype, f, count):
    """Rows scaled beforehand, as dgnn_spmm_weighted; and (fp32) scaled as they are gathered: value times dinv per entry."""
    torch.manual_seed(count)
    n, dt = 1 << 11, (B.DGNN_F32 if dtype == torch.float32 else B.DGNN_BF16)
    snaps = [DynamicGraph(graph("rmat", n, 4 + 12 * (k % 3), 2, 0, 0, seed=k), device=DEV).csr() for k in range(count)]
    nnz = [int(ci.numel()) for _, ci in snaps]
    val, dinv = [torch.rand(m, device=DEV) + 0.5 for m in nnz], [torch.rand(n, device=DEV) for _ in range(count)]
    h = [torch.randn(n, f, device=DEV).to(dtype) for _ in range(count)]
    z, z1 = (torch.zeros(count, n, f, dtype=dtype, device=DEV) for _ in range(2))
    b = SpmmTable(count)
    for k, col in ((b.ROWPTR, [s[0] for s in snaps]), (b.COLIDX, [s[1] for s in snaps]), (b.DINV, dinv), (b.VAL, val), (b.H, h), (b.Z, list(z))):
        b.column(k, pointers(col))
    b.column(b.NNZ, nnz)
    ws = torch.empty(B.spmm_batch_workspace(count, max(nnz), f), dtype=torch.uint8, device=DEV)
    ws1 = torch.empty(dg.spmm_workspace(n, max(nnz), f), dtype=torch.uint8, device=DEV)
    stream = torch.cuda.current_stream().cuda_stream
    B.spmm_batch(n, count, b.at(), f, dt, B.DGNN_RELU | B.DGNN_H_PRESCALED, ws, stream)
    for k, (rp, ci) in enumerate(snaps):
        dg.spmm_weighted(rp, ci, val[k], nnz[k], h[k], z1[k], ws1, flags=dg.DGNN_RELU | dg.DGNN_H_PRESCALED, dinv=dinv[k])
    assert torch.equal(z, z1)
    if dtype == torch.float32:
        B.spmm_batch(n, count, b.at(), f, dt, 0, ws, stream)
        for k, (rp, ci) in enumerate(snaps):
            dg.spmm_weighted(rp, ci, val[k] * dinv[k][ci.long()], nnz[k], h[k], z1[k], ws1)
            assert torch.equal(z[k], z1[k] * dinv[k][:, None]), k


@pytest.mark.parametrize("name,n,T,keep", [("c1", 1000, 8, None), ("c2", 20_000, 7, True), ("c3", 1 << 12, 5, False), ("c4", 3_001, 35, None)])
def test_pass_with_batched_steps_equals_the_pass_step_by_step(name, n, T, keep):
    wl = WORKLOADS[name] if WORKLOADS[name].n == n else WORKLOADS[name].scaled(n, T=T)
    runner = BlockRunner(make_block(wl, DEV, gen_device="cpu", T=T), keep_all_z=keep)
    assert runner.series
    runner.load_first()
    runner.run_resident(validate=True)                   # validation goes step by step
    want = runner.z.clone()
    for first in (1, 2):
        runner.z.fill_(float("nan"))
        runner.run_resident(first=first)
        torch.cuda.synchronize()
        if first == 1 or not runner.blk.window:
            assert torch.equal(runner.z[first - 1 if runner.keep_all_z else 0:], want[first - 1 if runner.keep_all_z else 0:])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("f_in,f_out,n", [(16, 16, 1), (32, 64, 333), (128, 128, 1000), (64, 16, 5000)])
def test_weight_gradient_through_the_relu(dtype, f_in, f_out, n):
    """x^T (z > 0 ? g : 0) in one call against the mask applied beforehand; zeros and negative zeros do not pass."""
    from paper_2109_07893_amd.batch import WeightGradTable
    torch.manual_seed(n)
    x, g, z = (torch.randn(2, n, f, device=DEV).to(dtype) for f in (f_in, f_out, f_out))
    z[:, ::3] = 0.0
    z[:, 1::7] = -0.0
    dw = torch.full((2, f_in, f_out), float("nan"), device=DEV)
    ws = torch.empty(B.weight_grad_workspace(f_in, f_out), dtype=torch.uint8, device=DEV)
    table = WeightGradTable(2)
    for k, t in ((table.X, x), (table.G, g), (table.Z, z), (table.DW, dw)):
        table.column(k, pointers(list(t)))
    B.weight_grad_batch(2, table.at(), n, f_in, f_out, False, B._dtype_code(x), ws, torch.cuda.current_stream().cuda_stream)
    want = x.double().transpose(1, 2).contiguous() @ torch.where(z > 0, g, torch.zeros_like(g)).double()
    assert torch.allclose(dw.double(), want, rtol=1e-4, atol=1e-4 * float(want.abs().max()) + 1e-6)


@pytest.mark.parametrize("name,layers", [("c1", 1), ("c1", 2), ("c3", 1), ("c3", 2), ("c4", 1)])
@pytest.mark.parametrize("what", ["SERIES_ENTRIES", "GATHERED_DINV_ROWS", "AGGREGATED_BYTES"])
def test_trainer_on_both_sides_of_its_size_rules(name, layers, what, monkeypatch):
    """The trainer at small sizes with the rules for large ones: rebuilds step by step, rows of X scaled beforehand, A~ X
    not kept."""
    from dtdg_synth import gradient
    from paper_2109_07893_amd import training
    wl = replace(WORKLOADS[name] if name == "c1" else WORKLOADS[name].scaled(1 << 11, T=5), layers=layers, window=3 if layers == 2 else 0)
    blk = make_block(wl, DEV, gen_device="cpu")
    g_y = torch.stack([gradient(wl, t) for t in range(1, wl.T + 1)]).to(DEV) + 1.0
    out = []
    for patched in (False, True):
        if patched:
            monkeypatch.setattr(training, what, 0)
        tr = training.make_trainer(wl, blk)
        assert tr.series == (not patched or what != "SERIES_ENTRIES")
        assert (tr.stack.p0 is not None) == (wl.dtype == "f32" and (not patched or what != "AGGREGATED_BYTES"))
        y = tr.forward()
        tr.backward(g_y.to(y.dtype))
        torch.cuda.synchronize()
        out.append((y.double().clone(), [d.double().clone() for d in tr.dw]))
    tol = 1e-5 if wl.dtype != "bf16" else 1e-2
    for a, b in zip([out[0][0]] + out[0][1], [out[1][0]] + out[1][1]):
        assert float((a - b).norm()) <= tol * float(b.norm())


@pytest.mark.parametrize("f,f2,T", [(16, 16, 1), (32, 32, 3), (64, 16, 5), (128, 32, 2), (16, 32, 130)])
def test_weight_recurrence_and_its_adjoint(f, f2, T):
    """All widths the one-launch recurrence takes; 130 steps: three launches of the adjoint."""
    import oracle
    from helpers import to_f64
    from paper_2109_07893_amd.evolve import EvolvingWeights
    gen = torch.Generator().manual_seed(T)
    w0 = torch.randn((f, f2), generator=gen) / f2 ** 0.5
    u_x, u_h = (torch.randn((f2, 4 * f2), generator=gen) / f2 ** 0.5 for _ in range(2))
    bias = torch.randn(4 * f2, generator=gen) * 0.1
    dw = [torch.randn((f, f2), generator=gen) for _ in range(T)]
    ev = EvolvingWeights(w0.to(DEV), u_x.to(DEV), u_h.to(DEV), bias.to(DEV), T)
    w_t = ev.forward()
    ev.backward([d.to(DEV) for d in dw])
    torch.cuda.synchronize()
    args = [to_f64(x) for x in (w0, u_x, u_h, bias)]
    ws, _ = oracle.evolve_weights(*args, T)
    for t in range(T):
        assert np.abs(to_f64(w_t[t]) - ws[t]).max() <= 1e-4, t
    want = oracle.evolve_weights_backward(*args, [to_f64(d) for d in dw])
    for got, exp in zip((ev.du_x, ev.du_h, ev.db, ev.dw0), want):
        assert np.abs(to_f64(got) - exp).max() <= 2e-4 * np.abs(exp).max()


def moved(t):
    """The same tensor object over other memory; what it lay in before is cleared."""
    old, new = t.view(-1), t.clone()
    t.set_(new)
    old.zero_()


def test_tensors_that_move_between_passes():
    """Nothing is kept of a call's tensors but the objects: features, lists, weights and frames that lie elsewhere in the next
    pass are found there."""
    blk = make_block(replace(WORKLOADS["c1"], layers=2), DEV, gen_device="cpu")
    runner = BlockRunner(blk)
    runner.load_first()
    runner.run_resident()
    want, want_rp = runner.z.clone(), runner.rowptr[runner.slot_of(blk.T)].clone()
    for t in [t for d in blk.deltas for t in d if t.numel()] + list(blk.x) + list(blk.w):
        moved(t)
    runner.z = torch.full_like(runner.z, float("nan"))
    runner.run_resident()
    torch.cuda.synchronize()
    assert torch.equal(runner.z, want) and torch.equal(runner.rowptr[runner.slot_of(blk.T)], want_rp)
    blk.x[0] = blk.x[0].double()
    with pytest.raises(ValueError):
        runner.run_resident()


def test_runner_whose_subclass_acts_per_snapshot():
    seen = []

    class Watching(BlockRunner):
        def snapshot_ready(self, t):
            seen.append(t)

    runner = Watching(make_block(WORKLOADS["c1"], DEV, gen_device="cpu"))
    runner.load_first()
    runner.run_resident()
    assert seen == list(range(1, runner.blk.T + 1))


@pytest.mark.parametrize("smoothed", [False, True])
def test_upstream_gradients_in_other_forms(smoothed):
    """Frames strided over the timesteps, and more of them than the block has, are taken; another type or place is refused."""
    from paper_2109_07893_amd import training
    wl = WORKLOADS["c3"].scaled(1 << 11, T=4)
    blk = make_block(wl, DEV, gen_device="cpu")
    tr = training.make_smoothed_trainer(wl, blk, 2) if smoothed else training.make_trainer(wl, blk)
    g = torch.randn((wl.T, wl.n, wl.f), device=DEV)
    spread = torch.empty((wl.T + 1, 2, wl.n, wl.f), device=DEV)
    spread[: wl.T, 0] = g
    out = []
    for form in (g, spread[:, 0], list(g)):
        tr.forward()
        tr.backward(form)
        torch.cuda.synchronize()
        out.append(tr.dw[0].clone())
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    for form in (g.double(), g.cpu(), g[:, :-1], g.transpose(1, 2).contiguous().transpose(1, 2)):
        with pytest.raises((ValueError, AssertionError)):
            tr.backward(form)


def test_cdgcn_layer_timestep_by_timestep():
    from paper_2109_07893_amd.cdgcn import CdgcnLayer
    gen = torch.Generator().manual_seed(3)
    wl = WORKLOADS["c1"]
    blk = make_block(wl, DEV, gen_device="cpu")
    w, w_x, w_h = (torch.randn(s, generator=gen).mul_(0.2).to(DEV) for s in ((16, 16), (32, 64), (16, 64)))
    layer = CdgcnLayer(blk, w, w_x, w_h, None, 16)
    layer.load_first()
    want = layer.run().clone()
    layer.h_all.zero_()
    layer.c.zero_()
    for t in range(1, blk.T + 1):
        if t >= 2:
            layer.rebuild(t, blk.deltas[t - 2])
        layer.step(t)
    torch.cuda.synchronize()
    assert torch.allclose(layer.h_all, want, rtol=1e-6, atol=1e-6)       # the same sums; a launch per step rounds the state alike


def test_long_series_of_dense_snapshots_go_step_by_step(monkeypatch):
    """Snapshots that would take too many bytes together: three slots again, the same frames and gradients."""
    from dtdg_synth import gradient
    from paper_2109_07893_amd import batch, training
    wl = replace(WORKLOADS["c1"], layers=2)
    blk = make_block(wl, DEV, gen_device="cpu")
    g_y = torch.stack([gradient(wl, t) for t in range(1, wl.T + 1)]).to(DEV)
    bytes_of_all = wl.T * (4 * max(blk.nnz) + 8 * wl.n)
    z, dw = [], []
    for limit in (bytes_of_all, bytes_of_all - 1):
        monkeypatch.setattr(batch, "SERIES_BYTES", limit)
        runner, tr = BlockRunner(blk, keep_all_z=True), training.make_trainer(wl, blk)
        assert runner.series == tr.series == (limit == bytes_of_all)
        assert len(runner.rowptr) == (wl.T if runner.series else 3)
        runner.load_first()
        runner.run_resident()
        tr.forward()
        tr.backward(g_y)
        torch.cuda.synchronize()
        z.append(runner.z.clone())
        dw.append([d.double().clone() for d in tr.dw])
    assert torch.equal(z[0], z[1])
    for a, b in zip(*dw):                                   # sums over timesteps in another order
        assert float((a - b).norm()) <= 1e-5 * float(b.norm())


@pytest.mark.parametrize("graph_kind,smoothed", [("er", False), ("rmat", False), ("rmat", True)])
def test_bf16_training_rounds_as_its_single_calls_do(graph_kind, smoothed):
    """A bf16 step, bit for bit: X W rounded per row and aggregated, going back G_H rounded per row and multiplied by X, one
    timestep after the other from the last one on.  (With A~ X rounded before the product, features of one sign leave the
    gradients up to three times as far from 64 bits.)"""
    from paper_2109_07893_amd import training
    wl = replace(graph(graph_kind, 1 << 11, 12, 5, 0.02, 0.03), f=64, dtype="bf16", layers=1, window=0)
    blk = make_block(wl, DEV, gen_device="cpu")
    blk.x = [x.abs() for x in blk.x]
    tr = training.make_smoothed_trainer(wl, blk, 3) if smoothed else training.make_trainer(wl, blk, keep_snapshots=True)
    g_y = torch.randn((wl.T, wl.n, wl.f), device=DEV).to(torch.bfloat16)
    y = tr.forward()
    tr.backward(g_y)
    h, gp, z = (torch.empty_like(blk.x[0]) for _ in range(3))
    dw = torch.zeros((wl.f, wl.f), device=DEV)
    ws_w = torch.empty(dg.weight_grad_workspace(wl.f, wl.f), dtype=torch.uint8, device=DEV)
    for t in range(wl.T - 1, -1, -1):
        if smoothed:
            (rp, ci, val), there, nnz, dinv = tr.s[t], tr.st[t], tr.s_nnz[t], tr.dinv_s[t]
        else:
            rp, ci, val, nnz, dinv = tr.a.rowptr[t], tr.a.colidx[t], None, blk.nnz[t], tr.a.dinv[t]
            there = (tr.at.rowptr[t], tr.at.colidx[t]) if tr.at is not None else (rp, ci)
        ws = torch.empty(dg.spmm_workspace(wl.n, nnz, wl.f), dtype=torch.uint8, device=DEV)

        def aggregate(snapshot, src, dst, flags):
            if val is None:
                dg.spmm(snapshot[0], snapshot[1], nnz, dinv, src, dst, ws, flags=flags | dg.DGNN_H_PRESCALED)
            else:
                dg.spmm_weighted(*snapshot, nnz, src, dst, ws, flags=flags | dg.DGNN_H_PRESCALED, dinv=dinv)
        dg.feature_transform(blk.x[t], blk.w[0], h, row_scale=dinv)
        aggregate((rp, ci, val), h, z, dg.DGNN_RELU)
        assert torch.equal(z, y[t]), t
        dg.relu_backward(g_y[t], z, gp, row_scale=dinv)
        aggregate(there, gp, h, 0)
        dg.weight_grad(blk.x[t], h, dw, ws_w, accumulate=t < wl.T - 1)
    assert torch.equal(dw, tr.dw[0])


@pytest.mark.parametrize("f_y,hidden", [(32, 32), (64, 32), (64, 64), (128, 64)])
def test_bf16_lstm_does_not_depend_on_the_steps_per_launch(f_y, hidden):
    """Every state is rounded to bf16 between two steps, whether or not they share a launch."""
    gen = torch.Generator(device=DEV).manual_seed(hidden + f_y)
    n, T = 333, 7
    y, h0, c0 = (torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16) for s in ((T, n, f_y), (n, hidden), (n, hidden)))
    w_x, w_h = (torch.randn(k, 4 * hidden, generator=gen, device=DEV).mul_(k ** -0.5).to(torch.bfloat16) for k in (f_y, hidden))
    bias = torch.randn(4 * hidden, generator=gen, device=DEV) * 0.1
    h, c, kept = torch.empty(T, n, hidden, dtype=y.dtype, device=DEV), torch.empty_like(c0), torch.empty(T, n, hidden, dtype=y.dtype, device=DEV)
    dg.lstm_series(y, h0, w_x, w_h, bias, c0, c, h)
    h_kept = torch.empty_like(h)
    dg.lstm_series(y, h0, w_x, w_h, bias, c0, kept, h_kept)
    state, prev, out = c0.clone(), h0, torch.empty_like(h)
    for t in range(T):
        dg.lstm_step(y[t], prev, w_x, w_h, bias, state, out[t])
        prev = out[t]
        assert torch.equal(kept[t], state), t
    assert torch.equal(h, out) and torch.equal(h_kept, out) and torch.equal(c, state)


def test_bf16_lstm_of_more_vertices_than_wavefronts_hold():
    """Wavefronts that walk several tiles of 32 vertices, a ragged last one among them: every vertex as in a call on its own slice."""
    gen = torch.Generator(device=DEV).manual_seed(5)
    n, T, f_y, hidden = 3 * 65536 + 45, 3, 128, 64
    y, h0, c0 = (torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16) for s in ((T, n, f_y), (n, hidden), (n, hidden)))
    w_x, w_h = (torch.randn(k, 4 * hidden, generator=gen, device=DEV).mul_(k ** -0.5).to(torch.bfloat16) for k in (f_y, hidden))
    c, h = torch.empty_like(c0), torch.empty(T, n, hidden, dtype=y.dtype, device=DEV)
    dg.lstm_series(y, h0, w_x, w_h, None, c0, c, h)
    for a in range(0, n, 50_000):
        rows = slice(a, min(a + 50_000, n))
        c_part, h_part = torch.empty_like(c0[rows]), torch.empty_like(h[:, rows])
        dg.lstm_series(y[:, rows].contiguous(), h0[rows], w_x, w_h, None, c0[rows], c_part, h_part)
        assert torch.equal(c[rows], c_part) and torch.equal(h[:, rows], h_part), a


def test_bf16_cdgcn_layer_does_not_depend_on_the_steps_per_launch():
    from paper_2109_07893_amd.cdgcn import CdgcnLayer
    gen = torch.Generator().manual_seed(4)
    wl = replace(WORKLOADS["c1"], f=32, dtype="bf16")
    blk = make_block(wl, DEV, gen_device="cpu")
    w, w_x, w_h = (torch.randn(s, generator=gen).mul_(0.2).to(torch.bfloat16).to(DEV) for s in ((32, 32), (64, 128), (32, 128)))
    layer = CdgcnLayer(blk, w, w_x, w_h, None, 32)
    layer.load_first()
    want, want_c = layer.run().clone(), layer.c.clone()
    layer.h_all.zero_()
    layer.c.zero_()
    for t in range(1, blk.T + 1):
        if t >= 2:
            layer.rebuild(t, blk.deltas[t - 2])
        layer.step(t)
    assert torch.equal(layer.h_all, want) and torch.equal(layer.c, want_c)


def test_rebinding_to_blocks_of_other_lengths():
    """A block, a shorter one with other weights, then one of full length again: every timestep takes the weights at hand."""
    from paper_2109_07893_amd.training import BlockTrainer
    wl = replace(graph("er", 700, 6, 6, 0.05, 0.05), f=32, layers=1, window=0)
    blk = make_block(wl, DEV, gen_device="cpu")

    def cut(T, w):
        return replace(blk, T=T, deltas=blk.deltas[:T - 1], x=blk.x[:T], nnz=blk.nnz[:T], w=[w])
    w = [torch.randn_like(blk.w[0]) for _ in range(2)]
    g_y = torch.randn((wl.T, wl.n, wl.f), device=DEV)
    tr = BlockTrainer(cut(6, w[0]), False)
    for T, k in ((6, 0), (2, 1), (6, 1), (3, 0), (5, 0)):
        part, fresh = cut(T, w[k]), BlockTrainer(cut(T, w[k]), False)
        tr.rebind(part)
        assert torch.equal(tr.forward(), fresh.forward()), (T, k)
        for t in (tr, fresh):
            t.backward(g_y[:T])
        assert torch.equal(tr.dw[0], fresh.dw[0]), (T, k)


@pytest.mark.parametrize("T,layers", [(5, 1), (5, 2), (34, 2)])
def test_smoothed_trainer_finds_its_first_snapshot_anew(T, layers):
    """A_1 (and its transpose) lies elsewhere in the next pass, or comes from the host with 64-bit indices.  34 timesteps: more
    than are smoothed in one call."""
    from paper_2109_07893_amd import training
    wl = replace(graph("rmat", 1 << 10, 8, T, 0.03, 0.03), f=16, layers=layers, window=0)
    blk = make_block(wl, DEV, gen_device="cpu")
    tr = training.make_smoothed_trainer(wl, blk, 3)
    g_y = torch.randn((wl.T, wl.n, wl.f), device=DEV)

    def step():
        y = tr.forward().clone()
        tr.backward(g_y)
        torch.cuda.synchronize()
        return [y] + [d.clone() for d in tr.dw]
    want = step()
    firsts = [blk.rowptr1, blk.colidx1] + (list(tr.t_first) if tr.t_first is not None else [])
    for t in firsts:
        moved(t)
    assert all(torch.equal(a, b) for a, b in zip(step(), want))
    blk.rowptr1, blk.colidx1 = blk.rowptr1.clone(), blk.colidx1.cpu().long()
    for t in firsts[:2]:
        t.zero_()
    assert all(torch.equal(a, b) for a, b in zip(step(), want))


def test_weight_recurrence_without_a_bias():
    from paper_2109_07893_amd.evolve import EvolvingWeights
    w0, u_x, u_h = torch.randn(32, 16, device=DEV), torch.randn(16, 64, device=DEV), torch.randn(16, 64, device=DEV)
    dw = [torch.randn(32, 16, device=DEV) for _ in range(4)]
    out = []
    for bias in (None, torch.zeros(64, device=DEV)):
        ev = EvolvingWeights(w0, u_x, u_h, bias, 4)
        ev.forward()
        ev.backward(dw)
        out.append((ev.w, ev.c, ev.dw0, ev.du_x, ev.du_h, ev.db))
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("kind", ["runner", "trainer", "smoothed", "checkpointed", "cdgcn"])
def test_memory_comes_back_with_the_last_reference(kind):
    """No driver holds itself: its buffers are free when it goes, without the garbage collector."""
    import gc
    from paper_2109_07893_amd import training
    from paper_2109_07893_amd.cdgcn import CdgcnTrainer
    wl = replace(graph("er", 2000, 6, 4, 0.05, 0.05), f=32, layers=2, window=0)
    blk = make_block(wl, DEV, gen_device="cpu")
    g_y = torch.randn((wl.T, wl.n, wl.f), device=DEV)
    weights = [torch.randn(s, device=DEV) for s in ((32, 32), (64, 128), (32, 128))]
    gc.collect()
    gc.disable()
    try:
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated(DEV)
        if kind == "runner":
            driver = BlockRunner(blk)
            driver.load_first()
            driver.run_resident()
        elif kind == "cdgcn":
            driver = CdgcnTrainer(blk, *weights, None, 32)
            driver.load_first()
        else:
            driver = {"trainer": training.make_trainer, "smoothed": lambda w, b: training.make_smoothed_trainer(w, b, 2),
                      "checkpointed": lambda w, b: training.CheckpointedTrainer(w, b, 2)}[kind](wl, blk)
        if kind != "runner":
            driver.forward()
            driver.backward(g_y)
        assert torch.cuda.memory_allocated(DEV) > before
        del driver
        assert torch.cuda.memory_allocated(DEV) == before
    finally:
        gc.enable()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("f", [16, 32, 128])
def test_a_nan_does_not_pass_the_relu(dtype, f):
    """The dense transform's ReLU gives 0 for a NaN of either sign, as the aggregation's does, and the gradient's mask is 0 there;
    infinities are ordinary values."""
    n, nan = 100, float("nan")
    x = torch.randn(n, f, device=DEV).to(dtype)
    x[3, 0], x[40, 1], x[41, 1] = nan, -nan, nan
    w, h = torch.eye(f, device=DEV).to(dtype), torch.empty_like(x)
    a = TransformTable(1)
    a.words[0] = (x.data_ptr(), w.data_ptr(), 0, h.data_ptr())
    dt = B.DGNN_F32 if dtype == torch.float32 else B.DGNN_BF16
    B.feature_transform_batch(1, a.at(), n, f, f, B.DGNN_RELU, dt, torch.cuda.current_stream().cuda_stream)
    want = torch.relu(x)
    want[[3, 40, 41]] = 0                                # a row with a NaN in it is all NaN behind the product
    assert torch.equal(h, want)
    z = torch.randn(n, f, device=DEV).to(dtype)
    g = torch.randn(n, f, device=DEV).to(dtype)
    z[5, :4] = torch.tensor([nan, -nan, float("inf"), -float("inf")], device=DEV).to(dtype)
    x = torch.randn(n, f, device=DEV).to(dtype)
    out, ws = [], torch.empty(dg.weight_grad_workspace(f, f), dtype=torch.uint8, device=DEV)
    for mask in (z, torch.nan_to_num(z, nan=0.0)):
        dw, table = torch.empty(f, f, device=DEV), WeightGradTable(1)
        table.words[0] = (x.data_ptr(), g.data_ptr(), mask.data_ptr(), dw.data_ptr())
        B.weight_grad_batch(1, table.at(), n, f, f, False, dt, ws, torch.cuda.current_stream().cuda_stream)
        out.append(dw)
    assert torch.equal(*out) and bool(torch.isfinite(out[0]).all())
    exp = x.double().T @ torch.where(torch.nan_to_num(z, nan=0.0) > 0, g, torch.zeros_like(g)).double()
    assert float((out[0] - exp).abs().max()) <= 1e-4 * n ** 0.5 * float(exp.abs().max())


@pytest.mark.parametrize("graph_kind", ["er", "rmat"])
@pytest.mark.parametrize("layers", [1, 2, 3])
def test_gradient_in_front_of_the_first_product(graph_kind, layers):
    """BlockTrainer.h after a step: A~_1^T of the first layer's masked gradient, whatever the number of layers."""
    from paper_2109_07893_amd import training
    wl = replace(graph(graph_kind, 512, 6, 4, 0.05, 0.05), f=16, layers=layers, window=0)
    blk = make_block(wl, DEV, gen_device="cpu")
    tr = training.make_trainer(wl, blk)
    g_y = torch.randn((wl.T, wl.n, wl.f), device=DEV)
    tr.forward()
    tr.backward(g_y)
    n, rows = wl.n, torch.repeat_interleave(torch.arange(wl.n, device=DEV), blk.rowptr1.diff())
    a = torch.zeros((n, n), dtype=torch.float64, device=DEV)
    a[rows, blk.colidx1.long()] = 1.0
    d = a.sum(1).rsqrt()
    a = d[:, None] * a * d[None, :]
    g = g_y[0].double()
    for layer in range(layers - 1, -1, -1):
        g = a.T @ torch.where(tr.z[layer, 0] > 0, g, torch.zeros_like(g))
        if layer > 0:
            g = g @ blk.w[layer].double().T
    assert float((tr.h - g).abs().max()) <= 1e-4 * float(g.abs().max())


@pytest.mark.parametrize("fused", [True, False])
def test_cdgcn_subclasses_are_asked_for_every_timestep(fused):
    from paper_2109_07893_amd.cdgcn import CdgcnLayer, CdgcnTrainer
    wl = replace(WORKLOADS["c1"], f=32)
    blk = make_block(wl, DEV, gen_device="cpu")
    weights = [torch.randn(s, device=DEV) * 0.2 for s in ((32, 32), (64, 128), (32, 128))]
    g_h = torch.randn((wl.T, wl.n, 32), device=DEV)
    seen = []

    class Steps(CdgcnLayer):
        def step(self, t):
            seen.append(t)
            super().step(t)

    class Forms:
        def form_y(self):
            seen.append(self.y.data_ptr())
            super().form_y()

    class FormsLayer(Forms, CdgcnLayer):
        pass

    class FormsTrainer(Forms, CdgcnTrainer):
        pass

    class SlotsOfItsOwn(BlockRunner):
        def slot_of(self, t):
            seen.append(t)
            return super().slot_of(t)
    plain = CdgcnLayer(blk, *weights, None, 32, fused=fused)
    plain.load_first()
    want = plain.run().clone()
    for kind in (Steps, FormsLayer):
        seen.clear()
        layer = kind(blk, *weights, None, 32, fused=fused)
        layer.load_first()
        assert torch.equal(layer.run(), want) and len(seen) == wl.T, kind
        assert kind is FormsLayer or seen == list(range(1, wl.T + 1))
    for keep in (True, False):
        grads = []
        for kind in (CdgcnTrainer, FormsTrainer):
            tr = kind(blk, *weights, None, 32, fused=fused, keep_activations=keep)
            tr.load_first()
            seen.clear()
            assert torch.equal(tr.forward(), want)
            tr.backward(g_h)
            grads.append([g.clone() for g in (tr.dw, tr.dw_x, tr.dw_h, tr.db)])
        assert len(seen) >= wl.T
        for a, b in zip(*grads):
            assert float((a - b).norm()) <= 1e-5 * float(a.norm())
    assert not SlotsOfItsOwn(blk).series and BlockRunner(blk).series


@pytest.mark.parametrize("hook", ["lstm_steps", "gcn_steps"])
def test_cdgcn_trainers_that_override_a_batch_of_steps_are_asked_in_turn(hook, monkeypatch):
    """Kept Y or not: the LSTM of a batch of timesteps right behind its GCN operations, before the next batch's."""
    from paper_2109_07893_amd import batch
    from paper_2109_07893_amd.cdgcn import CdgcnTrainer
    n, T = 1003, 7
    monkeypatch.setattr(batch, "BATCH_BYTES", 3 * n * 32 * 4)
    wl = replace(graph("er", n, 6, T, 0.05, 0.05), f=32, dtype="f32", layers=1, window=0)
    blk = make_block(wl, DEV, gen_device="cpu")
    weights = [torch.randn(s, device=DEV) * 0.2 for s in ((32, 32), (64, 128), (32, 128))]
    seen = []

    class Hooked(CdgcnTrainer):
        pass

    def asked(self, t, k, *rest):
        # h of the timesteps before is there
        seen.append((t, k, t == 0 or bool((self.h_all[t - 1] == want[t - 1]).all())))
        return getattr(CdgcnTrainer, hook)(self, t, k, *rest)
    for keep in (True, False):
        plain = CdgcnTrainer(blk, *weights, None, 32, keep_activations=keep)
        plain.load_first()
        want = plain.forward().clone()
        setattr(Hooked, hook, asked)
        tr = Hooked(blk, *weights, None, 32, keep_activations=keep)
        tr.h_all.fill_(float("nan"))
        tr.load_first()
        seen.clear()
        assert tr.together == 3 and torch.equal(tr.forward(), want)
        assert seen == [(0, 3, True), (3, 3, True), (6, 1, True)], keep


@pytest.mark.parametrize("dtype,f", [("f32", 32), ("f32", 16), ("bf16", 32)])
@pytest.mark.parametrize("n,T", [(1000, 5), (30_001, 7)])
def test_cdgcn_trainer_recomputes_what_it_was_not_asked_to_keep(dtype, f, n, T, monkeypatch):
    """Y0 and Y take memory only where they are asked for, and the gradients agree; 30 001 vertices: three timesteps together,
    several stretches going back."""
    from paper_2109_07893_amd import batch
    from paper_2109_07893_amd.cdgcn import CdgcnTrainer
    wl = replace(graph("er", n, 6, T, 0.05, 0.05), f=f, dtype=dtype, layers=1, window=0)
    blk = make_block(wl, DEV, gen_device="cpu")
    dt = blk.x[0].dtype
    weights = [(torch.randn(s, device=DEV) * 0.2).to(dt) for s in ((f, f), (2 * f, 4 * f), (f, 4 * f))]
    g_h = torch.randn((T, n, f), device=DEV).to(dt)
    if n > 1000:
        monkeypatch.setattr(batch, "BATCH_BYTES", 3 * n * f * weights[0].element_size())
    out, held = [], []
    for keep in (True, False):
        before = torch.cuda.memory_allocated(DEV)
        tr = CdgcnTrainer(blk, *weights, None, f, keep_activations=keep)
        assert tr.together == (T if n == 1000 else 3)
        tr.load_first()
        held.append(torch.cuda.memory_allocated(DEV) - before)
        h = tr.forward().clone()
        tr.backward(g_h)
        out.append([h] + [g.clone() for g in (tr.dw, tr.dw_x, tr.dw_h, tr.db)])
        del tr
    frames = n * 3 * f * weights[0].element_size()
    assert held[0] - held[1] >= (0 if n == 1000 else T * frames) // 2 and torch.equal(out[0][0], out[1][0])
    for a, b in zip(out[0][1:], out[1][1:]):
        assert float((a - b).norm()) <= 2e-5 * float(a.norm())


@pytest.mark.parametrize("layers,window", [(1, 0), (2, 3)])
def test_pinned_blocks_keep_three_slots_until_a_resident_pass(layers, window):
    """Passes over pinned lists need three snapshots' arrays; passes of either kind, in any order, give the same frames."""
    wl = replace(graph("er", 3000, 6, 9, 0.05, 0.05), f=16, layers=layers, window=window)
    blk = make_block(wl, DEV, pinned=True)
    plain = BlockRunner(replace(blk, pinned=None), keep_all_z=True)
    plain.load_first()
    plain.run_resident()
    runner = BlockRunner(blk, keep_all_z=True)
    assert runner.series and len(runner.rowptr) == 3 and len(plain.rowptr) == wl.T
    runner.load_first()
    for resident, overlap in ((False, False), (False, True), (True, True), (True, False), (False, False), (False, True), (True, False)):
        runner.z.zero_()
        (runner.run_resident if resident else runner.run_from_pinned)(overlap=overlap)
        torch.cuda.synchronize()
        assert torch.equal(runner.z, plain.z), (resident, overlap)
        a, b = runner.slot_of(wl.T), plain.slot_of(wl.T)
        assert torch.equal(runner.rowptr[a], plain.rowptr[b]) and torch.equal(runner.dinv[a], plain.dinv[b])
    assert len(runner.rowptr) == wl.T
    torch.cuda.synchronize()
    graph_ = runner.capture()
    for _ in range(3):
        runner.z.zero_()
        graph_.replay()
        torch.cuda.synchronize()
        assert torch.equal(runner.z, plain.z)


@pytest.mark.parametrize("graph_kind", ["er", "rmat"])
def test_checkpointed_blocks_decide_by_their_own_length(graph_kind, monkeypatch):
    """A~ X is kept where that of a block fits, whatever the length of the series."""
    from paper_2109_07893_amd import training
    wl = replace(graph(graph_kind, 1 << 10, 6, 9, 0.05, 0.05), f=16, layers=1, window=3)
    blk = make_block(wl, DEV, gen_device="cpu")
    g_y = torch.randn((wl.T, wl.n, wl.f), device=DEV)
    frame, grads = wl.n * wl.f * 4, []
    for limit, keeps in ((5 * frame, True), (4 * frame, False)):
        monkeypatch.setattr(training, "AGGREGATED_BYTES", limit)
        tr = training.CheckpointedTrainer(wl, blk, 5)
        assert (tr.trainer.stack.p0 is not None) == keeps
        tr.forward()
        tr.backward(g_y)
        grads.append(tr.dw[0].clone())
    assert float((grads[0] - grads[1]).norm()) <= 1e-5 * float(grads[0].norm())


@pytest.mark.parametrize("kind", ["trainer", "checkpointed", "evolving", "cdgcn"])
def test_trainers_find_moved_tensors(kind):
    """Features, weights and difference lists that lie elsewhere in the next step are found there, forward and back."""
    from paper_2109_07893_amd import training
    from paper_2109_07893_amd.cdgcn import CdgcnTrainer
    wl = replace(graph("rmat", 1 << 10, 8, 6, 0.05, 0.05), f=32, layers=1 if kind in ("cdgcn", "evolving") else 2, window=0)
    blk = make_block(wl, DEV, gen_device="cpu")
    g_y = torch.randn((wl.T, wl.n, wl.f), device=DEV)
    weights = [torch.randn(s, device=DEV) * 0.2 for s in ((32, 32), (64, 128), (32, 128), (128,))]
    if kind == "evolving":
        blk.w_t = [[torch.randn(32, 32, device=DEV)] for _ in range(wl.T)]
    if kind == "cdgcn":
        tr = CdgcnTrainer(blk, *weights, 32)
        tr.load_first()
        lists = blk.deltas
    else:
        tr = training.CheckpointedTrainer(wl, blk, 3) if kind == "checkpointed" else training.make_trainer(wl, blk)
        lists = list(blk.deltas) + list(getattr(tr, "t_deltas", None) or [])

    def step():
        tr.forward()
        tr.backward(g_y)
        torch.cuda.synchronize()
        grads = [tr.dw, tr.dw_x, tr.dw_h, tr.db] if kind == "cdgcn" else [d[0] for d in tr.dw_t] if kind == "evolving" else tr.dw
        return [g.clone() for g in grads]
    want = step()
    for t in [t for d in lists for t in d if t.numel()] + list(blk.x) + list(blk.w) + weights + [w[0] for w in blk.w_t or []]:
        moved(t)
    assert all(torch.equal(a, b) for a, b in zip(step(), want))
