"""Host-side checks of the C boundary that need no GPU: the library loads, exports every entry
point that include/dgnn.h declares, and turns bad arguments into error codes before anything is
enqueued."""
import ctypes
import os
import re

import pytest

import paper_2109_07893_amd as dg
from paper_2109_07893_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(dg.library_path()):
        dg.build_library()
    return dg.load_library()


def declared_entry_points():
    text = open(os.path.join(ROOT, "include", "dgnn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dgnn_[a-z0-9_]+)\s*\(", text)))


def test_header_and_library_agree(lib):
    names = declared_entry_points()
    assert set(names) == set(binding.EXPORTS)
    for name in names:
        assert getattr(lib, name) is not None


def test_strerror(lib):
    assert dg.strerror(0) == "ok"
    for code in range(-7, 0):
        assert dg.strerror(code) != "unknown dgnn status"
    assert dg.strerror(-99) == "unknown dgnn status"


P = ctypes.c_void_p
FAKE = 0x1000  # never dereferenced: every call below must fail on the host first


def test_workspace_queries(lib):
    out = ctypes.c_size_t(0)
    assert lib.dgnn_delta_rebuild_workspace(1000, 11000, 500, 500, ctypes.byref(out)) == 0
    assert out.value >= 4 * 1001
    assert lib.dgnn_delta_rebuild_workspace(1000, 11000, 500, 500, None) == -1
    assert lib.dgnn_delta_rebuild_workspace(0, 1, 0, 0, ctypes.byref(out)) == -2
    assert lib.dgnn_delta_rebuild_workspace(1 << 31, 1, 0, 0, ctypes.byref(out)) == -4
    assert lib.dgnn_delta_rebuild_workspace(10, (1 << 31) - 2, 5, 0, ctypes.byref(out)) == -4
    assert lib.dgnn_spmm_workspace(1000, 11000, 32, ctypes.byref(out)) == 0 and out.value > 0
    assert lib.dgnn_spmm_workspace(1000, 11000, 24, ctypes.byref(out)) == -2
    assert lib.dgnn_spmm_workspace(1000, 1 << 31, 32, ctypes.byref(out)) == -4
    limit = (1 << 31) - (1 << 16) - 1               # the largest accepted count: kernels add a tile to an index in int32
    assert lib.dgnn_spmm_workspace(1000, limit, 32, ctypes.byref(out)) == 0
    assert lib.dgnn_spmm_workspace(1000, limit + 1, 32, ctypes.byref(out)) == -4


def test_delta_rebuild_argument_errors(lib):
    nn = ctypes.c_int64(0)

    def call(n=10, rp=FAKE, ci=FAKE, nnz=20, ar=FAKE, ac=FAKE, na=2, dr=FAKE, dc=FAKE, nd=1, rpn=FAKE + 64,
             cin=FAKE + 128, cap=64, dinv=None, ws=FAKE + 256, wsb=1 << 20, flags=0):
        return lib.dgnn_delta_rebuild(n, rp, ci, nnz, ar, ac, na, dr, dc, nd, rpn, cin, cap, ctypes.byref(nn), dinv,
                                      ws, wsb, flags, None, None)

    assert call(rp=None) == -1 and call(cin=None) == -1 and call(ws=None) == -1
    assert call(ar=None) == -1 and call(dc=None) == -1
    assert call(n=0) == -2 and call(na=-1) == -2 and call(flags=8) == -2
    assert call(cap=20) == -3            # needs 21
    assert call(wsb=8) == -3
    assert call(n=1 << 31) == -4
    assert call(rpn=FAKE) == -5 and call(cin=FAKE) == -5


def test_feature_transform_argument_errors(lib):
    f = lib.dgnn_feature_transform
    assert f(None, 10, 32, FAKE, 32, None, FAKE + 4096, 0, None) == -1
    assert f(FAKE, 0, 32, FAKE, 32, None, FAKE + 4096, 0, None) == -2
    assert f(FAKE, 10, 24, FAKE, 32, None, FAKE + 4096, 0, None) == -2
    assert f(FAKE, 10, 32, FAKE, 32, None, FAKE + 4096, 7, None) == -2
    assert f(FAKE + 4, 10, 32, FAKE, 32, None, FAKE + 4096, 0, None) == -7
    assert f(FAKE, 10, 32, FAKE + 64, 32, None, FAKE, 0, None) == -5


def test_spmm_argument_errors(lib):
    f = lib.dgnn_spmm
    ok = dict(n=10, nnz=20, rp=FAKE, ci=FAKE, dinv=None, h=FAKE, f=32, z=FAKE + 4096, dt=0, flags=0, ws=FAKE + 8192,
              wsb=1 << 24)

    def call(**kw):
        a = dict(ok, **kw)
        return f(a["n"], a["nnz"], a["rp"], a["ci"], a["dinv"], a["h"], a["f"], a["z"], a["dt"], a["flags"], a["ws"],
                 a["wsb"], None)

    assert call(rp=None) == -1 and call(z=None) == -1 and call(ws=None) == -1
    assert call(f=20) == -2 and call(flags=4) == -2 and call(n=-1) == -2 and call(nnz=0) == -2
    assert call(wsb=16) == -3
    assert call(h=FAKE + 8) == -7
    assert call(z=FAKE) == -5
    assert call(nnz=1 << 31) == -4


def test_spmm_static_argument_errors(lib):
    """The variant without a workspace argument refuses bad arguments, and sizes its fixed scratch array cannot serve,
    on the host, before it touches the device."""
    f = lib.dgnn_spmm_static
    limit = ctypes.c_size_t(0)
    assert lib.dgnn_spmm_static_limit(ctypes.byref(limit)) == 0 and limit.value == 32 << 20
    assert lib.dgnn_spmm_static_limit(None) == -1
    assert f(10, 20, None, FAKE, None, FAKE, 32, FAKE + 4096, 0, 0, None) == -1
    assert f(10, 20, FAKE, FAKE, None, FAKE, 24, FAKE + 4096, 0, 0, None) == -2
    assert f(10, 20, FAKE, FAKE, None, FAKE, 32, FAKE + 4096, 0, 8, None) == -2
    assert f(10, 1 << 31, FAKE, FAKE, None, FAKE, 32, FAKE + 4096, 0, 0, None) == -4
    need = ctypes.c_size_t(0)
    assert lib.dgnn_spmm_workspace(1 << 20, 1 << 29, 128, ctypes.byref(need)) == 0 and need.value > limit.value
    assert f(1 << 20, 1 << 29, FAKE, FAKE, None, FAKE, 128, FAKE + 4096, 0, 0, None) == -3


def test_mproduct_argument_errors(lib):
    f = lib.dgnn_mproduct
    assert f(None, FAKE, 8, 10, 16, 3, None, 0, None) == -1
    assert f(FAKE, FAKE, 0, 10, 16, 3, None, 0, None) == -2
    assert f(FAKE, FAKE, 8, 10, 16, 0, None, 0, None) == -2
    assert f(FAKE, FAKE, 64, 10, 16, 33, None, 0, None) == -2           # window beyond the register ring
    assert f(FAKE, FAKE + 16, 8, 10, 16, 3, None, 0, None) == -5        # partial overlap
    assert f(FAKE, FAKE + 4, 8, 10, 16, 3, None, 0, None) == -7


def test_misc_argument_errors(lib):
    assert lib.dgnn_csr_dinv(10, None, FAKE, None) == -1
    assert lib.dgnn_csr_dinv(0, FAKE, FAKE, None) == -2
    assert lib.dgnn_delta_h2d(None, None, 3, None, None, 0, None, None, None, None, None) == -1
    assert lib.dgnn_delta_h2d(None, None, 0, None, None, 0, None, None, None, None, None) == 0
    assert lib.dgnn_delta_h2d(None, None, -1, None, None, 0, None, None, None, None, None) == -2


def test_python_binding_rejects_wrong_dtypes():
    import torch
    x = torch.zeros((4, 16), dtype=torch.float64)
    with pytest.raises(TypeError):
        dg.feature_transform(x, x, x)
    rp = torch.zeros(5, dtype=torch.int64)
    with pytest.raises(TypeError):
        dg.csr_dinv(rp, torch.zeros(4))


def test_backward_argument_errors(lib):
    out = ctypes.c_size_t(0)
    assert lib.dgnn_weight_grad_workspace(32, 64, ctypes.byref(out)) == 0 and out.value >= 32 * 64 * 4
    assert lib.dgnn_weight_grad_workspace(32, 64, None) == -1
    assert lib.dgnn_weight_grad_workspace(32, 48, ctypes.byref(out)) == -2
    big = 1 << 30
    f = lib.dgnn_weight_grad
    assert f(None, FAKE, 10, 32, 32, FAKE, 0, 0, FAKE, big, None) == -1
    assert f(FAKE, FAKE, 10, 32, 32, None, 0, 0, FAKE, big, None) == -1
    assert f(FAKE, FAKE, 0, 32, 32, FAKE, 0, 0, FAKE, big, None) == -2
    assert f(FAKE, FAKE, 10, 32, 20, FAKE, 0, 0, FAKE, big, None) == -2
    assert f(FAKE, FAKE, 10, 32, 32, FAKE, 0, 0, FAKE, 1024, None) == -3
    assert f(FAKE + 2, FAKE, 10, 32, 32, FAKE, 0, 0, FAKE, big, None) == -7
    f = lib.dgnn_relu_backward
    assert f(FAKE, None, None, FAKE, 10, 32, 0, None) == -1
    assert f(FAKE, FAKE, None, FAKE, 10, 33, 0, None) == -2
    assert f(FAKE, FAKE, None, FAKE, 10, 32, 5, None) == -2
    assert f(FAKE, FAKE + 8, None, FAKE, 10, 32, 0, None) == -7
    f = lib.dgnn_input_grad
    assert f(None, 10, 32, FAKE, 32, None, FAKE + 4096, 0, None) == -1
    assert f(FAKE, 10, 32, FAKE, 48, None, FAKE + 4096, 0, None) == -2
    assert f(FAKE, 10, 32, FAKE + 64, 32, None, FAKE, 0, None) == -5
    f = lib.dgnn_mproduct_backward
    assert f(None, FAKE, 8, 10, 16, 3, None, 0, None) == -1
    assert f(FAKE, FAKE, 8, 10, 16, 0, None, 0, None) == -2
    assert f(FAKE, FAKE + 16, 8, 10, 16, 3, None, 0, None) == -5
    f = lib.dgnn_mproduct_block
    assert f(FAKE, FAKE, 8, 10, 16, 3, None, 5, None, 2, 0, None) == -1          # frames promised but no pointer
    assert f(FAKE, FAKE, 8, 10, 16, 3, None, 5, FAKE + (1 << 20), 1, 0, None) == -2   # window 3 after 5 steps needs 2
    assert f(FAKE, FAKE, 8, 10, 16, 3, None, -1, None, 0, 0, None) == -2
    f = lib.dgnn_mproduct_backward_block
    assert f(FAKE, FAKE, 8, 10, 16, 3, None, 0, FAKE + (1 << 20), 3, 0, None) == -2
    assert f(FAKE, FAKE + (1 << 20), 8, 10, 16, 3, None, 0, FAKE + (1 << 20), 2, 0, None) == -5   # output over the hand-over
    f = lib.dgnn_mproduct_relu_backward_block
    far = [FAKE + (k << 20) for k in range(5)]
    assert f(far[0], None, far[2], far[3], 8, 10, 16, 3, 0, None, 0, 0, None) == -1
    assert f(far[0], far[1], None, far[3], 8, 10, 16, 3, 0, None, 0, 0, None) == -1
    assert f(far[0], far[1], far[2], far[3], 8, 10, 48, 3, 0, None, 0, 0, None) == -2
    assert f(far[0], far[1], far[2], far[3], 8, 10, 16, 33, 40, None, 0, 0, None) == -2           # the window is too long
    assert f(far[0], far[1] + 4, far[2], far[3], 8, 10, 16, 3, 0, None, 0, 0, None) == -7
    assert f(far[0], far[1], far[2], far[0], 8, 10, 16, 3, 0, None, 0, 0, None) == -5             # not in place
    assert f(far[0], far[3] + 16, far[2], far[3], 8, 10, 16, 3, 0, None, 0, 0, None) == -5
    assert f(far[0], far[1], far[2], far[3], 8, 10, 16, 3, 0, far[3], 2, 0, None) == -5
    for overlap in (0, 5120 - 4, -316):                                              # row_scale over g_p's first, over its last, from before it
        assert f(far[0], far[1], far[3] + overlap, far[3], 8, 10, 16, 3, 0, None, 0, 0, None) == -5


def test_weighted_argument_errors(lib):
    nn = ctypes.c_int64(0)

    def call(n=10, rp=FAKE, ci=FAKE, vp=FAKE, nnz=20, ar=FAKE, ac=FAKE, av=FAKE, na=2, dr=FAKE, dc=FAKE, nd=1, ur=FAKE,
             uc=FAKE, uv=FAKE, nu=1, rpn=FAKE + 64, cin=FAKE + 128, vn=FAKE + 256, cap=64, ws=FAKE + 512, wsb=1 << 20):
        return lib.dgnn_delta_rebuild_weighted(n, rp, ci, vp, nnz, ar, ac, av, na, dr, dc, nd, ur, uc, uv, nu, rpn, cin, vn,
                                               cap, ctypes.byref(nn), ws, wsb, 0, None, None)

    assert call(vp=None) == -1 and call(vn=None) == -1 and call(av=None) == -1 and call(uv=None) == -1
    assert call(nu=-1) == -2 and call(n=0) == -2
    assert call(cap=20) == -3
    assert call(vn=FAKE) == -5
    f = lib.dgnn_spmm_weighted
    assert f(10, 20, FAKE, FAKE, None, None, FAKE, 32, FAKE + 4096, 0, 0, FAKE + 8192, 1 << 24, None) == -1
    assert f(10, 20, FAKE, FAKE, FAKE, None, FAKE, 32, FAKE + 4096, 0, 2, FAKE + 8192, 1 << 24, None) == -2   # pre-scaled needs dinv
    assert f(10, 20, FAKE, FAKE, FAKE, FAKE, FAKE, 32, FAKE + 4096, 0, 0, FAKE + 8192, 1 << 24, None) == -2   # dinv needs pre-scaled h
    assert f(10, 20, FAKE, FAKE, FAKE, None, FAKE, 32, FAKE, 0, 0, FAKE + 8192, 1 << 24, None) == -5
    assert lib.dgnn_csr_weighted_dinv(10, 20, FAKE, None, FAKE, FAKE, 1 << 20, None) == -1
    assert lib.dgnn_csr_weighted_dinv(0, 20, FAKE, FAKE, FAKE, FAKE, 1 << 20, None) == -2
    assert lib.dgnn_csr_weighted_dinv(10, 1 << 20, FAKE, FAKE, FAKE, FAKE, 64, None) == -3


def test_cdgcn_argument_errors(lib):
    f = lib.dgnn_concat_relu
    assert f(None, 32, FAKE, 32, FAKE + 4096, 10, 0, None) == -1
    assert f(FAKE, 24, FAKE, 32, FAKE + 4096, 10, 0, None) == -2
    assert f(FAKE, 32, FAKE, 32, FAKE, 10, 0, None) == -5
    assert f(FAKE, 32, FAKE + 4, 32, FAKE + 4096, 10, 0, None) == -7
    f = lib.dgnn_transform_concat_relu
    assert f(None, 10, 32, FAKE, 32, FAKE + 4096, 0, None) == -1 and f(FAKE, 10, 32, FAKE, 32, None, 0, None) == -1
    assert f(FAKE, 0, 32, FAKE, 32, FAKE + 4096, 0, None) == -2 and f(FAKE, 10, 24, FAKE, 32, FAKE + 4096, 0, None) == -2
    assert f(FAKE, 10, 128, FAKE, 32, FAKE + 4096, 0, None) == -2          # a width pair it has no kernel for
    assert f(FAKE, 10, 32, FAKE, 16, FAKE + 4096, 0, None) == -2 and f(FAKE, 10, 64, FAKE, 128, FAKE + 4096, 1, None) == -2
    assert f(FAKE, 10, 32, FAKE, 32, FAKE + 4096, 7, None) == -2
    assert f(FAKE, 10, 32, FAKE, 32, FAKE, 0, None) == -5 and f(FAKE + 4, 10, 32, FAKE, 32, FAKE + 4096, 0, None) == -7
    f = lib.dgnn_lstm_cell
    assert f(FAKE, FAKE, None, None, FAKE, FAKE + 64, 10, 32, 0, None) == -1
    assert f(FAKE, FAKE + 64, None, FAKE + 128, FAKE + 128, FAKE + 256, 10, 20, 0, None) == -2
    assert f(FAKE, FAKE + 64, None, FAKE + 128, FAKE + 128, FAKE + 128, 10, 32, 0, None) == -5   # h_next over the state
    assert f(FAKE, FAKE + 64, None, FAKE + 128, FAKE + 128, FAKE + 256, 0, 32, 0, None) == -2


def test_lstm_step_argument_errors(lib):
    f = lib.dgnn_lstm_step
    ok = [FAKE, 64, FAKE + 0x1000, FAKE + 0x2000, FAKE + 0x3000, None, FAKE + 0x4000, FAKE + 0x5000, 10, 32, 0, None]
    def call(**kw):
        a = list(ok)
        for k, v in kw.items():
            a[{"y": 0, "f_y": 1, "h_prev": 2, "c": 6, "h_next": 7, "n": 8, "hidden": 9, "dt": 10}[k]] = v
        return f(*a)
    assert call(y=None) == -1 and call(c=None) == -1
    assert call(f_y=128) == -2 and call(hidden=64) == -2 and call(dt=1, hidden=16, f_y=32) == -2 and call(dt=2) == -2 and call(n=0) == -2
    assert call(f_y=16) == -2 and call(hidden=16, f_y=64) == -2
    assert call(h_next=FAKE + 0x4000) == -5 and call(h_next=FAKE + 0x1000) == -5
    assert call(y=FAKE + 8) == -7


def test_csr_combine_argument_errors(lib):
    f = lib.dgnn_csr_combine

    def call(n=10, rp_s=FAKE, ci_s=FAKE, nnz_s=20, rp_a=FAKE, ci_a=FAKE, nnz_a=5, rp_c=FAKE + 4096, ci_c=FAKE + 8192,
             val_c=FAKE + 12288, cap=100, ws=FAKE + 16384, ws_bytes=1 << 20):
        return f(n, rp_s, ci_s, None, nnz_s, rp_a, ci_a, nnz_a, 1.0, None, None, 0, -1.0, 0.0, rp_c, ci_c, val_c, cap, None, ws,
                 ws_bytes, None)

    assert call(rp_s=None) == -1 and call(ci_s=None) == -1 and call(ci_a=None) == -1 and call(val_c=None) == -1
    assert call(ws=None) == -1
    assert call(n=0) == -2 and call(nnz_s=-1) == -2 and call(cap=-1) == -2
    assert call(nnz_s=(1 << 31) - (1 << 16) - 10, nnz_a=100) == -4
    assert call(ws_bytes=4) == -3
    assert call(rp_c=FAKE) == -5 and call(ci_c=FAKE) == -5
    assert call(ws=FAKE + 16384 + 4) == -7
    b = ctypes.c_size_t(0)
    assert lib.dgnn_csr_combine_workspace(1 << 20, ctypes.byref(b)) == 0 and b.value >= 4 * ((1 << 10) + 1)
    assert lib.dgnn_csr_combine_workspace(-1, ctypes.byref(b)) == -2


def test_transpose_argument_errors(lib):
    """Bad arguments are refused on the host, before the device or its sort are asked anything."""
    f = lib.dgnn_csr_transpose
    b = ctypes.c_size_t(0)
    assert lib.dgnn_csr_transpose_workspace(0, 10, 0, ctypes.byref(b)) == -2
    assert lib.dgnn_csr_transpose_workspace(10, -1, 0, ctypes.byref(b)) == -2
    assert lib.dgnn_csr_transpose_workspace(10, 1 << 31, 0, ctypes.byref(b)) == -4
    assert lib.dgnn_csr_transpose_workspace(10, 10, 0, None) == -1
    assert lib.dgnn_coo_transpose_workspace(0, 10, ctypes.byref(b)) == -2 and lib.dgnn_coo_transpose_workspace(10, 10, None) == -1
    assert f(10, 20, None, FAKE, None, FAKE + 4096, FAKE + 8192, None, FAKE + 16384, 1 << 20, None) == -1
    assert f(10, 20, FAKE, FAKE, FAKE, FAKE + 4096, FAKE + 8192, None, FAKE + 16384, 1 << 20, None) == -1      # values in, none out
    assert f(0, 20, FAKE, FAKE, None, FAKE + 4096, FAKE + 8192, None, FAKE + 16384, 1 << 20, None) == -2
    assert f(10, 20, FAKE, FAKE, None, FAKE, FAKE + 8192, None, FAKE + 16384, 1 << 20, None) == -5
    assert f(10, 20, FAKE, FAKE, None, FAKE + 4096, FAKE + 8192, None, FAKE + 16384 + 4, 1 << 20, None) == -7
    g = lib.dgnn_coo_transpose
    assert g(10, 5, None, FAKE, FAKE + 4096, FAKE + 8192, FAKE + 16384, 1 << 20, None) == -1
    assert g(10, -1, FAKE, FAKE, FAKE + 4096, FAKE + 8192, FAKE + 16384, 1 << 20, None) == -2


def test_cdgcn_backward_argument_errors(lib):
    f = lib.dgnn_lstm_cell_backward
    a = [FAKE + 4096 * k for k in range(9)]
    assert f(None, a[1], None, a[3], a[4], None, None, a[7], a[8], 10, 32, 0, None) == -1
    assert f(a[0], a[1], None, a[3], None, None, None, a[7], a[8], 10, 32, 0, None) == -1        # no gradient arrives
    assert f(a[0], a[1], None, a[3], a[4], None, None, a[7], a[8], 10, 24, 0, None) == -2
    assert f(a[0], a[1], None, a[3], a[4], None, None, a[7], a[8], 10, 32, 5, None) == -2
    assert f(a[0], a[1], None, a[3], a[4], None, None, a[7], a[7], 10, 32, 0, None) == -5
    assert f(a[0], a[1], None, a[3], a[4], None, None, a[7], a[4], 10, 32, 0, None) == -5
    assert f(a[0], a[1], None, a[3], a[4] + 4, None, None, a[7], a[8], 10, 32, 0, None) == -7
    f = lib.dgnn_concat_relu_backward
    assert f(a[0], a[1], None, 32, None, 32, 10, 0, None) == -1
    assert f(a[0], a[1], None, 32, a[3], 20, 10, 0, None) == -2
    assert f(a[0], a[1], a[0], 32, a[3], 32, 10, 0, None) == -5
    f = lib.dgnn_bias_grad
    assert f(a[0], 10, 128, None, 0, 0, a[2], 1 << 20, None) == -1
    assert f(a[0], 10, 24, a[1], 0, 0, a[2], 1 << 20, None) == -2            # 6 pieces per row: not a power of two
    assert f(a[0], 10, 1024, a[1], 0, 0, a[2], 1 << 22, None) == -2
    assert f(a[0], 10, 128, a[1], 0, 0, a[2], 1024, None) == -3
    b = ctypes.c_size_t(0)
    assert lib.dgnn_bias_grad_workspace(128, ctypes.byref(b)) == 0 and b.value == 1024 * 128 * 4


def test_add_argument_errors(lib):
    f = lib.dgnn_add
    assert f(None, FAKE, FAKE, 10, 32, 0, None) == -1
    assert f(FAKE, FAKE, FAKE, 0, 32, 0, None) == -2 and f(FAKE, FAKE, FAKE, 10, 33, 0, None) == -2
    assert f(FAKE, FAKE + 8, FAKE, 10, 32, 0, None) == -7


def test_lstm_step_backward_argument_errors(lib):
    f = lib.dgnn_lstm_step_backward
    a = [FAKE + 4096 * k for k in range(12)]
    ok = dict(y=a[0], f_y=64, h=a[1], wx=a[2], wh=a[3], c=a[4], dh=a[5], da=a[6], dc=a[7], hidden=32, dt=0)

    def call(**kw):
        p = dict(ok, **kw)
        return f(p["y"], p["f_y"], p["h"], p["wx"], p["wh"], None, p["c"], p["dh"], None, None, p["da"], p["dc"], 10, p["hidden"],
                 p["dt"], None)

    assert call(y=None) == -1 and call(da=None) == -1 and call(dh=None) == -1
    assert call(f_y=16) == -2 and call(hidden=64) == -2 and call(dt=2) == -2 and call(dt=1, hidden=64) == -2
    assert call(da=a[0]) == -5 and call(dc=a[5]) == -5
    assert call(c=a[4] + 4) == -7


def test_csr_validate_argument_errors(lib):
    f = lib.dgnn_csr_validate
    assert f(10, None, FAKE, 20, 1, FAKE + 4096, None) == -1 and f(10, FAKE, FAKE, 20, 1, None, None) == -1
    assert f(10, FAKE, None, 20, 1, FAKE + 4096, None) == -1
    assert f(0, FAKE, FAKE, 20, 1, FAKE + 4096, None) == -2 and f(10, FAKE, FAKE, -1, 1, FAKE + 4096, None) == -2
    assert f(1 << 31, FAKE, FAKE, 20, 1, FAKE + 4096, None) == -4


def test_boundary_is_callable_from_plain_c(tmp_path):
    """A C99 program that includes include/dgnn.h, links libdgnn.so and calls it: host-side argument errors come back
    as codes without a GPU being touched (no compute call is made)."""
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    lib_dir = os.path.join(root, "paper_2109_07893_amd", "csrc")
    if not os.path.exists(os.path.join(lib_dir, "libdgnn.so")):
        pytest.skip("libdgnn.so has not been built")
    src = tmp_path / "use_dgnn.c"
    src.write_text(r'''
#include <stdio.h>
#include <string.h>
#include "dgnn.h"
int main(void) {
    size_t bytes = 0;
    int32_t fake[4] = {0, 0, 0, 0};
    if (strcmp(dgnn_strerror(DGNN_OK), "ok") != 0) return 1;
    if (dgnn_spmm_workspace(1000, 5000, 32, &bytes) != DGNN_OK || bytes == 0) return 2;
    if (dgnn_spmm_workspace(1000, 5000, 24, &bytes) != DGNN_ERR_SHAPE) return 3;
    if (dgnn_csr_combine_workspace(1 << 20, &bytes) != DGNN_OK || bytes < 4096) return 4;
    if (dgnn_csr_dinv(10, NULL, NULL, NULL) != DGNN_ERR_NULL) return 5;
    if (dgnn_csr_validate(0, fake, fake, 0, 1, fake, NULL) != DGNN_ERR_SHAPE) return 6;
    if (dgnn_mproduct(NULL, NULL, 4, 10, 32, 3, NULL, DGNN_F32, NULL) != DGNN_ERR_NULL) return 7;
    printf("boundary ok\n");
    return 0;
}
''')
    exe = tmp_path / "use_dgnn"
    subprocess.check_call(["gcc", "-std=c99", "-Wall", "-Werror", "-I", os.path.join(root, "include"), str(src), "-o", str(exe),
                           "-L", lib_dir, "-ldgnn", f"-Wl,-rpath,{lib_dir}", "-Wl,-rpath,/opt/rocm/lib"])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and "boundary ok" in out.stdout, (out.returncode, out.stdout, out.stderr)


def test_products_without_a_weight_take_no_flags(lib):
    """w NULL asks for the rows scaled and nothing else; a ReLU or a transposed w asked for beside it would be lost."""
    items = (ctypes.c_uint64 * 4)(FAKE, 0, FAKE + 4096, FAKE + 8192)
    for flags in (binding.DGNN_RELU, binding.DGNN_W_TRANSPOSED, binding.DGNN_RELU | binding.DGNN_W_TRANSPOSED):
        assert lib.dgnn_feature_transform_batch(1, items, 10, 32, 32, flags, 0, None) == -2
    assert lib.dgnn_feature_transform_batch(1, items, 10, 32, 64, 0, 0, None) == -2


def test_table_columns_follow_the_number_of_rows():
    """One weight stands for all timesteps of a pass, however many the passes before had."""
    from paper_2109_07893_amd.batch import Table
    table = Table(8, 2)
    for rows, value in ((4, 0xb), (8, 0xb), (3, 0xb), (8, 0xc), (2, 0xa), (8, 0xa)):
        table.refresh(1, [value], rows)
        assert (table.words[:rows, 1] == value).all(), (rows, value)
    table.refresh(1, [1, 2, 3], 3)
    table.refresh(1, [1, 2, 3, 4], 4)
    assert table.words[:4, 1].tolist() == [1, 2, 3, 4] and not table.words[:, 0].any()


def test_spmm_static_takes_as_many_ranges_as_fit(lib):
    """A record of 16 bytes and two partial rows per range of at most 8192 entries, whatever the width and type.  (The call
    that fits gets past the size check and is refused for its misaligned h, or without a device.)"""
    for f in (16, 32, 64, 128):
        most = ((32 << 20) - 512) // (16 + 8 * f) * 8192
        for dt in (0, 1):
            def call(nnz):
                return lib.dgnn_spmm_static(1 << 20, nnz, FAKE, FAKE, None, FAKE + 4, f, FAKE + 4096, dt, 0, None)
            assert call(most) in (-6, -7) and call(most + 1) == -3, (f, dt)


@pytest.mark.parametrize("before", [1, 30, 31])
def test_series_refuses_a_step_from_an_empty_snapshot(lib, before):
    """... as the single call does; 31 steps in front of it: the next launch would begin with it."""
    steps = before + 1
    table = (ctypes.c_uint64 * (9 * steps))()
    for k in range(steps):
        n_add, n_del = (0, 20) if k == before - 1 else (5, 0) if k == before else (0, 0)
        table[9 * k:9 * k + 9] = [FAKE, FAKE, FAKE, FAKE, n_add, n_del, FAKE + 64 * (2 * k + 1), FAKE + 64 * (2 * k + 2), 0]
    call = lib.dgnn_delta_rebuild_series
    assert call(10, FAKE, FAKE, 20, steps, table, 64, FAKE, 0, None) == -2
    assert call(10, FAKE, FAKE, 20, before, table, 64, FAKE, 0, None) == -3      # up to the empty one: on to the workspace, which is too small
    single = lib.dgnn_delta_rebuild(10, FAKE, FAKE, 0, FAKE, FAKE, 5, FAKE, FAKE, 0, FAKE + 64, FAKE + 128, 64, None, None, FAKE, 1 << 20, 0, None, None)
    assert single == -2


def test_batched_aggregations_are_checked_before_the_first_of_them(lib):
    """Faults of the 33rd item, which a second launch would take: a dinv that the others have not, a workspace too small."""
    def items(odd=None, count=33):
        table = (ctypes.c_uint64 * (7 * count))()
        for k in range(count):
            table[7 * k:7 * k + 7] = [FAKE, FAKE, odd if odd is not None and k == 32 else 0, 0, FAKE, FAKE + 4096, 20]
        return table
    call = lib.dgnn_spmm_batch
    assert call(10, 33, items(odd=FAKE), 32, 0, 0, FAKE, 1 << 24, None) == -2
    need, whole = ctypes.c_size_t(0), ctypes.c_size_t(0)
    assert lib.dgnn_spmm_batch_workspace(1, 20, 32, ctypes.byref(need)) == 0 and need.value > 0
    assert lib.dgnn_spmm_batch_workspace(33, 20, 32, ctypes.byref(whole)) == 0 and whole.value >= 33 * need.value
    assert call(10, 33, items(), 32, 0, 0, FAKE, 1000, None) == -3
    one = 256 + 256                                  # a record and two rows of 32 floats, each rounded up to 256 bytes
    assert call(10, 33, items(), 32, 0, 0, FAKE, 33 * one - 1, None) == -3


def test_scratch_of_many_dense_snapshots_on_few_vertices(lib):
    """Aggregations enqueued together: frames of 1 MB would let 512 of 4 M entries share a batch, whose scratch is that of 32."""
    import torch
    from paper_2109_07893_amd.batch import BATCH_BYTES, SpmmTable, steps_together
    from paper_2109_07893_amd.pipeline import BlockInputs
    from paper_2109_07893_amd.training import GcnStack
    n, f, entries = 2048, 128, 2048 * 2048
    assert steps_together(n * f * 4, 10_000) == BATCH_BYTES // (n * f * 4) == 512
    size = ctypes.c_size_t(0)
    for count in (1, 31, 32, 33, 512):
        assert lib.dgnn_spmm_batch_workspace(min(count, 32), entries, f, ctypes.byref(size)) == 0
        assert SpmmTable.workspace(count, entries, f) == size.value <= 32 * 35e6
    blk = BlockInputs(n=16, T=40, f=128, layers=1, window=0, rowptr1=torch.zeros(17, dtype=torch.int32), colidx1=torch.zeros(1, dtype=torch.int32),
                      deltas=[], x=[torch.zeros(16, 128)] * 40, w=[torch.zeros(128, 128)], nnz=[16] * 40)
    arrays = [[torch.zeros(17, dtype=torch.int32)] * 40 for _ in range(3)]
    stack = GcnStack(blk, 100_000, *arrays)
    assert stack.together == 40 and stack.ws_spmm.numel() == SpmmTable.workspace(32, 100_000, 128)


def test_a_series_needs_steps_enough_for_its_set_up(lib):
    """Blocks of one step are rebuilt as a series up to half the entries of longer ones."""
    import torch
    from paper_2109_07893_amd.batch import SERIES_ENTRIES, SERIES_ENTRIES_PER_STEP
    from paper_2109_07893_amd.pipeline import BlockInputs, BlockRunner
    lists = tuple(torch.zeros(1, dtype=torch.int32) for _ in range(4))
    for T, cap, series in ((2, SERIES_ENTRIES_PER_STEP, True), (2, SERIES_ENTRIES_PER_STEP + 1, False), (3, SERIES_ENTRIES, True),
                           (3, SERIES_ENTRIES + 1, False), (9, SERIES_ENTRIES, True), (1, 100, False)):
        blk = BlockInputs(n=10, T=T, f=16, layers=1, window=0, rowptr1=torch.zeros(11, dtype=torch.int32), colidx1=torch.zeros(1, dtype=torch.int32),
                          deltas=[lists] * (T - 1), x=[torch.zeros(10, 16)] * T, w=[torch.zeros(16, 16)], nnz=[cap] * T)
        assert BlockRunner(blk).series == series, (T, cap)
