"""The persistent LSTM kernels whatever wave of a workgroup runs first: lstm.hip compiled as host code (host_waves/), where the
order in which waves run between barriers is chosen by the test.  No GPU, and no timing that could hide a missing barrier."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from oracle import MIXED
from oracle import layers as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = os.environ.get("CLANG", "/opt/rocm/llvm/bin/clang++")

HOST = r"""
#include "lstm.hip"
namespace host {
int                 order[4] = {0, 1, 2, 3};
std::atomic<int>    worked[8];
thread_local Group* group    = nullptr;
}
namespace mp {
void set_error(const char* f, ...) { va_list v; va_start(v, f); vfprintf(stderr, f, v); va_end(v); }
int  hip_fail(hipError_t, const char*) { return -1; }
}
extern "C" int mp_fill_u32(size_t n, uint32_t value, void* dst, mp_stream) {
    std::fill_n(static_cast<uint32_t*>(dst), n, value);
    return MP_OK;
}
extern "C" void set_order(const int* o) { std::copy_n(o, 4, host::order); }
extern "C" void take_worked(int* n) { for (int i = 0; i < 8; ++i) n[i] = host::worked[i].exchange(0); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = str(tmp_path_factory.mktemp("waves"))
    src, so = os.path.join(tmp, "lstm_host.cpp"), os.path.join(tmp, "lstm_host.so")
    with open(src, "w") as f:
        f.write(HOST)
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-pthread", "-I", os.path.join(ROOT, "tests", "host_waves"),
                    "-I", os.path.join(ROOT, "paper_1805_10387_amd", "csrc"), "-I", os.path.join(ROOT, "include"), src, "-o", so], check=True)
    lib = C.CDLL(so)
    for n in ("mp_lstm_layer_workspace_bytes", "mp_lstm_layer_desc_workspace_bytes"):
        getattr(lib, n).restype = C.c_size_t
    return lib


def _aligned(shape, dtype, fill=0):
    n = int(np.prod(shape)) * np.dtype(dtype).itemsize
    raw = np.zeros(n + 64, np.uint8)
    lead = -raw.ctypes.data % 64
    a = raw[lead:lead + n].view(dtype).reshape(shape)
    a[...] = fill
    return a


def _layer(lib, order, T, Bn, I, H, x_seq, w, b, dh_seq, placed=False):
    """(gates, c, xh, h_up, dgates) of one layer through mp_lstm_layer_fwd and mp_lstm_layer_bwd, or the placed calls."""
    from paper_1805_10387_amd import _lib
    p = lambda a: a.ctypes.data_as(C.c_void_p)
    ld = I + H
    h = lambda shape: _aligned(shape, np.float16)
    wd, bd, dh, xh, up = h((4 * H, ld)), h(4 * H), h((T, Bn, H)), h((T, Bn, ld)), h((T, Bn, H))
    wd[...], bd[...], dh[...], xh[:, :, :I] = w, b, dh_seq, x_seq
    gx = _aligned((T, Bn, 4 * H), np.float32)
    gx[...] = x_seq.astype(np.float64) @ w[:, :I].astype(np.float64).T
    gates, c, dgates = h((T, Bn, 4 * H)), _aligned((T + 1, Bn, H), np.float32), h((T, Bn, 4 * H))
    status = _aligned(1, np.int32)
    d = _lib.LstmLayerDesc(T, Bn, I, H, ld, ld, H, 20_000_000, 0, Bn)
    n = lib.mp_lstm_layer_desc_workspace_bytes(C.byref(d))
    ws = _aligned(n, np.uint8)
    lib.set_order((C.c_int * 4)(*order))
    fwd, bwd = (lib.mp_lstm_layer_fwd_placed, lib.mp_lstm_layer_bwd_placed) if placed else (lib.mp_lstm_layer_fwd, lib.mp_lstm_layer_bwd)
    rest = (p(ws), C.c_size_t(n), *((0, None, C.c_size_t(0)) if placed else ()), None)
    assert fwd(C.byref(d), p(gx), p(wd), p(bd), p(gates), p(c), p(xh), p(up), p(status), *rest) == 0
    assert bwd(C.byref(d), p(wd), p(gates), p(c), p(dh), p(dgates), p(status), *rest) == 0
    assert status[0] == 0
    return gates, c, xh, up, dgates


def _inputs(T, Bn, I, H):
    r = np.random.default_rng(T * 100 + Bn + H)
    S = MIXED.store
    return (S(r.standard_normal((T, Bn, I))), S(r.uniform(-0.1, 0.1, (4 * H, I + H))), S(r.standard_normal(4 * H) * 0.1),
            S(r.standard_normal((T, Bn, H))))


@pytest.mark.parametrize("T,Bn,I,H", [(1, 3, 8, 64), (2, 8, 8, 64), (3, 11, 0, 64), (7, 5, 8, 128)])
def test_any_order_of_waves_gives_the_layer(lib, T, Bn, I, H):
    """Owners of cells ahead of the waves that fetch and store for them, and those ahead of the owners: the same bits, and the
    oracle's layer (fp16 storage: 1e-3, as for the device kernels)."""
    x_seq, w, b, dh_seq = _inputs(T, Bn, I, H)
    runs = [_layer(lib, o, T, Bn, I, H, x_seq, w, b, dh_seq) for o in ((0, 1, 2, 3), (2, 3, 0, 1), (3, 1, 2, 0))]
    runs.append(_layer(lib, (2, 3, 0, 1), T, Bn, I, H, x_seq, w, b, dh_seq, placed=True))
    f64 = lambda a: a.astype(np.float64)
    rel = lambda a, ref: np.linalg.norm(f64(a) - ref) / np.linalg.norm(ref)
    h_ref, (_, gates_ref, c_ref, _) = L.lstm_layer_fwd(MIXED, x_seq, w, b)
    for gates, c, xh, up, dgates in runs:
        assert rel(gates, gates_ref) <= 1e-3 and rel(up, h_ref) <= 1e-3 and rel(c, np.stack(c_ref)) <= 1e-3
        _, dw_ref, db_ref = L.lstm_layer_bwd(MIXED, dh_seq, (xh.astype(np.float32), gates.astype(np.float32), list(c), I), w)
        assert rel(f64(dgates).sum((0, 1)), db_ref) <= 1e-3
        assert rel(f64(dgates).reshape(T * Bn, -1).T @ f64(xh).reshape(T * Bn, -1), dw_ref) <= 1e-3
    for run in runs[1:]:
        for a, b_ in zip(runs[0], run):
            assert np.array_equal(a, b_, equal_nan=True)


@pytest.mark.parametrize("Bn,H", [(1, 192), (11, 128), (61, 64), (65, 64)])
def test_only_the_placed_calls_put_a_block_of_rows_on_one_xcd(lib, Bn, H):
    """Launches that together fit the device may run at the same time: the plain calls take the XCDs evenly, so that what fits the device
    fits every XCD, blocks of rows on one XCD or not.  The placed calls, which ask more of their caller, have all H / 16 workgroups of
    8 rows on one."""
    inputs, n = _inputs(1, Bn, 8, H), (C.c_int * 8)()
    units, groups = H // 16, -(-Bn // 8)
    for placed in (False, True):
        lib.take_worked(n)
        _layer(lib, (0, 1, 2, 3), 1, Bn, 8, H, *inputs, placed=placed)
        lib.take_worked(n)
        per = [k // 2 for k in n]                  # forward and backward
        assert sum(per) == units * groups
        if placed:
            assert all(k % units == 0 for k in per) and max(per) == -(-groups // 8) * units
        else:
            assert max(per) == -(-units * groups // 8)
