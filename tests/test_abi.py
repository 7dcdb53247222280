"""Host-side checks that need no GPU: the library loads, exports every symbol include/mp.h declares, the ctypes
mirror of the structs has the C layout, and argument validation rejects bad calls before anything is enqueued."""
import ctypes as C
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "mp.h")


def _declared():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(mp_[a-z0-9_]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    from paper_1805_10387_amd import _lib
    lib = _lib.load()
    names = _declared()
    assert len(names) >= 20
    for n in names:
        assert hasattr(lib, n), f"{n} declared in mp.h but not exported"
        assert n in _lib.SIGNATURES, f"{n} has no ctypes signature"
    assert set(_lib.SIGNATURES) == set(names)


def test_binding_has_the_same_names():
    import paper_1805_10387_amd as mp
    for n in _declared():
        if n == "mp_last_error":
            continue
        assert hasattr(mp, n), f"binding lacks {n}"


def test_the_package_imports_on_a_torch_without_gpu_entry_points():
    """What needs no stream (versions, sizes, descriptions) works on such a torch; only a call that launches something asks for one."""
    import subprocess
    code = ("import torch\n"
            "for n in ('_cuda_getCurrentRawStream', '_cuda_getDevice'):\n"
            "    if hasattr(torch._C, n): delattr(torch._C, n)\n"
            "import paper_1805_10387_amd as mp\n"
            "assert mp.mp_version() >= 1 and mp.mp_loss_workspace_bytes(8, 8) > 0\n"
            "try:\n"
            "    mp.binding._stream()\n"
            "except (RuntimeError, AssertionError, AttributeError, TypeError) as e:\n"
            "    assert 'GPU' in str(e) or 'CUDA' in str(e) or torch.cuda.is_available(), e\n"
            "else:\n"
            "    assert False\n")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT)


def test_struct_layouts_match_the_header():
    from paper_1805_10387_amd import _lib
    assert C.sizeof(_lib.ScaleState) == 12 * 4 + _lib.MP_HISTORY * 8
    assert _lib.ScaleState.found_inf.offset == 28 and _lib.ScaleState.opt_step.offset == 32
    assert _lib.ScaleState.hist_scale.offset == 48
    assert C.sizeof(_lib.GemmDesc) == 8 * 4 + 6 * 8 + 4 * 4
    assert _lib.GemmDesc.sx_outer.offset == 32 and _lib.GemmDesc.alpha.offset == 80
    assert C.sizeof(_lib.TensorDesc) == 48 and C.sizeof(_lib.OptCfg) == 48
    hdr = open(HEADER).read()
    assert f"#define MP_HISTORY {_lib.MP_HISTORY}" in hdr


def test_version_tells_a_recurrent_layer_description_with_step_rows():
    """Version 1 had an unused last field in mp_lstm_layer_desc; what it holds has a meaning since version 2, which header,
    library and binding agree on."""
    from paper_1805_10387_amd import _lib
    assert "#define MP_VERSION 2\n" in open(HEADER).read() and _lib.load().mp_version() == 2
    assert _lib.LstmLayerDesc.step_rows.offset + 4 == C.sizeof(_lib.LstmLayerDesc) == 40
    d = _lib.LstmLayerDesc(4, 8, 0, 128, 128, 128, 128)
    assert d.step_rows == 0


def test_validation_errors_enqueue_nothing():
    """NULL / malformed arguments are rejected on the host (no HIP call is made on these paths)."""
    from paper_1805_10387_amd import _lib
    lib = _lib.load()
    assert lib.mp_version() >= 1
    assert lib.mp_scale_state_init(None, 1, 2.0, 1, 1.0, 4.0, None) == _lib.MP_E_INVAL
    assert b"NULL" in lib.mp_last_error()
    assert lib.mp_loss_scale_update(None, None) == _lib.MP_E_INVAL
    d = _lib.GemmDesc()
    d.M, d.N, d.K, d.ldx, d.ldw, d.ldy, d.batch_outer, d.batch_inner, d.alpha = 8, 8, 8, 8, 8, 8, 1, 1, 1.0
    assert lib.mp_gemm_fwd(C.byref(d), None, None, None, None, None, None, None) == _lib.MP_E_INVAL
    d.ldx = 4
    assert lib.mp_gemm_bwd_dx(C.byref(d), 16, 16, None, None, 0, 16, None) == _lib.MP_E_INVAL
    assert b"leading dimension" in lib.mp_last_error()
    d.ldx = 8
    assert lib.mp_gemm_bwd_dw(C.byref(d), 16, 16, 16, None, None, None, 0, None) == _lib.MP_E_WORKSPACE
    cfg = _lib.OptCfg()
    cfg.kind = 7
    assert lib.mp_unscale_check_update(None, 0, C.byref(cfg), 16, 0, None) == _lib.MP_E_INVAL
    assert lib.mp_layernorm_fwd(4, 12, 16, None, 16, 16, 1e-5, 16, 16, 16, None) == _lib.MP_E_UNSUPPORTED
    assert lib.mp_mse_scaled(4, 8, 16, 16, 4, 16, 16, 16, None, 0, None) == _lib.MP_E_INVAL      # ld < cols
    # cross-entropy with the bias gradient: shape, NULL and workspace errors come before any launch
    assert lib.mp_softmax_xent_scaled_db(4, 8, 16, 4, 16, 16, 16, 16, 16, 16, 1 << 20, None) == _lib.MP_E_INVAL   # ld < vocab
    assert lib.mp_softmax_xent_scaled_db(4, 8, 16, 8, 16, 16, 16, 16, None, 16, 1 << 20, None) == _lib.MP_E_INVAL  # db NULL
    assert lib.mp_softmax_xent_scaled_db(4, 8, 16, 8, 16, 16, 16, 16, 16, 16, 8, None) == _lib.MP_E_WORKSPACE
    assert lib.mp_softmax_xent_db_workspace_bytes(0, 8) == 0
    assert lib.mp_softmax_xent_db_workspace_bytes(8192, 32768) >= 256 * 32768 * 4 + 8192 * 4
    assert C.sizeof(_lib.GemmGroupItem) == C.sizeof(_lib.GemmDesc) + 4 * 8
    # grouped weight gradients: empty / oversized lists, and shapes the grouped kernel does not take
    assert lib.mp_gemm_bwd_dw_grouped(None, 0, None, None) == _lib.MP_E_INVAL
    items = (_lib.GemmGroupItem * 9)()
    assert lib.mp_gemm_bwd_dw_grouped(items, 9, None, None) == _lib.MP_E_INVAL
    it = items[0]
    it.desc.M, it.desc.N, it.desc.K, it.desc.ldx, it.desc.ldw, it.desc.ldy = 128, 136, 128, 128, 128, 136
    it.desc.batch_outer = it.desc.batch_inner = 1
    it.desc.alpha = 1.0
    it.dY = it.X = it.dW = 256
    assert lib.mp_gemm_bwd_dw_grouped(items, 1, None, None) == _lib.MP_E_UNSUPPORTED     # 136 is not a multiple of 128
    assert b"mp_gemm_bwd_dw" in lib.mp_last_error()
    it.desc.N, it.desc.ldy, it.dW = 128, 128, None
    assert lib.mp_gemm_bwd_dw_grouped(items, 1, None, None) == _lib.MP_E_INVAL            # NULL operand
    # matrix-core rate probe: buffers are checked before anything is launched
    out = C.c_double(0.0)
    assert lib.mp_mfma_sustained_rate(None, 0, None, 0, 1, 1, C.byref(out), None) == _lib.MP_E_INVAL
    assert lib.mp_mfma_sustained_rate(256, 100, 256, 1 << 20, 256, 10, C.byref(out), None) == _lib.MP_E_INVAL   # too few operands
    assert lib.mp_mfma_sustained_rate(256, 16384, 256, 10, 256, 10, C.byref(out), None) == _lib.MP_E_INVAL      # sink too small
    assert lib.mp_mfma_sustained_rate(264, 16384, 256, 1 << 20, 256, 10, C.byref(out), None) == _lib.MP_E_INVAL  # misaligned


def test_workspace_queries_are_consistent():
    from paper_1805_10387_amd import _lib
    lib = _lib.load()
    d = _lib.GemmDesc()
    d.batch_outer = d.batch_inner = 1
    d.alpha = 1.0
    # big output, short contraction: no split, only the column-sum partials
    d.M, d.N, d.K, d.ldx, d.ldw, d.ldy = 8192, 4096, 1024, 1024, 1024, 4096
    no_db, with_db = lib.mp_gemm_bwd_dw_workspace_bytes(C.byref(d), 0), lib.mp_gemm_bwd_dw_workspace_bytes(C.byref(d), 1)
    assert with_db - no_db == lib.mp_colsum_workspace_bytes(8192, 4096) and no_db < (1 << 28)
    # small output, long contraction: split over K -> fp32 partials of (splits x N x K)
    d.M, d.N, d.K, d.ldx, d.ldw, d.ldy = 8192, 128, 256, 256, 256, 128
    split = lib.mp_gemm_bwd_dw_workspace_bytes(C.byref(d), 0)
    assert split >= 2 * 128 * 256 * 4 and (split - 256) % (128 * 256 * 4) == 0
    assert lib.mp_loss_workspace_bytes(8192, 32768) >= 8192 * 4
    assert lib.mp_layernorm_bwd_workspace_bytes(8192, 1024) % (2 * 1024 * 4) == 0


@pytest.mark.parametrize("d", [8, 192, 1024, 2048])
def test_a_layernorm_workspace_for_more_rows_is_enough_for_fewer(d):
    """What a call needs, mp_layernorm_bwd_nparts rows of partial sums, is in a workspace that was sized for a full batch."""
    from paper_1805_10387_amd import _lib
    lib = _lib.load()
    most = 0
    for rows in range(1, 9000):
        most = max(most, lib.mp_layernorm_bwd_nparts(rows, d) * 3 * d * 4)
        assert lib.mp_layernorm_bwd_workspace_bytes(rows, d) >= most


def test_joint_gradients_query_says_what_the_call_does():
    """mp_gemm_bwd_both_joint is 1 only where mp_gemm_bwd_both is one launch: a pair it names needs no workspace, and any
    other pair is refused without one before anything is launched."""
    from paper_1805_10387_amd import _lib
    lib = _lib.load()

    def desc(M, N, K, ldx=None, ldw=None, ldy=None, trans_w=0):
        d = _lib.GemmDesc()
        d.M, d.N, d.K, d.ldx, d.ldw, d.ldy = M, N, K, ldx or K, ldw or (N if trans_w else K), ldy or N
        d.batch_outer = d.batch_inner = 1
        d.trans_w, d.alpha = trans_w, 1.0
        return d

    joint = lambda x, w: lib.mp_gemm_bwd_both_joint(C.byref(x), C.byref(w))  # noqa: E731
    call = lambda x, w: lib.mp_gemm_bwd_both(C.byref(x), 256, 256, None, None, 0, 256, C.byref(w), 256, 256, None, None, None, 0, None)  # noqa: E731
    ok = desc(64, 256, 128)
    assert joint(ok, ok) == 1 and joint(desc(8, 8, 8), desc(8, 8, 8)) == 1 and joint(desc(100, 64, 40, ldw=104), desc(100, 64, 104)) == 1
    # rows of fewer than 8 elements, rows too far apart, a stored [K, N] weight, products that are not small
    for d in (desc(64, 256, 7), desc(64, 7, 256), desc(64, 4, 4), desc(64, 256, 128, ldx=1 << 24), desc(64, 256, 128, ldw=1 << 24),
              desc(64, 256, 128, ldy=1 << 24), desc(64, 256, 128, trans_w=1), desc(8192, 1024, 1024)):
        assert joint(d, d) == 0 and call(d, d) == _lib.MP_E_WORKSPACE
    assert joint(ok, desc(64, 256, 7)) == 0 and joint(desc(64, 256, 7), ok) == 0
    for w in (desc(65, 256, 128), desc(64, 248, 128, ldy=256), desc(64, 256, 128, ldy=264)):    # another dY: no pair
        assert joint(ok, w) == 0 and call(ok, w) == _lib.MP_E_INVAL


@pytest.mark.parametrize("cus", [256, 128, 32])
def test_recurrent_launches_leave_half_of_the_gpu(cus):
    """The blocks of batch rows that LSTMStep takes: in order, whole, each launch with at most one of the two workgroups
    per compute unit (16 units x 8 rows a workgroup), never many launches in a row; a batch of 32 always is persistent
    on the full chip."""
    from paper_1805_10387_amd.steps import lstm_row_blocks
    for hidden in range(64, 1025, 64):
        for batch in (1, 7, 8, 32, 33, 40, 64, 65, 100, 128, 200, 256, 500, 1024, 4096):
            blocks = lstm_row_blocks(batch, hidden, cus, 50)
            assert len(blocks) <= 4 and (blocks or batch > 32 or cus < 256)
            if blocks:
                assert [r for r, _ in blocks] == [sum(n for _, n in blocks[:k]) for k in range(len(blocks))]
                assert sum(n for _, n in blocks) == batch and all(n >= 1 for _, n in blocks)
                assert all(hidden // 16 * ((n + 7) // 8) <= cus and (r % 8 == 0) for r, n in blocks)
    # step by step is the faster plan beyond these
    assert lstm_row_blocks(128, 1024, 256, 50) and not lstm_row_blocks(129, 1024, 256, 50)
    assert lstm_row_blocks(256, 256, 256, 50) and not lstm_row_blocks(257, 256, 256, 50)
    # ... and several launches for sequences shorter than these
    for launches, steps in ((1, 1), (2, 3), (3, 5), (4, 9)):
        assert len(lstm_row_blocks(32 * launches, 1024, 256, steps)) == launches
        assert launches == 1 or not lstm_row_blocks(32 * launches, 1024, 256, steps - 1)


def test_product_never_imports_the_oracle():
    pkg = os.path.join(ROOT, "paper_1805_10387_amd")
    for fn in os.listdir(pkg):
        if fn.endswith(".py"):
            src = open(os.path.join(pkg, fn)).read()
            assert not re.search(r"^\s*(from|import)\s+oracle\b", src, flags=re.M), fn
    for fn in os.listdir(os.path.join(ROOT, "oracle")):
        if fn.endswith(".py"):
            src = open(os.path.join(ROOT, "oracle", fn)).read()
            assert "paper_1805_10387_amd" not in src, fn


def test_bench_refuses_more_than_one_gpu():
    """One GPU only: bench.py --gpus N with N > 1 exits with a message before touching any device."""
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0 and "ONE GPU" in r.stderr and r.stdout.strip() == ""
