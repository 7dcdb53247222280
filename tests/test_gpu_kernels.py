"""Per-kernel parity of the HIP library (through its C ABI) against the CPU oracle, element by element,
on seeded inputs whose sizes span several tiles and ragged tails.  Tolerances (north-star): contraction and
gradient outputs rel. Frobenius <= 1e-3, fp32 masters <= 1e-5, flags and scale sequence exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1805_10387_amd as mp
from paper_1805_10387_amd import _lib as ML
import mp_inputs as I
from oracle import MIXED
from oracle import layers as L
from oracle import optimizer as O
from oracle.numerics import half_bits
from gpu_util import *

RNG = lambda s: np.random.default_rng(1000 + s)
S16 = MIXED.store


def make_state(mode=ML.MP_SCALE_BACKOFF, scale=2.0 ** 15, interval=10, smin=1.0, smax=2.0 ** 24):
    st = mp.scale_state_alloc()
    mp.mp_scale_state_init(st, mode, scale, interval, smin, smax)
    return st


# ------------------------------------------------------------------ contractions
GEMM_SHAPES = [  # (M, N, K)
    (64, 1024, 256), (64, 256, 1024),          # config-1 layers
    (300, 200, 136), (257, 129, 72), (33, 520, 64), (512, 384, 1000), (8, 8, 8), (1, 40, 2048),
    (640, 512, 512),
]


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
@pytest.mark.parametrize("epi", ["none", "bias", "bias_relu"])
def test_gemm_fwd(M, N, K, epi):
    r = RNG(M + N + K)
    x, w, b = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K)) * 0.1), S16(r.standard_normal(N))
    ref = L.linear_fwd(MIXED, x, w, None if epi == "none" else b, relu=(epi == "bias_relu"))
    y = empty16(M, N)
    d = mp.gemm_desc(M, N, K, epilogue={"none": 0, "bias": 1, "bias_relu": 2}[epi])
    mp.mp_gemm_fwd(d, h16(x), h16(w), None if epi == "none" else h16(b), None, y)
    assert_close16(y, ref, 1e-3, max_ulp=1, what=f"fwd {M}x{N}x{K} {epi}")


@pytest.mark.parametrize("M,N,K", [(512, 384, 256), (300, 576, 136), (256, 192, 64), (1024, 3072, 128)])
def test_gemm_fwd_tile_256x192(M, N, K):
    """The 256 x 192 tile (contraction-contiguous operands only), forced: interior and ragged variants."""
    r = RNG(M + N + K + 5)
    x, w, b = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K)) * 0.1), S16(r.standard_normal(N))
    y = empty16(M, N)
    mp.mp_gemm_tuning_override(8, 1)
    try:
        mp.mp_gemm_fwd(mp.gemm_desc(M, N, K, epilogue=2), h16(x), h16(w), h16(b), None, y)
    finally:
        mp.mp_gemm_tuning_override(-1, 0)
    assert_close16(y, L.linear_fwd(MIXED, x, w, b, relu=True), 1e-3, max_ulp=1, what=f"fwd 256x192 tile {M}x{N}x{K}")


@pytest.mark.parametrize("tile,M,N,K", [(6, 1536, 1536, 1536), (6, 1536, 1536, 320), (6, 1536, 1536, 128),
                                        (3, 2560, 3456, 512), (0, 4352, 4096, 256)])
def test_gemm_workgroups_that_take_several_tiles(tile, M, N, K):
    """More tiles than resident workgroups: a workgroup goes on to a second tile, and with an even number (>= 4) of
    k-tiles the first k-tiles (and bias values) of that tile are fetched during the current one.  All three products,
    with the epilogues that read a second operand."""
    r = RNG(M + N + K + tile)
    x, w, b = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K)) * 0.1), S16(r.standard_normal(N))
    dy, src = S16(r.standard_normal((M, N))), S16(np.maximum(r.standard_normal((M, K)), 0))
    d = mp.gemm_desc(M, N, K, epilogue=2)
    y, dx, dw = empty16(M, N), empty16(M, K), empty16(N, K)
    st = make_state()
    ws = ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(d, False))
    mp.mp_gemm_tuning_override(tile, 1)
    try:
        mp.mp_gemm_fwd(d, h16(x), h16(w), h16(b), None, y)
        mp.mp_gemm_bwd_dx(mp.gemm_desc(M, N, K), h16(dy), h16(w), dx, relu_src=h16(src), ld_aux=K)
        mp.mp_gemm_bwd_dw(mp.gemm_desc(M, N, K), h16(dy), h16(x), dw, None, st, ws)
    finally:
        mp.mp_gemm_tuning_override(-1, 0)
    assert_close16(y, L.linear_fwd(MIXED, x, w, b, relu=True), 1e-3, max_ulp=1, what="fwd")
    assert_close16(dx, L.relu_mask(MIXED, MIXED.store(dy @ w), src), 1e-3, max_ulp=1, what="dx")
    assert_close16(dw, MIXED.store(dy.T @ x), 1e-3, max_ulp=1, what="dw")
    assert mp.scale_state_read(st).found_inf == 0


@pytest.mark.parametrize("tile,M,N,K", [(0, 4352, 4096, 256), (0, 512, 512, 32), (0, 256, 768, 1056), (1, 2304, 1152, 96),
                                        (2, 1152, 2304, 160), (3, 2560, 3456, 512), (3, 128, 128, 32), (4, 4352, 704, 320), (5, 704, 4352, 320),
                                        (8, 512, 384, 224)])
def test_gemm_direct_to_lds_kernels_all_layouts(tile, M, N, K):
    """The kernels whose operand tiles go from global memory straight into LDS (transposing LDS reads for output-contiguous
    operands), forced for every product they are built for: forward (both operands
    contraction-contiguous), dX (second operand output-contiguous) and dW (both output-contiguous), every tile shape,
    one and several tiles per workgroup (the load stream then runs on from tile to tile), contractions below (register-staged
    kernels), at and above the shortest they take, with the epilogues that read a second operand and the overflow flag."""
    r = RNG(M + N + K + tile + 3)
    x, w, b = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K)) * 0.1), S16(r.standard_normal(N))
    dy, src, other = S16(r.standard_normal((M, N))), S16(np.maximum(r.standard_normal((M, K)), 0)), S16(r.standard_normal((M, K)))
    d = mp.gemm_desc(M, N, K, epilogue=2)
    y, dx, dx2, dw = empty16(M, N), empty16(M, K), empty16(M, K), empty16(N, K)
    st = make_state()
    ws = ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(d, False))
    mp.mp_gemm_tuning_override(tile, 1)
    mp.mp_gemm_tuning_dtl(2)
    try:
        mp.mp_gemm_fwd(d, h16(x), h16(w), h16(b), None, y)
        mp.mp_gemm_bwd_dx(mp.gemm_desc(M, N, K), h16(dy), h16(w), dx, relu_src=h16(src), ld_aux=K)
        mp.mp_gemm_bwd_dx(mp.gemm_desc(M, N, K), h16(dy), h16(w), dx2, add=h16(other), ld_aux=K)
        mp.mp_gemm_bwd_dw(mp.gemm_desc(M, N, K), h16(dy), h16(x), dw, None, st, ws)
    finally:
        mp.mp_gemm_tuning_override(-1, 0)
        mp.mp_gemm_tuning_dtl(1)
    assert_close16(y, L.linear_fwd(MIXED, x, w, b, relu=True), 1e-3, max_ulp=1, what="fwd")
    base = MIXED.store(dy @ w)
    assert_close16(dx, L.relu_mask(MIXED, base, src), 1e-3, max_ulp=1, what="dx relu")
    assert_close16(dx2, L.add_store(MIXED, base, other), 1e-3, what="dx add")
    assert_close16(dw, MIXED.store(dy.T @ x), 1e-3, max_ulp=1, what="dw")
    assert mp.scale_state_read(st).found_inf == 0
    # the same weight gradient with the kernels switched off: the register-staged path stays covered
    dw0 = empty16(N, K)
    mp.mp_gemm_tuning_override(tile if tile != 8 else 0, 1)
    mp.mp_gemm_tuning_dtl(0)
    try:
        mp.mp_gemm_bwd_dw(mp.gemm_desc(M, N, K), h16(dy), h16(x), dw0, None, st, ws)
    finally:
        mp.mp_gemm_tuning_override(-1, 0)
        mp.mp_gemm_tuning_dtl(1)
    assert_close16(dw0, MIXED.store(dy.T @ x), 1e-3, max_ulp=1, what="dw, register-staged")
    with pytest.raises(mp.MPError):
        mp.mp_gemm_tuning_dtl(3)


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("rows,cols,depth,splits", [(264, 200, 192, 1), (1, 8, 256, 1), (257, 392, 320, 1), (3233, 1544, 448, 1),
                                                    (128, 256, 1024, 3), (136, 264, 1344, 4), (512, 384, 192, 1), (257, 256, 200, 1), (264, 392, 264, 1),
                                                    (4360, 4104, 192, 1), (4360, 4104, 200, 1), (136, 264, 1000, 3)])
def test_gemm_direct_to_lds_borders(tile, rows, cols, depth, splits):
    """The same kernels where output tiles stick out of the matrix (rows and columns just past a tile, far below one, several
    tiles per workgroup), at the shortest contraction they take (three k-tiles), with odd k-tile counts, with a last k-tile of 1, 5
    and 7 pieces, and with a split contraction whose last part is shorter.  Operands and outputs are blocks of larger arrays: NaN around the operands must not
    get in, nothing around an output may change.  mp_gemm_tuning_dtl(2) keeps the call on these kernels."""
    r = RNG(rows + cols + depth + tile)

    def block(a, pad):
        big = np.full((a.shape[0] + 3, a.shape[1] + pad), np.nan, np.float32)
        big[:a.shape[0], :a.shape[1]] = a
        return h16(big)[:a.shape[0], :a.shape[1]]

    def out(m, n, pad, dtype=torch.float16):
        big = torch.full((m + 3, n + pad), 7.0, dtype=dtype, device="cuda")
        return big, big[:m, :n]

    a, b, bias = S16(r.standard_normal((rows, depth))), S16(r.standard_normal((cols, depth)) * 0.1), S16(r.standard_normal(cols))
    other = S16(r.standard_normal((rows, cols)))
    ref = MIXED.store(a @ b.T)
    ws = ws_bytes(16 * rows * cols * 4 + 4096)
    mp.mp_gemm_tuning_override(tile, splits)
    mp.mp_gemm_tuning_dtl(2)
    try:
        big_y, y = out(rows, cols, 16)
        d = mp.gemm_desc(rows, cols, depth, ldx=depth + 8, ldw=depth + 16, ldy=cols + 16, epilogue=1)
        mp.mp_gemm_fwd_ws(d, block(a, 8), block(b, 16), h16(bias), None, y, ws=ws)
        big_x, dx = out(rows, cols, 8)
        d = mp.gemm_desc(rows, depth, cols, ldx=cols + 8, ldw=cols + 8, ldy=depth + 8)
        mp.mp_gemm_bwd_dx(d, block(a, 8), block(b.T, 8), dx, add=block(other, 24), ld_aux=cols + 24)
        dw_ok = rows % 8 == 0
        big_w, dw = out(rows, cols, 8)
        st = make_state()
        if dw_ok:
            d = mp.gemm_desc(depth, rows, cols, ldx=cols + 8, ldw=cols + 8, ldy=rows + 8)
            mp.mp_gemm_bwd_dw(d, block(a.T, 8), block(b.T, 8), dw, None, st, ws)
        f32 = torch.full((rows + 1, cols), 7.0, dtype=torch.float32, device="cuda")
        acc = torch.from_numpy(r.standard_normal((rows, cols)).astype(np.float32)).cuda()
        d = mp.gemm_desc(rows, cols, depth, ldx=depth + 8, ldw=depth + 16, alpha=0.5)
        mp.mp_gemm_fwd(d, block(a, 8), block(b, 16), None, acc, None, f32)
    finally:
        mp.mp_gemm_tuning_override(-1, 0)
        mp.mp_gemm_tuning_dtl(1)
    assert_close16(y, MIXED.store(a @ b.T + bias), 1e-3, max_ulp=1, what="fwd")
    assert_close16(dx, L.add_store(MIXED, ref, other), 1e-3, what="dx add")
    # fp32: sums of `depth` products in any order
    got, want = f32[:rows].cpu().numpy(), 0.5 * (a.astype(np.float64) @ b.T.astype(np.float64)) + acc.cpu().numpy()
    bound = 2.0 ** -24 * depth * (0.5 * (np.abs(a).astype(np.float64) @ np.abs(b).T) + np.abs(acc.cpu().numpy())) + 2.0 ** -23 * np.abs(want)
    assert np.all(np.abs(got - want) <= bound)
    assert torch.all(f32[rows:] == 7.0)
    for big in [big_y, big_x] + ([big_w] if dw_ok else []):
        assert torch.all(big[rows:] == 7.0) and torch.all(big[:, cols:] == 7.0)
    if dw_ok:
        assert_close16(dw, ref, 1e-3, max_ulp=1, what="dw")
        assert mp.scale_state_read(st).found_inf == 0


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("rows,cols,depth", [(33, 9, 192), (257, 391, 320), (1021, 2051, 256), (128, 258, 192)])
def test_gemm_direct_to_lds_ragged_outputs(tile, rows, cols, depth):
    """Forward products on aligned operands whose output has any width and element alignment (columns straddling a 16-byte piece
    by 1 to 7, odd leading dimensions, an odd bias address), with each epilogue, and no byte outside the
    output changes."""
    r = RNG(rows + cols + depth + tile)
    a, b, bias = S16(r.standard_normal((rows, depth))), S16(r.standard_normal((cols, depth)) * 0.1), S16(r.standard_normal(cols))
    bias_d = torch.zeros(cols + 1, dtype=torch.float16, device="cuda")
    bias_d[1:] = h16(bias)
    big = torch.full((rows + 2, cols + 3), 7.0, dtype=torch.float16, device="cuda")
    y = big.view(-1)[1:1 + rows * (cols + 3)].view(rows, cols + 3)[:, :cols]
    mp.mp_gemm_tuning_override(tile, 1)
    mp.mp_gemm_tuning_dtl(2)
    try:
        for epi, ref in ((0, a @ b.T), (1, a @ b.T + bias), (2, np.maximum(a @ b.T + bias, 0))):
            y.fill_(float("nan"))
            mp.mp_gemm_fwd(mp.gemm_desc(rows, cols, depth, ldy=cols + 3, epilogue=epi), h16(a), h16(b), bias_d[1:] if epi else None, None, y)
            assert_close16(y, MIXED.store(ref), 1e-3, max_ulp=1, what=f"epilogue {epi}")
        y.fill_(float("nan"))
        mp.mp_gemm_fwd(mp.gemm_desc(rows, cols, depth, ldy=cols + 3, alpha=0.5, epilogue=1), h16(a), h16(b), bias_d[1:], None, y)
    finally:
        mp.mp_gemm_tuning_override(-1, 0)
        mp.mp_gemm_tuning_dtl(1)
    assert_close16(y, MIXED.store(0.5 * (a @ b.T) + bias), 1e-3, max_ulp=1, what="scaled")
    flat = big.view(-1)
    keep = torch.ones(flat.numel(), dtype=torch.bool, device="cuda")
    keep[1:1 + rows * (cols + 3)].view(rows, cols + 3)[:, :cols] = False
    assert torch.all(flat[keep] == 7.0)


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("tokens,N,K,splits", [(193, 391, 264, 1), (255, 130, 8, 1), (321, 1, 200, 1), (1021, 2051, 392, 1), (1021, 135, 264, 3), (200, 256, 256, 1)])
def test_weight_gradients_of_any_token_count_direct_to_lds(tile, tokens, N, K, splits):
    """Weight gradients whose contraction is no multiple of 64 and whose output rows are no multiple of 8, on rows that are 16-byte
    pieces: NaN in the rows' padding and in the token rows beyond must not get in, nothing around the output may change."""
    r = RNG(tokens + N + K + tile)
    ld = (N + 7) // 8 * 8
    dy, x = S16(r.standard_normal((tokens, N)) * 0.1), S16(r.standard_normal((tokens, K)))

    def block(a, ldim):
        big = np.full((a.shape[0] + 70, ldim), np.nan, np.float32)
        big[:a.shape[0], :a.shape[1]] = a
        return h16(big)[:a.shape[0], :a.shape[1]]

    big = torch.full((N + 3, K + 8), 7.0, dtype=torch.float16, device="cuda")
    st = make_state()
    mp.mp_gemm_tuning_override(tile, splits)
    mp.mp_gemm_tuning_dtl(2)
    try:
        mp.mp_gemm_bwd_dw(mp.gemm_desc(tokens, N, K, ldx=K + 8, ldw=K + 8, ldy=ld), block(dy, ld), block(x, K + 8), big[:N, :K], None, st,
                          ws_bytes(16 * N * K * 4 + 4096))
    finally:
        mp.mp_gemm_tuning_override(-1, 0)
        mp.mp_gemm_tuning_dtl(1)
    assert_close16(big[:N, :K], MIXED.store(dy.T @ x), 1e-3, max_ulp=1, what="dw")
    assert torch.all(big[N:] == 7.0) and torch.all(big[:, K:] == 7.0)
    assert mp.scale_state_read(st).found_inf == 0


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_bwd_dx_and_dw(M, N, K):
    r = RNG(M * 3 + N + K)
    x, w = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K)) * 0.1)
    dy = S16(r.standard_normal((M, N)))
    dx_ref, dw_ref, db_ref = L.linear_bwd(MIXED, dy, x, w)
    d = mp.gemm_desc(M, N, K)
    dx = empty16(M, K)
    mp.mp_gemm_bwd_dx(d, h16(dy), h16(w), dx)
    assert_close16(dx, dx_ref, 1e-3, max_ulp=1, what="dx")
    dw, db = empty16(N, K), empty16(N)
    st = make_state()
    ws = ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(d, True))
    mp.mp_gemm_bwd_dw(d, h16(dy), h16(x), dw, db, st, ws)
    assert_close16(dw, dw_ref, 1e-3, max_ulp=1, what="dw")
    assert_close16(db, db_ref, 1e-3, max_ulp=1, what="db")
    assert mp.scale_state_read(st).found_inf == 0


@pytest.mark.parametrize("M,N,K", [(64, 128, 64), (300, 264, 136), (70, 90, 50), (70, 90, 10)])   # aligned, ragged, straddling, scalar kernel
def test_gemm_relu_epilogue_keeps_nonfinite_values(M, N, K):
    """max(x, 0) on a non-finite pre-activation: +inf stays +inf, -inf becomes 0 and NaN stays NaN, as in the
    oracle's definition.  A NaN that the epilogue dropped would hide a forward overflow from the gradient
    inspection (Section 3.1 item 1)."""
    r = RNG(M + N + K + 99)
    x, w, b = r.standard_normal((M, K)), r.standard_normal((N, K)) * 0.1, r.standard_normal(N)
    w[np.abs(w) < 1e-3] = 0.01                # (inf x 0 would make NaN on both sides, but keep the three cases apart)
    x[3, 5] = np.inf                          # row 3: +-inf by the sign of w[:, 5]
    x[7, 2] = np.nan                          # row 7: NaN everywhere
    x[9, 1], w[4, 1] = -np.inf, 0.0           # row 9: -+inf, and NaN where the weight is zero
    x, w, b = S16(x), S16(w), S16(b)
    with np.errstate(invalid="ignore"):
        ref = L.linear_fwd(MIXED, x, w, b, relu=True)
        ref_lin = L.linear_fwd(MIXED, x, w, b)
    assert np.isnan(ref[7]).all() and np.isnan(ref[9, 4]) and np.isposinf(ref[3]).any() and (ref[3] == 0).any()
    y = empty16(M, N)
    mp.mp_gemm_fwd(mp.gemm_desc(M, N, K, epilogue=2), h16(x), h16(w), h16(b), None, y)
    got = np32(y)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    assert not np.isneginf(got).any()
    assert_close16(y, ref, 1e-3, max_ulp=1, what="relu with non-finite inputs")
    mp.mp_gemm_fwd(mp.gemm_desc(M, N, K, epilogue=1), h16(x), h16(w), h16(b), None, y)
    got = np32(y)
    assert np.array_equal(np.isnan(got), np.isnan(ref_lin)) and np.array_equal(np.isneginf(got), np.isneginf(ref_lin))


def test_gemm_dx_relu_mask_and_residual_add():
    M, N, K = 200, 136, 264
    r = RNG(7)
    w, dy = S16(r.standard_normal((N, K)) * 0.1), S16(r.standard_normal((M, N)))
    src = S16(np.maximum(r.standard_normal((M, K)), 0))
    other = S16(r.standard_normal((M, K)))
    base = MIXED.store(dy @ w)
    d = mp.gemm_desc(M, N, K)
    out = empty16(M, K)
    mp.mp_gemm_bwd_dx(d, h16(dy), h16(w), out, relu_src=h16(src), ld_aux=K)
    assert_close16(out, L.relu_mask(MIXED, base, src), 1e-3, max_ulp=1, what="dx relu")
    assert np.all(np32(out)[src <= 0] == 0)
    mp.mp_gemm_bwd_dx(d, h16(dy), h16(w), out, add=h16(other), ld_aux=K)
    # one ulp of the intermediate rounding can exceed one ulp of the (possibly cancelling) sum: norm bound only
    assert_close16(out, L.add_store(MIXED, base, other), 1e-3, what="dx add")


@pytest.mark.parametrize("tile", [-1, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize("M,N,K", [(8, 8, 9), (65, 31, 63), (129, 257, 65), (260, 100, 71), (200, 523, 129)])
def test_gemm_extents_and_strides_of_any_parity(tile, M, N, K):
    """Extents that are no multiple of 8 (pieces that straddle the border, one to seven valid elements), odd leading
    dimensions and odd pointers, every tile shape: all three products with every epilogue, nothing written outside the
    output columns.  The bound is that of the aligned shapes: the sums differ from the oracle's in fp32 order only."""
    r = RNG(M + 3 * N + 7 * K)
    x, w, b = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K)) * 0.1), S16(r.standard_normal(N))
    dy, other = S16(r.standard_normal((M, N))), S16(r.standard_normal((M, K)))
    src = S16(np.maximum(other, 0))

    def odd(a):     # a matrix inside a wider one with an odd row length, starting at an odd element
        rows, cols = a.shape
        ld = cols + (3 if cols % 2 == 0 else 2)
        buf = torch.full((rows * ld + 9,), 7.0, dtype=torch.float16, device="cuda")
        v = buf[1:1 + rows * ld].view(rows, ld)
        v[:, :cols] = h16(a)
        return v, ld

    (xd, ldx), (wd, ldw), (dyd, ldy), (od, lda), (sd, _) = odd(x), odd(w), odd(dy), odd(other), odd(src)
    bd = torch.zeros(N + 1, dtype=torch.float16, device="cuda")
    bd[1:] = h16(b)
    outs = lambda rows, cols: odd(np.zeros((rows, cols)))[0]  # noqa: E731
    st = make_state()
    mp.mp_gemm_tuning_override(tile, 2)
    try:
        for epi in (0, 1, 2):
            y = outs(M, N)
            mp.mp_gemm_fwd(mp.gemm_desc(M, N, K, ldx=ldx, ldw=ldw, ldy=y.shape[1], epilogue=epi), xd, wd, bd[1:] if epi else None, None, y)
            assert_close16(y[:, :N], L.linear_fwd(MIXED, x, w, b if epi else None, relu=epi == 2), 1e-3, max_ulp=1, what=f"fwd {epi}")
            assert torch.all(y[:, N:] == 7.0)
        d = mp.gemm_desc(M, N, K, ldx=ldx, ldw=ldw, ldy=ldy)
        dx_ref, dw_ref, db_ref = L.linear_bwd(MIXED, dy, x, w)
        dx = outs(M, K)
        mp.mp_gemm_bwd_dx(d, dyd, wd, dx)
        assert_close16(dx[:, :K], dx_ref, 1e-3, max_ulp=1, what="dx")
        mp.mp_gemm_bwd_dx(d, dyd, wd, dx, relu_src=sd, ld_aux=lda)
        assert_close16(dx[:, :K], L.relu_mask(MIXED, dx_ref, src), 1e-3, max_ulp=1, what="dx relu")
        mp.mp_gemm_bwd_dx(d, dyd, wd, dx, add=od, ld_aux=lda)
        assert_close16(dx[:, :K], L.add_store(MIXED, dx_ref, other), 1e-3, what="dx add")
        assert torch.all(dx[:, K:] == 7.0)
        dw, db = outs(N, K), empty16(N)
        ws = ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(d, True))
        mp.mp_gemm_bwd_dw(d, dyd, xd, dw, db, st, ws)
        assert_close16(dw[:, :K], dw_ref, 1e-3, max_ulp=1, what="dw")
        assert_close16(db, db_ref, 1e-3, max_ulp=1, what="db")
        assert torch.all(dw[:, K:] == 7.0)
        # W stored [K, N] (the other orientation of the second operand), and an fp32 addend where N allows it
        wt, ldwt = odd(np.ascontiguousarray(w.T))
        y = outs(M, N)
        mp.mp_gemm_fwd(mp.gemm_desc(M, N, K, ldx=ldx, ldw=ldwt, ldy=y.shape[1], trans_w=1, alpha=0.5), xd, wt, None, None, y)
        assert_close16(y[:, :N], MIXED.store(np.float32(0.5) * (x @ w.T)), 1e-3, max_ulp=1, what="fwd, W[K,N], alpha")
        if N % 4 == 0:
            part = f32(dy)
            mp.mp_gemm_fwd(mp.gemm_desc(M, N, K, ldx=ldx, ldw=ldw, ldy=y.shape[1], epilogue=1), xd, wd, bd[1:], part, y)
            assert_close16(y[:, :N], MIXED.store((x @ w.T + dy) + b), 1e-3, max_ulp=1, what="fwd with addend")
    finally:
        mp.mp_gemm_tuning_override(-1, 1)
    assert mp.scale_state_read(st).found_inf == 0


@pytest.mark.parametrize("M,N,K", [(33, 45, 8), (33, 45, 12), (33, 45, 13), (17, 3855, 12), (17, 3856, 12), (1, 8, 9), (9, 40, 1)])
def test_gemm_short_ragged_contractions(M, N, K):
    """Contractions around the length, and outputs around the number, up to which ragged products take the scalar kernel, in
    each of the three products, at odd elements and leading dimensions; bounds as for the other shapes."""
    r = RNG(M + 3 * N + 7 * K)
    x, w, b = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K))), S16(r.standard_normal(N))
    (xd, ldx), (wd, ldw), (xt, ldxt), (wt, ldwt) = odd16(x), odd16(w), odd16(np.ascontiguousarray(x.T)), odd16(np.ascontiguousarray(w.T))
    ref = MIXED.store(x @ w.T)
    for what in ("fwd", "dx", "dw"):
        y, ldy = odd16(np.zeros((M, N)))
        y[:, :N] = float("nan")
        if what == "fwd":
            mp.mp_gemm_fwd(mp.gemm_desc(M, N, K, ldx=ldx, ldw=ldw, ldy=ldy, epilogue=1), xd, wd, h16(b), None, y)
        elif what == "dx":     # dY [M, K] W [K, N]
            mp.mp_gemm_bwd_dx(mp.gemm_desc(M, K, N, ldx=ldy, ldw=ldwt, ldy=ldx), xd, wt, y)
        else:                  # dY [K, M], X [K, N]
            d = mp.gemm_desc(K, M, N, ldx=ldwt, ldw=ldy, ldy=ldxt)
            mp.mp_gemm_bwd_dw(d, xt, wt, y, None, None, ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(d, False)))
        assert_close16(y[:, :N], L.linear_fwd(MIXED, x, w, b) if what == "fwd" else ref, 1e-3, max_ulp=1, what=what)
        assert torch.all(y[:, N:] == 7.0)


@pytest.mark.parametrize("outer,inner,M,N,K", [(3, 4, 13, 9, 16), (3, 4, 13, 9, 17), (16, 56, 16, 16, 9), (16, 57, 16, 16, 9)])
def test_gemm_short_ragged_batched_contractions(outer, inner, M, N, K):
    """The same rule over batches (outputs counted over all of them), batches side by side in rows of odd length."""
    r = RNG(outer + inner + M + K)
    x, w = S16(r.standard_normal((outer, M, inner * K))), S16(r.standard_normal((outer, N, inner * K)))
    pad = lambda a: np.concatenate([a, np.zeros(a.shape[:2] + (1 - a.shape[2] % 2,), np.float32)], 2)  # noqa: E731
    x, w = pad(x), pad(w)
    ld = x.shape[2]
    y = empty16(outer, inner, M, N)
    d = mp.gemm_desc(M, N, K, ldx=ld, ldw=ld, ldy=N, alpha=0.5, batch_outer=outer, batch_inner=inner, sx=(M * ld, K), sw=(N * ld, K),
                     sy=(inner * M * N, M * N))
    mp.mp_gemm_fwd(d, h16(x), h16(w), None, None, y)
    split = lambda a: a[:, :, :inner * K].reshape(outer, -1, inner, K).transpose(0, 2, 1, 3)  # noqa: E731
    assert_close16(y, MIXED.store(np.float32(0.5) * (split(x) @ split(w).transpose(0, 1, 3, 2))), 1e-3, max_ulp=1, what="batched")


def test_gemm_leading_dimensions_and_unaligned_fallback():
    r = RNG(8)
    M, N, K = 70, 90, 50                      # K, N not multiples of 8: pieces that straddle the rows' ends
    x, w = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K)))
    y = empty16(M, N)
    mp.mp_gemm_fwd(mp.gemm_desc(M, N, K), h16(x), h16(w), None, None, y)
    assert_close16(y, L.linear_fwd(MIXED, x, w), 1e-3, max_ulp=1, what="unaligned")
    # ld > cols, aligned: views into wider buffers
    M, N, K = 96, 72, 40
    xb, wb = S16(r.standard_normal((M, 64))), S16(r.standard_normal((N, 48)))
    yb = torch.full((M, 80), 7.0, dtype=torch.float16, device="cuda")
    mp.mp_gemm_fwd(mp.gemm_desc(M, N, K, ldx=64, ldw=48, ldy=80), h16(xb), h16(wb), None, None, yb)
    assert_close16(yb[:, :N], L.linear_fwd(MIXED, xb[:, :K], wb[:, :K]), 1e-3, max_ulp=1, what="ld")
    assert torch.all(yb[:, N:] == 7.0)        # nothing written outside the N columns


def test_gemm_fp32_addend_and_fp32_output():
    r = RNG(9)
    M, N, K1, K2 = 48, 264, 136, 72
    x1, x2 = S16(r.standard_normal((M, K1))), S16(r.standard_normal((M, K2)))
    w = S16(r.standard_normal((N, K1 + K2)) * 0.2)
    b = S16(r.standard_normal(N))
    ref = L.linear_fwd(MIXED, np.concatenate([x1, x2], 1), w, b)
    part = empty32(M, N)
    wd = h16(w)
    mp.mp_gemm_fwd(mp.gemm_desc(M, N, K1, ldw=K1 + K2), h16(x1), wd, None, None, None, part)
    y = empty16(M, N)
    mp.mp_gemm_fwd(mp.gemm_desc(M, N, K2, ldw=K1 + K2, epilogue=1), h16(x2), wd[:, K1:], h16(b), part, y)
    assert_close16(y, ref, 1e-3, max_ulp=1, what="split contraction")


@pytest.mark.parametrize("B,S,h,dk", [(3, 40, 4, 64), (2, 53, 3, 64), (2, 131, 2, 40), (3, 37, 2, 33), (1, 65, 5, 17), (2, 9, 3, 9)])
def test_gemm_attention_batched_strided(B, S, h, dk):
    """Q K^T, P V and their gradients on a fused qkv buffer, batch = (sequence, head), no copies.  Lengths and head sizes
    off 8: pieces that straddle the border, at odd batch strides and leading dimensions."""
    d_model, T = h * dk, B * S
    r = RNG(10)
    qkv = S16(r.standard_normal((T, 3 * d_model)))
    ctx_ref, cache = L.attention_fwd(MIXED, qkv, B, S, h)
    q, k, v, p, alpha = cache
    qkv_d = h16(qkv)
    s_d = empty16(B, h, S, S)
    ds = mp.gemm_desc(S, S, dk, ldx=3 * d_model, ldw=3 * d_model, ldy=S, alpha=float(alpha), batch_outer=B, batch_inner=h,
                      sx=(S * 3 * d_model, dk), sw=(S * 3 * d_model, dk), sy=(h * S * S, S * S))
    mp.mp_gemm_fwd(ds, qkv_d, qkv_d[:, d_model:], None, None, s_d)
    s_ref = MIXED.store(alpha * (q @ k.transpose(0, 1, 3, 2)))
    assert_close16(s_d, s_ref, 1e-3, max_ulp=1, what="scores")
    p_d = empty16(B, h, S, S)
    mp.mp_softmax_fwd(B * h * S, S, s_d, p_d, S)
    assert_close16(p_d, p, 1e-3, max_ulp=2, what="softmax")
    ctx_d = empty16(T, d_model)
    dc = mp.gemm_desc(S, dk, S, ldx=S, ldw=3 * d_model, ldy=d_model, trans_w=1, batch_outer=B, batch_inner=h,
                      sx=(h * S * S, S * S), sw=(S * 3 * d_model, dk), sy=(S * d_model, dk))
    mp.mp_gemm_fwd(dc, p_d, qkv_d[:, 2 * d_model:], None, None, ctx_d)
    assert_close16(ctx_d, ctx_ref, 1e-3, what="ctx")
    # backward (from the oracle's p so that the comparison isolates these kernels)
    dctx = S16(r.standard_normal((T, d_model)))
    dqkv_ref = L.attention_bwd(MIXED, dctx, cache)
    p_o, dctx_d = h16(p), h16(dctx)
    dp_d, dqkv_d = empty16(B, h, S, S), empty16(T, 3 * d_model)
    ws = ws_bytes(1 << 20)
    mp.mp_gemm_bwd_dx(dc, dctx_d, qkv_d[:, 2 * d_model:], dp_d)                     # dP = dctx V^T
    mp.mp_gemm_bwd_dw(dc, dctx_d, p_o, dqkv_d[:, 2 * d_model:], None, None, ws)      # dV = P^T dctx
    ds_d = empty16(B, h, S, S)
    mp.mp_softmax_bwd(B * h * S, S, p_o, dp_d, ds_d, S)
    mp.mp_gemm_bwd_dx(ds, ds_d, qkv_d[:, d_model:], dqkv_d)                          # dQ = alpha dS K
    mp.mp_gemm_bwd_dw(ds, ds_d, qkv_d, dqkv_d[:, d_model:], None, None, ws)          # dK = alpha dS^T Q
    assert_close16(dqkv_d, dqkv_ref, 1e-3, what="dqkv")


@pytest.mark.parametrize("B,S,h", [(3, 128, 2), (2, 40, 3), (5, 64, 1), (1, 8, 4), (2, 104, 2)])
def test_fused_attention_fwd_bwd(B, S, h):
    dk = 64
    d_model, T = h * dk, B * S
    r = RNG(B * 1000 + S + h)
    qkv = S16(r.standard_normal((T, 3 * d_model)))
    ctx_ref, cache = L.attention_fwd(MIXED, qkv, B, S, h)
    q, k, v, p_ref, alpha = cache
    qkv_d = h16(qkv)
    p_d = torch.zeros(B, h, S, S, dtype=torch.float16, device="cuda")
    ctx_d = torch.full((T, d_model + 8), 3.0, dtype=torch.float16, device="cuda")
    mp.mp_attention_fwd(B, h, S, dk, qkv_d, 3 * d_model, float(alpha), p_d, ctx_d, d_model + 8)
    assert_close16(p_d, p_ref, 1e-3, max_ulp=2, what="fused p")
    assert_close16(ctx_d[:, :d_model], ctx_ref, 1e-3, what="fused ctx")
    assert torch.all(ctx_d[:, d_model:] == 3.0)
    # backward from the GPU's own p (the stored tensor both sides would use)
    dctx = S16(r.standard_normal((T, d_model)))
    p_gpu = np32(p_d)
    dqkv_ref = L.attention_bwd(MIXED, dctx, (q, k, v, p_gpu, alpha))
    dqkv_d = torch.zeros(T, 3 * d_model, dtype=torch.float16, device="cuda")
    mp.mp_attention_bwd(B, h, S, dk, qkv_d, 3 * d_model, float(alpha), p_d, h16(dctx), d_model, dqkv_d, 3 * d_model)
    for name, lo in (("dq", 0), ("dk", d_model), ("dv", 2 * d_model)):
        assert_close16(dqkv_d[:, lo:lo + d_model], dqkv_ref[:, lo:lo + d_model], 1e-3, what=f"fused {name}")


@pytest.mark.parametrize("B,S,h,ld_p", [(3, 1, 2, 8), (2, 7, 1, 8), (2, 33, 3, 40), (3, 53, 2, 56), (2, 65, 1, 80), (2, 127, 2, 128),
                                        (2, 40, 2, 48)])
def test_fused_attention_rows_of_p_apart(B, S, h, ld_p):
    """Sequence lengths that are no multiple of 8, and rows of p further apart than needed: both directions against the
    oracle, zeros up to the next multiple of 8 behind a row of p and nothing written beyond; where the plain call takes the
    length, the same bits as it."""
    dk = 64
    d_model, T, pad = h * dk, B * S, (S + 7) // 8 * 8
    r = RNG(B * 1000 + S + h)
    qkv, dctx = S16(r.standard_normal((T, 3 * d_model))), S16(r.standard_normal((T, d_model)))
    ctx_ref, (q, k, v, p_ref, alpha) = L.attention_fwd(MIXED, qkv, B, S, h)
    qkv_d, p_d, ctx_d = h16(qkv), torch.full((B, h, S, ld_p), 3.0, dtype=torch.float16, device="cuda"), empty16(T, d_model)
    mp.mp_attention_fwd_ldp(B, h, S, dk, qkv_d, 3 * d_model, float(alpha), p_d, ld_p, ctx_d, d_model)
    assert_close16(p_d[..., :S], p_ref, 1e-3, max_ulp=2, what="p")
    assert torch.all(p_d[..., S:pad] == 0) and torch.all(p_d[..., pad:] == 3.0)
    assert_close16(ctx_d, ctx_ref, 1e-3, what="ctx")
    dqkv_ref = L.attention_bwd(MIXED, dctx, (q, k, v, np32(p_d[..., :S]), alpha))
    dqkv_d = empty16(T, 3 * d_model)
    mp.mp_attention_bwd_ldp(B, h, S, dk, qkv_d, 3 * d_model, float(alpha), p_d, ld_p, h16(dctx), d_model, dqkv_d, 3 * d_model)
    for name, lo in (("dq", 0), ("dk", d_model), ("dv", 2 * d_model)):
        # (one key: its probability is 1, dS and with it dq and dk are zero up to the rounding of dP and its sum)
        if S > 1 or name == "dv":
            assert_close16(dqkv_d[:, lo:lo + d_model], dqkv_ref[:, lo:lo + d_model], 1e-3, what=name)
        else:
            assert np.array_equal(np32(dqkv_d[:, lo:lo + d_model]), dqkv_ref[:, lo:lo + d_model])
    if S % 8 == 0:
        p2, ctx2, dqkv2 = empty16(B, h, S, S), empty16(T, d_model), empty16(T, 3 * d_model)
        mp.mp_attention_fwd(B, h, S, dk, qkv_d, 3 * d_model, float(alpha), p2, ctx2, d_model)
        mp.mp_attention_bwd(B, h, S, dk, qkv_d, 3 * d_model, float(alpha), p2, h16(dctx), d_model, dqkv2, 3 * d_model)
        assert torch.equal(p2, p_d[..., :S]) and torch.equal(ctx2, ctx_d) and torch.equal(dqkv2, dqkv_d)


def test_fused_attention_rejects_unsupported_shapes():
    x = empty16(64, 3 * 96)
    with pytest.raises(mp.MPError) as e:
        mp.mp_attention_fwd(1, 2, 64, 48, x, 3 * 96, 0.1, empty16(1, 2, 64, 64), empty16(64, 96), 96)
    assert e.value.code == ML.MP_E_UNSUPPORTED
    x = empty16(36, 3 * 64)
    with pytest.raises(mp.MPError):
        mp.mp_attention_fwd(1, 1, 36, 64, x, 3 * 64, 0.1, empty16(1, 1, 36, 36), empty16(36, 64), 64)


def test_gemm_overflow_gives_inf_and_dw_sets_flag():
    M, N, K = 64, 64, 64
    x = np.full((M, K), 200.0, np.float32)
    w = np.full((N, K), 200.0, np.float32)
    y = empty16(M, N)
    mp.mp_gemm_fwd(mp.gemm_desc(M, N, K), h16(x), h16(w), None, None, y)
    assert np.all(np.isposinf(np32(y)))                   # 64 * 4e4 overflows fp16: inf, never 65504
    st = make_state()
    d = mp.gemm_desc(M, N, K)
    dw = empty16(N, K)
    ws = ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(d, False))
    mp.mp_gemm_bwd_dw(d, h16(x), h16(w), dw, None, st, ws)
    assert mp.scale_state_read(st).found_inf == 1


def test_gemm_split_k_weight_gradient():
    M, N, K = 4096, 128, 256                  # small output, long token contraction: split over K
    r = RNG(11)
    x, dy = S16(r.standard_normal((M, K))), S16(r.standard_normal((M, N)) * 0.05)
    d = mp.gemm_desc(M, N, K)
    dw, db = empty16(N, K), empty16(N)
    ws = ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(d, True))
    mp.mp_gemm_bwd_dw(d, h16(dy), h16(x), dw, db, None, ws)
    _, dw_ref, db_ref = L.linear_bwd(MIXED, dy, x, np.zeros((N, K), np.float32))
    assert_close16(dw, dw_ref, 1e-3, max_ulp=1, what="split-K dw")
    assert_close16(db, db_ref, 1e-3, max_ulp=1, what="db")


def odd16(a):
    """A matrix inside a wider one of 7.0 with an odd row length, starting at an odd element -> (view, leading dimension)."""
    rows, cols = a.shape
    ld = cols + (3 if cols % 2 == 0 else 2)
    buf = torch.full((rows * ld + 9,), 7.0, dtype=torch.float16, device="cuda")
    v = buf[1:1 + rows * ld].view(rows, ld)
    v[:, :cols] = h16(a)
    return v, ld


@pytest.mark.parametrize("aligned", [False, True])
@pytest.mark.parametrize("joint,M,N,Kx,Kw", [
    (1, 8, 8, 8, 8), (1, 8, 9, 9, 8), (1, 1, 40, 33, 8),            # one tile, one straddling piece, one row
    (1, 65, 31, 63, 70), (1, 64, 256, 104, 128),                    # 4 waves: contractions of at most 512 ...
    (1, 521, 521, 321, 321), (1, 520, 520, 320, 328),               # ... or more than 256 tiles
    (1, 33, 523, 65, 129), (1, 600, 136, 72, 72), (1, 1500, 41, 29, 33),   # 8 waves; column sums in several rounds
    (1, 7, 40, 24, 24), (0, 70, 7, 24, 24), (0, 70, 24, 7, 24), (0, 70, 24, 24, 7),   # stored rows of fewer than 8 elements ...
    (0, 4128, 136, 520, 264),                                       # ... and products that are not small: separate calls
])
def test_gemm_both_gradients_of_a_layer(joint, M, N, Kx, Kw, aligned):
    """mp_gemm_bwd_both: input, weight and bias gradient against the oracle, with every epilogue of the input gradient,
    with and without the bias gradient, widths of the two products that differ, any extent, leading dimension and
    alignment, nothing written outside the output columns; one launch where mp_gemm_bwd_both_joint says so (it then takes
    no workspace), separate calls elsewhere.  Bounds as for the separate calls: fp32 order only."""
    r = RNG(M + 3 * N + 7 * Kx + 11 * Kw)
    x, w, dy = S16(r.standard_normal((M, Kw))), S16(r.standard_normal((N, Kx)) * 0.1), S16(r.standard_normal((M, N)) * 0.1)
    other = S16(r.standard_normal((M, Kx)))
    src = S16(np.maximum(other, 0))
    put = (lambda a: (h16(a), a.shape[1])) if aligned else odd16
    (xd, ldx), (wd, ldw), (dyd, ldy), (od, lda), (sd, _) = put(x), put(w), put(dy), put(other), put(src)
    (dx, ldo), (dw, ldg) = put(np.zeros((M, Kx))), put(np.zeros((N, Kw)))
    d_dx = mp.gemm_desc(M, N, Kx, ldx=ldo, ldw=ldw, ldy=ldy)
    d_dw = mp.gemm_desc(M, N, Kw, ldx=ldx, ldw=ldg, ldy=ldy)
    assert mp.mp_gemm_bwd_both_joint(d_dx, d_dw) == bool(joint)
    ws = None if joint else ws_bytes(max(mp.mp_gemm_bwd_dw_workspace_bytes(d_dw, True), mp.mp_gemm_split_workspace_bytes(d_dx)))
    dx_ref = MIXED.store(dy @ w)
    _, dw_ref, db_ref = L.linear_bwd(MIXED, dy, x, np.zeros((N, Kw), np.float32))
    st = make_state()
    bias = torch.full((N + 9,), 7.0, dtype=torch.float16, device="cuda")
    lead = 8 if aligned else 1
    for k, (kw, ref, ulp) in enumerate([({}, dx_ref, 1), (dict(relu_src=sd, ld_aux=lda), L.relu_mask(MIXED, dx_ref, src), 1),
                                        (dict(add=od, ld_aux=lda), L.add_store(MIXED, dx_ref, other), None)]):
        dx[:, :Kx] = float("nan")
        dw[:, :Kw] = float("nan")
        db = None if k == 1 else bias[lead:lead + N]
        mp.mp_gemm_bwd_both(d_dx, dyd, wd, dx, d_dw, xd, dw, db, st, ws, **kw)
        assert_close16(dx[:, :Kx], ref, 1e-3, max_ulp=ulp, what=f"dx {k}")
        assert_close16(dw[:, :Kw], dw_ref, 1e-3, max_ulp=1, what=f"dw {k}")
        if db is not None:
            assert_close16(db, db_ref, 1e-3, max_ulp=1, what=f"db {k}")
            bias[lead:lead + N] = 7.0
        assert torch.all(bias == 7.0)
    assert torch.all(dx[:, Kx:] == 7.0) and torch.all(dw[:, Kw:] == 7.0)
    assert mp.scale_state_read(st).found_inf == 0


@pytest.mark.parametrize("aligned", [False, True])
@pytest.mark.parametrize("M,N,Kx,Kw", [
    (1536, 24, 40, 72), (1537, 24, 40, 72), (1545, 41, 33, 29),     # the weight gradient's tiles last; first, 8 waves
    (1601, 131, 300, 90), (4096, 41, 97, 33),                       # first, 4 waves
    (700, 700, 700, 700), (333, 500, 1000, 900), (1001, 849, 500, 500),   # more than three workgroups per compute unit
])
def test_gemm_both_gradients_in_many_tiles(M, N, Kx, Kw, aligned):
    test_gemm_both_gradients_of_a_layer(1, M, N, Kx, Kw, aligned)


@pytest.mark.parametrize("M,N,K", [(128, 64, 40), (130, 65, 41), (640, 131, 67)])
def test_gemm_both_gradients_flag_what_the_separate_calls_flag(M, N, K):
    """A joint launch raises found_inf for the weight gradient alone and for the bias gradient alone, not for the input
    gradient (an activation gradient has no flag of its own), and not for finite results."""
    full = lambda rows, cols, v: torch.full((rows, cols), v, dtype=torch.float16, device="cuda")  # noqa: E731
    d = mp.gemm_desc(M, N, K)
    assert mp.mp_gemm_bwd_both_joint(d, d)
    for dy, w, x, flag, inf in ((60.0, 0.0, 2.0 ** 14, 1, "dw"), (600.0, 0.0, 0.0, 1, "db"), (60.0, 2.0 ** 14, 0.0, 0, "dx"),
                                (1.0, 1.0, 1.0, 0, "")):
        st = make_state()
        dx, dw, db = empty16(M, K), empty16(N, K), empty16(N)
        mp.mp_gemm_bwd_both(d, full(M, N, dy), full(N, K, w), dx, d, full(M, K, x), dw, db, st)
        assert mp.scale_state_read(st).found_inf == flag, inf
        for name, t in (("dx", dx), ("dw", dw), ("db", db)):
            assert bool(torch.isinf(t).all() if name == inf else torch.isfinite(t).all()), (inf, name)


@pytest.mark.parametrize("tile,shapes", GROUPED)
def test_gemm_grouped_weight_gradients(tile, shapes):
    """Several dW = dY^T X in one launch: each equals the oracle and, bit for bit, the single-problem entry point.
    `tile` is the shape the rule takes (of 256 x 256, 256 x 128 and 128 x 128 the one with the least estimated time)."""
    r = RNG(len(shapes) * 7 + shapes[0][1])
    items, refs, singles, db_refs = [], [], [], []
    st = make_state()
    for j, (M, N, K) in enumerate(shapes):
        x, dy = S16(r.standard_normal((M, K))), S16(r.standard_normal((M, N)) * 0.1)
        d = mp.gemm_desc(M, N, K)
        dw, dw1 = empty16(N, K), empty16(N, K)
        # every item but the second also asks for its bias gradient from the same launch
        items.append((d, h16(dy), h16(x), dw) + ((empty16(N),) if j != 1 else ()))
        _, dw_ref, db_ref = L.linear_bwd(MIXED, dy, x, np.zeros((N, K), np.float32))
        refs.append(dw_ref)
        db_refs.append(db_ref)
        mp.mp_gemm_tuning_override(tile, 1)                       # the tile the grouped launch takes, no k-split
        mp.mp_gemm_bwd_dw(d, items[-1][1], items[-1][2], dw1, None, None, ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(d, False)))
        mp.mp_gemm_tuning_override(-1, 0)
        singles.append(dw1)
    for mode in (1, 0):                                           # direct-to-LDS kernels (built-in choice), register-staged kernels
        mp.mp_gemm_tuning_dtl(mode)
        try:
            for it in items:
                for out in it[3:]:
                    out.fill_(float("nan"))
            mp.mp_gemm_bwd_dw_grouped(mp.gemm_group(items), st)
        finally:
            mp.mp_gemm_tuning_dtl(1)
        for k, (it, ref, one) in enumerate(zip(items, refs, singles)):
            assert_close16(it[3], ref, 1e-3, max_ulp=1, what=f"grouped dw {k} (mode {mode})")
            assert torch.equal(it[3], one), f"grouped dw {k} differs from the single-problem result (mode {mode})"
            if len(it) > 4:
                assert_close16(it[4], db_refs[k], 1e-3, max_ulp=1, what=f"grouped db {k} (mode {mode})")
    assert mp.scale_state_read(st).found_inf == 0


@pytest.mark.parametrize("rows,d,with_dz", [(3, 128, True), (200, 256, False), (4096, 512, True), (8191, 384, True), (8200, 1024, True),
                                            (300, 2048, True)])
def test_grouped_launch_finishes_layernorm_sums(rows, d, with_dz):
    """mp_layernorm_bwd_parts and the sums of a grouped launch (few and many partial rows, 4 and 8 waves to a workgroup, every
    register width) give the bits of mp_layernorm_bwd, and raise its flag: beside the tiles of a launch with as many idle workgroups as
    items, with a few (508 tiles of 128 x 128 on 512 workgroups: several items to each of them, the others behind the tiles), with idle
    ones in the second round only (600) and with none (1024), bias-gradient strips in front of the sums."""
    r = RNG(rows + d)
    up = lambda *s: h16(S16(r.standard_normal(s)))  # noqa: E731
    dy, x, a, gamma = up(rows, d), up(rows, d), up(rows, d), up(d)
    mean, rstd = torch.randn(rows, device="cuda") * 0.1, torch.rand(rows, device="cuda") + 0.5
    ws = ws_bytes(mp.mp_layernorm_bwd_workspace_bytes(rows, d))
    n = 3 if with_dz else 2
    want = [empty16(rows, d)] + [empty16(d) for _ in range(n)]
    st = make_state()
    mp.mp_layernorm_bwd(rows, d, dy, x, a, gamma, mean, rstd, want[0], want[1], want[2], st, ws, dz_colsum=want[3] if with_dz else None)
    for tiles in (1, 300, 508, 600, 1024):      # of 128 x 128
        M, N, K = 192, 128, 128 * tiles
        gy, gx, dw, db = up(M, N), up(M, K), empty16(N, K), empty16(N)
        for mode in (1, 0):
            db.fill_(float("nan"))
            got = [empty16(rows, d)] + [empty16(d) for _ in range(n)]
            part = ws_bytes(mp.mp_layernorm_bwd_workspace_bytes(rows, d))
            mp.mp_layernorm_bwd_parts(rows, d, dy, x, a, gamma, mean, rstd, got[0], with_dz, part)
            sums = mp.colsum_parts([(part, mp.mp_layernorm_bwd_nparts(rows, d), d, got[1:])] * 2)
            mp.mp_gemm_tuning_dtl(mode)
            try:
                mp.mp_gemm_bwd_dw_grouped_sums(mp.gemm_group([(mp.gemm_desc(M, N, K), gy, gx, dw, db)]), sums, st)
            finally:
                mp.mp_gemm_tuning_dtl(1)
            for k in range(n + 1):
                assert torch.equal(got[k], want[k]), (tiles, mode, k)
            assert_close16(db, MIXED.store(np32(gy).sum(0, dtype=np.float32)), 1e-3, max_ulp=1, what=f"db {tiles} {mode}")
    assert mp.scale_state_read(st).found_inf == 0
    dy[0, 0] = float("inf")
    mp.mp_layernorm_bwd_parts(rows, d, dy, x, a, gamma, mean, rstd, got[0], with_dz, part)
    mp.mp_gemm_bwd_dw_grouped_sums(mp.gemm_group([(mp.gemm_desc(M, N, K), gy, gx, dw)]), sums, st)
    assert mp.scale_state_read(st).found_inf != 0
    with pytest.raises(mp.MPError):             # columns off 128
        mp.mp_gemm_bwd_dw_grouped_sums(mp.gemm_group([(mp.gemm_desc(M, N, K), gy, gx, dw)]),
                                       mp.colsum_parts([(part, 1, d - 8, got[1:])]), st)


def test_gemm_grouped_transposed_weight_layout_with_bias_gradient():
    """A grouped item whose weight is stored [K, N] (trans_w): dW[K, N] = X^T dY, and db = column sums of dY, next to an
    ordinary item; both kernel families."""
    r = RNG(77)
    M, N, K = 192, 256, 384
    x, dy = S16(r.standard_normal((M, K))), S16(r.standard_normal((M, N)) * 0.1)
    _, dw_ref, db_ref = L.linear_bwd(MIXED, dy, x, np.zeros((N, K), np.float32))
    dt = mp.gemm_desc(M, N, K, ldw=N, trans_w=1)
    dn = mp.gemm_desc(M, N, K)
    for mode in (1, 0):
        dwt, dbt, dwn = empty16(K, N), empty16(N), empty16(N, K)
        for t in (dwt, dbt, dwn):
            t.fill_(float("nan"))
        mp.mp_gemm_tuning_dtl(mode)
        try:
            mp.mp_gemm_bwd_dw_grouped(mp.gemm_group([(dt, h16(dy), h16(x), dwt, dbt), (dn, h16(dy), h16(x), dwn)]), None)
        finally:
            mp.mp_gemm_tuning_dtl(1)
        assert_close16(dwt, dw_ref.T, 1e-3, max_ulp=1, what=f"grouped dw, [K, N] layout (mode {mode})")
        assert_close16(dwn, dw_ref, 1e-3, max_ulp=1, what=f"grouped dw (mode {mode})")
        assert_close16(dbt, db_ref, 1e-3, max_ulp=1, what=f"grouped db (mode {mode})")


@pytest.mark.parametrize("M", [128, 192])     # register-staged, straight into LDS
def test_gemm_grouped_flags_overflow_and_rejects_ragged_shapes(M):
    N, K = 128, 128
    big = torch.full((M, N), 300.0, dtype=torch.float16, device="cuda")
    x = torch.full((M, K), 300.0, dtype=torch.float16, device="cuda")
    ok_dy, ok_x = torch.ones(M, N, dtype=torch.float16, device="cuda"), torch.ones(M, K, dtype=torch.float16, device="cuda")
    st = make_state()
    d = mp.gemm_desc(M, N, K)
    dw0, dw1 = empty16(N, K), empty16(N, K)
    mp.mp_gemm_bwd_dw_grouped(mp.gemm_group([(d, ok_dy, ok_x, dw0), (d, big, x, dw1)]), st)
    assert mp.scale_state_read(st).found_inf == 1          # 128 * 300 * 300 overflows fp16
    assert torch.all(dw0 == float(M)) and torch.all(torch.isinf(dw1))
    # a bias gradient that overflows while the product stays finite: 128 rows of 600 sum to 76800 > 65504
    st2 = make_state()
    dy600 = torch.full((M, N), 600.0, dtype=torch.float16, device="cuda")
    zeros, db = torch.zeros(M, K, dtype=torch.float16, device="cuda"), empty16(N)
    mp.mp_gemm_bwd_dw_grouped(mp.gemm_group([(d, dy600, zeros, dw0, db)]), st2)
    assert mp.scale_state_read(st2).found_inf == 1 and torch.all(dw0 == 0.0) and torch.all(torch.isinf(db))
    bad = mp.gemm_desc(128, 136, 128)
    with pytest.raises(mp.MPError) as e:
        mp.mp_gemm_bwd_dw_grouped(mp.gemm_group([(bad, empty16(128, 136), ok_x, empty16(136, 128))]), st)
    assert e.value.code == ML.MP_E_UNSUPPORTED


def test_mfma_sustained_rate_probe_reads_sanely():
    """The ceiling probe: all-zero operands run near the top clock, N(0,1) operands clearly below it, both far above
    anything a memory-bound loop could show; the sink receives the (finite) accumulator sums."""
    sink = empty32(256 * 256)
    zeros = torch.zeros(16384, dtype=torch.float16, device="cuda")
    normal = torch.randn(16384, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).half()
    r0 = mp.mp_mfma_sustained_rate(zeros, sink, 256, 20000)
    assert torch.all(sink == 0)
    r1 = mp.mp_mfma_sustained_rate(normal, sink, 256, 20000)
    assert torch.isfinite(sink).all()
    assert r0 > 0 and 0.3 * r0 < r1 < r0, (r0, r1)       # ratios only: absolute rates depend on the box's clocks


@pytest.mark.parametrize("M,N,K", [(32, 4096, 2048), (32, 1024, 512), (8, 2048, 4096), (48, 520, 1000)])
def test_gemm_few_rows_with_workspace(M, N, K):
    """Products with few output rows (the recurrent products of config 5) given a workspace: the contraction may be
    split over more workgroups; forward with and without bias and dX against the oracle, also with a workspace that
    is too small (runs unsplit) and with an epilogue that is never split (ReLU)."""
    r = RNG(M + N + K + 17)
    x, w, b = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K)) * 0.05), S16(r.standard_normal(N))
    dy = S16(r.standard_normal((M, N)))
    d0, d1, d2 = mp.gemm_desc(M, N, K), mp.gemm_desc(M, N, K, epilogue=1), mp.gemm_desc(M, N, K, epilogue=2)
    need = mp.mp_gemm_split_workspace_bytes(d0)
    if (M, N, K) == (32, 4096, 2048):
        assert need > 0                                       # this one must split, or config 5 stays latency-bound
    xd, wd, bd, dyd = h16(x), h16(w), h16(b), h16(dy)
    for ws in (ws_bytes(max(need, 256)), ws_bytes(256), None):
        y = empty16(M, N)
        mp.mp_gemm_fwd_ws(d0, xd, wd, None, None, y, ws=ws)
        assert_close16(y, L.linear_fwd(MIXED, x, w), 1e-3, max_ulp=1, what="few rows fwd")
        mp.mp_gemm_fwd_ws(d1, xd, wd, bd, None, y, ws=ws)
        assert_close16(y, L.linear_fwd(MIXED, x, w, b), 1e-3, max_ulp=1, what="few rows fwd + bias")
        mp.mp_gemm_fwd_ws(d2, xd, wd, bd, None, y, ws=ws)
        assert_close16(y, L.linear_fwd(MIXED, x, w, b, relu=True), 1e-3, max_ulp=1, what="few rows fwd + bias + relu")
        dx = empty16(M, K)
        mp.mp_gemm_bwd_dx_ws(d0, dyd, wd, dx, ws=ws)
        assert_close16(dx, L.linear_bwd(MIXED, dy, x, w)[0], 1e-3, max_ulp=1, what="few rows dx")


@pytest.mark.parametrize("tokens,N,K", [(4096, 1024, 1024), (3240, 2048, 512), (8192, 384, 1024), (8192, 2048, 1024)])
def test_weight_gradient_takes_a_workspace_that_holds_its_plan(tokens, N, K):
    """The two kernel families split such a contraction differently.  A workspace that holds either plan of a call is taken, and no byte
    behind it changes; operands off 16 bytes, which only the register-staged kernels take, need their plan's; less is refused."""
    r = RNG(tokens + N)
    x, dy = S16(r.standard_normal((tokens, K))), S16(r.standard_normal((tokens, N)) * 0.1)
    ref, d = L.linear_bwd(MIXED, dy, x, np.zeros((N, K), np.float32))[1], mp.gemm_desc(tokens, N, K)

    def off(a, elements):
        t = torch.zeros(a.size + 8, dtype=torch.float16, device="cuda")[elements:elements + a.size].view(a.shape)
        return t.copy_(h16(a))

    both = mp.mp_gemm_bwd_dw_workspace_bytes(d, False)
    mp.mp_gemm_tuning_dtl(0)
    staged = mp.mp_gemm_bwd_dw_workspace_bytes(d, False)
    mp.mp_gemm_tuning_dtl(1)
    for elements, sizes in ((0, (both, staged)), (1, (staged,))):
        dyd, xd = off(dy, elements), off(x, elements)
        for size in sizes:
            ws = torch.full((size // 4 + 64,), 7.0, dtype=torch.float32, device="cuda")
            dw = empty16(N, K)
            mp.mp_gemm_bwd_dw(d, dyd, xd, dw, None, None, ws[:size // 4])
            assert_close16(dw, ref, 1e-3, max_ulp=1, what=f"dw {elements} {size}")
            assert torch.all(ws[size // 4:] == 7.0)
        with pytest.raises(mp.MPError):
            mp.mp_gemm_bwd_dw(d, dyd, xd, dw, None, None, ws[:staged // 4 - 1 if elements else 60])


def test_empty_and_degenerate_inputs():
    """Zero rows: nothing is launched and the output is untouched.  Zero-length contraction: the sum is empty, the
    epilogue still applies (Y = bias).  An empty tensor list and zero-length tensors in the optimizer wrapper: the step
    counts as clean and the scale state advances like the oracle's."""
    y = torch.full((4, 8), 3.0, dtype=torch.float16, device="cuda")
    x, w = empty16(4, 8), empty16(8, 8)
    mp.mp_gemm_fwd(mp.gemm_desc(0, 8, 8), x, w, None, None, y)
    torch.cuda.synchronize()
    assert torch.all(y == 3.0)
    b = h16(S16(RNG(3).standard_normal(8)))
    mp.mp_gemm_fwd(mp.gemm_desc(4, 8, 0, ldx=8, ldw=8, epilogue=1), x, w, b, None, y)
    assert torch.equal(y, b.expand(4, 8))
    dx = torch.full((4, 8), 5.0, dtype=torch.float16, device="cuda")
    mp.mp_gemm_bwd_dx(mp.gemm_desc(4, 0, 8, ldy=8), empty16(4, 8), empty16(8, 8), dx)     # no output columns to contract over
    assert torch.all(dx == 0)
    st = make_state(interval=2)
    cfg = mp.opt_cfg("adam", 1e-3)
    mp.mp_unscale_check_update(None, 0, cfg, st)
    mp.mp_loss_scale_update(st)
    one = dict(g16=h16(np.ones(16, np.float32)), w32=f32(np.ones(16, np.float32)), w16=empty16(16), m=f32(np.zeros(16, np.float32)),
               v=f32(np.zeros(16, np.float32)))
    lst = mp.tensor_list([one, one])
    lst[0].n = 0                                             # a zero-length tensor in front of a real one
    mp.mp_unscale_check_update(lst, 2, cfg, st)
    mp.mp_loss_scale_update(st)
    s = mp.scale_state_read(st)
    ost = O.ScaleState(scale=2.0 ** 15, growth_interval=2)
    O.loss_scale_update(ost, 0)
    O.loss_scale_update(ost, 0)
    assert (s.scale, s.good_steps, s.opt_step, s.skipped_steps) == (ost.scale, ost.good_steps, ost.opt_step, 0) and s.scale == 2.0 ** 16
    assert torch.all(one["w32"] < 1.0) and torch.equal(one["w16"], one["w32"].half())


def test_gemm_rejects_bad_arguments():
    d = mp.gemm_desc(8, 8, 8)
    with pytest.raises(mp.MPError) as e:
        mp.mp_gemm_fwd(d, None, None, None, None, None)
    assert e.value.code == ML.MP_E_INVAL
    d2 = mp.gemm_desc(8, 8, 8, ldx=4)
    with pytest.raises(mp.MPError):
        mp.mp_gemm_fwd(d2, empty16(8, 8), empty16(8, 8), None, None, empty16(8, 8))
    with pytest.raises(mp.MPError) as e:
        mp.mp_gemm_bwd_dw(d, empty16(8, 8), empty16(8, 8), empty16(8, 8), None, None, None)
    assert e.value.code == ML.MP_E_WORKSPACE


# ------------------------------------------------------------------ losses
@pytest.mark.parametrize("rows,cols", [(64, 256), (37, 100), (1, 8), (513, 1000)])
def test_mse_scaled(rows, cols):
    r = RNG(rows + cols)
    y, t = S16(r.standard_normal((rows, cols))), S16(r.standard_normal((rows, cols)))
    S = 2.0 ** 10
    loss_ref, dy_ref = L.mse_scaled(MIXED, y, t, S)
    st = make_state(scale=S)
    loss, dy = empty32(1), empty16(rows, cols)
    mp.mp_mse_scaled(rows, cols, h16(y), h16(t), cols, st, loss, dy, ws_bytes(mp.mp_loss_workspace_bytes(rows, cols)))
    assert abs(float(loss) - float(loss_ref)) <= 1e-5 * abs(float(loss_ref))
    assert_close16(dy, dy_ref, 1e-3, max_ulp=1, what="mse dy")


@pytest.mark.parametrize("rows", [1, 255, 257, 4095, 4096, 4097, 8449])   # the finish kernel takes 16 x 256 at a time
def test_softmax_xent_mean_over_any_number_of_rows(rows):
    r = RNG(rows)
    z, t = S16(r.standard_normal((rows, 8)) * 3), r.integers(0, 8, rows)
    z64 = z.astype(np.float64)
    ref = np.mean(np.log(np.exp(z64).sum(1)) - z64[np.arange(rows), t])
    loss, zd = empty32(1), h16(z)
    mp.mp_softmax_xent_scaled(rows, 8, zd, 8, i32(t.astype(np.int32)), make_state(scale=1.0), loss, zd, ws_bytes(mp.mp_loss_workspace_bytes(rows, 8)))
    # row losses: about 8 roundings of values up to 16; their sum, all terms >= 0: one rounding per addition of a chain
    assert abs(float(loss) - ref) <= 8 * 16 * 2.0 ** -24 + (rows / 256 + 10) * 2.0 ** -24 * ref


@pytest.mark.parametrize("rows,vocab", [(16, 32768), (33, 3000), (7, 1001), (5, 40000),
                                        (600, 32768), (300, 24584)])  # the last two: several rows per persistent workgroup
def test_softmax_xent_scaled(rows, vocab):
    r = RNG(rows + vocab)
    z = S16(r.standard_normal((rows, vocab)) * 3)
    t = r.integers(0, vocab, rows).astype(np.int32)
    if rows > 4:
        t[1], t[2] = -1, vocab                # out-of-range targets contribute nothing
    S = 2.0 ** 15
    loss_ref, g_ref = L.softmax_xent_scaled(MIXED, z, t, S)
    st = make_state(scale=S)
    loss, g = empty32(1), empty16(rows, vocab)
    ws = ws_bytes(mp.mp_loss_workspace_bytes(rows, vocab))
    zd = h16(z)
    mp.mp_softmax_xent_scaled(rows, vocab, zd, vocab, i32(t), st, loss, g, ws)
    assert abs(float(loss) - float(loss_ref)) <= 2e-6 * abs(float(loss_ref)) + 1e-6
    assert_close16(g, g_ref, 1e-3, max_ulp=2, what="xent grad")
    mp.mp_softmax_xent_scaled(rows, vocab, zd, vocab, i32(t), st, loss, zd, ws)   # in place
    assert np.array_equal(bits(zd), bits(g))


@pytest.mark.parametrize("rows,vocab", [(600, 32768), (300, 24584), (16, 32768), (33, 3000), (7, 1001)])
def test_softmax_xent_scaled_with_bias_gradient(rows, vocab):
    """The loss call that also sums the stored gradient per column (the bias gradient of the projection): same loss and
    the same gradient bits as the plain call, db equal to the oracle's column sums of that gradient; the first two shapes
    take the fused pass (several rows per persistent workgroup), the others the plain call followed by mp_colsum."""
    r = RNG(3 * rows + vocab)
    z = S16(r.standard_normal((rows, vocab)) * 3)
    t = r.integers(0, vocab, rows).astype(np.int32)
    t[1], t[2] = -1, vocab
    S = 2.0 ** 15
    loss_ref, g_ref = L.softmax_xent_scaled(MIXED, z, t, S)
    db_ref = L.linear_bwd(MIXED, g_ref, np.zeros((rows, 8), np.float32), np.zeros((vocab, 8), np.float32))[2]
    st = make_state(scale=S)
    loss, loss2, g, g2, db = empty32(1), empty32(1), empty16(rows, vocab), empty16(rows, vocab), empty16(vocab)
    db.fill_(float("nan"))
    zd = h16(z)
    mp.mp_softmax_xent_scaled(rows, vocab, zd, vocab, i32(t), st, loss, g, ws_bytes(mp.mp_loss_workspace_bytes(rows, vocab)))
    ws = ws_bytes(mp.mp_softmax_xent_db_workspace_bytes(rows, vocab))
    mp.mp_softmax_xent_scaled_db(rows, vocab, zd, vocab, i32(t), st, loss2, g2, db, ws)
    assert float(loss2) == float(loss) and np.array_equal(bits(g2), bits(g))
    assert abs(float(loss2) - float(loss_ref)) <= 2e-6 * abs(float(loss_ref)) + 1e-6
    # column sums of the gradient the GPU stored (its own bits), and of the oracle's gradient
    own = L.linear_bwd(MIXED, np32(g2), np.zeros((rows, 8), np.float32), np.zeros((vocab, 8), np.float32))[2]
    assert_close16(db, own, 1e-3, max_ulp=1, what="xent db vs sums of the stored gradient")
    assert_close16(db, db_ref, 2e-3, max_ulp=4, what="xent db vs oracle")
    assert mp.scale_state_read(st).found_inf == 0
    mp.mp_softmax_xent_scaled_db(rows, vocab, zd, vocab, i32(t), st, loss2, zd, db, ws)   # in place
    assert np.array_equal(bits(zd), bits(g))
    with pytest.raises(mp.MPError) as e:
        mp.mp_softmax_xent_scaled_db(rows, vocab, zd, vocab, i32(t), st, loss2, zd, db, ws_bytes(1024))
    assert e.value.code == ML.MP_E_WORKSPACE


@pytest.mark.parametrize("rows,vocab", [(3, 1), (5, 7), (6, 2 ** 13 + 1), (9, 2 ** 14 - 1), (70, 2 ** 14 + 3), (300, 2 ** 15 - 3),
                                        (4, 2 ** 15 + 1), (8, 2 ** 12), (300, 1280), (300, 1281)])
def test_softmax_xent_rows_at_any_alignment(rows, vocab):
    """Vocabularies that are no multiple of 8, in rows that start at odd elements, around the row lengths where the workgroup
    size changes: gradient and bias gradient against the oracle, in place too, nothing written between the rows, and rows
    with an out-of-range target get a zero gradient whatever their logits are."""
    r = RNG(rows + vocab)
    z = S16(r.standard_normal((rows, vocab)) * 3)
    t = r.integers(0, vocab, rows).astype(np.int32)
    t[1] = vocab
    z[1, 0] = np.inf
    S, ld = 2.0 ** 10, vocab + 3
    clean = z.copy()
    clean[1] = 0.0                                    # (what the row holds does not matter)
    loss_ref, g_ref = L.softmax_xent_scaled(MIXED, clean, t, S)
    buf = torch.full((rows * ld + 8,), 7.0, dtype=torch.float16, device="cuda")
    zd = buf[1:1 + rows * ld].view(rows, ld)
    zd[:, :vocab] = h16(z)
    gbuf = torch.full_like(buf, 5.0)
    gd = gbuf[1:1 + rows * ld].view(rows, ld)
    st = make_state(scale=S)
    loss, db = empty32(1), empty16(vocab)
    mp.mp_softmax_xent_scaled(rows, vocab, zd, ld, i32(t), st, loss, gd, ws_bytes(mp.mp_loss_workspace_bytes(rows, vocab)))
    assert abs(float(loss) - float(loss_ref)) <= 2e-6 * abs(float(loss_ref)) + 1e-6
    assert_close16(gd[:, :vocab], g_ref, 1e-3, max_ulp=2, what="gradient")
    assert torch.all(gd[:, vocab:] == 5.0) and float(gbuf[0]) == 5.0
    ws = ws_bytes(mp.mp_softmax_xent_db_workspace_bytes(rows, vocab))
    mp.mp_softmax_xent_scaled_db(rows, vocab, zd, ld, i32(t), st, loss, zd, db, ws)   # in place
    assert np.array_equal(bits(zd[:, :vocab].contiguous()), bits(gd[:, :vocab].contiguous()))
    assert torch.all(zd[:, vocab:] == 7.0) and float(buf[0]) == 7.0
    assert_close16(db, MIXED.store(np32(gd[:, :vocab]).sum(0, dtype=np.float32)), 1e-3, max_ulp=1, what="bias gradient")


@pytest.mark.parametrize("vocab", [8, 3000, 8200, 16384, 24584, 32768, 32776, 1001])   # each workgroup size, the fused sums, the generic kernel
def test_softmax_xent_rows_without_a_target_have_zero_gradient_whatever_they_hold(vocab):
    """Rows whose target lies outside the vocabulary, holding an infinity, a NaN, only infinities: zero gradient and no loss,
    as for finite rows, in rows of 16-byte pieces too; the bias gradient stays finite and no overflow is flagged."""
    rows, S = 6, 2.0 ** 10
    r = RNG(vocab)
    z, t = S16(r.standard_normal((rows, vocab)) * 3), r.integers(0, vocab, rows).astype(np.int32)
    t[1], t[2], t[3] = vocab, -1, vocab + 7
    clean = z.copy()
    clean[1:4] = 0.0
    z[1, 0], z[2, vocab - 1], z[3] = np.inf, np.nan, -np.inf
    loss_ref, g_ref = L.softmax_xent_scaled(MIXED, clean, t, S)
    st, loss, db = make_state(scale=S), empty32(1), empty16(vocab)
    g1, g2 = empty16(rows, vocab), empty16(rows, vocab)
    mp.mp_softmax_xent_scaled(rows, vocab, h16(z), vocab, i32(t), st, loss, g1, ws_bytes(mp.mp_loss_workspace_bytes(rows, vocab)))
    assert abs(float(loss) - float(loss_ref)) <= 2e-6 * abs(float(loss_ref)) + 1e-6
    mp.mp_softmax_xent_scaled_db(rows, vocab, h16(z), vocab, i32(t), st, loss, g2, db, ws_bytes(mp.mp_softmax_xent_db_workspace_bytes(rows, vocab)))
    assert abs(float(loss) - float(loss_ref)) <= 2e-6 * abs(float(loss_ref)) + 1e-6
    for g in (g1, g2):
        assert torch.all(g[1:4] == 0)
        assert_close16(g, g_ref, 1e-3, max_ulp=2, what="gradient")
    assert_close16(db, MIXED.store(np32(g2).sum(0, dtype=np.float32)), 1e-3, max_ulp=1, what="bias gradient")
    assert mp.scale_state_read(st).found_inf == 0


@pytest.mark.parametrize("rows,cols", [(1, 1), (65, 7), (64, 63), (200, 65), (1021, 1001), (3, 8), (300, 255), (65, 257), (70, 260),
                                       (1, 319), (130, 321)])
def test_colsum_rows_at_any_alignment(rows, cols):
    """Column counts around the 8-column pieces and 64-column workgroups, rows that start at odd elements."""
    r = RNG(rows + cols)
    dy, ld = S16(r.standard_normal((rows, cols))), cols + 3
    buf = torch.full((rows * ld + 8,), float("inf"), dtype=torch.float16, device="cuda")
    d = buf[1:1 + rows * ld].view(rows, ld)
    d[:, :cols] = h16(dy)
    db = empty16(cols)
    mp.mp_colsum(rows, cols, d, ld, db, None, ws_bytes(mp.mp_colsum_workspace_bytes(rows, cols)))
    assert_close16(db, MIXED.store(dy.sum(0, dtype=np.float32)), 1e-3, max_ulp=1, what="colsum")


def test_softmax_xent_bias_gradient_flags_overflow():
    """Every row has the same target and a dominant logit elsewhere: the column of the dominant class sums
    rows x S / rows = S = 2^17 > 65504, so db overflows while every stored gradient value is small."""
    rows, vocab = 512, 32768
    z = torch.zeros(rows, vocab, dtype=torch.float16, device="cuda")
    z[:, 7] = 30.0
    st = make_state(scale=2.0 ** 17)
    loss, db = empty32(1), empty16(vocab)
    mp.mp_softmax_xent_scaled_db(rows, vocab, z, vocab, i32(np.full(rows, 3)), st, loss, z, db,
                                 ws_bytes(mp.mp_softmax_xent_db_workspace_bytes(rows, vocab)))
    assert mp.scale_state_read(st).found_inf == 1
    assert torch.isinf(db[7]) and torch.isfinite(z).all()


@pytest.mark.parametrize("rows,vocab", [(60, 29), (7, 1279), (33, 5003), (100, 8192), (1021, 12001), (300, 20001), (5, 32771)])
def test_xent_gradient_also_side_by_side(rows, vocab):
    """mp_softmax_xent_scaled_db_copy: the bits of the plain call, and dlogits once more with rows `vocab` apart, in every kernel and row
    length (generic, cached, with the column sums), nothing around either changed; rows without a target are zero in both."""
    r = RNG(rows + vocab)
    ld = (vocab + 7) // 8 * 8
    t = r.integers(0, vocab, rows).astype(np.int32)
    t[rows // 2] = -1
    z = torch.full((rows, ld), 7.0, dtype=torch.float16, device="cuda")
    z[:, :vocab] = h16(S16(r.standard_normal((rows, vocab)) * 3))
    z2, st = z.clone(), make_state(scale=1024.0)
    loss, loss2, db, db2 = empty32(1), empty32(1), empty16(vocab), empty16(vocab)
    ws = ws_bytes(mp.mp_softmax_xent_db_workspace_bytes(rows, vocab))
    mp.mp_softmax_xent_scaled_db(rows, vocab, z, ld, i32(t), st, loss, z, db, ws)
    flat = torch.full((rows * vocab + 64,), 7.0, dtype=torch.float16, device="cuda")
    mp.mp_softmax_xent_scaled_db_copy(rows, vocab, z2, ld, i32(t), st, loss2, z2, flat[:rows * vocab], db2, ws)
    assert torch.equal(z2, z) and torch.equal(loss2, loss) and torch.equal(db2, db)
    assert torch.equal(flat[:rows * vocab].view(rows, vocab), z[:, :vocab]) and torch.all(flat[rows * vocab:] == 7.0)
    assert torch.all(z[rows // 2, :vocab] == 0) and torch.all(z[:, vocab:] == 7.0)


@pytest.mark.parametrize("vocab", [1000, 1001, 12001])
def test_xent_step_leaves_the_logits_gradient_contiguous(vocab):
    """XentStep.logits is one [T, V] block for every vocabulary, live over iterations."""
    import mp_inputs as I
    from dataclasses import replace
    from paper_1805_10387_amd import steps as St
    wl = replace(I.C4_SMALL, vocab=vocab)
    step = St.XentStep(wl)
    step.set_batch(wl.batch())
    held = step.logits
    assert held.is_contiguous() and held.shape == (wl.tokens, vocab)
    for _ in range(2):
        step.step()
        assert torch.equal(held.view(-1), step.rows16[:, :vocab].reshape(-1)) and torch.any(held != 0)
        held.fill_(1.0)


def test_xent_uniform_logits_closed_form():
    rows, vocab = 8, 32768
    st = make_state(scale=2.0 ** 15)
    loss, g = empty32(1), empty16(rows, vocab)
    z = torch.zeros(rows, vocab, dtype=torch.float16, device="cuda")
    mp.mp_softmax_xent_scaled(rows, vocab, z, vocab, i32(np.arange(rows)), st, loss, g,
                              ws_bytes(mp.mp_loss_workspace_bytes(rows, vocab)))
    assert abs(float(loss) - 10.39720770839918) < 1e-5          # ln 32768


# ------------------------------------------------------------------ LayerNorm / softmax / LSTM cell / colsum / cast
@pytest.mark.parametrize("rows,d", [(64, 512), (203, 1024), (5, 8), (130, 2048), (31, 200)])
def test_layernorm_fwd_bwd(rows, d):
    r = RNG(rows + d)
    x, a = S16(r.standard_normal((rows, d))), S16(r.standard_normal((rows, d)) * 0.5)
    gam, bet = S16(1 + 0.2 * r.standard_normal(d)), S16(0.1 * r.standard_normal(d))
    dy = S16(r.standard_normal((rows, d)))
    y_ref, cache = L.layernorm_fwd(MIXED, x, a, gam, bet)
    dz_ref, dg_ref, db_ref = L.layernorm_bwd(MIXED, dy, cache, gam)
    xd, ad, gd, bd = h16(x), h16(a), h16(gam), h16(bet)
    y, mean, rstd = empty16(rows, d), empty32(rows), empty32(rows)
    mp.mp_layernorm_fwd(rows, d, xd, ad, gd, bd, L.LN_EPS, y, mean, rstd)
    assert_close16(y, y_ref, 1e-3, max_ulp=1, what="ln y")
    assert np.allclose(np32(rstd), cache[1][:, 0], rtol=1e-5)
    dz, dg, db, dzs = empty16(rows, d), empty16(d), empty16(d), empty16(d)
    st = make_state()
    mp.mp_layernorm_bwd(rows, d, h16(dy), xd, ad, gd, mean, rstd, dz, dg, db, st,
                        ws_bytes(mp.mp_layernorm_bwd_workspace_bytes(rows, d)), dz_colsum=dzs)
    assert_close16(dz, dz_ref, 1e-3, what="ln dz")
    # the fused column sums are those of the dz the kernel stored
    assert_close16(dzs, MIXED.store(np32(dz).sum(0, dtype=np.float32)), 1e-3, max_ulp=1, what="ln dz colsum")
    dg2, db2 = empty16(d), empty16(d)
    mp.mp_layernorm_bwd(rows, d, h16(dy), xd, ad, gd, mean, rstd, dz, dg2, db2, None,
                        ws_bytes(mp.mp_layernorm_bwd_workspace_bytes(rows, d)))
    assert np.array_equal(bits(dg2), bits(dg)) and np.array_equal(bits(db2), bits(db))
    assert_close16(dg, dg_ref, 1e-3, max_ulp=1, what="ln dgamma")
    assert_close16(db, db_ref, 1e-3, max_ulp=1, what="ln dbeta")
    assert mp.scale_state_read(st).found_inf == 0


@pytest.mark.parametrize("rows,d", [(3, 8), (200, 264), (8200, 1024), (300, 2048)])
def test_layernorm_bwd_workspace_at_any_word(rows, d):
    """A workspace that starts at a 4-byte boundary which is no 16-byte boundary gives the bits of an aligned one, and nothing around it
    changes; 4 and 8 waves to a workgroup, every register width."""
    r = RNG(rows + d + 1)
    up = lambda *s: h16(S16(r.standard_normal(s)))  # noqa: E731
    dy, x, gam = up(rows, d), up(rows, d), up(d)
    mean, rstd = torch.randn(rows, device="cuda") * 0.1, torch.rand(rows, device="cuda") + 0.5
    words = mp.mp_layernorm_bwd_workspace_bytes(rows, d) // 4
    outs = []
    for at in (0, 1, 2, 3):
        ws = torch.full((words + 16,), 7.0, dtype=torch.float32, device="cuda")
        out = [empty16(rows, d)] + [empty16(d) for _ in range(3)]
        mp.mp_layernorm_bwd(rows, d, dy, x, None, gam, mean, rstd, out[0], out[1], out[2], None, ws[at:at + words], dz_colsum=out[3])
        assert torch.all(ws[:at] == 7.0) and torch.all(ws[at + words:] == 7.0)
        outs.append(out)
    for out in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out, outs[0]))


@pytest.mark.parametrize("rows,d", [(512, 192), (513, 1024), (200, 2048), (1100, 64)])
def test_layernorm_bwd_takes_any_workspace_that_holds_four_rows_to_a_wave(rows, d):
    """The sums are the same within fp32 order whether the workspace holds a row of partial sums per workgroup of the rule or only one
    per 16 rows (the least), nothing behind it is written, and less is refused."""
    r = RNG(rows + d)
    dy, x, gam = (h16(S16(r.standard_normal(s))) for s in ((rows, d), (rows, d), d))
    mean, rstd = torch.randn(rows, device="cuda") * 0.1, torch.rand(rows, device="cuda") + 0.5
    least, outs = (rows + 15) // 16 * 3 * d, []
    for words in (mp.mp_layernorm_bwd_workspace_bytes(rows, d) // 4, mp.mp_layernorm_bwd_nparts(rows, d) * 3 * d, least, least - 1):
        ws = torch.full((words + 64,), 7.0, dtype=torch.float32, device="cuda")
        out = [empty16(rows, d)] + [empty16(d) for _ in range(3)]
        call = lambda: mp.mp_layernorm_bwd(rows, d, dy, x, None, gam, mean, rstd, out[0], out[1], out[2], None, ws[:words], dz_colsum=out[3])  # noqa: B023,E731
        if words < least:
            with pytest.raises(RuntimeError):
                call()
        else:
            call()
            outs.append(out)
        assert torch.all(ws[words:] == 7.0)
    for out in outs[1:]:
        assert torch.equal(out[0], outs[0][0])
        for a, b in zip(out[1:], outs[0][1:]):
            assert_close16(a, np32(b), 1e-3, max_ulp=1)


@pytest.mark.parametrize("rows,cols", [(64, 64), (1000, 128), (77, 40), (50, 256), (9, 512), (13, 301), (6, 1000)])
def test_softmax_fwd_bwd(rows, cols):
    r = RNG(rows + cols)
    s = S16(r.standard_normal((rows, cols)) * 2)
    p_ref = MIXED.store(L.softmax_rows(MIXED, s))
    p = empty16(rows, cols)
    mp.mp_softmax_fwd(rows, cols, h16(s), p, cols)
    assert_close16(p, p_ref, 1e-3, max_ulp=2, what="softmax")
    dp = S16(r.standard_normal((rows, cols)))
    inner = (dp * p_ref).sum(-1, keepdims=True, dtype=np.float32)
    ds_ref = MIXED.store(p_ref * (dp - inner))
    ds = empty16(rows, cols)
    mp.mp_softmax_bwd(rows, cols, h16(p_ref), h16(dp), ds, cols)
    assert_close16(ds, ds_ref, 1e-3, what="softmax bwd")


@pytest.mark.parametrize("B,H", [(32, 1024), (8, 128), (3, 50)])
def test_lstm_cell_fwd_bwd(B, H):
    """The cell kernels against the oracle's LSTM layer itself.  With W = [I_4H | 0] (input width 4H) and b = 0 the
    layer's gate sums are its inputs (an exact copy), the recurrent gradient is zero and dx_t = dgates_t, so a
    two-step sequence exposes one cell update with c_prev = 0 and one with c_prev != 0, and backward steps with and
    without an incoming cell-state gradient."""
    r = RNG(B + H)
    T = 2
    x_seq = S16(r.standard_normal((T, B, 4 * H)) * 2)
    w = np.concatenate([np.eye(4 * H, dtype=np.float32), np.zeros((4 * H, H), np.float32)], axis=1)
    h_ref, cache = L.lstm_layer_fwd(MIXED, x_seq, w, np.zeros(4 * H, np.float32))
    _, gates_all, c_all, _ = cache
    assert np.array_equal(gates_all, x_seq)
    gd = h16(x_seq)
    c = [torch.zeros(B, H, dtype=torch.float32, device="cuda"), empty32(B, H), empty32(B, H)]
    h1 = empty16(T, B, H)
    h2 = torch.zeros(T, B, 2 * H + 8, dtype=torch.float16, device="cuda")
    for t in range(T):
        mp.mp_lstm_cell_fwd(B, H, gd[t], 4 * H, c[t], c[t + 1], h1[t], H, h2[t][:, H:], 2 * H + 8)
        assert np.allclose(np32(c[t + 1]), c_all[t + 1], rtol=2e-6, atol=2e-6)
        assert_close16(h1[t], h_ref[t], 1e-3, max_ulp=1, what=f"h[{t}]")
        assert np.array_equal(bits(h2[t][:, H:2 * H].contiguous()), bits(h1[t])) and float(h2[t][:, :H].abs().sum()) == 0
    # backward: dh = float(dh_a) + float(dh_b) on the device; the oracle receives that fp32 sum as the gradient from above
    dh_a, dh_b = S16(r.standard_normal((T, B, H))), S16(r.standard_normal((T, B, H)) * 0.3)
    dx_ref, _, _ = L.lstm_layer_bwd(MIXED, dh_a + dh_b, cache, w)      # = dgates of every step (W copies them)
    dcd, dg = torch.zeros(B, H, dtype=torch.float32, device="cuda"), empty16(T, B, 4 * H)
    # the device's own c would do as well; the oracle's keeps this an isolated check of the backward kernel
    for t in (1, 0):
        mp.mp_lstm_cell_bwd(B, H, gd[t], 4 * H, f32(c_all[t]), f32(c_all[t + 1]), h16(dh_a[t]), H, h16(dh_b[t]), H, dcd, dg[t])
        assert_close16(dg[t], dx_ref[t], 1e-3, what=f"dgates[{t}]")
    # one of the two addends may be absent
    dx_ref1, _, _ = L.lstm_layer_bwd(MIXED, dh_a, cache, w)
    dcd.zero_()
    for t in (1, 0):
        mp.mp_lstm_cell_bwd(B, H, gd[t], 4 * H, f32(c_all[t]), f32(c_all[t + 1]), h16(dh_a[t]), H, None, H, dcd, dg[t])
        assert_close16(dg[t], dx_ref1[t], 1e-3, what=f"dgates[{t}] single addend")


def _persistent_lstm_layer(T, Bn, I, H, x_seq, w, b, dh_seq, wait_limit_us=0, extra=0):
    """One LSTM layer through the persistent kernels: input half of the gate sums as one fp32 product, the recurrent
    kernel, and (backward) the recurrent kernel followed by the large input-gradient and weight-gradient products."""
    ld = I + H
    xh = torch.zeros(T, Bn, ld, dtype=torch.float16, device="cuda")
    xh[:, :, :I].copy_(h16(x_seq))
    wd, bd = h16(w), h16(b)
    gx = empty32(T * Bn, 4 * H)
    mp.mp_gemm_fwd(mp.gemm_desc(T * Bn, 4 * H, I, ldx=ld, ldw=ld), xh, wd, None, None, None, gx)
    gates, c = empty16(T, Bn, 4 * H), torch.zeros(T + 1, Bn, H, dtype=torch.float32, device="cuda")
    h_up = torch.full((T, Bn, H + 2), 5.0, dtype=torch.float16, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.zeros(mp.mp_lstm_layer_workspace_bytes() // 4, dtype=torch.int32, device="cuda")
    d = mp.lstm_layer_desc(T, Bn, I, H, ld, ld, H + 2, wait_limit_us, extra)
    mp.mp_lstm_layer_fwd(d, gx, wd, bd, gates, c, xh, h_up, status, ws)
    out = dict(xh=xh, gates=gates, c=c, h_up=h_up, status=status)
    if dh_seq is not None:
        dgates = empty16(T, Bn, 4 * H)
        mp.mp_lstm_layer_bwd(mp.lstm_layer_desc(T, Bn, I, H, ld, ld, H, wait_limit_us, extra), wd, gates, c, h16(dh_seq), dgates, status, ws)
        dx, dw, db = empty16(T * Bn, max(I, 8)), empty16(4 * H, ld), empty16(4 * H)
        if I > 0:
            dx = empty16(T * Bn, I)
            mp.mp_gemm_bwd_dx(mp.gemm_desc(T * Bn, 4 * H, I, ldx=I, ldw=ld), dgates, wd, dx)
        dall = mp.gemm_desc(T * Bn, 4 * H, ld)
        mp.mp_gemm_bwd_dw(dall, dgates, xh, dw, db, None, ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(dall, True)))
        out.update(dgates=dgates, dx=dx, dw=dw, db=db)
    return out


@pytest.mark.parametrize("T,Bn,I,H", [(6, 8, 96, 128), (5, 20, 64, 256), (3, 32, 8, 384), (4, 1, 0, 128), (1, 17, 8, 128),
                                      (10, 32, 1024, 1024)])
def test_lstm_persistent_layer_kernels(T, Bn, I, H):
    """All time steps of a layer in one launch per direction against the oracle's layer functions: every stored tensor
    of the forward pass (gate sums, h_t, fp32 cell states) and, from the GPU's own forward tensors, the gradients.
    Shapes: one and several workgroups, batch rows below / between / at the 16-row matrix-core blocks, no input half
    at all (I = 0), and config 5's layer at full width."""
    r = RNG(T * 1000 + Bn + I + H)
    x_seq = S16(r.standard_normal((T, Bn, I)))
    w, b = S16(r.uniform(-0.1, 0.1, (4 * H, I + H))), S16(r.standard_normal(4 * H) * 0.1)
    dh_seq = S16(r.standard_normal((T, Bn, H)))
    h_ref, cache = L.lstm_layer_fwd(MIXED, x_seq, w, b)
    xh_ref, gates_ref, c_ref, _ = cache
    o = _persistent_lstm_layer(T, Bn, I, H, x_seq, w, b, dh_seq)
    assert int(o["status"].item()) == 0
    assert_close16(o["gates"][0], gates_ref[0], 1e-3, max_ulp=1, what="gate sums of step 0")   # same inputs on both sides
    assert_close16(o["gates"], gates_ref, 1e-3, what="gate sums")      # later steps see the device's own h_{t-1}
    assert_close16(o["h_up"][:, :, :H], h_ref, 1e-3, what="h")
    assert torch.all(o["h_up"][:, :, H:] == 5.0)
    assert_close16(o["xh"], xh_ref, 1e-3, what="[x, h_prev] row blocks")
    assert rel_fro(np32(o["c"]), np.stack(c_ref)) <= 1e-3
    # backward from the device's own stored forward tensors (what a training step differentiates)
    cache_gpu = (np32(o["xh"]), np32(o["gates"]), list(np32(o["c"])), I)
    dx_ref, dw_ref, db_ref = L.lstm_layer_bwd(MIXED, dh_seq, cache_gpu, w)
    if I > 0:
        assert_close16(o["dx"].view(T, Bn, I), dx_ref, 1e-3, what="dx")
    assert_close16(o["dw"], dw_ref, 1e-3, what="dW")
    assert_close16(o["db"], db_ref, 1e-3, what="db")


@pytest.mark.parametrize("ld", [(1 << 21) - 1, 1 << 21, (1 << 21) + 3])
def test_gemm_leading_dimension_beyond_the_large_tiles(ld):
    """Leading dimensions around 2^21, where an offset inside a 256-row tile comes near the end of the buffer range and the
    rule changes to 64 x 64 tiles: a product over rows and one over columns of the same wide matrix."""
    M, N, K = 300, 40, 72
    r = RNG(ld % 1000)
    x, w, dy = S16(r.standard_normal((M, K))), S16(r.standard_normal((N, K)) * 0.1), S16(r.standard_normal((M, N)))
    buf = torch.zeros(M * ld, dtype=torch.float16, device="cuda")
    xd = buf.view(M, ld)
    xd[:, :K] = h16(x)
    y, dw = empty16(M, N), empty16(N, K)
    for tile in (-1, 0):
        mp.mp_gemm_tuning_override(tile, 1)
        try:
            mp.mp_gemm_fwd(mp.gemm_desc(M, N, K, ldx=ld), xd, h16(w), None, None, y)
            mp.mp_gemm_bwd_dw(mp.gemm_desc(M, N, K, ldx=ld), h16(dy), xd, dw, None, None, ws_bytes(1 << 20))
        finally:
            mp.mp_gemm_tuning_override(-1, 1)
        assert_close16(y, L.linear_fwd(MIXED, x, w, None), 1e-3, max_ulp=1, what="fwd")
        assert_close16(dw, L.linear_bwd(MIXED, dy, x, w)[1], 1e-3, max_ulp=1, what="dw")


@pytest.mark.parametrize("T,Bn,I,H", [(9, 9, 8, 640), (6, 31, 16, 896), (8, 3, 8, 512), (5, 24, 0, 768), (12, 32, 32, 1024)])
def test_lstm_persistent_layer_exchange_ring(T, Bn, I, H):
    """More time steps than the exchange ring has slots, every kind of k-step count per wave, batches that fill their
    8-row blocks and batches that do not, against the oracle layer."""
    test_lstm_persistent_layer_kernels(T, Bn, I, H)


@pytest.mark.parametrize("T,Bn,I,H,block", [(6, 40, 24, 64, 40), (7, 65, 8, 192, 33), (5, 20, 16, 320, 8), (6, 64, 40, 1024, 64)])
def test_lstm_persistent_layer_step_rows(T, Bn, I, H, block):
    """Calls that give step_rows: widths that are multiples of 64 only (waves with unequal or no shares of the
    contraction), batches of more than 32 rows, and a batch in blocks of rows, against the oracle layer."""
    r = RNG(T * 1000 + Bn + I + H)
    x_seq, dh_seq = S16(r.standard_normal((T, Bn, I))), S16(r.standard_normal((T, Bn, H)))
    w, b = S16(r.uniform(-0.1, 0.1, (4 * H, I + H))), S16(r.standard_normal(4 * H) * 0.1)
    h_ref, (xh_ref, gates_ref, c_ref, _) = L.lstm_layer_fwd(MIXED, x_seq, w, b)
    ld = I + H
    xh = torch.zeros(T, Bn, ld, dtype=torch.float16, device="cuda")
    xh[:, :, :I].copy_(h16(x_seq))
    wd, bd, gx, up = h16(w), h16(b), empty32(T * Bn, 4 * H), empty16(T, Bn, H)
    mp.mp_gemm_fwd(mp.gemm_desc(T * Bn, 4 * H, I, ldx=ld, ldw=ld), xh, wd, None, None, None, gx)
    gates, c, dgates = empty16(T, Bn, 4 * H), torch.zeros(T + 1, Bn, H, dtype=torch.float32, device="cuda"), empty16(T, Bn, 4 * H)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    dh = h16(dh_seq)
    for r0 in range(0, Bn, block):
        d = mp.lstm_layer_desc(T, min(block, Bn - r0), I, H, ld, ld, H, step_rows=Bn)
        ws = torch.zeros(mp.mp_lstm_layer_desc_workspace_bytes(d) // 4, dtype=torch.int32, device="cuda")
        mp.mp_lstm_layer_fwd(d, gx[r0:], wd, bd, gates[0, r0:], c[0, r0:], xh[0, r0:], up[0, r0:], status, ws)
        mp.mp_lstm_layer_bwd(d, wd, gates[0, r0:], c[0, r0:], dh[0, r0:], dgates[0, r0:], status, ws)
    assert int(status.item()) == 0
    assert_close16(gates[0], gates_ref[0], 1e-3, max_ulp=1, what="gate sums of step 0")
    for name, got, ref in (("gates", gates, gates_ref), ("h", up, h_ref), ("xh", xh, xh_ref)):
        assert_close16(got, ref, 1e-3, what=name)
    assert rel_fro(np32(c), np.stack(c_ref)) <= 1e-3
    _, dw_ref, db_ref = L.lstm_layer_bwd(MIXED, dh_seq, (np32(xh), np32(gates), list(np32(c)), I), w)
    dw, db, dall = empty16(4 * H, ld), empty16(4 * H), mp.gemm_desc(T * Bn, 4 * H, ld)
    mp.mp_gemm_bwd_dw(dall, dgates, xh, dw, db, None, ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(dall, True)))
    assert_close16(dw, dw_ref, 1e-3, what="dW")
    assert_close16(db, db_ref, 1e-3, what="db")


@pytest.mark.parametrize("T,Bn,H", [(9, 64, 512), (9, 65, 512), (2, 8, 64), (1, 9, 64), (6, 24, 192), (5, 64, 384), (5, 72, 384), (7, 128, 256)])
def test_lstm_persistent_layer_places(T, Bn, H):
    """Groups of workgroups on one XCD each, several to an XCD, and one group more than that allows; a workspace that holds the
    exchange rings but not the words in which workgroups tell where they run gives the same bits, and both the oracle's."""
    r = RNG(T + Bn + H)
    I, ld = 8, 8 + H
    x_seq, dh_seq = S16(r.standard_normal((T, Bn, I))), S16(r.standard_normal((T, Bn, H)))
    w, b = S16(r.uniform(-0.1, 0.1, (4 * H, ld))), S16(r.standard_normal(4 * H) * 0.1)
    wd, bd, dh = h16(w), h16(b), h16(dh_seq)
    d = mp.lstm_layer_desc(T, Bn, I, H, ld, ld, H, step_rows=Bn)
    full = mp.mp_lstm_layer_desc_workspace_bytes(d) // 4
    rings = (Bn + 7) // 8 * 4 * 4 * 1024 * (H // 64) // 4 + 4
    assert full >= rings and (full > rings) == (H // 16 * ((Bn + 63) // 64) <= 32)
    outs = []
    for words in (full, rings):
        xh = torch.zeros(T, Bn, ld, dtype=torch.float16, device="cuda")
        xh[:, :, :I].copy_(h16(x_seq))
        gx, up = empty32(T * Bn, 4 * H), empty16(T, Bn, H)
        mp.mp_gemm_fwd(mp.gemm_desc(T * Bn, 4 * H, I, ldx=ld, ldw=ld), xh, wd, None, None, None, gx)
        gates, c, dgates = empty16(T, Bn, 4 * H), torch.zeros(T + 1, Bn, H, dtype=torch.float32, device="cuda"), empty16(T, Bn, 4 * H)
        status, ws = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(words, dtype=torch.int32, device="cuda")
        mp.mp_lstm_layer_fwd_placed(d, gx, wd, bd, gates, c, xh, up, status, ws)
        mp.mp_lstm_layer_bwd_placed(d, wd, gates, c, dh, dgates, status, ws)
        assert int(status.item()) == 0
        outs.append((gates, c, xh, up, dgates))
    for a, b_ in zip(*outs):
        assert torch.equal(a, b_)
    gates, c, xh, up, dgates = outs[0]
    h_ref, (_, gates_ref, c_ref, _) = L.lstm_layer_fwd(MIXED, x_seq, w, b)
    assert_close16(gates, gates_ref, 1e-3, what="gates")
    assert_close16(up, h_ref, 1e-3, what="h")
    assert rel_fro(np32(c), np.stack(c_ref)) <= 1e-3
    _, _, db_ref = L.lstm_layer_bwd(MIXED, dh_seq, (np32(xh), np32(gates), list(np32(c)), I), w)
    db = empty16(4 * H)
    mp.mp_colsum(T * Bn, 4 * H, dgates, 4 * H, db, None, ws_bytes(mp.mp_colsum_workspace_bytes(T * Bn, 4 * H)))
    assert_close16(db, db_ref, 1e-3, what="db")


@pytest.mark.parametrize("T,Bn,H", [(9, 64, 512), (9, 65, 512), (2, 8, 64), (1, 9, 64), (6, 24, 192), (5, 64, 384), (5, 72, 384), (7, 128, 256), (4, 32, 1024)])
def test_lstm_persistent_layer_placed_calls(T, Bn, H):
    """The calls that put each group of workgroups on one XCD, several groups to an XCD, and one group or width more than that
    allows, with the words in which workgroups tell where they run and without: the bits of the plain calls."""
    r = RNG(T + Bn + H)
    I, ld = 8, 8 + H
    x_seq, wd, bd = h16(r.standard_normal((T, Bn, I))), h16(r.uniform(-0.1, 0.1, (4 * H, ld))), h16(r.standard_normal(4 * H) * 0.1)
    dh, gx = h16(r.standard_normal((T, Bn, H))), f32(r.standard_normal((T * Bn, 4 * H)))
    d = mp.lstm_layer_desc(T, Bn, I, H, ld, ld, H, step_rows=Bn)
    full = mp.mp_lstm_layer_desc_workspace_bytes(d) // 4
    rings = (Bn + 7) // 8 * 4 * 4 * 1024 * (H // 64) // 4 + 4
    outs = []
    for placed, words in ((False, full), (True, full), (True, rings)):
        xh = torch.zeros(T, Bn, ld, dtype=torch.float16, device="cuda")
        xh[:, :, :I].copy_(x_seq)
        gates, up, dgates = empty16(T, Bn, 4 * H), empty16(T, Bn, H), empty16(T, Bn, 4 * H)
        c, status = torch.zeros(T + 1, Bn, H, dtype=torch.float32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        a, b = (torch.zeros(words, dtype=torch.int32, device="cuda") for _ in range(2))
        if placed:
            mp.mp_lstm_layer_fwd_placed(d, gx, wd, bd, gates, c, xh, up, status, a, False, b)
            mp.mp_lstm_layer_bwd_placed(d, wd, gates, c, dh, dgates, status, b, True)
        else:
            mp.mp_lstm_layer_fwd(d, gx, wd, bd, gates, c, xh, up, status, a)
            mp.mp_lstm_layer_bwd(d, wd, gates, c, dh, dgates, status, b)
        assert int(status.item()) == 0
        outs.append((gates, c, xh, up, dgates))
    for other in outs[1:]:
        for a, b in zip(outs[0], other):
            assert torch.equal(a, b)


def test_lstm_persistent_layer_workspace_at_any_word():
    """A workspace of the stated size at a 4-byte boundary that is no 16-byte boundary is enough."""
    T, Bn, I, H = 6, 32, 8, 1024
    r = RNG(78)
    w = h16(r.uniform(-0.05, 0.05, (4 * H, I + H)))
    gx, bias = f32(r.standard_normal((T * Bn, 4 * H))), h16(np.zeros(4 * H))
    got = []
    for lead in (0, 1):
        words = mp.mp_lstm_layer_workspace_bytes() // 4
        buf = torch.zeros(words + lead + 64, dtype=torch.int32, device="cuda")
        gates, c, status = empty16(T, Bn, 4 * H), torch.zeros(T + 1, Bn, H, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        xh, up = torch.zeros(T, Bn, I + H, dtype=torch.float16, device="cuda"), empty16(T, Bn, H)
        d = mp.lstm_layer_desc(T, Bn, I, H, I + H, I + H, H)
        mp.mp_lstm_layer_fwd(d, gx, w, bias, gates, c, xh, up, status, buf[lead:lead + words])
        assert int(status.item()) == 0 and torch.all(buf[lead + words:] == 0)
        got.append(up)
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("T,Bn,H", [(9, 32, 1024), (2, 3, 64), (5, 65, 192), (1, 8, 128)])
def test_lstm_persistent_layer_chain(T, Bn, H):
    """Calls that empty the next call's workspace: forward and backward calls in a chain of two workspaces that start full of
    other values, the same bits as the plain calls, twice; a workspace that overlaps the call's own is refused."""
    I = 8
    r = RNG(T + Bn + H)
    ld = I + H
    w, bias, gx = h16(r.uniform(-0.1, 0.1, (4 * H, ld))), h16(np.zeros(4 * H)), f32(r.standard_normal((T * Bn, 4 * H)))
    dh = h16(r.standard_normal((T, Bn, H)))
    d = mp.lstm_layer_desc(T, Bn, I, H, ld, ld, H, step_rows=Bn)
    words = mp.mp_lstm_layer_desc_workspace_bytes(d) // 4
    # (in one buffer, at 4-byte boundaries that are no 16-byte boundaries, with guard words around them)
    buf = torch.full((2 * words + 3,), 0x3C003C00, dtype=torch.int32, device="cuda")
    two = [buf[1:1 + words], buf[2 + words:2 + 2 * words]]
    status = torch.zeros(1, dtype=torch.int32, device="cuda")

    def run(chain):
        out = []
        a, b, ready = two[0], two[1], False
        for _ in range(2):
            gates, c = empty16(T, Bn, 4 * H), torch.zeros(T + 1, Bn, H, device="cuda")
            xh, up, dgates = torch.zeros(T, Bn, ld, dtype=torch.float16, device="cuda"), empty16(T, Bn, H), empty16(T, Bn, 4 * H)
            if chain:
                mp.mp_lstm_layer_fwd_chain(d, gx, w, bias, gates, c, xh, up, status, a, ready, b)
                mp.mp_lstm_layer_bwd_chain(d, w, gates, c, dh, dgates, status, b, True, a)
                ready = True
            else:
                mp.mp_lstm_layer_fwd(d, gx, w, bias, gates, c, xh, up, status, a)
                mp.mp_lstm_layer_bwd(d, w, gates, c, dh, dgates, status, a)
            out += [gates, c, xh, up, dgates]
        return out

    plain = run(False)
    buf.fill_(0x3C003C00)
    for got, ref in zip(run(True), plain):
        assert torch.equal(got, ref)
    assert int(status.item()) == 0
    assert all(int(buf[k]) == 0x3C003C00 for k in (0, 1 + words, 2 + 2 * words))
    with pytest.raises(mp.MPError) as e:
        mp.mp_lstm_layer_bwd_chain(d, w, plain[0], plain[1], dh, plain[4], status, two[0], False, buf[words // 2:words // 2 + words])
    assert e.value.code == ML.MP_E_INVAL


def test_lstm_persistent_layer_timeout_path_and_rejections():
    """The step barrier's wait is bounded: asked to wait for a flag nobody raises (debug_extra_participants) with a
    2 ms limit, every workgroup gives up, the kernels end normally and *status reports it; a poisoned status makes the
    next launch stop at its first barrier; after clearing it the same buffers give the right answer again."""
    T, Bn, I, H = 4, 8, 32, 256
    r = RNG(77)
    x_seq, w, b = S16(r.standard_normal((T, Bn, I))), S16(r.uniform(-0.1, 0.1, (4 * H, I + H))), S16(np.zeros(4 * H))
    o = _persistent_lstm_layer(T, Bn, I, H, x_seq, w, b, S16(r.standard_normal((T, Bn, H))), wait_limit_us=2000, extra=1)
    torch.cuda.synchronize()
    assert int(o["status"].item()) != 0
    h_ref, _ = L.lstm_layer_fwd(MIXED, x_seq, w, b)
    good = _persistent_lstm_layer(T, Bn, I, H, x_seq, w, b, None)
    assert int(good["status"].item()) == 0
    assert_close16(good["h_up"][:, :, :H], h_ref, 1e-3, what="h after a timed-out launch")
    # unsupported shapes are refused before anything is launched
    ws = torch.zeros(mp.mp_lstm_layer_workspace_bytes() // 4, dtype=torch.int32, device="cuda")
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    for (Bx, Hx, Ix) in ((33, 128, 8), (8, 192, 8), (8, 2048, 8), (8, 128, 4)):
        with pytest.raises(mp.MPError) as e:
            mp.mp_lstm_layer_fwd(mp.lstm_layer_desc(2, Bx, Ix, Hx, Ix + Hx, Ix + Hx, Hx), empty32(2 * Bx, 4 * Hx), empty16(4 * Hx, Ix + Hx),
                                 empty16(4 * Hx), empty16(2, Bx, 4 * Hx), empty32(3, Bx, Hx), empty16(2, Bx, Ix + Hx), None, st, ws)
        assert e.value.code == ML.MP_E_UNSUPPORTED
    with pytest.raises(mp.MPError) as e:
        mp.mp_lstm_layer_fwd(mp.lstm_layer_desc(2, 8, 8, 128, 136, 136, 128), empty32(16, 512), empty16(512, 136), empty16(512),
                             empty16(2, 8, 512), empty32(3, 8, 128), empty16(2, 8, 136), None, None, ws)
    assert e.value.code == ML.MP_E_INVAL


@pytest.mark.parametrize("rows,cols", [(4096, 512), (100, 40), (1, 8), (777, 1001), (8192, 64)])
def test_colsum(rows, cols):
    r = RNG(rows + cols)
    dy = S16(r.standard_normal((rows, cols)))
    db = empty16(cols)
    mp.mp_colsum(rows, cols, h16(dy), cols, db, None, ws_bytes(mp.mp_colsum_workspace_bytes(rows, cols)))
    assert_close16(db, MIXED.store(dy.sum(0, dtype=np.float32)), 1e-3, max_ulp=1, what="colsum")


def test_gradient_producers_flag_their_own_overflow():
    """The column-sum and LayerNorm-backward kernels write fp16 gradients (bias, gamma, beta): when a sum leaves the
    fp16 range the stored value is inf as in the oracle, and the overflow flag of the state they are given is set
    (what MP_UPDATE_PRECHECKED relies on)."""
    rows, cols = 4096, 264
    dy = np.full((rows, cols), 2.0, np.float32)
    dy[:, 5] = 100.0                                           # column 5 sums to 409600: beyond fp16
    dy[:, 9] = -100.0
    ref = MIXED.store(dy.sum(0, dtype=np.float32))
    assert np.isposinf(ref[5]) and np.isneginf(ref[9]) and np.isfinite(np.delete(ref, [5, 9])).all()
    st = make_state()
    db = empty16(cols)
    ws = ws_bytes(mp.mp_colsum_workspace_bytes(rows, cols))
    mp.mp_colsum(rows, cols, h16(dy), cols, db, st, ws)
    assert np.array_equal(bits(db), half_bits(ref)) and mp.scale_state_read(st).found_inf == 1
    st = make_state()
    mp.mp_colsum(rows, cols, h16(np.full((rows, cols), 2.0, np.float32)), cols, db, st, ws)
    assert mp.scale_state_read(st).found_inf == 0 and torch.all(db == 8192.0)
    # a NaN in the input reaches the sum and the flag
    dyn = np.full((rows, cols), 1.0, np.float32)
    dyn[77, 3] = np.nan
    mp.mp_colsum(rows, cols, h16(dyn), cols, db, st, ws)
    assert mp.scale_state_read(st).found_inf == 1 and np.isnan(np32(db)[3]) and np.isfinite(np.delete(np32(db), 3)).all()
    # the weight-gradient entry point with db: flag from the bias gradient alone (dW itself stays finite)
    d = mp.gemm_desc(rows, cols, 64)
    x = np.zeros((rows, 64), np.float32)
    st = make_state()
    dw, db2 = empty16(cols, 64), empty16(cols)
    mp.mp_gemm_bwd_dw(d, h16(dy), h16(x), dw, db2, st, ws_bytes(mp.mp_gemm_bwd_dw_workspace_bytes(d, True)))
    assert torch.all(dw == 0) and np.array_equal(bits(db2), half_bits(ref)) and mp.scale_state_read(st).found_inf == 1

    # LayerNorm backward: dgamma = sum_rows dy xhat, dbeta = sum_rows dy, dz column sums
    rows, d_ = 2048, 256
    r = RNG(5)
    x_, a_ = S16(r.standard_normal((rows, d_))), S16(r.standard_normal((rows, d_)) * 0.5)
    gam = S16(np.ones(d_))
    y_ref, cache = L.layernorm_fwd(MIXED, x_, a_, gam, np.zeros(d_, np.float32))
    xd, ad, gd = h16(x_), h16(a_), h16(gam)
    y, mean, rstd = empty16(rows, d_), empty32(rows), empty32(rows)
    mp.mp_layernorm_fwd(rows, d_, xd, ad, gd, h16(np.zeros(d_)), L.LN_EPS, y, mean, rstd)
    for case in ("dbeta", "dgamma", "clean"):
        dy_ = S16(r.standard_normal((rows, d_)))
        if case == "dbeta":
            dy_[:, 11] = 64.0                                   # 2048 x 64 = 131072 -> inf in dbeta[11]
        elif case == "dgamma":
            dy_[:, 13] = S16(600.0 * np.sign(cache[0][:, 13]))  # sum |xhat| 600 ~ 1e6 -> inf in dgamma[13]
        dz_ref, dg_ref, db_ref = L.layernorm_bwd(MIXED, dy_, cache, gam)
        bad_ref = not (np.isfinite(dg_ref).all() and np.isfinite(db_ref).all()
                       and np.isfinite(MIXED.store(dz_ref.sum(0, dtype=np.float32))).all())
        assert bad_ref == (case != "clean")
        st = make_state()
        dz, dg, dbt, dzs = empty16(rows, d_), empty16(d_), empty16(d_), empty16(d_)
        mp.mp_layernorm_bwd(rows, d_, h16(dy_), xd, ad, gd, mean, rstd, dz, dg, dbt, st,
                            ws_bytes(mp.mp_layernorm_bwd_workspace_bytes(rows, d_)), dz_colsum=dzs)
        assert mp.scale_state_read(st).found_inf == int(bad_ref), case
        assert np.array_equal(np.isfinite(np32(dg)), np.isfinite(dg_ref)) and np.array_equal(np.isfinite(np32(dbt)), np.isfinite(db_ref))


def test_cast_is_rne_and_overflows_to_inf():
    r = RNG(12)
    x = np.concatenate([r.standard_normal(100003).astype(np.float32) * np.float32(s) for s in (1e-7, 1e-3, 1, 7e4)])
    x[:6] = [65520.0, 65519.99, 2.0 ** -25, np.nextafter(np.float32(2.0 ** -25), np.float32(1)), -1e9, np.nan]
    out = empty16(x.size)
    mp.mp_cast_f32_to_f16(x.size, f32(x), out)
    ref = half_bits(MIXED.store(x))
    got = bits(out)
    nan = np.isnan(x)
    assert np.array_equal(got[~nan], ref[~nan]) and np.all((got[nan] & 0x7C00) == 0x7C00)


# ------------------------------------------------------------------ optimizer wrapper and scale policy
def _tensors(r, sizes, adam=True):
    out = []
    for n in sizes:
        out.append(dict(w=r.standard_normal(n).astype(np.float32) * 0.05, g=S16(r.standard_normal(n) * 100),
                        m=r.standard_normal(n).astype(np.float32) * 0.01, v=np.abs(r.standard_normal(n)).astype(np.float32) * 1e-4))
    return out


def _run_update(ts, kind, S, t_prev, wd=0.0, poison=None, flags=0, lr=1e-3):
    host = [dict(g16=t["g"].copy(), w32=t["w"].copy(), w16=MIXED.store(t["w"]), m=t["m"].copy(), v=t["v"].copy()) for t in ts]
    if poison is not None:
        host[poison[0]]["g16"][poison[1]] = poison[2]
    ost = O.ScaleState(scale=S, opt_step=t_prev, growth_interval=3)
    ocfg = I.OptCfg(kind=kind, lr=lr, weight_decay=wd)
    dev = [dict(g16=h16(h["g16"]), w32=f32(h["w32"]), w16=h16(h["w16"]), m=f32(h["m"]), v=f32(h["v"])) for h in host]
    found_ref = O.unscale_check_update(MIXED, host, ocfg, ost)
    O.loss_scale_update(ost, found_ref)
    st = make_state(scale=S, interval=3)
    # bring the device state to the same optimizer step count
    words = st.cpu()
    words[8] = t_prev
    st.copy_(words)
    mp.mp_unscale_check_update(mp.tensor_list(dev), len(dev), mp.opt_cfg(kind, lr, weight_decay=wd), st, flags)
    mp.mp_loss_scale_update(st)
    return host, dev, ost, mp.scale_state_read(st), found_ref


@pytest.mark.parametrize("kind", ["adam", "sgd"])
@pytest.mark.parametrize("t_prev,wd", [(0, 0.0), (1, 1e-4), (57, 1e-2), (3, 0.3)])
def test_update_matches_oracle(kind, t_prev, wd):
    """Unscale + SGD / Adam on the masters + fp16 re-cast, with and without the fp32-side weight decay of Section 3.3
    (g += wd * w32 after unscaling, for both optimizers)."""
    sizes = [8192 * 3 + 5, 1, 7, 4096, 100000, 33] + [64] * 40          # > 32 tensors: several launches
    ts = _tensors(RNG(20 + t_prev), sizes)
    host, dev, ost, dst, found = _run_update(ts, kind, 2.0 ** 7, t_prev, wd=wd)
    assert found == 0 and dst.opt_step == ost.opt_step == t_prev + 1
    for h, d in zip(host, dev):
        assert rel_fro(np32(d["w32"]), h["w32"]) <= 1e-5
        assert np.abs(np32(d["w32"]) - h["w32"]).max() <= 1e-5 * np.abs(h["w32"]).max()
        if kind == "adam":
            assert rel_fro(np32(d["m"]), h["m"]) <= 1e-6 and rel_fro(np32(d["v"]), h["v"]) <= 1e-6
        # the fp16 copy is exactly RNE16 of the master the device holds
        assert np.array_equal(bits(d["w16"]), half_bits(MIXED.store(np32(d["w32"]))))


@pytest.mark.parametrize("poison", [False, True])
@pytest.mark.parametrize("n", [2048 * 1024 - 2, 2048 * 1024 + 5, 2 * 2048 * 1024 + 1023, 4 * 2048 * 1024 + 4])
def test_update_workgroup_shares(n, poison):
    """Parameter counts around the lines where a workgroup takes 1, 2, 4 or 8 pieces, in two tensors: every element is
    updated once, and a value that is not finite is found in the last element of the list."""
    sizes = [n - 1500, 1500]
    ts = _tensors(RNG(24), sizes)
    host, dev, ost, dst, found = _run_update(ts, "adam", 2.0 ** 7, 3, poison=(1, 1499, np.inf) if poison else None)
    assert found == int(poison) and dst.opt_step == ost.opt_step == 3 + (not poison)
    for h, d in zip(host, dev):
        if poison:
            assert np.array_equal(np32(d["w32"]), h["w32"]) and np.array_equal(np32(d["v"]), h["v"])
        else:  # tolerances as in test_update_matches_oracle
            assert rel_fro(np32(d["w32"]), h["w32"]) <= 1e-5 and np.abs(np32(d["w32"]) - h["w32"]).max() <= 1e-5 * np.abs(h["w32"]).max()
            assert rel_fro(np32(d["m"]), h["m"]) <= 1e-6 and rel_fro(np32(d["v"]), h["v"]) <= 1e-6


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("where", [(0, 0), (2, 4095), (5, 32), (45, 63)])
def test_update_skips_on_nonfinite_and_halves_scale(bad, where):
    sizes = [8192 * 3 + 5, 1, 4096, 7, 100000, 33] + [64] * 40
    ts = _tensors(RNG(30), sizes)
    host, dev, ost, dst, found = _run_update(ts, "adam", 2.0 ** 15, 4, poison=(where[0], where[1], bad))
    assert found == 1
    assert (dst.scale, dst.good_steps, dst.opt_step, dst.skipped_steps, dst.found_inf) == (2.0 ** 14, 0, 4, 1, 0)
    assert (ost.scale, ost.good_steps, ost.opt_step, ost.skipped_steps) == (2.0 ** 14, 0, 4, 1)
    assert dst.hist_scale[0] == 2.0 ** 15 and dst.hist_found_inf[0] == 1
    for t, d in zip(ts, dev):                 # every buffer byte-identical to before the call
        assert np.array_equal(np32(d["w32"]).view(np.uint32), t["w"].view(np.uint32))
        assert np.array_equal(np32(d["m"]).view(np.uint32), t["m"].view(np.uint32))
        assert np.array_equal(np32(d["v"]).view(np.uint32), t["v"].view(np.uint32))
        assert np.array_equal(bits(d["w16"]), half_bits(MIXED.store(t["w"])))


def test_update_prechecked_flag_trusts_state():
    ts = _tensors(RNG(31), [5000])
    host, dev, ost, dst, found = _run_update(ts, "sgd", 4.0, 0, poison=(0, 17, np.inf), flags=ML.MP_UPDATE_PRECHECKED)
    # the inspection pass was skipped and nobody had set the flag: the step is applied (inf reaches the master)
    assert found == 1 and dst.opt_step == 1 and not np.isfinite(np32(dev[0]["w32"])[17])


@pytest.mark.parametrize("name", ["c1", "c2", "c4", "c5", "floor"])
def test_scale_policy_sequences(name):
    from test_oracle_optimizer import _golden
    g = _golden()[name]
    st = make_state(scale=g["s0"], interval=g["n"])
    flag = torch.ones(1, dtype=torch.int32, device="cuda")
    for step in range(g["steps"]):
        if step in g["ovf"]:
            st[7:8].copy_(flag)               # found_inf word, as a gradient-producing kernel would set it
        mp.mp_loss_scale_update(st)
    s = mp.scale_state_read(st)
    assert list(s.hist_scale[:g["steps"]]) == g["seq"]
    assert list(s.hist_found_inf[:g["steps"]]) == [int(i in g["ovf"]) for i in range(g["steps"])]
    assert (s.scale, s.good_steps, s.opt_step, s.skipped_steps, s.total_steps) == (g["final"], g["good"], g["t"], g["skipped"], g["steps"])
    assert s.inv_scale == 1.0 / g["final"]


def test_scale_state_static_mode_and_validation():
    st = make_state(mode=ML.MP_SCALE_STATIC, scale=10.0, interval=1)
    flag = torch.ones(1, dtype=torch.int32, device="cuda")
    for f in (0, 1, 0, 0):
        if f:
            st[7:8].copy_(flag)
        mp.mp_loss_scale_update(st)
    s = mp.scale_state_read(st)
    assert s.scale == 10.0 and s.skipped_steps == 1 and s.opt_step == 3 and s.inv_scale == np.float32(1.0) / np.float32(10.0)
    with pytest.raises(mp.MPError):
        mp.mp_scale_state_init(st, 1, 2.0, 0)
    with pytest.raises(mp.MPError):
        mp.mp_scale_state_init(st, 7, 2.0, 1)


@pytest.mark.parametrize("tile,splits", [(1, 1), (3, 1), (4, 1), (5, 1), (1, 3), (3, 2), (4, 3), (5, 4), (9, 1), (10, 1), (9, 2)])
@pytest.mark.parametrize("T,N,K", [(192, 256, 512), (193, 520, 456), (1000, 264, 392), (640, 1024, 40), (65, 36, 24), (700, 29, 36)])
def test_bias_gradient_from_the_weight_gradient(T, N, K, tile, splits):
    """Both gradients from one launch in every tile shape that carries the sums (9 and 10: the small kernel), split or not, with rows,
    columns and a contraction that stick out of the tiles and rows at any alignment, and (few inputs) where the waves beside each other do not cover a tile's rows and the sums
    are launches of their own; a sum that overflows raises the flag."""
    r = RNG(T + N + K)
    dy, x, w = S16(r.standard_normal((T, N))), S16(r.standard_normal((T, K))), S16(r.standard_normal((N, K)))
    d, st = mp.gemm_desc(T, N, K), mp.scale_state_alloc()
    mp.mp_scale_state_init(st, ML.MP_SCALE_BACKOFF, 2.0, 100, 1.0, 2.0 ** 24)
    ws = ws_bytes(8 << 20)
    xd = h16(x)
    _, dw_ref, db_ref = L.linear_bwd(MIXED, dy, x, w)
    mp.mp_gemm_tuning_override(tile, splits)
    try:
        for bad in (False, True):
            dyd, dw, db = h16(dy), empty16(N, K), empty16(N)
            if bad:
                dyd[:, N - 1] = 30000.0
            mp.mp_gemm_bwd_dw(d, dyd, xd, dw, db, st, ws)
            if not bad:
                # (fp32 sums in another order: one ulp of the result, and of the summed magnitudes where they cancel)
                assert_close16(dw, dw_ref, 1e-3, max_ulp=1, what="dw")
                assert_close16(db, db_ref, 1e-3, max_ulp=1, what="db")
                assert mp.scale_state_read(st).found_inf == 0
            else:
                assert torch.isinf(db[N - 1]) and torch.equal(db[:N - 1], good) and mp.scale_state_read(st).found_inf == 1
            good = db[:N - 1]
    finally:
        mp.mp_gemm_tuning_override(-1, 1)


@pytest.mark.parametrize("tile,splits", [(1, 1), (3, 1), (4, 1), (5, 1), (1, 3), (3, 2), (4, 3), (5, 4), (9, 1), (10, 1), (9, 2), (0, 1), (-1, 1)])
@pytest.mark.parametrize("T,N,K", [(640, 264, 392), (193, 520, 456), (700, 29, 36)])
def test_bias_gradient_of_subnormal_gradients(T, N, K, tile, splits):
    """Gradients below the least normal half (multiples of 2^-24, what loss scaling is about), and beside them one row of 2^-3: every
    partial sum is a multiple of 2^-24 below 2^-2, exact in fp32 in any order, so the bias gradient is the sum's one rounding.  Every
    tile shape that carries the sums, one that leaves them to launches of their own (0), and the joint launch (-1)."""
    r = RNG(T + N + K)
    k = r.integers(-1023, 1024, (T, N))
    k[1, :] = 1                            # a lone least subnormal is not lost beside the large row either
    big = k.copy()
    big[0, ::2] = 1 << 21
    d, x, w = mp.gemm_desc(T, N, K), h16(r.standard_normal((T, K))), h16(r.standard_normal((N, K)))
    ws = ws_bytes(8 << 20)
    mp.mp_gemm_tuning_override(tile, splits)
    try:
        for units in (k, big, np.where(np.arange(T)[:, None] == 1, k, 0)):
            dy, dw, db = h16(units * 2.0 ** -24), empty16(N, K), empty16(N)
            if tile < 0:
                assert mp.mp_gemm_bwd_both_joint(d, d)
                mp.mp_gemm_bwd_both(d, dy, w, empty16(T, K), d, x, dw, db, None, ws)
            else:
                mp.mp_gemm_bwd_dw(d, dy, x, dw, db, None, ws)
            assert np.abs(units).sum(0).max() < 1 << 22
            want = h16(units.sum(0).astype(np.float64) * 2.0 ** -24)
            assert torch.equal(db, want) and torch.count_nonzero(db) > 0
    finally:
        mp.mp_gemm_tuning_override(-1, 1)


@pytest.mark.parametrize("kind,rows,cols,ld", [("mse", 3, 8, 8), ("mse", 300, 29, 31), ("mse", 4096, 512, 512), ("xent", 5, 40, 40),
                                               ("xent", 257, 1001, 1008), ("xent", 600, 17000, 17000), ("xent", 9000, 264, 264)])
def test_loss_finished_with_the_scale_update(kind, rows, cols, ld):
    """A loss left as partial sums and finished by the launch that updates the scale: the bits of the plain call, the state that
    mp_loss_scale_update leaves, for one and for many partial sums per thread, with and without the bias gradient."""
    r = RNG(rows + cols)
    y, t = h16(r.standard_normal((rows, ld))), h16(r.standard_normal((rows, ld)))
    tgt, ws = i32(r.integers(0, cols, rows)), ws_bytes(mp.mp_softmax_xent_db_workspace_bytes(rows, cols))
    for with_db in ((False, True) if kind == "xent" else (False,)):
        out = []
        for parts in (False, True):
            st, loss, g, db = mp.scale_state_alloc(), empty32(1), empty16(rows, ld), empty16(cols)
            mp.mp_scale_state_init(st, ML.MP_SCALE_BACKOFF, 2.0 ** 12, 1, 1.0, 2.0 ** 24)
            g.zero_(), db.zero_()
            if kind == "mse" and parts:
                p = mp.mp_mse_scaled_parts(rows, cols, y, t, ld, st, g, ws)
            elif kind == "mse":
                mp.mp_mse_scaled(rows, cols, y, t, ld, st, loss, g, ws)
            elif parts:
                p = mp.mp_softmax_xent_scaled_parts(rows, cols, y, ld, tgt, st, g, None, db if with_db else None, ws)
            elif with_db:
                mp.mp_softmax_xent_scaled_db(rows, cols, y, ld, tgt, st, loss, g, db, ws)
            else:
                mp.mp_softmax_xent_scaled(rows, cols, y, ld, tgt, st, loss, g, ws)
            if parts:
                mp.mp_loss_scale_update_mean(st, p, loss)
            else:
                mp.mp_loss_scale_update(st)
            out.append((loss, st, g, db))
        for a, b in zip(*out):
            assert torch.equal(a, b)
        assert float(out[0][0]) > 0 and mp.scale_state_read(out[1][1]).scale == 2.0 ** 13


@pytest.mark.parametrize("kind", ["adam", "sgd"])
@pytest.mark.parametrize("sizes", [(5,), (1000, 40000), (31 * 1024 + 1,), (1024 * 1024,), (1024 * 1024 + 1,), (3000,) * 33])
def test_iteration_ended_by_the_update(sizes, kind):
    """mp_unscale_check_update_end against the calls it stands for: one workgroup, fewer and more than there are counters, the most
    it counts and one more, more tensors than a launch takes; clean and overflowing iterations in turn, as calls and as a replayed
    graph; the counters are clear afterwards."""
    r = RNG(sum(sizes))
    cfg = mp.opt_cfg(kind, 1e-3, 0.9, 0.999, 1e-8, 0.01)
    part, part_n = torch.from_numpy(r.random(300).astype(np.float32)).cuda(), 300
    parts = ML.MeanParts()
    parts.part, parts.denom, parts.n = part.data_ptr(), 7.0, part_n
    g0, w0 = [h16(r.standard_normal(n)) for n in sizes], [torch.from_numpy(r.standard_normal(n).astype(np.float32)).cuda() for n in sizes]
    outs = []
    for how in ("apart", "end", "graph"):
        t = [dict(g16=g.clone(), w32=w.clone(), w16=w.half(), m=torch.zeros_like(w), v=torch.zeros_like(w)) for g, w in zip(g0, w0)]
        tl, st, loss, counters = mp.tensor_list(t), mp.scale_state_alloc(), empty32(1), mp.update_counters_alloc()
        mp.mp_scale_state_init(st, ML.MP_SCALE_BACKOFF, 2.0 ** 10, 2, 1.0, 2.0 ** 24)

        def one(p):
            if how == "apart":
                mp.mp_unscale_check_update(tl, len(t), cfg, st)
                mp.mp_loss_scale_update_mean(st, p, loss) if p is not None else mp.mp_loss_scale_update(st)
            else:
                mp.mp_unscale_check_update_end(tl, len(t), cfg, st, counters, ML.MP_UPDATE_DEFAULT, p, None if p is None else loss)
        one(None)
        run = lambda: one(parts)  # noqa: E731
        if how == "graph":
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                one(parts)
            run = graph.replay
        seen = []
        for k in range(5):
            t[-1]["g16"][-1:].fill_(float("inf") if k == 2 else 0.5)
            run()
            torch.cuda.synchronize()
            seen.append([loss.clone(), st.clone()] + [x[f].clone() for x in t for f in ("w32", "w16", "m", "v")])
            assert int(counters.abs().max()) == 0
        outs.append(seen)
        s = mp.scale_state_read(st)
        assert s.total_steps == 6 and s.skipped_steps == 1 and s.opt_step == 5 and s.found_inf == 0
    for a, b, c in zip(*outs):
        for x, y, z in zip(a, b, c):
            assert torch.equal(x, y) and torch.equal(x, z)
