// Contractions: split-K finish, generic fallback and the C entry points.  The matrix-core kernel templates are in gemm_kernels.hpp and
// are instantiated in gemm_kk.hip / gemm_ko.hip / gemm_oo.hip; gemm_plan.hpp picks among them.
#include "gemm_dtl.hpp"
#include "gemm_small.hpp"

#include <algorithm>
#include <cstdlib>
#include <cstring>

namespace mp {

extern template int launch_tile<true, true>(int, const GemmArgs&, dim3, hipStream_t);
extern template int launch_tile<true, false>(int, const GemmArgs&, dim3, hipStream_t);
extern template int launch_tile<false, false>(int, const GemmArgs&, dim3, hipStream_t);
extern template int launch_dtl_tile<true, true>(int, const GemmArgs&, dim3, hipStream_t);
extern template int launch_dtl_tile<true, false>(int, const GemmArgs&, dim3, hipStream_t);
extern template int launch_dtl_tile<false, false>(int, const GemmArgs&, dim3, hipStream_t);
extern template int launch_grouped<256, 256>(const GroupArgs&, hipStream_t);
extern template int launch_grouped<128, 128>(const GroupArgs&, hipStream_t);
extern template int launch_dtl_grouped<256, 256>(const GroupArgs&, hipStream_t);
extern template int launch_dtl_grouped<256, 128>(const GroupArgs&, hipStream_t);
extern template int launch_dtl_grouped<128, 128>(const GroupArgs&, hipStream_t);

// Sum split-K partials in split order, scale, round once, optional non-finite flag.  db (may be NULL): the same for the
// sums of the first operand, db_part[splits][db_n], which have no scale.
__global__ __launch_bounds__(256) void splitk_finish_kernel(const float* __restrict__ part, int splits, long long mn,
                                                            int N, int ldc, float alpha, const uint16_t* __restrict__ bias,
                                                            uint16_t* __restrict__ C, int* found_inf, const float* __restrict__ db_part,
                                                            int db_n, uint16_t* __restrict__ db) {
    bool bad = false;
    if (db) {
        for (int m = blockIdx.x * 256 + threadIdx.x; m < db_n; m += gridDim.x * 256) {
            float s = db_part[m];
            for (int p = 1; p < splits; ++p) s += db_part[(long long)p * db_n + m];
            const uint16_t h = f2h(s);
            db[m]            = h;
            bad |= half_nonfinite(h);
        }
    }
    for (long long v = (long long)blockIdx.x * 256 + threadIdx.x; v * 4 < mn; v += (long long)gridDim.x * 256) {
        const long long e = v * 4;  // N % 4 == 0 on this path
        float4          s = *reinterpret_cast<const float4*>(part + e);
        for (int p = 1; p < splits; ++p) {
            const float4 t = *reinterpret_cast<const float4*>(part + (long long)p * mn + e);
            s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
        }
        const long long m = e / N, n = e - m * N;
        s.x *= alpha; s.y *= alpha; s.z *= alpha; s.w *= alpha;
        if (bias) {
            s.x += h2f(bias[n]); s.y += h2f(bias[n + 1]); s.z += h2f(bias[n + 2]); s.w += h2f(bias[n + 3]);
        }
        const uint16_t h0 = f2h(s.x), h1 = f2h(s.y), h2 = f2h(s.z), h3 = f2h(s.w);
        *reinterpret_cast<u32x2_u*>(C + m * ldc + n) = u32x2g{(unsigned)h0 | ((unsigned)h1 << 16), (unsigned)h2 | ((unsigned)h3 << 16)};
        bad |= half_nonfinite(h0) | half_nonfinite(h1) | half_nonfinite(h2) | half_nonfinite(h3);
    }
    if (found_inf && __any(bad)) {
        if ((threadIdx.x & 63) == 0) atomicOr(found_inf, 1);
    }
}

// Scalar kernel with the same contract, for the few shapes the matrix-core path does not take or is slower on (see
// matrix_path_ok, scalar_wins).
__global__ __launch_bounds__(256) void gemm_generic_kernel(GemmArgs g, int a_kc, int b_kc) {
    const long long mn  = (long long)g.M * g.N;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    bool            bad = false;
    if (idx < mn) {
        const int       m = (int)(idx / g.N), n = (int)(idx - (long long)m * g.N);
        const int       bo = blockIdx.y / g.batch_inner, bi = blockIdx.y - bo * g.batch_inner;
        const uint16_t* A = g.A + bo * g.sa_o + bi * g.sa_i;
        const uint16_t* B = g.B + bo * g.sb_o + bi * g.sb_i;
        float           acc = 0.f;
        for (int k = 0; k < g.K; ++k) {
            const float a = h2f(a_kc ? A[(long long)m * g.lda + k] : A[(long long)k * g.lda + m]);
            const float b = h2f(b_kc ? B[(long long)n * g.ldb + k] : B[(long long)k * g.ldb + n]);
            acc += a * b;
        }
        acc *= g.alpha;
        if (g.acc_in) acc += g.acc_in[(long long)m * g.N + n];
        if (g.C32) {
            g.C32[(long long)m * g.N + n] = acc;
        } else {
            if (g.bias) acc += h2f(g.bias[n]);
            if (g.relu) acc = (acc < 0.f) ? 0.f : acc;  // keeps a NaN, like the definition max(x, 0) on the reals extended by NaN
            uint16_t        h = f2h(acc);
            const long long coff = bo * g.sc_o + bi * g.sc_i;
            if (g.relu_src) {
                if (!(h2f(g.relu_src[coff + (long long)m * g.ld_aux + n]) > 0.f)) h = 0;
            } else if (g.add) {
                h = f2h(h2f(h) + h2f(g.add[coff + (long long)m * g.ld_aux + n]));
            }
            g.C[coff + (long long)m * g.ldc + n] = h;
            bad = half_nonfinite(h);
        }
    }
    if (g.found_inf && __any(bad)) {
        if ((threadIdx.x & 63) == 0) atomicOr(g.found_inf, 1);
    }
}

// ------------------------------------------------------------------------------------ host side
static PlanTuning g_tuning;

static bool fast_path_ok(const GemmArgs& g) {
    auto m8 = [](long long v) { return (v & 7) == 0; };
    if (!aligned16(g.A) || !aligned16(g.B)) return false;
    if (g.C && !aligned16(g.C)) return false;
    if (!m8(g.lda) || !m8(g.ldb) || !m8(g.ldc)) return false;
    if (!m8(g.sa_o) || !m8(g.sa_i) || !m8(g.sb_o) || !m8(g.sb_i) || !m8(g.sc_o) || !m8(g.sc_i)) return false;
    if ((g.relu_src || g.add) && (!m8(g.ld_aux) || !aligned16(g.relu_src) || !aligned16(g.add))) return false;
    if (g.bias && !aligned16(g.bias)) return false;
    if ((g.N & 7) != 0) return false;  // the epilogue moves 8 columns at a time
    if ((g.acc_in || g.C32) && (!aligned16(g.acc_in) || !aligned16(g.C32))) return false;
    return true;
}

// Leading dimensions up to which an offset inside a tile of 256 (of 64) rows stays inside the buffer size.
constexpr int LD_BUFFER_256 = 1 << 21, LD_BUFFER_64 = 1 << 24;

// What the matrix-core kernels take: a straddling piece of 8 elements is loaded so that it ends at the border, so the
// stored direction of an operand must hold at least 8 elements; fp32 outputs and addends move 4 columns at a time; and
// an offset inside a tile must fit the buffer size.  Alignment and multiples of 8 do not matter.
static bool matrix_path_ok(const GemmArgs& g, bool a_kc, bool b_kc) {
    if (g.K == 0 || (a_kc ? g.K : g.M) < 8 || (b_kc ? g.K : g.N) < 8) return false;
    if ((g.acc_in || g.C32) && (g.N & 3) != 0) return false;
    const bool interior = g.aligned && g.M % 64 == 0 && g.N % 64 == 0 && g.K % BK == 0;  // (no buffer offsets in 64 x 64 tiles)
    return interior || std::max(g.lda, g.ldb) < LD_BUFFER_64;
}

// What the direct-to-LDS kernels take: operand rows that are whole 16-byte pieces (the output's too unless both operands are
// contraction-contiguous), a contraction of whole pieces (any where both are output-contiguous: what lies beyond it reads as
// zero) and long enough for the load stream's lead, offsets inside a tile within the buffer size.  Output tiles may stick out
// of the matrix.
static bool dtl_ok(const GemmArgs& g, bool a_kc, bool b_kc, long long batches) {
    const bool operands = aligned16(g.A) && aligned16(g.B) && g.lda % 8 == 0 && g.ldb % 8 == 0;
    return g_tuning.dtl != 0 && (g.aligned || (operands && a_kc && b_kc)) && batches == 1 && g.K >= DTL_MIN_K && (a_kc ? g.K % 8 == 0 : !b_kc) &&
           std::max(g.lda, g.ldb) < LD_BUFFER_256;
}

// Few ragged outputs over a contraction that short cost the scalar kernel less than the matrix cores' chain of loads, LDS and
// final sum (us, matrix cores / scalar, forward: 1500 x 29 over 9 4.2 / 3.3, over 12 4.2 / 3.6, over 17 4.2 / 4.1; 512 x 512 over 9
// 4.0 / 4.3; 64 products 37 x 37 over 9 4.6 / 3.3, over 17 4.7 / 4.2; 512 of 20 x 20 over 9 5.5 / 5.2.  Input gradients:
// 1500 x 29 over 12 4.0 / 3.5, over 17 4.0 / 4.0; 512 products 9 x 40 over 9 5.7 / 4.1, 20 x 40 over 20 5.8 / 7.1).
static bool scalar_wins(const GemmArgs& g, long long batches) {
    const long long outs = (long long)g.M * g.N * batches;
    return g_tuning.tile < 0 && !g.aligned && (batches == 1 ? g.K <= 12 && outs <= 65536 : g.K <= 16 && outs * g.K <= 1 << 21);
}

// Column sums of dY as launches of their own: two, 2.5 + 2 us by themselves, 4.6 each behind a product in a captured chain.
constexpr double SUMS_APART_US = 6.;

// ws: split-K partial buffer (may be NULL when !allow_split).  sums_ws: room for the partial sums of g.db where the
// contraction is split.  *sums_done: whether g.db was written; else it is the caller's to compute.
static int run_gemm(GemmArgs g, bool a_kc, bool b_kc, long long batches, bool allow_split, float* ws, size_t ws_floats,
                    hipStream_t hs, float* sums_ws = nullptr, size_t sums_floats = 0, bool* sums_done = nullptr) {
    uint16_t* const db       = g.db;
    const double    apart_us = db ? SUMS_APART_US : 0.;
    g.db = nullptr;
    if (sums_done) *sums_done = false;
    if (g.M == 0 || g.N == 0 || batches == 0) return MP_OK;
    g.aligned = fast_path_ok(g);
    if (!matrix_path_ok(g, a_kc, b_kc) || scalar_wins(g, batches) || batches > 65535) {
        if (batches > 65535) {
            set_error("gemm: more than 65535 batches");
            return MP_E_UNSUPPORTED;
        }
        const long long mn = (long long)g.M * g.N;
        g.k_per_split      = g.K;
        hipLaunchKernelGGL(gemm_generic_kernel, dim3((unsigned)((mn + 255) / 256), (unsigned)batches), dim3(256), 0, hs, g,
                           (int)a_kc, (int)b_kc);
        MP_LAUNCH_CHECK("gemm (generic)");
        return MP_OK;
    }
    const bool dtl = dtl_ok(g, a_kc, b_kc, batches);
    Plan p = make_plan(g.M, g.N, g.K, batches, allow_split && ws != nullptr && (g.N & 3) == 0 && batches == 1, a_kc, b_kc, dtl, g_tuning, apart_us);
    // a workspace too small for that: the register-staged kernel's plan if it holds that one, else unsplit
    const auto too_small = [&] { return p.splits > 1 && (size_t)p.splits * g.M * g.N > ws_floats; };
    if (dtl && too_small()) {
        p = make_plan(g.M, g.N, g.K, batches, true, a_kc, b_kc, false, g_tuning, apart_us);
        if (p.splits == 1) p = make_plan(g.M, g.N, g.K, batches, false, a_kc, b_kc, dtl, g_tuning, apart_us);
    }
    if (too_small()) p = make_plan(g.M, g.N, g.K, batches, false, a_kc, b_kc, dtl, g_tuning, apart_us);
    // very long rows: 64 x 64 tiles, unless all loads are plain ones
    if (std::max(g.lda, g.ldb) >= LD_BUFFER_256 && !(g.aligned && g.M % 256 == 0 && g.N % 256 == 0 && g.K % BK == 0 && p.tile < kTileKcOnly))
        p = Plan{6, 1, (g.K + BK - 1) / BK * BK, false};
    g.k_per_split = p.k_per_split;
    if (p.tile >= kTileSmall4 && (batches != 1 || (!a_kc && b_kc))) p.tile = 6;
    const bool    small = p.tile >= kTileSmall4;
    const int     waves = p.tile == kTileSmall4 ? 4 : 8;
    const TileCfg tile  = small ? TileCfg{32, 32, {}, {}} : kTiles[p.tile];
    g.tiles_m     = (g.M + tile.bm - 1) / tile.bm;
    g.tiles_n     = (g.N + tile.bn - 1) / tile.bn;
    // persistent along x: at most as many workgroups as fit on the chip at once (a multiple of 8, see the tile
    // mapping); batches and splits keep their own grid dimensions
    const int  ntiles   = g.tiles_m * g.tiles_n;
    const int  resident = small ? ntiles : kCUs * ((p.dtl ? tile.dtl : tile.reg).per_kt2 > 0.f ? 2 : 1);
    const long long others = batches * p.splits;
    const int  gx = (others == 1 && ntiles > resident) ? resident : ntiles;
    const dim3 grid((unsigned)gx, (unsigned)batches, (unsigned)p.splits);

    GemmArgs   k    = g;
    const bool sums = db && !a_kc && !b_kc && sums_ride(p.tile, p.dtl, g.N) && (p.splits == 1 || (size_t)p.splits * g.M <= sums_floats);
    if (sums) {
        k.db       = db;
        k.db_part  = sums_ws;
        *sums_done = true;
    }
    if (p.splits > 1) {  // partials to workspace, epilogue (scale, bias, rounding, flag) in the finish kernel
        k.C32       = ws;
        k.C         = nullptr;
        k.found_inf = nullptr;
        k.bias      = nullptr;
    }
    int rc;
    if (small) rc = launch_small_tile(waves, a_kc, b_kc, k, p.splits, hs);
    else if (p.dtl && a_kc && b_kc) rc = launch_dtl_tile<true, true>(p.tile, k, grid, hs);
    else if (p.dtl && a_kc) rc = launch_dtl_tile<true, false>(p.tile, k, grid, hs);
    else if (sums) rc = launch_dtl_sums_tile(p.tile, k, grid, hs);
    else if (p.dtl) rc = launch_dtl_tile<false, false>(p.tile, k, grid, hs);
    else if (a_kc && b_kc) rc = launch_tile<true, true>(p.tile, k, grid, hs);
    else if (a_kc && !b_kc) rc = launch_tile<true, false>(p.tile, k, grid, hs);
    else if (!a_kc && !b_kc) rc = launch_tile<false, false>(p.tile, k, grid, hs);
    else {
        set_error("gemm: operand layout combination not built");
        return MP_E_UNSUPPORTED;
    }
    if (rc != MP_OK) return rc;
    if (p.splits > 1) {
        const long long mn = (long long)g.M * g.N;
        long long       nb = (mn / 4 + 255) / 256;
        if (nb > 4096) nb = 4096;
        hipLaunchKernelGGL(splitk_finish_kernel, dim3((unsigned)nb), dim3(256), 0, hs, ws, p.splits, mn, g.N, g.ldc, g.alpha,
                           g.bias, g.C, g.found_inf, sums_ws, g.M, sums ? db : nullptr);
        MP_LAUNCH_CHECK("gemm (split-K finish)");
    }
    return MP_OK;
}

static int check_desc(const mp_gemm_desc* d, const char* who) {
    MP_REQUIRE(d != nullptr, "%s: desc is NULL", who);
    MP_REQUIRE(d->M >= 0 && d->N >= 0 && d->K >= 0, "%s: negative dimension", who);
    MP_REQUIRE(d->batch_outer >= 1 && d->batch_inner >= 1, "%s: batch counts must be >= 1", who);
    MP_REQUIRE(d->trans_w == 0 || d->trans_w == 1, "%s: trans_w must be 0 or 1", who);
    MP_REQUIRE(d->ldx >= d->K && d->ldy >= d->N && d->ldw >= (d->trans_w ? d->N : d->K),
               "%s: leading dimension smaller than the row length (ldx=%d ldw=%d ldy=%d)", who, d->ldx, d->ldw, d->ldy);
    MP_REQUIRE(d->sx_outer >= 0 && d->sx_inner >= 0 && d->sw_outer >= 0 && d->sw_inner >= 0 && d->sy_outer >= 0 &&
                   d->sy_inner >= 0,
               "%s: negative batch stride", who);
    return MP_OK;
}

static void zero_args(GemmArgs& g) { g = GemmArgs{}; }

}  // namespace mp

using namespace mp;

// fp32 partial-sum floats the product [M,N] with contraction K uses (0 when the plan does not split the contraction)
static size_t splitk_floats(int M, int N, int K, bool a_kc, bool b_kc, bool dtl, bool with_sums = false) {
    if (M <= 0 || N <= 0 || (N & 3) != 0) return 0;
    const int splits = make_plan(M, N, K, 1, true, a_kc, b_kc, dtl, g_tuning, with_sums ? SUMS_APART_US : 0.).splits;
    return splits > 1 ? (size_t)splits * (size_t)M * (size_t)N : 0;
}
// ... where the pointers and leading dimensions, which decide between the kernels, are not known yet
static size_t splitk_floats_any(int M, int N, int K, bool a_kc, bool b_kc, bool with_sums = false) {
    const size_t staged = splitk_floats(M, N, K, a_kc, b_kc, false, with_sums);
    return g_tuning.dtl != 0 && K >= DTL_MIN_K ? std::max(staged, splitk_floats(M, N, K, a_kc, b_kc, true, with_sums)) : staged;
}

extern "C" int mp_gemm_tuning_override(int tile, int splits) {
    MP_REQUIRE(tile <= kTileSmall8, "mp_gemm_tuning_override: tile index %d out of range (%d shapes)", tile, kTileSmall8 + 1);
    MP_REQUIRE(tile < 0 || (splits >= 0 && splits <= 16), "mp_gemm_tuning_override: splits %d outside 0..16", splits);
    g_tuning.tile   = tile;
    g_tuning.splits = splits > 0 ? splits : 1;
    return MP_OK;
}

extern "C" int mp_gemm_tuning_dtl(int mode) {
    MP_REQUIRE(mode >= 0 && mode <= 2, "mp_gemm_tuning_dtl: mode %d outside 0..2", mode);
    g_tuning.dtl = mode;
    return MP_OK;
}

extern "C" size_t mp_gemm_bwd_dw_workspace_bytes(const mp_gemm_desc* d, int with_db) {
    if (!d) return 0;
    const int rows = d->trans_w ? d->K : d->N, cols = d->trans_w ? d->N : d->K;
    size_t    b    = 0;
    if (d->batch_outer * (long long)d->batch_inner == 1) b = splitk_floats_any(rows, cols, d->M, false, false, with_db && !d->trans_w) * sizeof(float);
    if (with_db) b += mp_colsum_workspace_bytes(d->M, d->N);
    return b + 256;
}

// A product may split its contraction over grid.z (fp32 partials in `ws`, summed in split order by a finish launch)
// when the epilogue is one the finish launch can do: scale, bias, one rounding, overflow flag.
static bool split_ok(const GemmArgs& g, long long batches, const void* ws) {
    return ws != nullptr && aligned16(ws) && batches == 1 && !g.relu && !g.relu_src && !g.add && !g.acc_in && !g.C32;
}

extern "C" size_t mp_gemm_split_workspace_bytes(const mp_gemm_desc* d) {
    if (!d || d->M <= 0 || d->N <= 0 || d->K <= 0) return 0;
    // the larger of the forward (M x N over K) and dX (M x K over N) plans; 0 when neither would split
    const size_t a = splitk_floats_any(d->M, d->N, d->K, true, d->trans_w == 0);
    const size_t b = splitk_floats_any(d->M, d->K, d->N, true, d->trans_w == 1);
    return (a > b ? a : b) * sizeof(float);
}

extern "C" int mp_gemm_fwd(const mp_gemm_desc* d, const mp_half* X, const mp_half* W, const mp_half* bias,
                           const float* acc_in, mp_half* Y, float* y_f32, mp_stream stream) {
    return mp_gemm_fwd_ws(d, X, W, bias, acc_in, Y, y_f32, nullptr, 0, stream);
}

extern "C" int mp_gemm_fwd_ws(const mp_gemm_desc* d, const mp_half* X, const mp_half* W, const mp_half* bias,
                              const float* acc_in, mp_half* Y, float* y_f32, void* ws, size_t ws_bytes, mp_stream stream) {
    int rc = check_desc(d, "mp_gemm_fwd");
    if (rc) return rc;
    MP_REQUIRE(X && W && (Y || y_f32), "mp_gemm_fwd: NULL operand");
    MP_REQUIRE(d->epilogue >= MP_EPI_NONE && d->epilogue <= MP_EPI_BIAS_RELU, "mp_gemm_fwd: bad epilogue %d", d->epilogue);
    MP_REQUIRE((d->epilogue == MP_EPI_NONE) == (bias == nullptr), "mp_gemm_fwd: bias must be given iff the epilogue uses it");
    MP_REQUIRE(!(y_f32 && d->epilogue != MP_EPI_NONE), "mp_gemm_fwd: y_f32 needs MP_EPI_NONE");
    const long long batches = (long long)d->batch_outer * d->batch_inner;
    MP_REQUIRE(batches == 1 || (!acc_in && !y_f32), "mp_gemm_fwd: acc_in / y_f32 are not available for batched problems");
    GemmArgs g;
    zero_args(g);
    g.A = X; g.B = W; g.C = y_f32 ? nullptr : Y; g.C32 = y_f32; g.acc_in = acc_in; g.bias = bias;
    g.relu = d->epilogue == MP_EPI_BIAS_RELU;
    g.M = d->M; g.N = d->N; g.K = d->K;
    g.lda = d->ldx; g.ldb = d->ldw; g.ldc = d->ldy;
    g.sa_o = d->sx_outer; g.sa_i = d->sx_inner; g.sb_o = d->sw_outer; g.sb_i = d->sw_inner;
    g.sc_o = d->sy_outer; g.sc_i = d->sy_inner;
    g.batch_inner = d->batch_inner; g.alpha = d->alpha;
    const bool sp = split_ok(g, batches, ws);
    return run_gemm(g, true, d->trans_w == 0, batches, sp, sp ? static_cast<float*>(ws) : nullptr, sp ? ws_bytes / sizeof(float) : 0,
                    as_stream(stream));
}

extern "C" int mp_gemm_bwd_dx(const mp_gemm_desc* d, const mp_half* dY, const mp_half* W, const mp_half* relu_src,
                              const mp_half* add, int32_t ld_aux, mp_half* dX, mp_stream stream) {
    return mp_gemm_bwd_dx_ws(d, dY, W, relu_src, add, ld_aux, dX, nullptr, 0, stream);
}

extern "C" int mp_gemm_bwd_dx_ws(const mp_gemm_desc* d, const mp_half* dY, const mp_half* W, const mp_half* relu_src,
                                 const mp_half* add, int32_t ld_aux, mp_half* dX, void* ws, size_t ws_bytes, mp_stream stream) {
    int rc = check_desc(d, "mp_gemm_bwd_dx");
    if (rc) return rc;
    MP_REQUIRE(dY && W && dX, "mp_gemm_bwd_dx: NULL operand");
    MP_REQUIRE(!(relu_src && add), "mp_gemm_bwd_dx: relu_src and add may not both be given");
    MP_REQUIRE(!(relu_src || add) || ld_aux >= d->K, "mp_gemm_bwd_dx: ld_aux=%d smaller than K", ld_aux);
    GemmArgs g;
    zero_args(g);
    g.A = dY; g.B = W; g.C = dX; g.relu_src = relu_src; g.add = add; g.ld_aux = ld_aux;
    g.M = d->M; g.N = d->K; g.K = d->N;
    g.lda = d->ldy; g.ldb = d->ldw; g.ldc = d->ldx;
    g.sa_o = d->sy_outer; g.sa_i = d->sy_inner; g.sb_o = d->sw_outer; g.sb_i = d->sw_inner;
    g.sc_o = d->sx_outer; g.sc_i = d->sx_inner;
    g.batch_inner = d->batch_inner; g.alpha = d->alpha;
    // W[N,K] read as B(n'=k, k'=n) is output-contiguous; W[K,N] is contraction-contiguous.
    const long long batches = (long long)d->batch_outer * d->batch_inner;
    const bool      sp      = split_ok(g, batches, ws);
    return run_gemm(g, true, d->trans_w == 1, batches, sp, sp ? static_cast<float*>(ws) : nullptr, sp ? ws_bytes / sizeof(float) : 0,
                    as_stream(stream));
}

extern "C" int mp_gemm_bwd_dw(const mp_gemm_desc* d, const mp_half* dY, const mp_half* X, mp_half* dW, mp_half* db,
                              mp_scale_state* st, void* ws, size_t ws_bytes, mp_stream stream) {
    int rc = check_desc(d, "mp_gemm_bwd_dw");
    if (rc) return rc;
    MP_REQUIRE(dY && X && dW, "mp_gemm_bwd_dw: NULL operand");
    const long long batches = (long long)d->batch_outer * d->batch_inner;
    MP_REQUIRE(!(db && batches != 1), "mp_gemm_bwd_dw: db is not available for batched problems");
    GemmArgs g;
    zero_args(g);
    g.C = dW; g.found_inf = st ? &st->found_inf : nullptr;
    g.K = d->M;
    g.ldc = d->ldw;
    g.sc_o = d->sw_outer; g.sc_i = d->sw_inner;
    g.batch_inner = d->batch_inner; g.alpha = d->alpha;
    if (!d->trans_w) {  // dW[N,K] = dY^T X
        g.A = dY; g.lda = d->ldy; g.sa_o = d->sy_outer; g.sa_i = d->sy_inner; g.M = d->N;
        g.B = X;  g.ldb = d->ldx; g.sb_o = d->sx_outer; g.sb_i = d->sx_inner; g.N = d->K;
    } else {  // dW[K,N] = X^T dY
        g.A = X;  g.lda = d->ldx; g.sa_o = d->sx_outer; g.sa_i = d->sx_inner; g.M = d->K;
        g.B = dY; g.ldb = d->ldy; g.sb_o = d->sy_outer; g.sb_i = d->sy_inner; g.N = d->N;
    }
    // the partial sums of the plan that runs, or of the register-staged kernel's plan where the workspace holds only those (run_gemm)
    const bool   sums     = db && !d->trans_w;   // (dY is the first operand)
    const size_t cs_bytes = db ? mp_colsum_workspace_bytes(d->M, d->N) : 0;
    const auto   need = [&](size_t floats) { return floats * sizeof(float) + cs_bytes + 256; };
    size_t       sk_floats = 0;
    if (batches == 1) {
        g.aligned = fast_path_ok(g);
        sk_floats = splitk_floats(g.M, g.N, g.K, false, false, dtl_ok(g, false, false, 1), sums);
        if (ws_bytes < need(sk_floats)) sk_floats = std::min(sk_floats, splitk_floats(g.M, g.N, g.K, false, false, false, sums));
    }
    if (!ws || ws_bytes < need(sk_floats) || !aligned16(ws)) {
        set_error("mp_gemm_bwd_dw: 16-byte aligned workspace of %zu bytes needed, %zu given", need(sk_floats), ws_bytes);
        return MP_E_WORKSPACE;
    }
    char* const  cs_ws     = static_cast<char*>(ws) + ((sk_floats * sizeof(float) + 255) / 256) * 256;
    const size_t cs_b      = ws_bytes - (size_t)(cs_ws - static_cast<char*>(ws));
    bool         sums_done = false;
    if (sums) g.db = db;
    rc = run_gemm(g, false, false, batches, sk_floats > 0, sk_floats > 0 ? static_cast<float*>(ws) : nullptr, sk_floats, as_stream(stream),
                  reinterpret_cast<float*>(cs_ws), cs_b / sizeof(float), &sums_done);
    if (rc) return rc;
    if (db && !sums_done) {
        return mp_colsum(d->M, d->N, dY, d->ldy, db, st, cs_ws, cs_b, stream);
    }
    return MP_OK;
}

// One launch for both gradients: each product for the small kernel by itself (so together at most four workgroups per compute
// unit).  us, separate calls / one launch, with the bias gradient, M x N x K: 616 x 240 x 112 8.1 / 4.8, 824 x 440 x 592 (760
// workgroups) 12.8 / 8.8, 1000 x 848 x 504 (944) 17.2 / 13.5, 1604 x 889 x 304 (792) 24.0 / 16.4, 1681 x 1690 x 255 (848) 30.2 / 27.8;
// of 310 random sizes the geometric mean is 0.75, the worst 20.9 / 22.0 (3668 x 15 x 67, a long chain in few tiles).  Two encoder
// layers 320 wide (a width that the grouped launch does not take) on 384 tokens: 218 us an iteration with a product each and
// 187 so.  (An iteration of a 64 x 256 -> 1024 -> 256 network 84 -> 57 us with this launch and the small tiles, of a ragged
// 192-wide encoder layer 191 -> 144 us, both with the host's part of the time that remained then.)
static bool both_joint(const mp_gemm_desc* dx, const mp_gemm_desc* dw) {
    const auto plain = [](const mp_gemm_desc* d) { return d->batch_outer == 1 && d->batch_inner == 1 && d->trans_w == 0 && d->M > 0 && d->N > 0 && d->K > 0; };
    if (g_tuning.tile >= 0 || !plain(dx) || !plain(dw) || dx->M != dw->M || dx->N != dw->N || dx->ldy != dw->ldy) return false;
    // (as matrix_path_ok, for both: stored rows of at least 8 elements, offsets inside a tile within the buffer size)
    if (dx->N < 8 || dx->K < 8 || dw->K < 8 || std::max(std::max(dx->ldy, dx->ldw), dw->ldx) >= LD_BUFFER_64) return false;
    return small_wins(dx->M, dx->K, dx->N) && small_wins(dw->N, dw->K, dw->M);
}

extern "C" int mp_gemm_bwd_both_joint(const mp_gemm_desc* d_dx, const mp_gemm_desc* d_dw) {
    return d_dx && d_dw && both_joint(d_dx, d_dw) ? 1 : 0;
}

extern "C" int mp_gemm_bwd_both(const mp_gemm_desc* d_dx, const mp_half* dY, const mp_half* W, const mp_half* relu_src,
                                const mp_half* add, int32_t ld_aux, mp_half* dX, const mp_gemm_desc* d_dw, const mp_half* X,
                                mp_half* dW, mp_half* db, mp_scale_state* st, void* ws, size_t ws_bytes, mp_stream stream) {
    int rc = check_desc(d_dx, "mp_gemm_bwd_both");
    if (rc == MP_OK) rc = check_desc(d_dw, "mp_gemm_bwd_both");
    if (rc) return rc;
    MP_REQUIRE(d_dx->M == d_dw->M && d_dx->N == d_dw->N && d_dx->ldy == d_dw->ldy, "mp_gemm_bwd_both: the products do not share dY");
    MP_REQUIRE(dY && W && dX && X && dW, "mp_gemm_bwd_both: NULL operand");
    MP_REQUIRE(!(relu_src && add), "mp_gemm_bwd_both: relu_src and add may not both be given");
    MP_REQUIRE(!(relu_src || add) || ld_aux >= d_dx->K, "mp_gemm_bwd_both: ld_aux=%d smaller than K", ld_aux);
    if (both_joint(d_dx, d_dw)) {
        BothArgs b{};
        GemmArgs& x = b.dx;
        x.A = dY; x.B = W; x.C = dX; x.relu_src = relu_src; x.add = add; x.ld_aux = ld_aux;
        x.M = d_dx->M; x.N = d_dx->K; x.K = d_dx->N;
        x.lda = d_dx->ldy; x.ldb = d_dx->ldw; x.ldc = d_dx->ldx; x.alpha = d_dx->alpha; x.batch_inner = 1;
        GemmArgs& w = b.dw;
        w.A = dY; w.B = X; w.C = dW; w.db = db; w.found_inf = st ? &st->found_inf : nullptr;
        w.M = d_dw->N; w.N = d_dw->K; w.K = d_dw->M;
        w.lda = d_dw->ldy; w.ldb = d_dw->ldx; w.ldc = d_dw->ldw; w.alpha = d_dw->alpha; w.batch_inner = 1;
        for (GemmArgs* g : {&x, &w}) {
            g->tiles_m = (g->M + 31) / 32;
            g->tiles_n = (g->N + 31) / 32;
        }
        return launch_small_both(small_waves((long long)x.tiles_m * x.tiles_n + (long long)w.tiles_m * w.tiles_n, std::max(x.K, w.K)), b,
                                 as_stream(stream));
    }
    rc = mp_gemm_bwd_dw(d_dw, dY, X, dW, db, st, ws, ws_bytes, stream);
    if (rc) return rc;
    return mp_gemm_bwd_dx_ws(d_dx, dY, W, relu_src, add, ld_aux, dX, ws, ws_bytes, stream);
}

extern "C" int mp_gemm_bwd_dw_grouped(const mp_gemm_group_item* items, int count, mp_scale_state* st, mp_stream stream) {
    return mp_gemm_bwd_dw_grouped_sums(items, count, nullptr, 0, st, stream);
}

extern "C" int mp_gemm_bwd_dw_grouped_sums(const mp_gemm_group_item* items, int count, const mp_colsum_parts* sums, int nsums,
                                           mp_scale_state* st, mp_stream stream) {
    MP_REQUIRE(nsums >= 0 && nsums <= SUMS_MAX && (nsums == 0 || sums != nullptr), "mp_gemm_bwd_dw_grouped_sums: 0..%d sums", SUMS_MAX);
    MP_REQUIRE(items != nullptr && count >= 1 && count <= GROUP_MAX, "mp_gemm_bwd_dw_grouped: 1..%d items", GROUP_MAX);
    GemmArgs args[GROUP_MAX];
    bool     dtl = g_tuning.dtl != 0;
    for (int i = 0; i < count; ++i) {
        const mp_gemm_desc* d = &items[i].desc;
        int rc = check_desc(d, "mp_gemm_bwd_dw_grouped");
        if (rc) return rc;
        MP_REQUIRE(items[i].dY && items[i].X && items[i].dW, "mp_gemm_bwd_dw_grouped: item %d has a NULL operand", i);
        GemmArgs& g = args[i];
        zero_args(g);
        g.C = items[i].dW;
        g.K = d->M; g.ldc = d->ldw; g.batch_inner = 1; g.alpha = d->alpha;
        if (!d->trans_w) {  // dW[N,K] = dY^T X
            g.A = items[i].dY; g.lda = d->ldy; g.M = d->N;
            g.B = items[i].X;  g.ldb = d->ldx; g.N = d->K;
        } else {  // dW[K,N] = X^T dY
            g.A = items[i].X;  g.lda = d->ldx; g.M = d->K;
            g.B = items[i].dY; g.ldb = d->ldy; g.N = d->N;
        }
        g.k_per_split = g.K;
        const bool ok = d->batch_outer == 1 && d->batch_inner == 1 && fast_path_ok(g) && g.K > 0 && g.K % BK == 0 &&
                        g.M % 128 == 0 && g.N % 128 == 0;
        if (!ok) {
            set_error("mp_gemm_bwd_dw_grouped: item %d is batched, unaligned, or its shape is not a multiple of 128 "
                      "(weights) / 64 (rows); use mp_gemm_bwd_dw", i);
            return MP_E_UNSUPPORTED;
        }
        dtl  = dtl && g.K >= DTL_MIN_K && std::max(g.lda, g.ldb) < LD_BUFFER_256;
    }
    // what rides along: strips of bias gradients and columns of the other sums
    GroupArgs ga{};
    int       strips = 0, strip_rows = 0, sum_rows = 0, k_max = 0;
    for (int i = 0; i < count; ++i) {
        k_max = std::max(k_max, args[i].K);
        if (!items[i].db) continue;
        strips += items[i].desc.N / BIAS_COLS;      // N is a multiple of 128 here (checked above for either orientation)
        strip_rows = std::max(strip_rows, items[i].desc.M);
    }
    for (int i = 0; i < nsums; ++i) {
        const mp_colsum_parts& c = sums[i];
        MP_REQUIRE(c.part && aligned16(c.part) && c.nparts > 0 && c.cols > 0 && c.cols % BIAS_COLS == 0 && c.nseg >= 1 && c.nseg <= 3,
                   "mp_gemm_bwd_dw_grouped_sums: sum %d: bad shape or pointer", i);
        SumItem& s = ga.s[i];
        s.part = c.part; s.nparts = c.nparts; s.cols = c.cols; s.nseg = c.nseg;
        for (int k = 0; k < c.nseg; ++k) {
            MP_REQUIRE(c.out[k], "mp_gemm_bwd_dw_grouped_sums: sum %d has a NULL output", i);
            s.out[k] = reinterpret_cast<unsigned short*>(c.out[k]);
        }
        ga.sum_start[i + 1] = ga.sum_start[i] + c.nseg * (c.cols / BIAS_COLS);
        sum_rows            = std::max(sum_rows, c.nparts);
    }
    ga.nsums = nsums;
    for (int i = nsums; i < SUMS_MAX; ++i) ga.sum_start[i + 1] = ga.sum_start[i];
    const int columns = ga.sum_start[nsums];
    int m_of[GROUP_MAX], n_of[GROUP_MAX];
    for (int i = 0; i < count; ++i) {
        m_of[i] = args[i].M;
        n_of[i] = args[i].N;
    }
    const GroupPlan plan = group_plan(m_of, n_of, count, k_max, dtl, strips, strip_rows, columns, sum_rows);
    MP_REQUIRE(plan.tile >= 0, "mp_gemm_bwd_dw_grouped: too many tiles");
    const int bm = kTiles[plan.tile].bm, bn = kTiles[plan.tile].bn;
    ga.share = plan.share;
    // longest contraction first, so that the tiles that take longest start first
    int order[GROUP_MAX];
    for (int i = 0; i < count; ++i) order[i] = i;
    for (int i = 1; i < count; ++i)
        for (int j = i; j > 0 && args[order[j]].K > args[order[j - 1]].K; --j) std::swap(order[j], order[j - 1]);
    ga.count = count;
    long long total = 0;
    for (int i = 0; i < count; ++i) {
        const GemmArgs& g = args[order[i]];
        ga.p[i]          = GroupItem{g.A, g.B, g.C, g.M, g.N, g.K, g.lda, g.ldb, g.ldc, g.M / bm, g.N / bn, g.alpha};
        ga.tile_start[i] = (int)total;
        total += (long long)(g.M / bm) * (g.N / bn);
    }
    ga.found_inf = st ? &st->found_inf : nullptr;
    for (int i = count; i <= GROUP_MAX; ++i) ga.tile_start[i] = (int)total;
    // bias gradients: strips of BIAS_COLS columns of dY[M, N], numbered after the product tiles (same item order)
    strips = 0;
    for (int i = 0; i < count; ++i) {
        const mp_gemm_group_item& it = items[order[i]];
        if (!it.db) continue;
        BiasItem& b = ga.b[ga.nbias];
        b.dY = reinterpret_cast<const unsigned short*>(it.dY);
        b.db = reinterpret_cast<unsigned short*>(it.db);
        b.ld = it.desc.ldy; b.rows = it.desc.M;
        ga.strip_start[ga.nbias++] = strips;
        strips += it.desc.N / BIAS_COLS;
    }
    for (int i = ga.nbias; i <= GROUP_MAX; ++i) ga.strip_start[i] = strips;
    if (dtl) {
        if (bn == 256) return launch_dtl_grouped<256, 256>(ga, as_stream(stream));
        return bm == 256 ? launch_dtl_grouped<256, 128>(ga, as_stream(stream)) : launch_dtl_grouped<128, 128>(ga, as_stream(stream));
    }
    return bm == 256 ? launch_grouped<256, 256>(ga, as_stream(stream)) : launch_grouped<128, 128>(ga, as_stream(stream));
}
