// Contraction kernel for small problems: 32 x 32 output tiles whose CONTRACTION is dealt to the NW (4 or 8) waves of a
// workgroup (wave w takes the 64-deep k-tiles w, w + NW, ...), each with the whole tile in its accumulators and its own
// LDS; the partial sums are added once at the end, in wave order.  Same arithmetic and results contract as gemm_kernels.hpp
// (paper Section 3.1: fp16 operands, fp32 sums, one rounding); the fp32 summation order differs.
//
// What bounds a small product is the chain launch - first operands - k-tile after k-tile - results, not bandwidth.  In
// the kernels of gemm_kernels.hpp the waves share each k-tile behind a workgroup barrier, 0.2 us a k-tile; here no wave
// waits for another inside the loop and the chain is a quarter or an eighth as long (us alone, before and now:
// 64 x 1024 over 256 4.1 -> 3.0, 64 x 256 over 1024 6.7 -> 4.4, 520 x 256 over 3000 16.3 -> 8.3).
// Operands come through buffer loads, so ragged borders cost no branches (see EDGE and TAIL there); an operand stored
// along the output direction is turned by byte permutes on its way to LDS.
#pragma once
#include "gemm_kernels.hpp"

namespace mp {

constexpr int E        = 32;            // tile edge
// k-tiles a wave has on their way (32 registers each).  The joint launch of both gradients has two or three workgroups to a
// compute unit, which its registers have to leave room for; a product alone has one or two.  us, depth 4 / 3 / 2:
// both gradients of 2000 x 256 x 256 11.2 / 11.2 / 9.3, of 1200 x 512 x 320 10.0 / 10.0 / 8.3, of 1500 x 1024 x 161 13.8 / 13.4 / 12.9;
// alone, where the chain is short, forward 200 x 576 over 192 3.64 / 3.61 / 3.74, input gradient 64 x 1024 over 256 3.67 / 3.64 /
// 3.74, and where it is long, input gradient 520 x 256 over 3000 9.0 / 8.6 / 8.0: a product alone has the depth of the short
// ones whatever its contraction.
constexpr int SM_DEPTH = 3, SM_DEPTH_BOTH = 2;
constexpr int SM_WAVE  = 2 * E * 128;   // LDS bytes of one wave: a k-tile of both operands, later its partial sums
constexpr int sm_lds(int waves) { return waves * SM_WAVE; }

// One k-tile (E rows x 64 k) of an operand, loaded and staged by one wave.
template <bool KC, int MODE>
struct WaveOperand {
    static constexpr int NV = E / 8;          // 16-byte pieces per lane
    static constexpr int RG = E / 8;          // output-contiguous: groups of 8 rows; a lane owns NV k x 8 rows
    u32x4    v[NV];
    unsigned lane_off;  // elements from the k-tile's origin
    int      sh;        // TAIL: how far the pieces now in v were loaded early
    // KC: row hi + 8 i, k-piece lo; else: k = NV hi + i, row piece lo
    static __device__ __forceinline__ int lo() { return KC ? threadIdx.x & 7 : threadIdx.x & (RG - 1); }
    static __device__ __forceinline__ int hi() { return KC ? (threadIdx.x & 63) >> 3 : (threadIdx.x & 63) / RG; }
    __device__ __forceinline__ void init(int ld) {
        lane_off = (unsigned)(KC ? hi() : NV * hi()) * (unsigned)ld + lo() * 8;
        sh       = 0;
    }
    __device__ __forceinline__ void load(const uint16_t* tile, int ld, int rows_left, int k_left) {
        const int c = (KC ? k_left : rows_left) - lo() * 8;       // elements of this lane's pieces that exist
        if (MODE == TAIL) sh = tail_shift(c);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            unsigned off = 2u * (lane_off + (unsigned)(KC ? 8 * i : i) * (unsigned)ld);
            if (MODE == TAIL) off += 16 - 2 * sh;
            const bool in = c > 0 && (KC ? hi() < rows_left - 8 * i : NV * hi() < k_left - i);
            v[i]          = buffer_piece(MODE == TAIL ? tile - 8 : tile, in ? off : BUF_OUT);
        }
    }
    // into LDS rows of 64 k (128 bytes), 16-byte slot ^ swz(row)
    __device__ __forceinline__ void store(char* lds) {
        if (MODE == TAIL) {
#pragma unroll
            for (int i = 0; i < NV; ++i) v[i] = shift_down(v[i], sh);
        }
        if constexpr (KC) {
            static_for<NV>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                *reinterpret_cast<u32x4*>(lds + i * 1024 + hi() * 128 + ((lo() ^ hi() ^ i) << 4)) = v[i];
            });
        } else {
            static_for<8>([&](auto ic) {  // row 8 lo + i: its halves at k = NV hi ... NV hi + NV - 1
                constexpr int i = decltype(ic)::value;
                unsigned      t[NV / 2];
#pragma unroll
                for (int p = 0; p < NV / 2; ++p)
                    t[p] = __builtin_amdgcn_perm(v[2 * p + 1][i >> 1], v[2 * p][i >> 1], (i & 1) ? 0x07060302u : 0x05040100u);
                char* const row = lds + lo() * 1024 + i * 128;
                *reinterpret_cast<u32x2g*>(row + (((hi() >> 1) ^ i ^ lo()) << 4) + (hi() & 1) * 8) = u32x2g{t[0], t[1]};
            });
        }
    }
};

// Output tile (tm, tn) of problem g, k-tiles [kt0, kt1).  split: leave the raw sums in C32 (partials of a split
// contraction, or the fp32 result with scale and addend when !split).
template <int NW, bool A_KC, bool B_KC, int MODE, bool SUMS, int DEPTH>
__device__ __forceinline__ void small_tile(const GemmArgs& g, const int tm, const int tn, const int kt0, const int kt1, float* C32,
                                           const bool split, char* smem, bool& bad) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int m0 = tm * E, n0 = tn * E;
    char* const own = smem + wave * SM_WAVE;

    f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    WaveOperand<A_KC, MODE> a[DEPTH];  // k-tiles on their way
    WaveOperand<B_KC, MODE> b[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
        a[d].init(g.lda);
        b[d].init(g.ldb);
    }
    auto load = [&](auto& a, auto& b, const int kt) {
        const long long k = (long long)kt * BK;
        a.load(A_KC ? g.A + (long long)m0 * g.lda + k : g.A + k * g.lda + m0, g.lda, g.M - m0, g.K - (int)k);
        b.load(B_KC ? g.B + (long long)n0 * g.ldb + k : g.B + k * g.ldb + n0, g.ldb, g.N - n0, g.K - (int)k);
    };
    // fragment of slice kk: row r, k-slot 2 kk + h
    int off[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) off[c] = r * 128 + ((((2 * c) | h) ^ swz(r)) << 4);
    // SUMS: sums of the first operand over the contraction (a weight gradient's bias gradient) where g.db is given.  The first tile
    // of a tile row has its rows' fragments anyway: 16 dot products of two per k-tile; a lane sums the k of its own slots of row r.
    const bool sums = SUMS && g.db != nullptr && tn == 0;
    float      rsum = 0.f;
    auto step = [&](auto& a, auto& b, const int kt) {
        a.store(own);
        b.store(own + E * 128);
        if (kt + NW * DEPTH < kt1) load(a, b, kt + NW * DEPTH);
        static_for<4>([&](auto kc) {
            constexpr int kk = decltype(kc)::value;
            const f16x8   af = *reinterpret_cast<const f16x8*>(own + off[kk]);
            const f16x8   bf = *reinterpret_cast<const f16x8*>(own + E * 128 + off[kk]);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf, af, acc, 0, 0, 0);
            if (sums) {
#pragma unroll
                for (int e = 0; e < 8; e += 2) rsum = __builtin_amdgcn_fdot2(f16x2{af[e], af[e + 1]}, f16x2{(f16)1.f, (f16)1.f}, rsum, false);
            }
        });
    };
    int kt = kt0 + wave;
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (kt + NW * d < kt1) load(a[d], b[d], kt + NW * d);
    for (; kt < kt1; kt += NW * DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
            if (kt + NW * d < kt1) step(a[d], b[d], kt + NW * d);
    }

    // partial sums, row-major fp32 in 16-byte slots ^ (row % 8): lane (r, h) holds row r, columns 8 q + 4 h ...
    constexpr int SX = E / 4 - 1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4*>(own + r * (4 * E) + (((2 * q + h) ^ (r & SX)) << 4)) =
            f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    if (sums) {   // (behind the 4 KB of partial sums)
        rsum += __shfl_xor(rsum, 32, 64);
        *reinterpret_cast<float*>(own + 4 * E * E + 4 * r) = rsum;
    }
    __syncthreads();
    if (sums && wave == NW - 1 && lane < E && m0 + lane < g.M) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += *reinterpret_cast<const float*>(smem + w * SM_WAVE + 4 * E * E + 4 * lane);
        if (split) {
            g.db_part[m0 + lane] = s;
        } else {
            const uint16_t hv = f2h(s);
            g.db[m0 + lane]   = hv;
            bad |= half_nonfinite(hv);
        }
    }
    // wave w finishes rows E / NW w ..., a lane (of the first E E / 8 / NW) 8 consecutive columns of one
    const uint16_t* const aux = g.relu_src ? g.relu_src : g.add;
    constexpr int         CG = E / 8;  // column groups
    const int             cg = lane % CG, n = n0 + 8 * cg;
    {
        const int row = E / NW * wave + lane / CG, m = m0 + row;
        if (m >= g.M || n >= g.N || lane / CG >= E / NW) return;
        float x[8];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const char* s = smem + row * (4 * E) + (((2 * cg + q) ^ (row & SX)) << 4);
            f32x4       t = *reinterpret_cast<const f32x4*>(s);
#pragma unroll
            for (int w = 1; w < NW; ++w) t += *reinterpret_cast<const f32x4*>(s + w * SM_WAVE);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * q + e] = t[e];
        }
        const long long mn = (long long)m * g.N + n;
        const int       left = g.N - n;
        if (!split && (g.alpha != 1.f || g.acc_in)) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x[e] *= g.alpha;
                if (g.acc_in && e < left) x[e] += g.acc_in[mn + e];
            }
        }
        if (C32) {  // (N is a multiple of 4)
            *reinterpret_cast<f32x4_u*>(C32 + mn) = f32x4{x[0], x[1], x[2], x[3]};
            if (left > 4) *reinterpret_cast<f32x4_u*>(C32 + mn + 4) = f32x4{x[4], x[5], x[6], x[7]};
            return;
        }
        if (g.bias) {
            const u32x4 b = MODE == TAIL ? load8_guard(g.bias + n, left) : *reinterpret_cast<const u32x4_u*>(g.bias + n);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] += h2f((uint16_t)((e & 1) ? (b[e >> 1] >> 16) : (b[e >> 1] & 0xFFFFu)));
        }
        if (g.relu) {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = (x[e] < 0.f) ? 0.f : x[e];  // (keeps a NaN)
        }
        uint16_t o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = f2h(x[e]);
        if (aux) {
            const uint16_t* ap = aux + (long long)m * g.ld_aux + n;
            const u32x4     av = MODE == TAIL ? load8_guard(ap, left) : *reinterpret_cast<const u32x4_u*>(ap);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint16_t t = (uint16_t)((e & 1) ? (av[e >> 1] >> 16) : (av[e >> 1] & 0xFFFFu));
                if (g.relu_src) o[e] = h2f(t) > 0.f ? o[e] : (uint16_t)0;
                else o[e] = f2h(h2f(o[e]) + h2f(t));
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) bad |= half_nonfinite(o[e]) && (MODE != TAIL || e < left);
        const u32x4 out = {(unsigned)o[0] | ((unsigned)o[1] << 16), (unsigned)o[2] | ((unsigned)o[3] << 16),
                           (unsigned)o[4] | ((unsigned)o[5] << 16), (unsigned)o[6] | ((unsigned)o[7] << 16)};
        uint16_t* const dst = g.C + (long long)m * g.ldc + n;
        if (MODE != TAIL || left >= 8) *reinterpret_cast<u32x4_u*>(dst) = out;
        else store8_tail(dst, out, left);
    }
}

// workgroup id -> output tile: an XCD (consecutive workgroup ids go round the 8 of them) gets a contiguous run of tiles,
// numbered along the shorter side of the output, so that what a run reads (a few panels of either operand) fits its L2.
// A run of whole tile rows of a wide output reads most of its second operand (us, 256 x 2048 over 1536, forward / input
// gradient / weight gradient: 11.8 / 15.6 / 16.5 that way, 8.7 / 10.1 / 11.3 this way; the larger tiles 9.7 / 10.5 / 12.1).
__device__ __forceinline__ int2 small_tile_of(const int id, const int tiles_m, const int tiles_n) {
    const int n = tiles_m * tiles_n, x = id & 7;
    const int t = x * (n >> 3) + min(x, n & 7) + (id >> 3);
    return tiles_n > tiles_m ? make_int2(t % tiles_m, t / tiles_m) : make_int2(t / tiles_n, t % tiles_n);
}

// grid: (tiles, 1, splits of the contraction); g.k_per_split is a multiple of BK
template <int NW, bool A_KC, bool B_KC, int MODE, bool SUMS = false>
__global__ __launch_bounds__(64 * NW) void gemm_small_kernel(GemmArgs g) {
    extern __shared__ __align__(16) char smem[];
    bool      bad = false;
    if (SUMS && gridDim.z > 1) g.db_part += (long long)blockIdx.z * g.M;
    const int2 t = small_tile_of(blockIdx.x, g.tiles_m, g.tiles_n);
    const int  per = g.k_per_split / BK, nkt = (g.K + BK - 1) / BK;
    const bool split = gridDim.z > 1;
    small_tile<NW, A_KC, B_KC, MODE, SUMS, SM_DEPTH>(g, t.x, t.y, blockIdx.z * per, min(nkt, (int)(blockIdx.z + 1) * per),
                                 g.C32 ? g.C32 + (long long)blockIdx.z * g.M * g.N : nullptr, split, smem, bad);
    if (g.found_inf && __any(bad)) {
        if ((threadIdx.x & 63) == 0) atomicOr(g.found_inf, 1);
    }
}

// Both gradients of a linear layer in one launch: tiles of dX, then tiles of dW, which have the bias gradient with them.  They
// share dY and depend on nothing else, and each alone leaves most of a small layer's time to launches.  (With the column sums of
// dY as workgroups of their own, 32 columns each, their rounds of rows were the longest chain: 3000 x 512 x 96 14.4 us,
// 12.0 with them in the tiles.)
// Either product's tiles go to the XCDs as those of a product alone do (small_tile_of; a run of ids that starts anywhere still has
// every eighth on one XCD): M x N x K 3033 x 2525 x 78 31.4 -> 27.9 us, 1424 x 1584 x 232 16.5 -> 14.8, 2744 x 2352 x 8 11.6 -> 9.7,
// small ones as before.  The tiles of dW come first where their chain is long: 3033 x 2525 x 78 27.9 -> 24.6, 1848 x 1272 x 248 19.2 ->
// 16.9, 1604 x 889 x 304 19.8 -> 16.4, at worst 13.0 -> 13.3 (1544 x 944 x 264); below the line it loses where the tiles are many:
// 1216 x 1144 x 384 14.3 -> 16.8, 544 x 472 x 920 9.6 -> 11.3.
constexpr int SM_DW_FIRST = 1536;
struct BothArgs {
    GemmArgs dx, dw;
};

template <int NW, int MODE>
__global__ __launch_bounds__(64 * NW) void gemm_small_both_kernel(BothArgs b) {
    extern __shared__ __align__(16) char smem[];
    bool      bad = false;
    const int ndx = b.dx.tiles_m * b.dx.tiles_n;
    const int id = b.dw.K > SM_DW_FIRST ? (int)blockIdx.x - b.dw.tiles_m * b.dw.tiles_n : (int)blockIdx.x;   // (dX: 0 ... ndx - 1)
    if (id >= 0 && id < ndx) {
        const int2 t = small_tile_of(id, b.dx.tiles_m, b.dx.tiles_n);
        small_tile<NW, true, false, MODE, false, SM_DEPTH_BOTH>(b.dx, t.x, t.y, 0, (b.dx.K + BK - 1) / BK, nullptr, false, smem, bad);
        return;  // (dX has no overflow flag)
    }
    const int2 t = small_tile_of(id < 0 ? (int)blockIdx.x : id - ndx, b.dw.tiles_m, b.dw.tiles_n);
    small_tile<NW, false, false, MODE, true, SM_DEPTH_BOTH>(b.dw, t.x, t.y, 0, (b.dw.K + BK - 1) / BK, nullptr, false, smem, bad);
    if (b.dw.found_inf && __any(bad)) {
        if ((threadIdx.x & 63) == 0) atomicOr(b.dw.found_inf, 1);
    }
}

// ------------------------------------------------------------------------------------ launches
template <int NW, bool AKC, bool BKC>
int launch_small(const GemmArgs& g, int splits, hipStream_t hs) {
    const bool tail = (AKC ? g.K : g.M) % 8 != 0 || (BKC ? g.K : g.N) % 8 != 0 || g.N % 8 != 0;
    const dim3 grid(g.tiles_m * g.tiles_n, 1, splits);
    if constexpr (!AKC && !BKC) {   // (a kernel of its own: the branch costs a product without sums 0.1 to 0.3 us)
        if (g.db) {
            if (tail) hipLaunchKernelGGL((gemm_small_kernel<NW, false, false, TAIL, true>), grid, dim3(64 * NW), sm_lds(NW), hs, g);
            else hipLaunchKernelGGL((gemm_small_kernel<NW, false, false, EDGE, true>), grid, dim3(64 * NW), sm_lds(NW), hs, g);
            MP_LAUNCH_CHECK("gemm launch (small)");
            return MP_OK;
        }
    }
    if (tail) hipLaunchKernelGGL((gemm_small_kernel<NW, AKC, BKC, TAIL>), grid, dim3(64 * NW), sm_lds(NW), hs, g);
    else hipLaunchKernelGGL((gemm_small_kernel<NW, AKC, BKC, EDGE>), grid, dim3(64 * NW), sm_lds(NW), hs, g);
    MP_LAUNCH_CHECK("gemm launch (small)");
    return MP_OK;
}
int launch_small_tile(int waves, bool a_kc, bool b_kc, const GemmArgs& g, int splits, hipStream_t hs);
int launch_small_both(int waves, const BothArgs& b, hipStream_t hs);

}  // namespace mp
