// Which tile shape, kernel and split count a contraction takes.  Plain C++, so that a test can ask without a GPU.
#pragma once
#include <algorithm>

namespace mp {

constexpr int BK = 64;              // a k-tile: halves per LDS row = 128 bytes = 8 slots of 16 bytes
constexpr int DTL_MIN_K = 3 * BK;   // least contraction straight into LDS: the loads run two k-tiles ahead and cross at most one tile border

// Tile shapes and what they cost.  A workgroup's time is fixed + per_kt x its k-tiles (of 64), us, with one workgroup on every
// compute unit; fixed2 + per_kt2 is that of a pair sharing one.  Fitted to 3000 launches of one card (M 512 to 8192, N and K 320 to
// 4096, the three products, N(0,1) operands, every shape forced in turn): 3 us + the sum over the rounds is off by 5 to 9 % on
// average.  (The two six-stage shapes, 128 x 64 and 64 x 128 straight into LDS: fixed time raised by 0.3 so that they start where
// they win, 1718 x 768 over 256 5.9 register-staged / 6.8, 802 x 1536 over 384 6.4 / 7.0, 4096 x 512 over 512 7.3 / 6.8.)
struct TileTime {
    float fixed, per_kt, fixed2, per_kt2;   // (per_kt2 0: a pair does not fit)
};
struct TileCfg {
    int      bm, bn;
    TileTime reg, dtl;  // register-staged kernel; kernel that loads straight into LDS (gemm_dtl.hpp; per_kt 0: not built)
};
static const TileCfg kTiles[] = {{256, 256, {6.45f, 1.15f}, {5.96f, 1.03f}},
                                 {256, 128, {3.68f, 0.75f}, {3.13f, 0.63f}},
                                 {128, 256, {3.75f, 0.76f}, {3.30f, 0.64f}},
                                 {128, 128, {1.99f, 0.50f, 3.02f, 1.08f}, {1.26f, 0.42f, 2.69f, 0.88f}},
                                 {128, 64, {1.09f, 0.38f, 1.73f, 0.70f}, {2.05f, 0.27f}},
                                 {64, 128, {1.08f, 0.39f, 1.84f, 0.69f}, {1.80f, 0.27f}},
                                 {64, 64, {0.57f, 0.30f, 1.00f, 0.46f}, {}},
                                 {32, 128, {1.00f, 0.34f, 1.60f, 0.63f}, {}},   // (not fitted: 0.9 of 128 x 64)
                                 // only when both operands are stored contraction-contiguous (the transposing loader
                                 // wants a power-of-two tile edge): fills the chip evenly when N is a multiple of 192 only
                                 {256, 192, {5.98f, 0.88f}, {6.19f, 0.81f}}};
constexpr int kCUs = 256;
// us of `wgs` workgroups with k_tiles k-tiles each, without the launch
inline double rounds_us(const TileTime& t, int wgs, double k_tiles) {
    const double one = t.fixed + t.per_kt * k_tiles, two = t.fixed2 + t.per_kt2 * k_tiles;
    if (t.per_kt2 == 0.f) return (double)((wgs + kCUs - 1) / kCUs) * one;
    const int rest = wgs % (2 * kCUs);
    return (double)(wgs / (2 * kCUs)) * two + (rest == 0 ? 0. : rest <= kCUs ? one : two);
}
constexpr int   kTileKcOnly = 8;  // first index of the shapes restricted to that operand layout
constexpr int   kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
// then 32 x 32 with the contraction dealt to 4 or to 8 waves (gemm_small.hpp), unbatched only
constexpr int   kTileSmall4 = kNumTiles, kTileSmall8 = kNumTiles + 1;

// Products for the small kernel: up to two workgroups per compute unit, and not so long a contraction that reading the
// operand panels anew for every 32 x 32 tile outweighs the short chain.  us alone, larger tiles against this kernel:
// 64 x 1024 over 256 4.1 / 3.0, 64 x 256 over 1024 6.7 / 4.4, 520 x 256 over 3000 16.3 / 8.3, 1024 x 161 over 1500 15.2 / 7.9.
// At the line, forward, input gradient, weight gradient: 512 x 512 over 3072 14.9 / 8.9, 16.6 / 10.7, 12.1 / 11.9;
// 256 x 2048 over 1536 9.7 / 8.7, 10.5 / 10.1, 12.1 / 11.3; the least gain of 288 sizes inside it: 1024 x 512 over 1024 7.7 / 7.0,
// 8.3 / 8.6, 10.9 / 9.5.  Beyond it 512 x 512 over 4096 13.0 / 16.8, 1024 x 1024 over 1024 7.3 / 10.0.
inline long long small_tiles(int M, int N) { return ((M + 31) / 32) * (long long)((N + 31) / 32); }
inline bool      small_wins(int M, int N, int K) {
    const long long t = small_tiles(M, N);
    return t <= 2 * kCUs && K <= 4096 && t * K <= 3072ll * kCUs;
}
// 8 waves (64 KB of LDS) when a workgroup has its compute unit to itself and each wave several k-tiles: 512 x 512 over
// 4096 20.7 -> 16.8 us, 1500 x 29 over 1024 6.6 -> 5.7; shorter contractions lose 0.2 us in the longer final sum.
inline int small_waves(long long tiles, int K) { return tiles <= kCUs && K > 512 ? 8 : 4; }

struct Plan {
    int  tile, splits, k_per_split;
    bool dtl;  // on the kernel that loads straight into LDS
};
// What the tuning calls set: a tile shape and a split count for every product (tile < 0: none), and which products take the
// direct-to-LDS kernels: 0 = none, 1 = where the plan finds them the faster ones, 2 = every product they are built for.
struct PlanTuning {
    int tile = -1, splits = 1, dtl = 1;
};

// (contraction K in parts of kps: each has to hold the load stream's lead)
inline bool dtl_takes(int tile, int K, int splits, int kps) {
    return tile < kNumTiles && kTiles[tile].dtl.per_kt > 0.f && (splits == 1 ? K : std::min(kps, K - (splits - 1) * kps)) >= DTL_MIN_K;
}

// Factor on the estimate of a direct-to-LDS shape whose operands arrive more slowly than in the fitted range.  Chosen on 20000
// forced launches of input and weight gradients (500 to 16384 tokens, vocabularies of 3000 to 65536, 128 to 1024 wide, every
// shape and split count).  What it moves, us, without / with it:
//   input gradients over more than 4096, where each row of the first operand lies in pages of its own: 7949 x 768 over 16440
//     300 / 210, 8075 x 320 over 14864 141 / 117, 6130 x 192 over 23552 108 / 90, 8192 x 128 over 16384 70 / 62; without a
//     workspace 7260 x 128 over 27448 234 / 199.  344 sizes of 500 to 8192 rows, 128 to 1024 wide, up to 400 MB: 1.7 % from the best
//     of all launches on average, without the factor 3.8;
//   of more than 400 MB, where the fewest bytes count: 256 x 256 tiles however few (75 sizes of up to 16384 rows, rows no multiple of 32
//     KB apart: 1.0 % from the best, 2.6 % behind the register-staged kernel's best at most; without the factor 3.0 and 20 %);
//   of more than 500 MB with rows a multiple of 32 KB apart, where the memory channels are met unevenly: the register-staged kernel
//     up to 512 columns, whose loads are further apart (8192 over 32768, straight into LDS / staged: 320 wide 246-266 / 230, 384
//     249 / 235, 192 184 / 180, 512 251 / 254, 256 182 / 192; 640 and wider 365 / 385);
//   weight gradients on operands of more than 200 MB (the memory-side cache holds 256): 32768 x 128 over 8192 118 / 112, 20000 x 192
//     over 8192 132 / 117, 31864 x 192 over 4677 102 / 87;
//   forward products in the six-stage shapes: where rows are no multiple of 128 bytes apart, 64 elements of a row lie in two cache
//     lines, for which their short k-tile leaves no time (1564 x 320 over 3928 30.4 / 21.5, 680 x 1216 over 3760 28.1 / 21.2, 954 x 1152
//     over 400 7.9 / 6.9); other rows 205 x 1216 over 3008 16.5 / 14.3.  311 forward products of 200 to 8192 rows, 192 to 4096 wide, over
//     192 to 4096: 1.0 % from the best of all launches on average, 5 % behind the register-staged kernel's best at most; without
//     the factor 2.0 and 42 %.  (Input and weight gradients, 589, need none there: 2 % behind at most.)
inline double arrival(const int t, const int M, const int N, const int K, const bool a_kc, const bool b_kc, const bool allow_split) {
    const double mb = 2e-6 * ((double)M + N) * K;
    if (b_kc) return t != 4 && t != 5 ? 1. : K % 64 == 0 ? 1.08 : 1.35;
    if (a_kc) {
        if (K <= 4096) return 1.;
        if (!allow_split && t == 5 && mb > 400. && N <= 192) return 1.2;
        if (mb > 500. && K % 16384 == 0 && N <= 512) return 1.3;
        if (t == 4) return 1.2;
        return t == 1 || (t != 0 && mb > 400.) ? 1.1 : 1.;
    }
    if (mb < 200.) return 1.;
    if (mb < 256. || N > 192) return t == 3 ? 1.15 : 1.;
    return t == 3 ? 1.3 : t == 1 ? 1.1 : t == 4 ? 1.2 : 1.;
}

// The direct-to-LDS kernels of weight gradients also sum their first operand over the contraction (the bias gradient), 16 rows
// to a wave, so the waves beside each other have to cover a tile's rows; 256 x 256 has no registers for it, and 128 x 256 is
// hardly ever the best shape.  us of a weight gradient with its bias gradient, column sums apart / riding (rows x outputs x
// inputs, in a captured chain): 1600 x 4096 x 2048 36.2 / 33.0, 1600 x 2048 x 1024 19.1 / 15.0, 1024 x 8000 x 512 19.9 / 15.6,
// 1021 x 12008 x 512 29.9 / 22.8, 520 x 3000 x 256 10.8 / 8.1, 8000 x 640 x 640 26.8 / 19.8, 8192 x 3072 x 1024 76.0 / 67.6; in
// the small kernel (the first tile of a row of tiles sums) 1500 x 29 x 1024 12.0 / 8.5, 1200 x 512 x 320 11.0 / 6.4, 64 x 1024 x 256
// 7.4 / 3.9.
inline bool sums_ride(int tile, bool dtl, int N) {
    if (tile >= kTileSmall4) return true;
    return dtl && (tile == 1 || (tile >= 3 && tile <= 5)) && 2 * ((N + kTiles[tile].bn - 1) / kTiles[tile].bn) >= kTiles[tile].bm / 32;
}

// Pick the tile shape (and split count when allowed) that minimises the estimate of run time.  a_kc, b_kc: contraction-contiguous
// operands; dtl: the operands are fit for the direct-to-LDS kernels; apart_us: what a kernel that does not sum its first operand
// leaves to launches of their own
inline Plan make_plan(int M, int N, int K, long long batches, bool allow_split, bool a_kc, bool b_kc, bool dtl, const PlanTuning& tuning,
                      double apart_us = 0.) {
    const bool kc_kc = a_kc && b_kc;
    if (tuning.tile >= 0) {
        int t = tuning.tile < (kc_kc ? kNumTiles : kTileKcOnly) || tuning.tile >= kTileSmall4 ? tuning.tile : 0, sp = allow_split ? tuning.splits : 1;
        if (sp < 1) sp = 1;
        if (sp > 16) sp = 16;
        // every split must own at least one k-tile: (sp - 1) * k_per_split < K, as in the planner's own search
        int kps = ((K + sp - 1) / sp + BK - 1) / BK * BK;
        while (sp > 1 && (long long)(sp - 1) * kps >= K) {
            --sp;
            kps = ((K + sp - 1) / sp + BK - 1) / BK * BK;
        }
        return Plan{t, sp, kps > 0 ? kps : BK, dtl && dtl_takes(t, K, sp, kps)};
    }
    const bool dtl_only = dtl && tuning.dtl == 2;
    if (!dtl_only && batches == 1 && small_wins(M, N, K) && (!allow_split || K <= 3072))  // (longer ones: split over more workgroups)
        return Plan{small_waves(small_tiles(M, N), K) == 8 ? kTileSmall8 : kTileSmall4, 1, (K + BK - 1) / BK * BK, false};
    Plan   best{0, 1, 0, false};
    double best_cost = 1e300;
    for (int t = 0; t < (kc_kc ? kNumTiles : kTileKcOnly); ++t) {
        const long long tm = (M + kTiles[t].bm - 1) / kTiles[t].bm, tn = (N + kTiles[t].bn - 1) / kTiles[t].bn;
        const long long tiles = tm * tn * batches;
        const int       max_s = allow_split ? 16 : 1;
        for (int s = 1; s <= max_s; s *= 2) {
            const int kps = ((K + s - 1) / s + BK - 1) / BK * BK;
            if (s > 1 && (kps < 4 * BK || (long long)(s - 1) * kps >= K || tiles > 2 * kCUs)) break;
            // the finish launch, and the fp32 partials written and read again (1024 x 1024 over 8192 in 4: 10.5 us, 512 x 512 in 8: 6.7)
            const double parts = s > 1 ? 2.5 + 2.0e-6 * M * N * s : 0.;
            for (int v = 0; v < 2; ++v) {
                const bool d = v == 0;
                if (d ? !dtl || !dtl_takes(t, K, s, kps) : dtl_only) continue;
                const TileTime& time = d ? kTiles[t].dtl : kTiles[t].reg;
                const double    cost = parts + (sums_ride(t, d, N) ? 0. : apart_us) + (d && batches == 1 ? arrival(t, M, N, K, a_kc, b_kc, allow_split) : 1.) *
                                                rounds_us(time, (int)std::min(tiles * s, 1ll << 30), kps / (double)BK);
                if (cost < best_cost) {
                    best_cost = cost;
                    best      = Plan{t, s, kps, d};
                }
            }
        }
    }
    if (best.splits == 1) best.k_per_split = (K + BK - 1) / BK * BK;
    if (best.k_per_split == 0) best.k_per_split = BK;
    return best;
}

}  // namespace mp
