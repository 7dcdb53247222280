// Which workgroup of a grouped launch does what: the product tiles and the small items (strips of a bias gradient, columns of
// other column sums) that ride along.  Plain C++, so that a test can walk it without a GPU.
#pragma once
#include "gemm_plan.hpp"

#if defined(__HIPCC__)
#define MP_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define MP_HOST_DEVICE inline
#endif

namespace mp {

// Tiles go round the workgroups, so the first `busy` of them have one tile more than the others, which are idle in the last
// round; these take the small items 0 .. first - 1.  What they have no time for goes round all workgroups, behind their tiles.
struct GroupShare {
    int wgs, busy, first;
};

// tile(t) for every tile of workgroup wg, then item(j) for every small item of it
template <typename TILE, typename ITEM>
MP_HOST_DEVICE void group_walk(const GroupShare& s, const int tiles, const int items, const int wg, TILE&& tile, ITEM&& item) {
    for (int t = wg; t < tiles; t += s.wgs) tile(t);
    if (wg >= s.busy) {
        for (int j = wg - s.busy; j < s.first; j += s.wgs - s.busy) item(j);
    }
    for (int j = s.first + wg; j < items; j += s.wgs) item(j);
}

// us of a small item (a strip of `rows` rows, a column of `rows` partial sums) while the matrix cores work, and on a chip that is
// done with its tiles.  128-column strips of 8192 rows: 70 to 150 beside tiles of 128 x 128, 51 alone.
inline double item_us_beside(const int rows) { return 2. + 0.0085 * rows; }
inline double item_us_alone(const int rows) { return 1. + 0.0062 * rows; }

// `strips` items of strip_rows rows come first, then `sums` items of sum_rows; round_us: a tile's time.  Idle workgroups take
// items for about as long as a tile lasts, one at least.  us, 8192 rows, all items to the idle workgroups however few / this
// rule: 510 tiles of 128 x 128 with 56 strips 1438 / 185, 504 with 43 352 / 181, 496 with 39 214 / 172, 484 with 42 159 / 159
// (without the strips 148, 146, 153, 139).  Where all have a tile and some two, items from workgroup 0 on / this rule: 588 tiles
// with 49 strips 256 / 209.
inline GroupShare group_share(const int tiles, const int strips, const int strip_rows, const int sums, const int sum_rows, const int resident,
                              const double round_us) {
    const int  items = strips + sums;
    GroupShare s;
    s.wgs  = std::max(1, tiles < resident ? std::min(resident, tiles + items) : resident);
    s.busy = tiles % s.wgs;
    s.first = 0;
    if (s.busy == 0 && tiles > 0) return s;
    const int    idle = s.wgs - s.busy;
    const double time = 1.25 * round_us, strip_us = item_us_beside(strip_rows), sum_us = item_us_beside(sum_rows);
    const int    n = std::max(1, (int)std::min(time / strip_us, 1e6));   // strips of an idle workgroup
    if ((long long)n * idle < strips) {
        s.first = n * idle;
    } else {
        const int    have = (strips + idle - 1) / idle;
        const double left = time - have * strip_us;
        const int    more = std::max(have ? 0 : 1, (int)std::min(std::max(left, 0.) / sum_us, 1e6));
        s.first = (int)std::min<long long>(items, (long long)(have + more) * idle);
    }
    return s;
}
// us of the launch whose tiles take tiles_us: items beside tiles cost nothing, those behind them a round each
inline double group_us(const GroupShare& s, const int strips, const int strip_rows, const int sums, const int sum_rows, const double tiles_us) {
    const int left = strips + sums - s.first;
    return tiles_us + (left + s.wgs - 1) / s.wgs * item_us_alone(s.first < strips ? strip_rows : sum_rows);
}

// Tile shape of a grouped launch of weight gradients M[i] x N[i] (multiples of 128) over at most k_max: the one with the least
// estimated time; tile < 0: too many tiles.  dtl: on the kernels that load straight into LDS (the others have no 256 x 128).
// Large tiles win once they fill the chip (a layer with d_model 1024: 192 tiles of 256 x 256 in one round, the strips beside
// them); with fewer, most compute units would idle through a long contraction (d_model 512, 4096 tokens: 48 such tiles, 92 us
// with the register-staged kernels, against 192 of 128 x 128, 49 us).
// Strips beside tiles count nothing (us, 256 x 256 / 256 x 128 / 128 x 128, 8192 rows: d_model 1024, 4096 wide 171 / 217 / 267,
// with a bias gradient for each of the four 199 / - / 236; d_model 768, 3072 wide - / 167 / 150; d_model 512, 2048 wide, 4096
// rows 75 / 52 / 36).
struct GroupPlan {
    int        tile;
    GroupShare share;
};
inline GroupPlan group_plan(const int* M, const int* N, const int count, const int k_max, const bool dtl, const int strips, const int strip_rows,
                            const int sums, const int sum_rows) {
    GroupPlan best{-1, {}};
    double    best_us = 1e300;
    for (int t : {0, 1, 3}) {
        const int tm = kTiles[t].bm, tn = kTiles[t].bn;
        long long tiles = 0;
        bool      fits = t != 1 || dtl;
        for (int i = 0; i < count; ++i) {
            fits = fits && M[i] % tm == 0 && N[i] % tn == 0;
            tiles += (long long)(M[i] / tm) * (N[i] / tn);
        }
        if (!fits || tiles >= (1 << 24)) continue;
        const TileTime&  time     = dtl ? kTiles[t].dtl : kTiles[t].reg;
        const int        resident = kCUs * (time.per_kt2 > 0.f ? 2 : 1);
        const double     kt = k_max / (double)BK, all_us = rounds_us(time, (int)tiles, kt), last_us = rounds_us(time, ((int)tiles - 1) % resident + 1, kt);
        const GroupShare share = group_share((int)tiles, strips, strip_rows, sums, sum_rows, resident, last_us);
        const double     us = group_us(share, strips, strip_rows, sums, sum_rows, all_us);
        if (us < best_us) {
            best_us = us;
            best    = GroupPlan{t, share};
        }
    }
    return best;
}

}  // namespace mp
