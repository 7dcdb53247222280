"""The rules that deal work to kernels and workgroups, checked on the CPU: the headers that hold them are plain C++ and are
compiled here with g++."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_10387_amd", "csrc")

GROUP = r"""
#include "group_rule.hpp"
extern "C" int walk(int tiles, int strips, int strip_rows, int sums, int sum_rows, int resident, double round_us,
                    int* tile_wg, int* item_wg, double* us) {
    const mp::GroupShare s = mp::group_share(tiles, strips, strip_rows, sums, sum_rows, resident, round_us);
    for (int w = 0; w < s.wgs; ++w)
        mp::group_walk(s, tiles, strips + sums, w, [&](int t) { tile_wg[t] = tile_wg[t] == -1 ? w : -2; },
                       [&](int j) { item_wg[j] = item_wg[j] == -1 ? w : -2; });
    us[0] = mp::item_us_beside(strip_rows); us[1] = mp::item_us_beside(sum_rows); us[2] = mp::item_us_alone(strip_rows); us[3] = mp::item_us_alone(sum_rows);
    us[4] = mp::group_us(s, strips, strip_rows, sums, sum_rows, 1000. * round_us);
    return s.wgs;
}
"""


def _compile(tmp, name, source):
    src, lib = os.path.join(tmp, name + ".cpp"), os.path.join(tmp, name + ".so")
    with open(src, "w") as f:
        f.write(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    return C.CDLL(lib)


@pytest.fixture(scope="module")
def group(tmp_path_factory):
    lib = _compile(str(tmp_path_factory.mktemp("rules")), "group", GROUP)
    lib.walk.argtypes = [C.c_int] * 6 + [C.c_double] + [C.c_void_p] * 3
    return lib


@pytest.mark.parametrize("rows", [64, 2048, 8192])
@pytest.mark.parametrize("resident,round_fixed,round_row", [(256, 6.0, 0.016), (512, 2.7, 0.0137)])
@pytest.mark.parametrize("strips,sums", [(0, 0), (1, 0), (0, 48), (43, 42), (56, 30), (49, 42), (400, 0), (2000, 96)])
def test_small_items_of_a_grouped_launch(group, strips, sums, resident, round_fixed, round_row, rows):
    """Every tile and every small item exactly once, whatever the counts.  An idle workgroup's items last no longer than 1.25 tiles, or are one;
    a workgroup that is not idle takes items only where the idle ones have their share, and then no more than
    one more than any other; so the launch ends soon after its tiles."""
    round_us = round_fixed + round_row * rows
    for tiles in (1, 48, 192, 255, 256, 257, 432, 496, 504, 510, 511, 512, 513, 588, 600, 1023, 1024, 5000):
        tile_wg, item_wg, us = (C.c_int * tiles)(*[-1] * tiles), (C.c_int * (strips + sums + 1))(*[-1] * (strips + sums + 1)), (C.c_double * 5)()
        wgs = group.walk(tiles, strips, rows, sums, 256, resident, round_us, tile_wg, item_wg, us)
        assert 1 <= wgs <= resident and all(0 <= w < wgs for w in tile_wg) and all(0 <= w < wgs for w in item_wg[:strips + sums])
        n_tiles, n_strips, n_sums = [0] * wgs, [0] * wgs, [0] * wgs
        for w in tile_wg:
            n_tiles[w] += 1
        for j, w in enumerate(item_wg[:strips + sums]):
            (n_strips if j < strips else n_sums)[w] += 1
        full = max(n_tiles)
        assert min(n_tiles) >= full - 1
        idle = [w for w in range(wgs) if n_tiles[w] < full]
        busy = [w for w in range(wgs) if n_tiles[w] == full]
        beside = max((n_strips[w] * us[0] + n_sums[w] * us[1] for w in idle), default=0.0)
        behind = max(n_strips[w] + n_sums[w] for w in busy)
        items = strips + sums
        if not behind:                   # nothing waits for the tiles
            assert beside <= max(1.25 * round_us + us[1], us[0], us[1]) + 1e-9
        else:
            assert behind <= -(-items // wgs)
        if idle and -(-strips // len(idle)) * us[0] + -(-sums // len(idle)) * us[1] <= round_us:
            assert behind == 0           # the idle ones have the time
        # the estimate the tile shape is chosen by: items beside tiles cost nothing (strips counted as tiles made a second round of
        # 192 tiles of 256 x 256 and 72 strips), items behind them a round each
        assert us[4] >= 1000 * round_us - 1e-9 and (us[4] <= 1000 * round_us + 1e-9) == (behind == 0 or items == 0)
        assert us[4] <= 1000 * round_us + -(-items // wgs) * max(us[2], us[3]) + 1e-9


PLAN = r"""
#include "gemm_plan.hpp"
extern "C" void plan(int M, int N, int K, int allow_split, int a_kc, int b_kc, int dtl, int* out) {
    const mp::Plan p = mp::make_plan(M, N, K, 1, allow_split, a_kc, b_kc, dtl, mp::PlanTuning{});
    out[0] = p.tile; out[1] = p.splits; out[2] = p.dtl; out[3] = p.k_per_split;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = _compile(str(tmp_path_factory.mktemp("rules")), "plan", PLAN)
    out = (C.c_int * 4)()

    def ask(M, N, K, split, a_kc, b_kc, dtl):
        lib.plan(M, N, K, int(split), int(a_kc), int(b_kc), int(dtl), out)
        return tuple(out)
    return ask


# us of forced plans (tile, splits) straight into LDS, and of the register-staged kernel's plan without those kernels
SLOW_ARRIVAL = [  # input gradients M x N over K (with a workspace or without), weight gradients, forward products
    ("dx", True, 6130, 192, 23552, 96.9, {(0, 8): 87.7, (2, 4): 89.5}),
    ("dx", True, 8192, 128, 16384, 66.7, {(3, 4): 62.4, (5, 2): 64.5, (4, 2): 66.9}),
    ("dx", True, 8075, 320, 14864, 125.9, {(3, 1): 111.8, (0, 4): 116.8, (2, 2): 121.6}),
    ("dx", True, 7949, 768, 16440, 232.9, {(0, 2): 210.1, (2, 1): 222.6, (2, 4): 226.9}),
    ("dx", True, 4096, 128, 32768, 67.6, {(3, 8): 63.8, (5, 4): 66.4}),
    ("dx", True, 8192, 512, 32768, 263.4, {(1, 2): 252.9}),
    ("dx", True, 8192, 384, 32000, 224.6, {(0, 4): 207.6}),
    ("dx", True, 8192, 192, 32760, 157.3, {(0, 8): 148.3, (2, 4): 148.2}),
    ("dx", True, 7900, 512, 32128, 245.3, {(0, 4): 220.9, (2, 2): 239.6, (0, 8): 241.0}),
    ("dx", True, 8192, 320, 30016, 205.9, {(0, 4): 194.2}),
    ("dx", True, 7000, 256, 32768, 159.4, {(0, 8): 154.7, (1, 4): 160.2}),
    ("dx", True, 8192, 320, 32768, 229.9, {}),
    ("dx", True, 8192, 384, 32768, 235.3, {}),
    ("dx", False, 7260, 128, 27448, 199.2, {}),
    ("dx", False, 8192, 128, 32768, 236.2, {(4, 1): 222.4}),
    ("dw", True, 32768, 128, 8192, 112.2, {}),
    ("dw", True, 20000, 192, 8192, 127.3, {(0, 2): 105.1, (2, 1): 116.6, (2, 4): 125.9}),
    ("dw", True, 23432, 192, 8010, 146.7, {(0, 2): 116.7, (2, 1): 136.1, (2, 4): 139.6}),
    ("dw", True, 31864, 192, 4677, 97.0, {(2, 1): 86.8}),
    ("fwd", False, 1564, 320, 3928, 21.3, {}),
    ("fwd", False, 680, 1216, 3760, 20.5, {}),
    ("fwd", False, 215, 2304, 3680, 18.5, {}),
    ("fwd", False, 5067, 384, 392, 7.7, {}),
    ("fwd", False, 954, 1152, 400, 6.8, {}),
    ("fwd", False, 205, 1216, 3008, 14.3, {}),
    ("fwd", False, 3965, 576, 2096, 22.6, {(3, 1): 22.7}),
]


@pytest.mark.parametrize("product,split,M,N,K,staged,dtl", SLOW_ARRIVAL)
def test_plan_of_products_whose_operands_arrive_slowly(plan, product, split, M, N, K, staged, dtl):
    """Long contractions of narrow products out of memory, and forward products on rows that straddle cache lines: the plan
    is not slower (1 % for the scatter of these times) than what the register-staged kernel alone would take."""
    tile, splits, direct, _ = plan(M, N, K, split, product != "dw", product == "fwd", True)
    assert not direct or dtl.get((tile, splits), 1e9) <= 1.01 * staged, (tile, splits)


@pytest.mark.parametrize("a_kc,b_kc", [(True, True), (True, False), (False, False)])
def test_plan_parts_hold_the_contraction(plan, a_kc, b_kc):
    """Parts of a split contraction are whole k-tiles, none is empty, and each is long enough for the kernel that takes it."""
    for M in (1, 40, 264, 1021, 8192, 32768):
        for N in (8, 128, 392, 1024, 12001):
            for K in (1, 63, 192, 200, 1000, 4096, 4104, 12001, 32768):
                for split in (False, True):
                    for dtl in (False, True):
                        tile, splits, direct, per = plan(M, N, K, split, a_kc, b_kc, dtl and K >= 192)
                        assert 0 <= tile <= 10 and 1 <= splits <= (16 if split else 1) and per % 64 == 0 and per > 0
                        assert (splits - 1) * per < K <= splits * per
                        if direct:
                            assert min(per, K - (splits - 1) * per) >= 192
                        if not (a_kc and b_kc):
                            assert tile != 8


GROUPED_TILE = r"""
#include "group_rule.hpp"
extern "C" int grouped_tile(const int* M, const int* N, int count, int k_max, int dtl, int strips, int strip_rows, int* wgs) {
    const mp::GroupPlan p = mp::group_plan(M, N, count, k_max, dtl, strips, strip_rows, 0, 0);
    wgs[0] = p.share.wgs; wgs[1] = p.share.busy; wgs[2] = p.share.first;
    return p.tile;
}
"""


def test_tile_of_a_grouped_launch(tmp_path):
    """The tile shape that each case of the GPU test of grouped launches is there for, and that the cases cover what a launch can
    do: every shape of both kernel families, in one round and in several, items beside the tiles only, behind them as well, and
    behind them only."""
    from gpu_util import GROUPED
    lib, share = _compile(str(tmp_path), "tile", GROUPED_TILE), (C.c_int * 3)()
    seen = set()
    for tile, shapes in GROUPED:
        rows, n = shapes[0][0], len(shapes)
        assert all(s[0] == rows for s in shapes)
        ints = lambda k: (C.c_int * n)(*[s[k] for s in shapes])  # noqa: E731
        strips = sum(s[1] // 128 for j, s in enumerate(shapes) if j != 1)
        for dtl in ([1, 0] if rows >= 192 else [0]):
            got = lib.grouped_tile(ints(1), ints(2), n, rows, dtl, strips, rows, share)
            assert got == tile or (not dtl and rows >= 192 and got in (0, 3)), (shapes, dtl, got)
            wgs, busy, first = share
            tm, tn = {0: (256, 256), 1: (256, 128), 3: (128, 128)}[got]
            several = sum(s[1] // tm * (s[2] // tn) for s in shapes) > wgs
            seen |= {(dtl, got, several), "beside" if first >= strips else "both" if first else "behind"}
    assert seen >= {(1, 0, False), (1, 0, True), (1, 1, False), (1, 1, True), (1, 3, False), (1, 3, True), (0, 0, False), (0, 0, True),
                    (0, 3, False), (0, 3, True), "beside", "both", "behind"}, seen
