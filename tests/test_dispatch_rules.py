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
