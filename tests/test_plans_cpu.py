"""Which kernel and tile a call takes, on the side of each rule where a slower one was taken before.  No GPU: the
plan is asked for through heinsen_kernel_name and heinsen_tile_shape; rules that do not show there stand in
scan_rules.hpp and are compiled by themselves."""
import os
import subprocess

import pytest

from paper_2311_06281_amd import binding as hb

BDN, BND = hb.HEINSEN_LAYOUT_BDN, hb.HEINSEN_LAYOUT_BND
LOGS = hb.HEINSEN_LOG_INPUTS | hb.HEINSEN_LOG_OUTPUT
CLOG = hb.HEINSEN_LOG_OUTPUT | hb.HEINSEN_OUT_COMPLEX


# rows, n, flags -> kernel, rows per workgroup, steps (four waves per workgroup)
@pytest.mark.parametrize("rows,n,flags,kernel,tile", [
    (512, 200, 0, "rows_wave", (4, 200)),              # one wave per SIMD: a row each
    (4096, 100, 0, "rows_packed", (4 * 4, 100)),       # eight steps per lane: 13 lanes per row
    (131072, 100, 0, "rows_packed", (4 * 9, 100)),     # the chip is full: 16 steps, 7 lanes
    (4096, 300, 0, "rows_wave", (4, 300)),
    (32768, 300, 0, "rows_packed", (4 * 3, 300)),
    (16384, 508, 0, "rows_wave", (4, 508)),
    (63, 16, CLOG, "rows_packed", (4 * 32, 16)),       # two lanes of eight steps
    (512, 4096, LOGS, "tiles", (1, 4 * 64 * 16)),
    (2048, 4096, 0, "tiles", (1, 2 * 64 * 32)),
    (2048, 12000, 0, "tiles", (1, 8 * 64 * 32)),
    (600, 12000, 0, "tiles", (1, 6 * 64 * 32)),
    (600, 1022, 0, "rows_wave", (4, 1022)),
])
def test_plans_of_rows(rows, n, flags, kernel, tile):
    assert hb.heinsen_kernel_name(1, rows, n, BDN, flags) == "heinsen_scan_" + kernel
    assert hb.heinsen_tile_shape(1, rows, n, BDN, flags) == tile


# B, n, D -> channels a tile takes: of several items where an item's do not fill it
@pytest.mark.parametrize("B,n,D,channels", [
    (1, 300, 5, 64), (13, 300, 5, 40), (256, 4096, 19, 38), (256, 4096, 16, 64), (7, 300, 40, 64), (3, 300, 1024, 64),
])
def test_channels_of_a_tile(B, n, D, channels):
    assert hb.heinsen_tile_shape(B, D, n, BND, 0) == (channels, 256)


# B, n, D -> kernel for a few steps
@pytest.mark.parametrize("B,n,D,kernel", [(64, 1, 4096, "steps"), (64, 8, 8, "steps"), (64, 4, 3, "steps"), (64, 8, 3, "steps"), (1 << 21, 8, 3, "bnd"), (64, 9, 4096, "bnd")])
def test_kernel_of_a_few_steps(B, n, D, kernel):
    assert hb.heinsen_kernel_name(B, D, n, BND, 0) == "heinsen_scan_" + kernel


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """Values of C++ expressions over scan_rules.hpp."""
    folder = tmp_path_factory.mktemp("rules")
    csrc = os.path.join(os.path.dirname(os.path.abspath(hb.__file__)), "csrc")

    def values(expressions):
        lines = "".join(f'    std::printf("%lld\\n", (long long)({e}));\n' for e in expressions)
        (folder / "rules.cpp").write_text(f'#include "scan_rules.hpp"\n#include <cstdio>\nusing namespace hs;\nint main()\n{{\n{lines}}}\n')
        subprocess.run(["g++", "-std=c++17", "-I", csrc, str(folder / "rules.cpp"), "-o", str(folder / "rules")], check=True)
        return [int(v) for v in subprocess.run([str(folder / "rules")], check=True, capture_output=True, text=True).stdout.split()]

    return values


def test_only_tiles_that_share_a_compute_unit_are_paced(rules):
    # moved as vectors, complex output, bf16, tiles per row, tiles
    assert rules(["pace_ns(true, false, false, 5000, 5000)", "pace_ns(true, false, true, 5000, 5000)"]) == [12, 8]
    assert rules([f"pace_ns({v}, {c}, {h}, {r}, {t})" for v, c in (("false", "false"), ("true", "true"), ("false", "true"))
                  for h in ("false", "true") for r, t in ((3, 600), (5000, 5000), (16, 1024))]) == [0] * 18
    assert rules(["pace_ns(true, false, false, 2, 5000)", "pace_ns(true, false, false, 100, 100)"]) == [0, 0]  # rows of two tiles; a launch that fits the chip


def test_launches_of_up_to_two_rounds_are_paced_only_in_long_rows(rules):
    tiles = (511, 512, 519, 520, 760, 819, 820, 960, 1024, 1025, 1600, 100000)
    for half, ns in (("false", 12), ("true", 8)):
        assert rules([f"pace_ns(true, false, {half}, 16, {t})" for t in tiles]) == [0] * 9 + [ns] * 3
    assert rules([f"pace_ns(true, false, false, 64, {t})" for t in tiles]) == [0, 0, 0, 12, 12, 12, 0, 0, 0, 12, 12, 12]
    assert rules([f"pace_ns(true, false, true, 500, {t})" for t in tiles]) == [0] * 9 + [8] * 3


def test_ticket_queues_go_by_columns_alone(rules):
    assert rules([f"ticket_queues(8, {c}, true)" for c in (128, 255, 256, 511, 512, 1023, 1024, 4096)]) == [1, 1, 2, 2, 4, 4, 8, 8]
    assert rules([f"ticket_queues(8, {c}, false)" for c in (1, 15, 16, 31, 32, 63, 64, 1000)]) == [1, 1, 2, 2, 4, 4, 8, 8]


def test_only_tiles_that_wait_keep_ordinary_stores(rules):
    # waves of a tile, columns, tiles of a column, second carry level, without logarithms, runs of narrow items
    assert rules([f"waits_behind_stores(8, {c}, {k}, false, false, false)" for c, k in ((64, 4), (257, 1), (129, 2), (128, 4), (96, 8), (769, 1), (385, 2))]) == [0, 0, 1, 1, 1, 0, 0]
    assert rules([f"waits_behind_stores({w}, 500, 1, false, false, false)" for w in (1, 2, 4, 8)]) == [0] * 4  # one tile each
    assert rules(["waits_behind_stores(16, 125, 4, false, false, false)", "waits_behind_stores(8, 125, 4, false, false, true)"]) == [0, 0]


def test_two_carry_levels_keep_ordinary_stores_only_without_logarithms(rules):
    assert rules([f"waits_behind_stores(8, {c}, {k}, true, false, false)" for c, k in ((8, 40), (15, 30), (3, 100), (12, 37))]) == [0] * 4
    assert rules([f"waits_behind_stores(8, {c}, {k}, true, true, false)" for c, k in ((7, 60), (8, 32), (8, 33), (12, 37), (8, 64), (9, 57), (14, 60))]) == [0, 0, 1, 1, 1, 0, 0]


def test_runs_that_cut_lines_are_written_through_up_to_96_mb(rules):
    mb = 1 << 20
    assert rules([f"runs_in_lines(true, 250, 994 * 17, {m * mb})" for m in (49, 96, 97, 120)]) == [1, 1, 0, 0]
    assert rules([f"runs_in_lines({o}, {b}, {e}, {200 * mb})" for o, b, e in (("true", 9, 4096 * 16), ("true", 1, 4097 * 13), ("false", 9, 4096 * 16), ("false", 1, 4096))]) == [1, 1, 0, 0]


def test_tall_tiles_are_for_few_columns_and_few_rounds(rules):
    def tall(pairs, channels=64, runs="false", bf16="false", steps=512):  # columns, tiles of 512 steps per column (or one of 256 fewer)
        return rules([f"tall_tiles({c}, {2 * k - (steps < 512)}, {channels}, {runs}, {bf16}, 8)" for c, k in pairs])

    few = ((1, 128), (1, 129), (1, 768), (1, 769), (3, 256), (3, 257), (15, 8), (15, 51), (15, 52))
    assert tall(few) == tall(few, 2, "true", "true") == tall(few, steps=256) == [0, 1, 1, 0, 1, 0, 0, 1, 0]
    assert tall(((16, 8), (16, 9), (16, 32), (16, 33), (24, 21), (24, 22), (25, 10), (32, 8), (32, 9))) == [0, 1, 1, 0, 1, 0, 0, 1, 0]
    assert tall(((16, 32), (19, 12), (19, 26), (24, 20), (24, 21), (32, 8)), 3, "true") == [1, 1, 0, 0, 1, 1]
    assert tall(((16, 30), (16, 31), (17, 28)), 3, "true", "true") == [0, 1, 0]
    assert tall(((28, 5), (29, 5), (16, 9)), steps=256) == [0, 1, 1]  # more than 256 tiles of 256 steps
    assert tall(((16, 32), (17, 10), (20, 9), (32, 8), (17, 16)), 2, "true") == [0, 0, 1, 1, 0]
    # one round of the chip, as the queues deal the columns (33 to 63 columns in four, from 64 in eight)
    one = ((44, 5), (48, 5), (49, 5), (64, 4), (65, 4), (85, 3))
    assert tall(one) == tall(one, bf16="true") == [1, 1, 0, 1, 0, 0]
    assert tall(one, 65) == tall(one, 16, "true") == [1, 1, 0, 0, 0, 0]
    assert tall(one, 65, bf16="true") == tall(one, 16, "true", "true") == [0] * 6
    # two rounds
    two = ((64, 8), (72, 7), (65, 7), (48, 9), (48, 8), (80, 6), (85, 5), (56, 9), (57, 9), (32, 16), (32, 12))
    assert tall(two) == tall(two, 16, "true", "true") == [0] * len(two)
    assert tall(two, 65) == [1, 1, 1, 1, 0, 1, 0, 1, 0, 1, 0]
    assert tall(two, 65, bf16="true") == [1, 1, 1, 1, 0, 0, 0, 1, 0, 1, 0]
    assert tall(two, 16, "true") == [0, 0, 0, 0, 0, 0, 0, 0, 0, 1, 0]


# B, n, D, flags -> steps of a tile
@pytest.mark.parametrize("B,n,D,flags,steps", [
    (2, 131072, 96, 0, 512), (2, 131072, 96, hb.HEINSEN_LINEAR, 256), (2, 131072, 96, CLOG, 256), (1, 512 * 128, 64, 0, 256), (1, 512 * 129, 64, 0, 512),
    (16, 8192, 64, LOGS, 512), (16, 16384 + 1, 64, LOGS, 256), (40, 512 * 45, 5, 0, 512),
    (6, 3001, 770, 0, 512), (6, 3001, 768, 0, 256), (4, 1996, 896, 0, 512), (64, 4096, 64, 0, 256), (128, 8192, 16, 0, 512), (128, 8192, 16, hb.HEINSEN_LINEAR, 256),
])
def test_steps_of_a_tile(B, n, D, flags, steps):
    assert hb.heinsen_tile_shape(B, D, n, BND, flags)[1] == steps


def test_few_short_runs_keep_tiles_of_eight_waves(rules):
    # columns and tiles of 512 steps per column: as runs (float32, bf16) and not
    sizes = ((8, 17), (8, 20), (7, 20), (6, 23), (8, 24), (6, 24), (5, 26), (4, 40), (9, 15), (12, 11), (15, 9))
    for half in ("false", "true"):
        assert rules([f"tall_tiles({c}, {2 * k}, 5, true, {half}, 8)" for c, k in sizes]) == [0] * 4 + [1] * 7
        assert rules([f"tall_tiles({c}, {2 * k}, 64, false, {half}, 8)" for c, k in sizes]) == [1] * 11
