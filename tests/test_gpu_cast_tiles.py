"""The radix cast (more than 8192 pairs) at the sizes where its code changes,
against the CPU oracle, every index bit for bit: each digit width, pair counts
around the tile (4096 pairs) and around full groups of 16 tiles, digit counts
in the batch's own arrays and (more tables than full tiles) in the plan's
area, and keys that are all equal or all in one digit."""
import numpy as np
import pytest

from tests.test_gpu_cast_layouts import check, gpu_cast, oracle_cast

pytestmark = pytest.mark.gpu

TILE, GROUP = 4096, 16


# 1..31 key bits, in one to three passes: every width of digit
@pytest.mark.parametrize("bits", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 15, 17, 19, 20, 21, 22,
                                  23, 26, 28, 31])
def test_digit_widths(bits):
    check(f"{bits} bits", [2 ** bits - (bits > 3)], [3 * TILE - 5], bags_per_table=97, seed=bits,
          bounds=[0])


@pytest.mark.parametrize("tiles", [GROUP - 1, GROUP, GROUP + 1, 2 * GROUP, 3 * GROUP + 1,
                                   9 * GROUP + 2])
def test_groups_of_tiles(tiles):
    n = tiles * TILE
    check(f"{tiles} tiles", [70_000, 50, 900], [n, n - 1, TILE + 1], bags_per_table=333,
          seed=tiles)


# digits of 11 bits up to 512 tiles, of 10 at most above
@pytest.mark.parametrize("bits", [11, 21, 22, 31])
@pytest.mark.parametrize("tiles", [512, 513])
def test_widest_digits(bits, tiles):
    check(f"{bits} bits, {tiles} tiles", [2 ** bits - 1], [tiles * TILE], bags_per_table=700,
          seed=bits + tiles, bounds=[0])


# sorts whose group sums are scanned (one segment: from 512 tiles; three: from
# 887) and not, table-local and global
@pytest.mark.parametrize("groups", [31, 32, 55, 56])
def test_long_segments(groups):
    n = groups * GROUP * TILE + 37
    check(f"{groups} groups", [3000, 40_000, 70], [TILE + 1, n, 5], bags_per_table=2000,
          seed=groups)


# in a scanned sort, segments on both sides of the 8 groups that are added up
# one by one
def test_segments_of_a_scanned_sort():
    n = GROUP * TILE
    check("scanned sort", [900, 5000, 30, 70_000], [8 * n + 5, 9 * n, 60 * n - 1, 9],
          bags_per_table=999, seed=1)


# the segment build in one launch (up to 96 tiles) and in two
@pytest.mark.parametrize("pairs", [95 * TILE + 1, 96 * TILE, 96 * TILE + 1])
def test_segment_build_launches(pairs):
    check(f"{pairs} pairs", [300_000], [pairs], bags_per_table=1000, seed=pairs % 97)


@pytest.mark.parametrize("tables,pairs", [(256, 40), (256, 700), (200, 4097), (37, 230)])
def test_many_tables(tables, pairs):
    check(f"{tables} tables", [1000 + 13 * k for k in range(tables)],
          [pairs + k % 3 for k in range(tables)], bags_per_table=3, seed=tables)


@pytest.mark.parametrize("rows,index", [(1, 0), (70_000, 69_999), (2 ** 20, 2 ** 19 + 1)])
def test_one_row_takes_all(rows, index):
    n, bags = 17 * TILE + 3, 50
    off = np.array([0, rows], np.int64)
    bo = np.linspace(0, n, bags + 1).astype(np.int32)
    idx = np.full(n, index, np.int32)
    ref, got = oracle_cast(off, bo, idx, bags), gpu_cast(off, bo, idx, bags, rows)
    assert got["num_unique"] == ref["num_unique"] == 1
    for k in ("unique_rows", "seg_offsets", "casted_src", "casted_dst"):
        assert np.array_equal(got[k], ref[k][:len(got[k])]), k
