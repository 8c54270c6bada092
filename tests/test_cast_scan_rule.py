"""The rule by which a sort scans its group sums, and the rows of them that the
scatter reads, on the CPU with the source's own text: at most 2^17 rows a pass
without the scan, in whatever way the segments share the tiles, so that the
scatter's work never grows with the square of a segment's length; and the
segments' first tiles fit behind the tile records."""
import pytest

from tests import host_kernel as hk

MAIN = r"""
int main(int argc, char **argv) {
    const int32_t num_tables = atoi(argv[1]);
    for (int64_t n = 8193; n < int64_t(1) << 31; n += n / 7) {
        const CastPlan p = cast_plan(n, num_tables);
        const bool scan = scan_groups(p.seg_tiles, num_tables);
        const int64_t groups = p.seg_tiles / kGroupTiles, rows = p.seg_tiles * groups;
        if (!scan && rows >= 1 << 17) return 3;
        if (scan && p.seg_tiles < 512) return 4;
        const size_t firsts = (p.off_recs + size_t(p.sort_tiles) * sizeof(TileRec)) +
                              size_t(num_tables + 1) * sizeof(int32_t);
        if (scan && firsts > p.bytes) return 5;
    }
    return 0;
}
"""


@pytest.mark.parametrize("tables", [1, 3, 32, 256])
def test_rows_read_without_the_scan(tmp_path, tables):
    src = hk.source("tc_cast.hip")
    parts = ["#include <cstddef>\nconstexpr int kSortTile = 4096, kMaxSegTables = 256;\n",
             hk.const(src, "kGroupTiles"), hk.block(src, "struct alignas(16) TileRec {"),
             hk.const(src, "kAlign"), hk.block(src, "inline size_t align_up("),
             hk.block(src, "inline int32_t seg_capacity("), hk.block(src, "struct CastPlan {"),
             hk.block(src, "inline CastPlan cast_plan("), hk.block(src, "inline bool scan_groups(")]
    hk.run(hk.program(tmp_path, parts, MAIN), tables)
