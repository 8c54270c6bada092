"""The backward's list kernel on the CPU: which entries of seg_offsets it
reads (0 .. *num_unique, whatever the capacities are: max_unique is that of
the coalesced rows alone), and that every long segment the workspace covers is
listed once."""
import pytest

from tests import host_kernel as hk

MAIN = r"""
// num segments; cap segments of room, cap_pairs covered, blocks workgroups.
// of 1 to 3 pairs, with one of 48 or more now and then; `empty` percent
// of them without pairs instead
int main(int argc, char **argv) {
    const int64_t num = atoll(argv[1]), cap = atoll(argv[2]), cap_pairs = atoll(argv[3]);
    const int blocks = atoi(argv[4]), empty = atoi(argv[5]);
    std::vector<int32_t> offs(num + 1, 0);
    uint32_t s = 12345u + uint32_t(num);
    auto next = [&] { return s = s * 1664525u + 1013904223u, s >> 8; };
    for (int64_t u = 0; u < num; ++u) {
        const uint32_t r = next() % 97;
        int32_t len = r == 0 ? 48 + next() % 700 : r == 1 && !empty ? 2048 + next() % 9000 : 1 + r % 3;
        if (empty && int(next() % 100) < empty) len = 0;
        offs[u + 1] = offs[u] + len;
    }
    const int32_t n = int32_t(num);
    SplitWs ws{};
    ws.cap_pairs = cap_pairs;
    ws.list_blocks = blocks;
    ws.parts = 2;
    const int64_t pairs = std::max<int64_t>(cap_pairs, offs[num]);
    std::vector<int4> heads(blocks);
    std::vector<int2> big(pairs / kBigLong + 2, int2{-1, -1}), longs(pairs / kListLong + 2, int2{-1, -1});
    std::vector<int32_t> done((pairs / kSplitPairs + 2) * ws.parts, -1), turns(kXcds * kTurnStride);
    ws.heads = heads.data(), ws.big = big.data(), ws.longs = longs.data();
    ws.seg_done = done.data(), ws.turns = turns.data();
    const int grid = int(std::max<int64_t>(1, std::min<int64_t>(blocks, (cap + kListThreads - 1) / kListThreads)));
    run_grid(grid, kListThreads, [&] { k_backward_list(Checked{offs.data(), num + 1}, &n, cap, ws); });
    // the entries, by the heads' slots, against the segments
    std::vector<int32_t> listed(num, 0);
    int64_t sum = 0, covered = 0;
    for (int b = 0; b < blocks; ++b) {
        const int4 h = heads[b];
        for (int i = 0; i < h.x; ++i) {
            const int2 e = big[h.z / kBigLong + i];
            if (e.x < 0 || e.x >= num) return 4;
            listed[e.x] += e.y < 0 ? 1000 : 1;
        }
        for (int i = 0; i < h.y; ++i) {
            const int2 e = longs[h.z / kListLong + i];
            if (e.x < 0 || e.x >= num || offs[e.x] != e.y) return 5;
            listed[e.x] += 1000;
        }
        sum += h.w;
    }
    for (int64_t u = 0; u < num; ++u) {
        const int32_t len = offs[u + 1] - offs[u];
        const bool is = len >= kListLong && offs[u + 1] <= cap_pairs;
        const int32_t want = !is ? 0 : len >= kSplitPairs ? num_pieces(len) : 1000;
        if (listed[u] != want) {
            std::printf("segment %lld of %d pairs: %d listed, not %d\n", (long long)u, len, listed[u], want);
            return 6;
        }
        if (is) covered += len;
    }
    if (sum != covered) return 7;
    std::printf("%lld pairs in long segments\n", (long long)covered);
    return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    src, internal = hk.source("tc_backward.hip"), hk.source("tc_internal.h")
    consts = "".join(hk.const(src, c) for c in ("kListLong", "kPieceMin", "kMaxPieces", "kBigLong",
                                                "kTurnStride"))
    consts += "constexpr int kListThreads = 256;\n"  # of the 1024, to be quick
    kernel = hk.block(src, "__global__ __launch_bounds__(kListThreads) void k_backward_list(")
    kernel = kernel.replace("const int32_t *__restrict__ offsets", "Checked offsets", 1)
    assert "Checked offsets" in kernel
    # the grid, as launch_backward has it
    assert "grid_for(cap, kListThreads, ws.list_blocks)" in src
    return hk.program(tmp_path_factory.mktemp("list"), [
        "constexpr int32_t kSplitPairs = 2048;\n", hk.const(internal, "kXcds"), consts,
        hk.block(src, "struct SplitWs {"), hk.block(src, "__device__ __forceinline__ int32_t num_pieces("),
        kernel], MAIN)


# segments against the capacities: full, a few segments in room for many (the
# largest batch's, or the fixed scratch's cover), none at all, one, and more
# segments than threads
@pytest.mark.parametrize("num,cap,cap_pairs,blocks", [
    (0, 1, 80, 16), (0, 5000, 10 ** 7, 256), (1, 1, 80, 16), (1, 200_000, 10 ** 7, 256),
    (300, 300, 40_000, 16), (300, 8_000, 8_000, 16), (1_500, 100_000, 35_800_000, 256),
    (5_000, 5_000, 10 ** 6, 256), (5_000, 5_001, 3_000, 16), (40_000, 40_000, 10 ** 7, 16),
    (3_000, 300_000, 10 ** 7, 256)])
def test_reads_only_the_batch_s_offsets(exe, num, cap, cap_pairs, blocks):
    hk.run(exe, num, cap, cap_pairs, blocks, 0)


# segments without pairs, more of them than the workspace covers pairs
@pytest.mark.parametrize("num,cap_pairs,blocks,empty", [
    (50_000, 6_000, 16, 99), (9_000, 4_000, 16, 98), (400_000, 100_000, 256, 99),
    (2_500, 2_400, 16, 80)])
def test_segments_without_pairs(exe, num, cap_pairs, blocks, empty):
    out = hk.run(exe, num, num, cap_pairs, blocks, empty)
    assert int(out.split()[0]) > 0
