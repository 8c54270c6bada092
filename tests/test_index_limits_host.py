"""Index arithmetic at the largest sizes the calls take (num_pairs and
num_bags up to 2^31 - 1), on the CPU with the kernels' own text: tiles of a
sort segment, tiles of the plain slices, the pair build's walk over a bag and
the gather-reduce's over an index range. Arrays are stand-ins that check every
index."""
import pytest

from tests import host_kernel as hk

STANDINS = r"""
static int64_t seen;
[[noreturn]] static void bad(const char *what, int64_t i) {
    std::printf("%s %lld\n", what, (long long)i);
    std::fflush(stdout);
    std::_Exit(3);
}
struct Range {  // entries [lo, hi) of an array, all 0
    int64_t lo, hi;
    int32_t operator[](int64_t i) const {
        if (i < lo || i >= hi) bad("read of entry", i);
        return 0;
    }
};
struct Out {  // counts the stores into [lo, hi)
    int64_t lo, hi;
    struct Ref {
        int64_t n;
        Ref &operator=(int64_t) { return __atomic_fetch_add(&seen, n, __ATOMIC_RELAXED), *this; }
    };
    Ref operator[](int64_t i) const {
        if (i < lo || i >= hi) bad("store to entry", i);
        return {1};
    }
};
constexpr int64_t kTop = (int64_t(1) << 31) - 1;
"""


def cast_source():
    return hk.source("tc_cast.hip")


TILES = r"""
int main() {
    for (int64_t n : {int64_t(1), int64_t(kSortTile), int64_t(kSortTile + 1), kTop - 4096, kTop - 4095, kTop - 1, kTop}) {
        const int64_t want = (n + kSortTile - 1) / kSortTile;
        if (tiles_of(int32_t(n)) != want) bad("tiles of", n);
        static SegLayout L;  // an empty table, then one that ends at pair kTop
        L.pstart[0] = L.pstart[1] = int32_t(kTop - n), L.pstart[2] = int32_t(kTop);
        L.tstart[0] = L.tstart[1] = 0, L.tstart[2] = int32_t(want);
        for (int64_t b = 0; b < want; b += b + 3 < want && b > 2 ? std::max<int64_t>(1, (want - b) / 2) : 1) {
            const TileRec r = tile_record(L, 2, int32_t(want), int32_t(b));
            const int64_t p0 = kTop - n + b * kSortTile;
            if (r.s != 1 || r.p0 != p0 || r.p1 != std::min(p0 + kSortTile, kTop)) bad("record of tile", b);
            const TileRec t = tile_of(int32_t(b), int32_t(want), nullptr, int32_t(n));
            if (t.s != 0 || t.p0 != b * kSortTile || t.p1 != std::min<int64_t>((b + 1) * kSortTile, n))
                bad("slice", b);
        }
        if (tile_of(int32_t(want), int32_t(want) + 1, nullptr, int32_t(n)).s >= 0) bad("slice past", n);
    }
}
"""


def test_tiles_up_to_the_last_pair(tmp_path):
    src = cast_source()
    parts = [STANDINS, "constexpr int kSortTile = 4096, kMaxSegTables = 256;\n",
             hk.block(src, "struct alignas(16) TileRec {"), hk.block(src, "struct SegLayout {")]
    for head in ("__device__ __forceinline__ int32_t tiles_of(", "__device__ TileRec tile_record(",
                 "__device__ __forceinline__ TileRec tile_of("):
        parts.append(hk.block(src, head))
    hk.run(hk.program(tmp_path, parts, TILES))


BUILD = r"""
int main() {
    for (int len : {1, 15, 16, 17, 40, 4000}) {
        seen = 0;
        const int32_t bo[2] = {int32_t(kTop - len), int32_t(kTop)};
        const int64_t off[2] = {0, 1};
        const Range idx{kTop - len, kTop};
        const Out out{kTop - len, kTop};
        run_grid(1, kBlock, [&] {
            build_pairs(0, 1, idx, bo, off, 1, 1, 1, false, false, SortPrep{}, out, out);
        });
        if (seen != 2 * len) bad("stores", seen);
    }
}
"""


def test_bag_that_ends_at_the_last_pair(tmp_path):
    fn = hk.block(cast_source(), "__device__ __forceinline__ void build_pairs(")
    for a, b in (("const int32_t *__restrict__ indices", "Range indices"),
                 ("int32_t *__restrict__ keys", "Out keys"), ("int32_t *__restrict__ vals", "Out vals")):
        assert a in fn
        fn = fn.replace(a, b)
    parts = [STANDINS, "constexpr int kBlock = 16;\nstruct SortPrep {};\n",
             "template <class... A> static void prepare_sort(A...) {}\n", fn]
    hk.run(hk.program(tmp_path, parts, BUILD))


WALK = r"""
int main() {
    for (int len : {1, 3, 4, 5, 40, 63}) {
        const float row[4] = {1.f, 2.f, 3.f, 4.f};
        const Range ids{kTop - len, kTop};
        static float4 got[kLanes];
        run_grid(1, kLanes, [&] {
            float4 acc[1] = {{0.f, 0.f, 0.f, 0.f}};
            group_range_sum<kLanes, 1>(row, 4, ids, 0, int32_t(kTop - len), int32_t(kTop),
                                       threadIdx.x, acc);
            got[threadIdx.x] = acc[0];
        });
        if (got[0].x != len || got[0].w != 4 * len) bad("sum", len);
    }
}
"""


@pytest.mark.parametrize("lanes", [4, 16])
def test_range_that_ends_at_the_last_pair(tmp_path, lanes):
    src = hk.source("tc_group_sum.h")
    fn = hk.block(src, "template <int LANES, int CHUNKS>\n__device__ __forceinline__ void group_range_sum(")
    a = "const int32_t *__restrict__ ids"
    assert a in fn
    parts = [STANDINS, f"constexpr int kLanes = {lanes};\n", """
struct alignas(16) float4 { float x, y, z, w; };
static float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
static float4 f4_add(float4 a, float4 b) { return {a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w}; }
static int32_t shuffle[kLanes];
static int32_t __shfl(int32_t v, int lane, int) {
    shuffle[threadIdx.x] = v;
    __syncthreads();
    const int32_t r = shuffle[lane];
    __syncthreads();
    return r;
}
""", hk.const(src, "kUnroll"), fn.replace(a, "Range ids")]
    hk.run(hk.program(tmp_path, parts, WALK))


def test_small_cast_walk_over_bags_does_not_wrap():
    # its stride past the last of 2^31 - 1 bags stays in range
    assert "for (uint32_t g = tid + kSmallPairs; g < uint32_t(num_bags); g += kSmallThreads)" \
        in cast_source()
