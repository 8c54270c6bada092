// Tensor Casting (Algorithm 2) on CDNA4.
//
//  1. k_build_keys   -- (src, dst) pairs from the bag-major CSR index:
//                       key = row, value = bag id. Also writes the tile
//                       records of the sort segments (below) and clears the
//                       group sums of the passes' digit counts.
//  2. LSD radix sort by key, stable, at most kMaxRadixBits bits per pass over
//     the key bits that can be set. Each pass is
//       k_radix_hist    per-tile digit counts (LDS histograms), and their
//                       sums over full groups of kGroupTiles tiles
//       k_radix_scan    for long segments: prefixes of those sums
//       k_radix_scatter stable scatter: the tile's place in each digit from
//                       the counts of the tiles before it; a wave finds the
//                       lanes holding equal digits with ballots, counts them
//                       into its running per-digit count in LDS, waves are
//                       combined in tile order, and the tile is laid out in
//                       sorted order in LDS and stored in that order.
//     A pass reads and writes 8 bytes per pair plus a 4-byte read for the
//     histogram. The last pass writes the values straight into casted_src.
//  3. Segment build (the scan and cumulative sum of Algorithm 2):
//       k_segments   counts the heads (key differs from its predecessor) per
//                    tile, then casted_dst, unique_rows, seg_offsets and
//                    *num_unique from the counts of the tiles before; for
//                    large batches in two launches, k_seg_count, k_seg_write
//
// What bounds it at a batch of a million pairs is not bandwidth (a pass moves
// 20 bytes per pair, 4 us) but the number of launches and, in each, a chain of
// dependent steps of 4-10 us that every workgroup goes through once: so few
// passes with wide digits, and no kernel between a histogram and its scatter
// until segments are long.
// Measured (us, the cast's kernels): 8 tables of 1M rows, 1.3M pairs: 49,
// against 70 with three passes of 7-bit digits over 2048-pair tiles with a
// scan kernel each; 16 tables, 91k pairs each: 61 against 84; 13 tables, 139k
// pairs: 32 against 50; one table of 50M rows, 1.6M pairs: 79 against 104;
// 32 tables, 5.2M pairs (bandwidth: 10-bit digits leave runs of 16 bytes): 111
// against 145.
//
// Sort segments. The pairs of table t are contiguous in the input
// (bag-major CSR, tables in order) and so are their rows in the output. When
// the caller bounds the table sizes, each table is sorted on its
// table-local row, which needs fewer key bits than the global row (32 tables
// of 2^20 rows: 20 bits, two passes, instead of 25 bits and three), and the
// last pass adds the table's row offset back. A segment is cut into tiles of
// kSortTile pairs (its last tile may be short), tiles of all segments are
// numbered in segment order, and a digit's position inside its segment comes
// from the counts of the segment's tiles. The build writes one record per
// tile (its pair range and its segment's), so a pass kernel finds its tile
// with a single load. Without a bound there is one segment, all pairs on
// global rows, and tiles are plain slices of kSortTile pairs.
//
// Within a tile, wave w owns positions [w*kWaveSpan, (w+1)*kWaveSpan) and
// walks them 64 at a time, lane l taking position base + 64*i + l, so tile
// order = (wave, iteration, lane) order and every pass is stable. The only
// atomics on global memory are the group sums' (whole numbers, whose order
// does not matter) and the segment build's; no result depends on scheduling
// order.
//
// tc_embed_forward_cast runs the forward gather-reduce in the cast's
// launches: k_forward_build (workgroups building pairs, then workgroups of the
// forward) or, for a small batch, beside the one k_cast_small workgroup.
#include "tc_group_sum.h"

namespace tc {
namespace {

// Tiles of the sort: kSortThreads threads, kItems positions per lane, digits of
// up to kMaxRadixBits bits. Wide digits save passes and cost bookkeeping
// (counts written and read back for every digit of every tile); tiles of 4096
// pairs carry that and still spread a batch of a million pairs over all CUs,
// whose wavefronts rank their pairs four SIMDs at a time.
constexpr int kMaxRadixBits = 11;
constexpr int kSortThreads = 512;
constexpr int kItems = 8;
constexpr int kSortWaves = kSortThreads / kWave;      // 8
constexpr int kWaveSpan = kWave * kItems;             // 512
constexpr int kSortTile = kSortWaves * kWaveSpan;     // 4096
// Full groups of this many tiles of a segment have their digit counts summed.
constexpr int kGroupTiles = 16;
// Table-local sorting for at most this many tables (one thread per table
// lays the segments out).
constexpr int kMaxSegTables = kBlock;

// Exclusive scan over a workgroup of one value per thread; returns the prefix
// and writes the workgroup's total to *total.
template <int THREADS>
__device__ __forceinline__ int32_t block_scan(int32_t v, int32_t *total) {
    constexpr int kWaves = THREADS / kWave;
    __shared__ int32_t wsum[kWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int32_t incl = wave_prefix(v);
    if (lane == kWave - 1) wsum[w] = incl;
    __syncthreads();
    int32_t wbase = 0, tot = 0;
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
        const int32_t s = wsum[ww];
        if (ww < w) wbase += s;
        tot += s;
    }
    __syncthreads();  // wsum may be reused by the next call
    *total = tot;
    return wbase + incl - v;
}

// One tile of a radix pass: pairs [p0, p1) of segment s, whose tiles are
// [first, next), whose pairs start at pstart, and whose keys get rowoff added
// by the last pass. Tiles past the last one have p0 = p1 = 0 and s = -1.
struct alignas(16) TileRec {
    int32_t p0, p1, first, next, pstart, rowoff, s, pad;
};
// Tiles of `pairs` pairs. (Positions go up to 2^31 - 1: no sum here exceeds it.)
__device__ __forceinline__ int32_t tiles_of(int32_t pairs) {
    return pairs / kSortTile + (pairs % kSortTile != 0);
}
// ---------------------------------------------------------------------------
// 1. key build. The segments of the table-local sort, in LDS: segment s has
// tiles [tstart[s], tstart[s+1]) and pairs [pstart[s], pstart[s+1]), and
// rowoff[s] is its table's first row. seg_layout fills it (whole workgroup)
// and returns the number of tiles; tile_record reads tile b's record off it.
struct SegLayout {
    int32_t tstart[kMaxSegTables + 1], pstart[kMaxSegTables + 1], rowoff[kMaxSegTables];
};

__device__ int32_t seg_layout(SegLayout &L, const int32_t *__restrict__ bag_offsets,
                              const int64_t *__restrict__ table_row_offset, int64_t num_bags,
                              int32_t bags_per_table, int32_t num_tables) {
    const int t = threadIdx.x;
    int32_t p0 = 0, n_t = 0;
    if (t < num_tables) {
        p0 = bag_offsets[int64_t(t) * bags_per_table];
        n_t = bag_offsets[int64_t(t + 1) * bags_per_table] - p0;
        L.rowoff[t] = int32_t(table_row_offset[t]);
    }
    int32_t total;
    const int32_t ts = block_scan<kBlock>(tiles_of(n_t), &total);
    if (t < num_tables) {
        L.tstart[t] = ts;
        L.pstart[t] = p0;
    }
    if (t == 0) {
        L.tstart[num_tables] = total;
        L.pstart[num_tables] = bag_offsets[num_bags];
    }
    __syncthreads();
    return total;
}

__device__ TileRec tile_record(const SegLayout &L, int32_t num_tables, int32_t total, int32_t b) {
    TileRec r{0, 0, 0, 0, 0, 0, -1, 0};
    if (b < total) {
        // the segment holding tile b: last s with tstart[s] <= b (segments
        // without pairs have no tiles and are passed over)
        int32_t lo = 0, hi = num_tables - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) / 2;
            if (L.tstart[mid] <= b) lo = mid; else hi = mid - 1;
        }
        const int32_t sg = lo;
        r.s = sg;
        r.first = L.tstart[sg];
        r.next = L.tstart[sg + 1];
        r.pstart = L.pstart[sg];
        r.rowoff = L.rowoff[sg];
        r.p0 = L.pstart[sg] + (b - r.first) * kSortTile;
        const int32_t end = L.pstart[sg + 1];
        r.p1 = end - r.p0 > kSortTile ? r.p0 + kSortTile : end;
    }
    return r;
}

// The records of all num_tile_slots tile slots, written by one workgroup, and
// the segments' first tiles to seg_first (if not null).
__device__ void write_tile_records(const int32_t *__restrict__ bag_offsets,
                                   const int64_t *__restrict__ table_row_offset,
                                   int64_t num_bags, int32_t bags_per_table, int32_t num_tables,
                                   TileRec *__restrict__ tiles, int32_t num_tile_slots,
                                   int32_t *__restrict__ seg_first) {
    __shared__ SegLayout L;
    const int32_t total = seg_layout(L, bag_offsets, table_row_offset, num_bags, bags_per_table,
                                     num_tables);
    for (int32_t b = threadIdx.x; b < num_tile_slots; b += kBlock)
        tiles[b] = tile_record(L, num_tables, total, b);
    if (seg_first)
        for (int32_t t = threadIdx.x; t <= num_tables; t += kBlock) seg_first[t] = L.tstart[t];
}

// Where the sort's bookkeeping is, for the kernels before its first pass:
// tile records to write (null: none), and words to clear.
struct SortPrep {
    TileRec *recs;
    int32_t tile_slots;
    int32_t *groups;
    int64_t group_words;
    int32_t *state;  // of the segment build, cleared too
    int64_t state_words;
    int32_t *seg_first;  // for k_radix_scan (null: it does not run)
};
// The share of workgroup `b` of `blocks` in that; workgroup 0 also writes the
// records.
__device__ __forceinline__ void prepare_sort(const SortPrep &sp, int64_t b, int64_t blocks,
                                             const int32_t *__restrict__ bag_offsets,
                                             const int64_t *__restrict__ table_row_offset,
                                             int64_t num_bags, int32_t bags_per_table,
                                             int32_t num_tables) {
    for (int64_t i = b * kBlock + threadIdx.x; i < sp.group_words; i += blocks * kBlock)
        sp.groups[i] = 0;
    for (int64_t i = b * kBlock + threadIdx.x; i < sp.state_words; i += blocks * kBlock)
        sp.state[i] = 0;
    if (sp.recs && b == 0)
        write_tile_records(bag_offsets, table_row_offset, num_bags, bags_per_table, num_tables,
                           sp.recs, sp.tile_slots, sp.seg_first);
}

// (src, dst) pairs by a walk over the bags, and the share of workgroup `b` of
// `blocks` in prepare_sort: one group of 16 lanes per bag writes that bag's
// pairs. Keys are table-local rows when `local`, else global rows; values are
// bag ids (dst), or pair positions when `positions` (an argsort).
__device__ __forceinline__ void build_pairs(int64_t b, int64_t blocks,
                                            const int32_t *__restrict__ indices,
                                            const int32_t *__restrict__ bag_offsets,
                                            const int64_t *__restrict__ table_row_offset,
                                            int64_t num_bags, int32_t bags_per_table,
                                            int32_t num_tables, bool local, bool positions,
                                            const SortPrep &sp, int32_t *__restrict__ keys,
                                            int32_t *__restrict__ vals) {
    prepare_sort(sp, b, blocks, bag_offsets, table_row_offset, num_bags, bags_per_table,
                 num_tables);
    constexpr int kLanes = 16, kGroups = kBlock / kLanes;
    const int sub = threadIdx.x & (kLanes - 1);
    for (int64_t g = b * kGroups + threadIdx.x / kLanes; g < num_bags; g += blocks * kGroups) {
        const int32_t beg = bag_offsets[g], end = bag_offsets[g + 1];
        const int64_t base = local ? 0 : table_row_offset[g / bags_per_table];
        for (uint32_t j = beg + sub; j < uint32_t(end); j += kLanes) {  // may pass 2^31
            keys[j] = int32_t(base + indices[j]);
            vals[j] = positions ? int32_t(j) : int32_t(g);
        }
    }
}
// Workgroups for it.
inline unsigned build_grid(int64_t num_bags) {
    return grid_for(num_bags, kBlock / 16, int64_t(device_cus()) * 8);
}

// The pair build alone (tc_cast_index, tc_argsort_rows).
__global__ __launch_bounds__(kBlock) void k_build_keys(
    const int32_t *__restrict__ indices, const int32_t *__restrict__ bag_offsets,
    const int64_t *__restrict__ table_row_offset, int64_t num_bags, int32_t bags_per_table,
    int32_t num_tables, bool local, bool positions, SortPrep sp, int32_t *__restrict__ keys,
    int32_t *__restrict__ vals) {
    build_pairs(blockIdx.x, gridDim.x, indices, bag_offsets, table_row_offset, num_bags,
                bags_per_table, num_tables, local, positions, sp, keys, vals);
}

// The pair build with the forward gather-reduce in one launch
// (tc_embed_forward_cast): the first `builders` workgroups build pairs, the
// others run the forward (as k_forward). Both read the index array; the pairs'
// stores stay out of the forward's chains of dependent loads, and their
// latency hides behind the forward's.
template <int LANES, int CHUNKS>
__global__ __launch_bounds__(kBlock) void k_forward_build(
    FwdSlice f, int32_t num_tables, bool local, SortPrep sp, int32_t builders,
    int32_t *__restrict__ keys, int32_t *__restrict__ vals) {
    if (int32_t(blockIdx.x) < builders) {  // uniform
        build_pairs(blockIdx.x, builders, f.ids, f.offsets, f.table_row_offset, f.bag_hi,
                    f.bags_per_table, num_tables, local, false, sp, keys, vals);
        return;
    }
    constexpr int64_t kWaves = kBlock / kWave;
    forward_bags<LANES, CHUNKS>(f, (int64_t(blockIdx.x) - builders) * kWaves + threadIdx.x / kWave,
                                (int64_t(gridDim.x) - builders) * kWaves);
}

// The tile of this workgroup of a pass: consecutive tiles on one XCD
// (workgroups go round-robin over the XCDs; any mapping gives the same
// results), so that the short runs that neighbouring tiles write side by side
// meet in one L2. Measured with 10-bit digits (us): 5.2M pairs 50.3 -> 35.6,
// 1.3M pairs 15.7 -> 14.2.
__device__ __forceinline__ int32_t tile_index() {
    return int32_t(blockIdx.x % kXcds * (gridDim.x / kXcds) + blockIdx.x / kXcds);
}
inline unsigned tile_grid(int32_t tiles) { return unsigned((tiles + kXcds - 1) / kXcds * kXcds); }

// Tile b: its record (table-local sort) or a plain slice of the n pairs
// (global sort: one segment, tiles 0 .. ceil(n/kSortTile)-1); s < 0 past the
// last tile.
__device__ __forceinline__ TileRec tile_of(int32_t b, int32_t tiles,
                                           const TileRec *__restrict__ recs, int32_t n) {
    TileRec r{0, 0, 0, 0, 0, 0, -1, 0};
    if (b >= tiles) return r;
    if (recs) return recs[b];
    r.next = tiles_of(n);
    if (b < r.next) {
        r.s = 0;
        r.p0 = b * kSortTile;
        r.p1 = n - r.p0 < kSortTile ? n : r.p0 + kSortTile;
    }
    return r;
}

// Lanes of a wavefront whose digit equals this lane's, among the lanes where
// ok holds. One ballot per digit bit; a lane's mismatches gather as lanes |
// (ballot ^ its own bit, spread), one three-input operation on each half.
__device__ __forceinline__ uint32_t add_mismatch(uint32_t lanes, uint32_t ballot, uint32_t mine) {
    return __builtin_amdgcn_bitop3_b32(ballot, mine, lanes, (0xf0 ^ 0xcc) | 0xaa);
}
template <int BITS>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool ok) {
    const uint64_t out = ~__ballot(ok);
    uint32_t lo = uint32_t(out), hi = uint32_t(out >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        uint32_t mine = uint32_t(__builtin_amdgcn_sbfe(int32_t(d), b, 1));
        asm("" : "+v"(mine));  // else the ballot tests d << (31 - b), one more instruction
        const uint64_t m = __ballot(mine != 0);
        lo = add_mismatch(lo, uint32_t(m), mine);
        hi = add_mismatch(hi, uint32_t(m >> 32), mine);
    }
    return ~(uint64_t(hi) << 32 | lo);
}
// Lanes of mask below this one.
__device__ __forceinline__ int32_t count_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0));
}

// The same with the digit width known only at run time (uniform branches).
__device__ __forceinline__ uint64_t match_digit_n(uint32_t d, bool ok, int bits) {
    const uint64_t out = ~__ballot(ok);
    uint32_t lo = uint32_t(out), hi = uint32_t(out >> 32);
#pragma unroll
    for (int b = 0; b < kMaxRadixBits; ++b) {
        if (b < bits) {
            uint32_t mine = uint32_t(__builtin_amdgcn_sbfe(int32_t(d), b, 1));
            asm("" : "+v"(mine));
            const uint64_t m = __ballot(mine != 0);
            lo = add_mismatch(lo, uint32_t(m), mine);
            hi = add_mismatch(hi, uint32_t(m >> 32), mine);
        }
    }
    return ~(uint64_t(hi) << 32 | lo);
}

// Whether every item of the wavefront where ok holds has the same digit (a
// run of one hot row, common in the later passes under skewed keys); *act
// gets those lanes. Two ballots, against one per digit bit for a match.
__device__ __forceinline__ bool all_same_digit(uint32_t d, bool ok, uint64_t *act) {
    const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
    *act = __ballot(ok);
    return __ballot(ok && d == d0) == *act;
}

// ---------------------------------------------------------------------------
// Digit counts of the tiles: a tile's row of `counts` holds digits 2t and
// 2t + 1 in one word (a count is at most kSortTile), and a row of `groups`
// the sums, one word per digit, over a full group of kGroupTiles tiles of one
// segment, tiles first + 16 g ... first + 16 g + 15. Groups are disjoint runs
// of 16 tiles, so (their first tile) / 16 names the row.

// 2a. per-tile digit histogram. Every item adds one to its wave's copy of the
// histogram (an LDS atomic; the order of the adds does not matter here),
// except that a wavefront whose items share one digit adds them all at once.
template <int BITS>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(
    const int32_t *__restrict__ keys, int32_t n, int shift, const TileRec *__restrict__ recs,
    int32_t tiles, uint32_t *__restrict__ counts, int32_t *__restrict__ groups) {
    constexpr int R = 1 << BITS;
    constexpr int kHistCopies = R > 1024 ? 2 : 4;
    __shared__ int32_t hist[kHistCopies][R];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    constexpr uint32_t mask = R - 1u;
    for (int i = tid; i < kHistCopies * R; i += kSortThreads) (&hist[0][0])[i] = 0;
    const int32_t b = tile_index();
    const TileRec tr = tile_of(b, tiles, recs, n);
    if (tr.s < 0) return;  // uniform: past the last tile
    const int32_t in_tile = tr.p1 - tr.p0;  // at least 1
    const int32_t base = w * kWaveSpan + lane;
    const int32_t *tile_keys = keys + tr.p0;
    int32_t key[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i)
        key[i] = tile_keys[uint32_t(min(base + i * kWave, in_tile - 1))];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const bool ok = base + i * kWave < in_tile;
        const uint32_t d = (uint32_t(key[i]) >> shift) & mask;
        uint64_t act;
        if (all_same_digit(d, ok, &act)) {
            if (lane == 0 && act) atomicAdd(&hist[w % kHistCopies][d], __popcll(act));
        } else if (ok) {
            atomicAdd(&hist[w % kHistCopies][d], 1);
        }
    }
    __syncthreads();
    const int32_t group = tr.first + (b - tr.first) / kGroupTiles * kGroupTiles;
    const bool full = group + kGroupTiles <= tr.next;
    for (int t = tid; t < R / 2; t += kSortThreads) {
        int32_t c[2] = {0, 0};
#pragma unroll
        for (int k = 0; k < kHistCopies; ++k) {
            c[0] += hist[k][2 * t];
            c[1] += hist[k][2 * t + 1];
        }
        counts[int64_t(b) * (R / 2) + t] = uint32_t(c[0]) | uint32_t(c[1]) << 16;
        if (full) {
            int32_t *row = groups + int64_t(group / kGroupTiles) * R + 2 * t;
            if (c[0]) atomicAdd(row, c[0]);
            if (c[1]) atomicAdd(row + 1, c[1]);
        }
    }
}

// 2b. where segments can be long (scan_groups): in those of more than
// kScanGroups full groups, the groups' digit sums become their inclusive
// prefixes over the groups, in place, so that the scatter reads two rows
// however long its segment is (all rows, read by every tile, cost the square of
// the segment's length). A workgroup takes 32 digits of every gridDim.y-th
// segment, in chunks of rows side by side. seg_first: the segments' first tiles
// and the last one's end; null for one segment of `tiles` tiles.
constexpr int kScanGroups = 8;
constexpr int kScanThreads = 1024;
constexpr int kScanDigits = 32, kScanChunks = kScanThreads / kScanDigits;
__global__ __launch_bounds__(kScanThreads) void k_radix_scan(
    int32_t *__restrict__ groups, int radix, const int32_t *__restrict__ seg_first,
    int32_t num_segs, int32_t tiles) {
    __shared__ int32_t sums[kScanChunks][kScanDigits];
    const int32_t d = threadIdx.x % kScanDigits, chunk = threadIdx.x / kScanDigits;
    const int32_t digit = blockIdx.x * kScanDigits + d;
    for (int32_t s = blockIdx.y; s < num_segs; s += gridDim.y) {  // uniform
        const int32_t first = seg_first ? seg_first[s] : 0;
        const int32_t full = ((seg_first ? seg_first[s + 1] : tiles) - first) / kGroupTiles;
        if (full <= kScanGroups) continue;
        int32_t *rows = groups + int64_t(first / kGroupTiles) * radix;
        const int32_t per = (full + kScanChunks - 1) / kScanChunks;
        const int32_t g0 = min(chunk * per, full), g1 = min(g0 + per, full);
        int32_t sum = 0;
        if (digit < radix)
#pragma unroll 8
            for (int32_t g = g0; g < g1; ++g) sum += rows[int64_t(g) * radix + digit];
        sums[chunk][d] = sum;
        __syncthreads();
        int32_t run = 0;
#pragma unroll
        for (int k = 0; k < kScanChunks; ++k) run += k < chunk ? sums[k][d] : 0;
        if (digit < radix)
#pragma unroll 8
            for (int32_t g = g0; g < g1; ++g) {
                run += rows[int64_t(g) * radix + digit];
                rows[int64_t(g) * radix + digit] = run;
            }
        __syncthreads();  // sums is written again
    }
}

// 2c. stable scatter of one tile. Where the tile's run of each digit goes
// comes straight from the counts: the segment's full groups (two rows of their
// prefixes if k_radix_scan has run, else all of them), and at most two partial
// groups tile by tile. Within a wavefront the lanes holding equal digits are
// found with ballots; each reads the wave's running count of its digit and the
// lowest of them then adds their number to it. The tile is then laid out in
// sorted order in LDS, keys and then values, and written back thread by thread
// in that order, so neighbouring threads write neighbouring addresses of the
// same digit run (coalesced stores instead of one scattered store per pair).
// With add_rowoff the keys leave with the segment's row offset added.
template <int BITS>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const int32_t *__restrict__ keys_in, const int32_t *__restrict__ vals_in,
    int32_t *__restrict__ keys_out, int32_t *__restrict__ vals_out, int32_t n, int shift,
    const TileRec *__restrict__ recs, int32_t tiles, const uint32_t *__restrict__ counts,
    const int32_t *__restrict__ groups, bool scanned, bool add_rowoff) {
    constexpr int R = 1 << BITS;
    constexpr int H = R / 2;  // words of two digits
    constexpr int WPT = H > kSortThreads ? H / kSortThreads : 1;  // consecutive ones per thread
    constexpr uint32_t mask = R - 1u;
    // wave w's running counts, two digits per word, then the tile-local starts
    // of its runs
    __shared__ uint32_t wcount[kSortWaves][H];
    __shared__ int32_t run_shift[R];  // global position - tile-local position
    __shared__ int32_t stage[kSortTile];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int32_t b = tile_index();
    const TileRec tr = tile_of(b, tiles, recs, n);
    if (tr.s < 0) return;  // uniform: past the last tile

    const int32_t in_tile = tr.p1 - tr.p0;  // at least 1
    const int32_t base = w * kWaveSpan + lane;
    const int32_t *tile_keys = keys_in + tr.p0, *tile_vals = vals_in + tr.p0;
    int32_t key[kItems], val[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) key[i] = tile_keys[uint32_t(min(base + i * kWave, in_tile - 1))];
    for (int i = tid; i < kSortWaves * H; i += kSortThreads) (&wcount[0][0])[i] = 0;
    // where this tile's runs of the thread's digits start
    int32_t digit_base[2 * WPT];
    {
        int32_t before[2 * WPT], total[2 * WPT], my = 0;
#pragma unroll
        for (int k = 0; k < 2 * WPT; ++k) before[k] = total[k] = 0;
        if (tid * WPT < H) {
            const int32_t full = (tr.next - tr.first) / kGroupTiles;  // full groups
            const int32_t mine = (b - tr.first) / kGroupTiles;
            const bool sums = scanned && full > kScanGroups;  // uniform
            if (sums) {  // inclusive prefixes already
                const int32_t *row = groups + int64_t(tr.first / kGroupTiles) * R + 2 * WPT * tid;
#pragma unroll
                for (int k = 0; k < 2 * WPT; ++k) {
                    before[k] = row[int64_t(max(mine - 1, 0)) * R + k];
                    total[k] = row[int64_t(full - 1) * R + k];
                    before[k] = mine > 0 ? before[k] : 0;
                }
            }
            for (int32_t g0 = 0; g0 < full && !sums; g0 += 8) {
                int32_t c[8][2 * WPT];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int32_t *row =
                        groups + int64_t((tr.first + min(g0 + i, full - 1) * kGroupTiles) /
                                         kGroupTiles) * R;
#pragma unroll
                    for (int k = 0; k < 2 * WPT; ++k) c[i][k] = row[uint32_t(2 * WPT * tid + k)];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int32_t any = g0 + i < full ? -1 : 0, in = g0 + i < mine ? -1 : 0;
#pragma unroll
                    for (int k = 0; k < 2 * WPT; ++k) {
                        total[k] += c[i][k] & any;
                        before[k] += c[i][k] & in;
                    }
                }
            }
            // the tiles of this one's group before it, and those past the
            // full groups (rows past them are read as the last one, and masked)
            const auto rows = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint32_t *>(counts), 0, -1, 0x00020000);
            auto add_tiles = [&](int32_t from, int32_t to, int32_t (&sum)[2 * WPT]) {
#pragma unroll
                for (int k = 0; k < WPT; ++k) {
                    uint32_t c[kGroupTiles];
#pragma unroll
                    for (int i = 0; i < kGroupTiles; ++i)
                        c[i] = __builtin_amdgcn_raw_buffer_load_b32(
                            rows, (tid * WPT + k) * 4,
                            uint32_t(min(from + i, tr.next - 1)) * uint32_t(H * 4), 0);
#pragma unroll
                    for (int i = 0; i < kGroupTiles; ++i) {
                        c[i] &= from + i < to ? ~0u : 0u;
                        sum[2 * k] += c[i] & 0xffff, sum[2 * k + 1] += c[i] >> 16;
                    }
                }
            };
            add_tiles(tr.first + mine * kGroupTiles, b, before);
            add_tiles(tr.first + full * kGroupTiles, tr.next, total);
        }
#pragma unroll
        for (int k = 0; k < 2 * WPT; ++k) my += total[k];
        int32_t tot;
        int32_t p = block_scan<kSortThreads>(my, &tot) + tr.pstart;
#pragma unroll
        for (int k = 0; k < 2 * WPT; ++k) {
            digit_base[k] = p + before[k];
            p += total[k];
        }
    }

    // every lane reads its digit's count before the lowest peer adds the item's
    // to it: a wave's LDS operations complete in order
    int32_t rank[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const bool ok = base + i * kWave < in_tile;
        const uint32_t d = (uint32_t(key[i]) >> shift) & mask;
        const uint64_t peers = match_digit<BITS>(d, ok);
        const int32_t below = count_below(peers);
        const int sh = 16 * (d & 1);
        uint32_t *count = &wcount[w][d >> 1];
        rank[i] = int32_t(__hip_atomic_load(count, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_WAVEFRONT) >> sh & 0xffff) + below;
        if (ok && below == 0) atomicAdd(count, uint32_t(__popcll(peers)) << sh);
    }
#pragma unroll
    for (int i = 0; i < kItems; ++i) val[i] = tile_vals[uint32_t(min(base + i * kWave, in_tile - 1))];
    __syncthreads();
    {
        // per digit: tile-local start of each wave's run (digit order, then
        // wave order) and the shift from tile-local to global positions
        const bool mine = tid * WPT < H;
        int32_t sum = 0;
        if (mine)
#pragma unroll
            for (int k = 0; k < WPT; ++k)
#pragma unroll
                for (int ww = 0; ww < kSortWaves; ++ww) {
                    const uint32_t c = wcount[ww][tid * WPT + k];
                    sum += (c & 0xffff) + (c >> 16);
                }
        int32_t tot;
        int32_t start = block_scan<kSortThreads>(sum, &tot);
        if (mine)
#pragma unroll
            for (int k = 0; k < WPT; ++k) {
                uint32_t c[kSortWaves];
                int32_t n0 = 0, n1 = 0;
#pragma unroll
                for (int ww = 0; ww < kSortWaves; ++ww) {
                    c[ww] = wcount[ww][tid * WPT + k];
                    n0 += c[ww] & 0xffff, n1 += c[ww] >> 16;
                }
                int32_t r0 = start, r1 = start + n0;
                start += n0 + n1;
                run_shift[2 * (tid * WPT + k)] = digit_base[2 * k] - r0;
                run_shift[2 * (tid * WPT + k) + 1] = digit_base[2 * k + 1] - r1;
#pragma unroll
                for (int ww = 0; ww < kSortWaves; ++ww) {
                    wcount[ww][tid * WPT + k] = uint32_t(r0) | uint32_t(r1) << 16;
                    r0 += c[ww] & 0xffff, r1 += c[ww] >> 16;
                }
            }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint32_t d = (uint32_t(key[i]) >> shift) & mask;
        rank[i] += wcount[w][d >> 1] >> (16 * (d & 1)) & 0xffff;
        if (base + i * kWave < in_tile) stage[rank[i]] = key[i];
    }
    __syncthreads();
    const int32_t koff = add_rowoff ? tr.rowoff : 0;
    int32_t pos[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int32_t lp = i * kSortThreads + tid;
        if (lp < in_tile) {
            const int32_t k = stage[lp];
            pos[i] = run_shift[(uint32_t(k) >> shift) & mask] + lp;
            keys_out[pos[i]] = k + koff;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; ++i)
        if (base + i * kWave < in_tile) stage[rank[i]] = val[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int32_t lp = i * kSortThreads + tid;
        if (lp < in_tile) vals_out[pos[i]] = stage[lp];
    }
}

// ---------------------------------------------------------------------------
// Segment heads of the sorted keys, whose tiles are plain slices of kSortTile:
// the wavefront's keys (position base + 64 i + lane) and, per i, the lanes
// whose key differs from its predecessor's.
struct Heads {
    int32_t key[kItems];
    uint64_t lanes[kItems];
    int32_t count;
};
__device__ __forceinline__ Heads segment_heads(const int32_t *__restrict__ keys, int64_t base,
                                               int64_t n) {
    Heads h;
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int64_t j = base + i * kWave + lane;
        h.key[i] = keys[j < n ? j : n - 1];
    }
    int32_t before = base > 0 && base <= n ? keys[base - 1] : 0;  // the key before item i
    h.count = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int64_t j = base + i * kWave + lane;
        // wave_shr:1, lane 0 taking the one before
        const int32_t prev =
            __builtin_amdgcn_update_dpp(before, h.key[i], 0x138, 0xf, 0xf, false);
        h.lanes[i] = __ballot(j < n && (j == 0 || h.key[i] != prev));
        h.count += __popcll(h.lanes[i]);
        before = __builtin_amdgcn_readlane(h.key[i], kWave - 1);
    }
    return h;
}

// casted_dst, unique_rows and seg_offsets of one wavefront's span, `run` heads
// coming before it.
__device__ __forceinline__ void write_segments(const Heads &h, int64_t base, int64_t n,
                                               int32_t run, int32_t *__restrict__ unique_rows,
                                               int32_t *__restrict__ seg_offsets,
                                               int32_t *__restrict__ casted_dst) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int64_t j = base + i * kWave + lane;
        const bool head = h.lanes[i] >> lane & 1u;
        const int32_t incl = run + count_below(h.lanes[i]) + head;
        if (j < n) {
            if (casted_dst) casted_dst[j] = incl - 1;
            if (head) {
                unique_rows[incl - 1] = h.key[i];
                seg_offsets[incl - 1] = int32_t(j);
            }
            if (j == n - 1) seg_offsets[incl] = int32_t(n);
        }
        run += __popcll(h.lanes[i]);
    }
}

// 3a. casted_dst (inclusive head count - 1), unique_rows and seg_offsets in one
// launch, up to kOneLaunchTiles tiles: a workgroup counts its tile's heads and
// publishes the count, then adds up the counts of the tiles before it, waiting
// for those still missing. Tiles are handed out in the order in which
// workgroups start (state[0]), and each publishes before it waits, so whatever
// a workgroup waits for comes from one that has started and waits for nothing
// first: every wait ends, however many workgroups are resident. A count is one
// word, state[1 + tile] = count + 1, zero until published (cleared by the pair
// build), stored and loaded at agent scope, so nothing else needs ordering.
// The workgroup of the last tile writes *num_unique.
// The tickets cost 12 ns each, one after another, so two launches take less
// time for many tiles. Measured (us in one launch and in two; tables of 1M x 64, the
// cast and the whole step): 20 tiles 29.1 and 30.4, 50.0 and 50.9; 64 tiles 32.0
// and 32.4, 76.2 and 76.4; 96 tiles 33.6 and 33.7, 97.3 and 97.0; 112 tiles 34.5
// and 34.3, 105.7 and 105.2; 160 tiles 41.7 and 40.0, 141.6 and 140.0; 320 tiles
// 56.7 and 52.4, 251 and 247.
constexpr int kOneLaunchTiles = 96;
__global__ __launch_bounds__(kSortThreads) void k_segments(
    const int32_t *__restrict__ keys, int64_t n, int32_t tiles, int32_t *__restrict__ state,
    int32_t *__restrict__ unique_rows, int32_t *__restrict__ seg_offsets,
    int32_t *__restrict__ casted_dst, int32_t *__restrict__ num_unique) {
    __shared__ int32_t wsum[kSortWaves];
    __shared__ int32_t s_tile;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    if (tid == 0)
        s_tile = __hip_atomic_fetch_add(&state[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int32_t b = __builtin_amdgcn_readfirstlane(s_tile);
    const int64_t base = int64_t(b) * kSortTile + int64_t(w) * kWaveSpan;
    const Heads h = segment_heads(keys, base, n);
    if (lane == 0) wsum[w] = h.count;
    __syncthreads();
    int32_t run = 0, total = 0;
#pragma unroll
    for (int ww = 0; ww < kSortWaves; ++ww) {
        if (ww < w) run += wsum[ww];
        total += wsum[ww];
    }
    if (tid == 0)
        __hip_atomic_store(&state[1 + b], total + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int32_t part = 0;
    for (int32_t t = tid; t < b; t += kSortThreads) {
        int32_t c;
        while ((c = __hip_atomic_load(&state[1 + t], __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT)) == 0)
            __builtin_amdgcn_s_sleep(1);
        part += c - 1;
    }
    int32_t before;
    block_scan<kSortThreads>(part, &before);
    run += before;
    if (b == tiles - 1 && tid == 0) *num_unique = before + total;
    write_segments(h, base, n, run, unique_rows, seg_offsets, casted_dst);
}

// 3b. the same in two launches, for more tiles: number of heads per tile,
__global__ __launch_bounds__(kSortThreads) void k_seg_count(const int32_t *__restrict__ keys,
                                                            int64_t n, int32_t tiles,
                                                            int32_t *__restrict__ tile_heads) {
    __shared__ int32_t wsum[kSortWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int32_t b = tile_index();
    if (b >= tiles) return;  // uniform
    const Heads h = segment_heads(keys, int64_t(b) * kSortTile + int64_t(w) * kWaveSpan, n);
    if (lane == 0) wsum[w] = h.count;
    __syncthreads();
    if (tid == 0) {
        int32_t s = 0;
#pragma unroll
        for (int ww = 0; ww < kSortWaves; ++ww) s += wsum[ww];
        tile_heads[b] = s;
    }
}

// then the writes, where each workgroup adds up the head counts of the tiles
// before it (a few loads per thread even for thousands of tiles, so no separate
// scan kernel); the last tile's writes *num_unique.
__global__ __launch_bounds__(kSortThreads) void k_seg_write(
    const int32_t *__restrict__ keys, int64_t n, int32_t tiles,
    const int32_t *__restrict__ tile_heads, int32_t *__restrict__ unique_rows,
    int32_t *__restrict__ seg_offsets, int32_t *__restrict__ casted_dst,
    int32_t *__restrict__ num_unique) {
    __shared__ int32_t wsum[kSortWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int32_t b = tile_index();
    if (b >= tiles) return;  // uniform
    const int64_t base = int64_t(b) * kSortTile + int64_t(w) * kWaveSpan;
    int32_t part = 0;
#pragma unroll 4
    for (int32_t t = tid; t < b; t += kSortThreads) part += tile_heads[t];
    const Heads h = segment_heads(keys, base, n);
    if (lane == 0) wsum[w] = h.count;
    int32_t before;
    block_scan<kSortThreads>(part, &before);  // (and wsum is written)
    int32_t run = before, total = before;
#pragma unroll
    for (int ww = 0; ww < kSortWaves; ++ww) {
        if (ww < w) run += wsum[ww];
        total += wsum[ww];
    }
    if (b == tiles - 1 && tid == 0) *num_unique = total;
    write_segments(h, base, n, run, unique_rows, seg_offsets, casted_dst);
}

// ---------------------------------------------------------------------------
// Small batches (at most kSmallPairs pairs): the whole cast in one workgroup
// of kSmallThreads threads, without the kernel chain: for a few thousand pairs
// the multi-kernel cast is all launch and memory latency. Same stable LSD
// passes and segment build, the pairs in registers and LDS: they are spread
// evenly over the wavefronts in whole trips of 64, wave w owning positions
// [w*span, (w+1)*span), walked 64 at a time. All of it is one CU's issue rate,
// so what counts is instructions per pair: bags come from one prefix sum over
// marks at the bags' first pairs (not a walk over the bags), ranks from four
// instructions a digit bit and one LDS read and add, a digit's counts of two
// digits per word, and prefixes from DPP adds. Measured (5120 pairs in 256
// bags, 17-bit keys, the forward beside it): 16.5 us, against 22.1 with a walk
// over the bags, shuffled ranks and a digit per word.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;  // 16
constexpr int kSmallItems = 8;
constexpr int kSmallPairs = kSmallThreads * kSmallItems;  // 8192
constexpr int kSmallWords = 1 << (kMaxRadixBits - 1);  // of two digits' counts per wave
static_assert(kSmallWords <= kSmallThreads, "one word per thread in the digit scan");

// With FL > 0 (tc_embed_forward_cast) the workgroups after the first run the
// forward gather-reduce beside it, FL lanes per bag: a small cast keeps one
// CU busy and leaves the others to the forward.
template <int FL>
__global__ __launch_bounds__(kSmallThreads) void k_cast_small(
    const int32_t *__restrict__ indices, const int32_t *__restrict__ bag_offsets,
    const int64_t *__restrict__ table_row_offset, int32_t num_tables, int32_t num_bags,
    int32_t bags_per_table, int32_t n, int bits, bool positions, int32_t *__restrict__ unique_rows,
    int32_t *__restrict__ seg_offsets, int32_t *__restrict__ casted_src,
    int32_t *__restrict__ casted_dst, int32_t *__restrict__ num_unique, FwdSlice fs) {
    // every item of a pass is in registers before the pass writes any
    // (barriers between), so one buffer each does
    __shared__ int32_t keys[kSmallPairs];
    __shared__ int32_t vals[kSmallPairs];
    __shared__ uint32_t wcount[kSmallWaves][kSmallWords];
    __shared__ int32_t wsum[kSmallWaves];
    if constexpr (FL > 0) {
        if (blockIdx.x > 0) {  // uniform: a forward workgroup
            constexpr int64_t kWaves = kSmallThreads / kWave;
            forward_bags<FL, 1>(fs, (int64_t(blockIdx.x) - 1) * kWaves + threadIdx.x / kWave,
                                (int64_t(gridDim.x) - 1) * kWaves);
            return;
        }
    }
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    // trips of 64 positions per wavefront (at most kSmallItems), so that
    // every wavefront holds a share of the pairs
    const int trips = (n + kSmallThreads - 1) / kSmallThreads;
    const int32_t base = w * trips * kWave + lane;
    int32_t key[kSmallItems], val[kSmallItems];

    // (src, dst) pairs from the bag-major CSR index. All loads that can be
    // are issued together; marks[j] then counts the bags that start at pair j,
    // and the sum of the marks up to j, less one, is j's bag (the last one
    // starting at or before it).
    {
        int32_t *marks = vals, *row_off = reinterpret_cast<int32_t *>(&wcount[0][0]);
        constexpr int kOffs = kSmallWaves * kSmallWords;
        int32_t start[kSmallItems];
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i) {
            const int32_t j = base + i * kWave, g = tid + i * kSmallThreads;
            key[i] = i < trips ? indices[min(j, n - 1)] : 0;
            start[i] = g < num_bags ? bag_offsets[g] : n;
        }
        for (int32_t t = tid; t < num_tables && t < kOffs; t += kSmallThreads)
            row_off[t] = int32_t(table_row_offset[t]);
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i) marks[tid + i * kSmallThreads] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i)
            if (start[i] < n) atomicAdd(&marks[start[i]], 1);
        for (uint32_t g = tid + kSmallPairs; g < uint32_t(num_bags); g += kSmallThreads) {
            const int32_t b = bag_offsets[g];  // bags without pairs beyond the first 8192
            if (b < n) atomicAdd(&marks[b], 1);
        }
        __syncthreads();
        int32_t run = 0;
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i) {
            if (i >= trips) continue;  // uniform
            const int32_t j = base + i * kWave;
            val[i] = wave_prefix(j < n ? marks[j] : 0) + run;
            run = __builtin_amdgcn_readlane(val[i], kWave - 1);
        }
        if (lane == 0) wsum[w] = run;
        __syncthreads();
        int32_t before = -1;
#pragma unroll
        for (int ww = 0; ww < kSmallWaves; ++ww)
            if (ww < w) before += wsum[ww];
        const float inv = 1.0f / float(bags_per_table);
        const bool small_ids = num_bags < (1 << 22);  // exact in fp32
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i) {
            if (i >= trips) continue;  // uniform
            const int32_t g = val[i] + before;
            int32_t t;
            if (small_ids) {  // the quotient is off by one at most
                t = int32_t(float(g) * inv);
                const int32_t r = g - t * bags_per_table;
                t += (r >= bags_per_table) - (r < 0);
            } else {
                t = g / bags_per_table;
            }
            key[i] += num_tables <= kOffs ? row_off[t] : int32_t(table_row_offset[t]);
            val[i] = positions ? base + i * kWave : g;
        }
        __syncthreads();  // the marks and row offsets have been read
    }

    const int passes = (bits + kMaxRadixBits - 1) / kMaxRadixBits;
    const int per_pass = (bits + passes - 1) / passes;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * per_pass;
        const int pbits = shift + per_pass <= bits ? per_pass : bits - shift;
        const uint32_t mask = (1u << pbits) - 1u;
        const int words = 1 << (pbits - 1);  // pbits >= 1
        for (int i = tid; i < kSmallWaves << (pbits - 1); i += kSmallThreads)
            wcount[i >> (pbits - 1)][i & (words - 1)] = 0;
        if (p > 0) {
#pragma unroll
            for (int i = 0; i < kSmallItems; ++i)
                if (i < trips) {
                    const int32_t j = min(base + i * kWave, n - 1);
                    key[i] = keys[j];
                    val[i] = vals[j];
                }
        }
        __syncthreads();
        // every lane reads its digit's count before the lowest peer adds the
        // item's to it: a wave's LDS operations complete in order
        int32_t rank[kSmallItems];
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i) {
            if (i >= trips) continue;  // uniform
            const bool ok = base + i * kWave < n;
            const uint32_t d = (uint32_t(key[i]) >> shift) & mask;
            const uint64_t peers = match_digit_n(d, ok, pbits);
            const int32_t below = count_below(peers);
            const int sh = 16 * (d & 1);
            uint32_t *count = &wcount[w][d >> 1];
            rank[i] = int32_t(__hip_atomic_load(count, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_WAVEFRONT) >> sh & 0xffff) +
                      below;
            if (ok && below == 0) atomicAdd(count, uint32_t(__popcll(peers)) << sh);
        }
        __syncthreads();
        {
            // digits 2 tid and 2 tid + 1: start of each wave's run, in digit
            // order then wave order
            uint32_t c[kSmallWaves];
            int32_t n0 = 0, n1 = 0;
#pragma unroll
            for (int ww = 0; ww < kSmallWaves; ++ww) {
                c[ww] = tid < words ? wcount[ww][tid] : 0;
                n0 += c[ww] & 0xffff, n1 += c[ww] >> 16;
            }
            int32_t tot;
            int32_t r0 = block_scan<kSmallThreads>(n0 + n1, &tot), r1 = r0 + n0;
            if (tid < words) {
#pragma unroll
                for (int ww = 0; ww < kSmallWaves; ++ww) {
                    wcount[ww][tid] = uint32_t(r0) | uint32_t(r1) << 16;
                    r0 += c[ww] & 0xffff, r1 += c[ww] >> 16;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i) {
            if (i < trips && base + i * kWave < n) {
                const uint32_t d = (uint32_t(key[i]) >> shift) & mask;
                const int32_t lp = int32_t(wcount[w][d >> 1] >> (16 * (d & 1)) & 0xffff) + rank[i];
                keys[lp] = key[i];
                vals[lp] = val[i];
            }
        }
        __syncthreads();
    }

    // segment build, on the sorted positions in the same trips
    uint64_t heads[kSmallItems];
    int32_t prev = base >= kWave ? keys[min(base - lane, n) - 1] : 0;  // the key before item i
    int32_t count = 0;
#pragma unroll
    for (int i = 0; i < kSmallItems; ++i) {
        if (i >= trips) continue;  // uniform
        const int32_t j = base + i * kWave;
        key[i] = keys[min(j, n - 1)];
        val[i] = vals[min(j, n - 1)];
        // wave_shr:1, lane 0 taking the one before
        const int32_t before = __builtin_amdgcn_update_dpp(prev, key[i], 0x138, 0xf, 0xf, false);
        heads[i] = __ballot(j < n && (j == 0 || key[i] != before));
        count += __popcll(heads[i]);
        prev = __builtin_amdgcn_readlane(key[i], kWave - 1);
    }
    if (lane == 0) wsum[w] = count;
    __syncthreads();
    int32_t run = 0, total = 0;
#pragma unroll
    for (int ww = 0; ww < kSmallWaves; ++ww) {
        if (ww < w) run += wsum[ww];
        total += wsum[ww];
    }
#pragma unroll
    for (int i = 0; i < kSmallItems; ++i) {
        if (i >= trips) continue;  // uniform
        const int32_t j = base + i * kWave;
        if (j < n) {
            const bool head = heads[i] >> lane & 1u;
            const int32_t incl = run + count_below(heads[i]) + head;
            casted_src[j] = val[i];
            if (casted_dst) casted_dst[j] = incl - 1;
            if (head) {
                unique_rows[incl - 1] = key[i];
                seg_offsets[incl - 1] = j;
            }
        }
        run += __popcll(heads[i]);
    }
    if (tid == 0) {
        seg_offsets[total] = n;
        *num_unique = total;
    }
}

// No pairs: zero segments, seg_offsets[0] = 0.
__global__ void k_cast_empty(int32_t *seg_offsets, int32_t *num_unique) {
    if (threadIdx.x == 0) {
        seg_offsets[0] = 0;
        *num_unique = 0;
    }
}

// One LSD pass over `bits` (1..kMaxRadixBits) digit bits starting at `shift`.
tc_status launch_radix_pass(int bits, const int32_t *kin, const int32_t *vin, int32_t *kout,
                            int32_t *vout, int32_t n, int shift, const TileRec *recs,
                            uint32_t *counts, int32_t *groups, int32_t tiles, bool scan,
                            const int32_t *seg_first, int32_t num_segs, bool last,
                            hipStream_t stream) {
#define TC_PASS_CASE(B)                                                                      \
    case B:                                                                                  \
        k_radix_hist<B><<<tile_grid(tiles), kSortThreads, 0, stream>>>(                      \
            kin, n, shift, recs, tiles, counts, groups);                                     \
        if (check_launch("k_radix_hist") != TC_OK) return TC_ERR_HIP;                        \
        if (scan) {                                                                          \
            k_radix_scan<<<dim3(((1 << B) + kScanDigits - 1) / kScanDigits,                  \
                                num_segs < 8 ? num_segs : 8),                                \
                           kScanThreads, 0, stream>>>(groups, 1 << B, seg_first, num_segs,   \
                                                      (n - 1) / kSortTile + 1);              \
            if (check_launch("k_radix_scan") != TC_OK) return TC_ERR_HIP;                    \
        }                                                                                    \
        k_radix_scatter<B><<<tile_grid(tiles), kSortThreads, 0, stream>>>(                   \
            kin, vin, kout, vout, n, shift, recs, tiles, counts, groups, scan, last);        \
        return check_launch("k_radix_scatter");
    switch (bits) {
        TC_PASS_CASE(1)
        TC_PASS_CASE(2)
        TC_PASS_CASE(3)
        TC_PASS_CASE(4)
        TC_PASS_CASE(5)
        TC_PASS_CASE(6)
        TC_PASS_CASE(7)
        TC_PASS_CASE(8)
        TC_PASS_CASE(9)
        TC_PASS_CASE(10)
        TC_PASS_CASE(11)
        default:
            break;
    }
#undef TC_PASS_CASE
    set_error("no radix pass for %d bits", bits);
    return TC_ERR_UNSUPPORTED;
}
static_assert(kMaxRadixBits == 11, "launch_radix_pass instantiates 1..11 bits");

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Sort segments available to a call with num_tables tables.
inline int32_t seg_capacity(int32_t num_tables) {
    return num_tables >= 1 && num_tables <= kMaxSegTables ? num_tables : 1;
}

struct CastPlan {
    int64_t sort_tiles;  // tile slots of a radix pass (all segments)
    int64_t seg_tiles;   // tiles of the segment build (plain tiles of kSortTile)
    size_t off_ka, off_va, off_kb, off_vb, off_counts, counts_bytes, off_state, off_recs, bytes;
};

inline CastPlan cast_plan(int64_t n, int32_t num_tables) {
    CastPlan p{};
    const int32_t nseg = seg_capacity(num_tables);
    p.seg_tiles = (n + kSortTile - 1) / kSortTile;
    p.sort_tiles = p.seg_tiles + nseg;  // each segment adds at most one short tile
    const size_t arr = align_up(size_t(n) * 4);
    const int64_t slots = (n + 2047) / 2048 + nseg;  // a KB of counts each
    size_t o = 0;
    p.off_ka = o; o += arr;
    p.off_va = o; o += arr;
    p.off_kb = o; o += arr;
    p.off_vb = o; o += arr;
    // group sums, and digit counts where the batch's own arrays are too small
    // for them (sort_digits)
    p.counts_bytes = align_up(size_t(slots) * 1024) + 1024;
    p.off_counts = o; o += p.counts_bytes;
    p.off_state = o; o += align_up(size_t(slots - nseg) * 4);
    p.off_recs = o; o += align_up(size_t(slots) * sizeof(TileRec));
    p.bytes = o;
    return p;
}

// The passes over `bits` key bits. A pass has counts of a word per two digits
// and tile, which go where its values are not: the last pass, which writes the
// values to the caller's array, leaves one of the plan's two value arrays
// free, and the passes before it the caller's. When the batch is too small for
// that (n words), as with many more tables than full tiles, they go into the
// plan's own area. The group sums, one set per pass, are there in any case.
// The fewest passes that fit are taken; those of 1 bit always do.
//
// Digits of kMaxRadixBits bits are for up to kWideTiles tiles, as many as the
// scatter's workgroups of that width that are resident at once (two per CU): a
// second round of them takes longer than a third pass of 7 or 8 bits, which keys
// of 21 and 22 bits have instead. Measured (us of the cast, in two and in three
// passes; pairs): one table of 4M rows 43.6 and 44.7 (0.4M), 60.0 and 56.6
// (1.0M), 88.0 and 72.4 (2.0M), 104 and 88.5 (2.2M), 158 and 120 (5M), 2680 and
// 2000 (100M); of 2M rows 54.4 and 55.2 (1.0M), 77.2 and 71.2 (2.0M), 92.0 and
// 86.5 (2.2M); 16 ragged tables of up to 2M, Zipf lookups: 57.4 and 60.6 (1.4M).
constexpr int64_t kWideTiles = 512;
struct SortDigits {
    int passes, per_pass;
    bool own_counts;      // counts in the plan's area
    size_t counts_bytes;  // there, before the group sums
    size_t group_words;   // of one pass
};
inline SortDigits sort_digits(const CastPlan &p, int64_t n, int bits) {
    SortDigits d{};
    const int most = p.seg_tiles <= kWideTiles ? kMaxRadixBits : kMaxRadixBits - 1;
    for (d.passes = (bits + most - 1) / most;; ++d.passes) {
        d.per_pass = (bits + d.passes - 1) / d.passes;
        const size_t radix = size_t(1) << d.per_pass;
        const size_t counts = size_t(p.sort_tiles) * radix * 2;
        d.own_counts = counts > size_t(n) * 4;
        d.counts_bytes = d.own_counts ? align_up(counts) : 0;
        d.group_words = size_t(p.sort_tiles / kGroupTiles) * radix;
        if (d.per_pass == 1 || d.counts_bytes + d.passes * d.group_words * 4 <= p.counts_bytes)
            return d;
    }
}

// Whether k_radix_scan runs in a sort of `tiles` tiles and num_segs segments,
// whose own lengths only the device knows. Its launch takes 2.2 us a pass. Against
// that stand the rows of group sums that the tiles read without it: tiles x
// (groups of their segment). It runs from 2^14 rows at the mean length of a
// segment, and from 2^17 (5.9M pairs) if one segment could have all pairs.
// Measured (us of the cast, without and with; pairs): one table of 4M rows 72.5
// and 76.7 (2.0M), 91.7 and 88.9 (2.2M), 149.5 and 120.3 (5M), 2239 and 684
// (35M), 15500 and 2000 (100M); 4 tables of 2M 82.5 and 86.9 (3M), 119.2 and
// 117.2 (5M); 32 tables of 1M 119.8 and 124.3 (5.2M), 434 and 428 (20M). One of
// many tables having nearly all of up to 5.9M pairs is what the rule leaves: at
// most 170 and 130.
inline bool scan_groups(int64_t tiles, int32_t num_segs) {
    const int64_t rows = tiles * (tiles / kGroupTiles);
    return rows / num_segs >= 1 << 14 || rows >= 1 << 17;
}

// bits needed for keys in [0, rows)
inline int key_bits(int64_t rows) {
    int b = 0;
    while (b < 31 && (int64_t(1) << b) < rows) ++b;
    return b < 1 ? 1 : b;  // at least one pass, so the values are always moved
}

}  // namespace
}  // namespace tc

using namespace tc;

extern "C" size_t tc_cast_workspace_bytes(int64_t num_pairs, int64_t total_rows,
                                          int32_t num_tables) {
    (void)total_rows;
    if (num_pairs < 0) return 0;
    return cast_plan(num_pairs, num_tables).bytes;
}

namespace {
// The forward over all bags of fwd as its own kernel.
tc_status forward_alone(const FwdSlice &fwd, hipStream_t stream) {
    return launch_forward(fwd.W, fwd.dim, fwd.ids, fwd.offsets, fwd.table_row_offset,
                          fwd.bags_per_table, fwd.bag_hi, fwd.out, stream);
}

// The sort and segment build behind tc_cast_index (values = bag ids) and
// tc_argsort_rows (values = pair positions). `what` names the entry point in
// error messages. With fwd (tc_embed_forward_cast; values = bag ids), the
// forward gather-reduce of all fwd->bag_hi bags runs too: beside the
// single-workgroup cast (or, for rows of several chunks a lane, before it), or
// in the key-building kernel of the radix sort.
tc_status cast_impl(const char *what, bool positions, const int64_t *table_row_offset,
                    int32_t num_tables, int32_t bags_per_table, int64_t total_rows,
                    int64_t max_table_rows, const int32_t *indices, const int32_t *bag_offsets,
                    int64_t num_pairs, int32_t *unique_rows, int32_t *seg_offsets,
                    int32_t *casted_src, int32_t *casted_dst, int32_t *num_unique,
                    void *workspace, size_t workspace_bytes, hipStream_t stream,
                    const FwdSlice *fwd = nullptr) {
    TC_REQUIRE(num_tables >= 0 && bags_per_table >= 0 && total_rows >= 0 && num_pairs >= 0 &&
                   max_table_rows >= 0,
               TC_ERR_INVALID_ARG, "%s: negative size", what);
    TC_REQUIRE(total_rows < (int64_t(1) << 31) && num_pairs < (int64_t(1) << 31),
               TC_ERR_INVALID_ARG, "%s: total_rows and num_pairs must be below 2^31", what);
    const int64_t num_bags = int64_t(num_tables) * bags_per_table;
    TC_REQUIRE(num_bags < (int64_t(1) << 31), TC_ERR_INVALID_ARG,
               "%s: more than 2^31-1 bags", what);
    TC_REQUIRE(seg_offsets && num_unique, TC_ERR_INVALID_ARG, "%s: null pointer", what);
    if (num_pairs == 0) {
        if (fwd) {
            const tc_status st = forward_alone(*fwd, stream);
            if (st != TC_OK) return st;
        }
        k_cast_empty<<<1, kWave, 0, stream>>>(seg_offsets, num_unique);
        return check_launch("k_cast_empty");
    }
    TC_REQUIRE(num_bags > 0 && total_rows > 0, TC_ERR_INVALID_ARG,
               "%s: pairs without bags or rows", what);
    TC_REQUIRE(table_row_offset && indices && bag_offsets && unique_rows && casted_src,
               TC_ERR_INVALID_ARG, "%s: null pointer", what);
    const CastPlan plan = cast_plan(num_pairs, num_tables);
    TC_REQUIRE(workspace && workspace_bytes >= plan.bytes, TC_ERR_WORKSPACE,
               "%s: workspace of %zu bytes, %zu needed", what, workspace_bytes, plan.bytes);
    TC_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) == 0, TC_ERR_WORKSPACE,
               "%s: workspace must be 256-byte aligned", what);

    const RowShape shape = row_shape(fwd ? int(fwd->dim) : 4);
    if (num_pairs <= kSmallPairs) {
        // one workgroup in LDS (the workspace is not touched); the forward's
        // workgroups, if any, run beside it (one per CU at most: each holds
        // the kernel's LDS), one bag per lane group
        // (rows of several chunks a lane have the forward first, as its own
        // kernel: it needs more registers than 1024 threads have)
        const int fl = fwd && shape.chunks == 1 ? shape.lanes : 0;
        if (fwd && fl == 0) {
            const tc_status st = forward_alone(*fwd, stream);
            if (st != TC_OK) return st;
        }
        unsigned fb = 0;
        if (fl) {
            const int64_t per_block = int64_t(kSmallThreads / kWave) * (kWave / fl);
            fb = grid_for(num_bags, per_block, device_cus() > 1 ? device_cus() - 1 : 1);
        }
        const FwdSlice fs = fl ? *fwd : FwdSlice{};
#define TC_SMALL(FL)                                                                         \
    k_cast_small<FL><<<1 + fb, kSmallThreads, 0, stream>>>(                                  \
        indices, bag_offsets, table_row_offset, num_tables, int32_t(num_bags), bags_per_table, \
        int32_t(num_pairs), key_bits(total_rows), positions, unique_rows, seg_offsets,        \
        casted_src, casted_dst, num_unique, fs)
        if (fl == 1) TC_SMALL(1);
        else if (fl == 2) TC_SMALL(2);
        else if (fl == 4) TC_SMALL(4);
        else if (fl == 8) TC_SMALL(8);
        else if (fl == 16) TC_SMALL(16);
        else if (fl == 32) TC_SMALL(32);
        else if (fl == 64) TC_SMALL(64);
        else TC_SMALL(0);
#undef TC_SMALL
        return check_launch("k_cast_small");
    }
    // Table-local keys when the tables are known to be small enough to save
    // key bits; otherwise one segment of global rows.
    const int global_bits = key_bits(total_rows);
    const bool local = max_table_rows > 0 && num_tables <= kMaxSegTables &&
                       key_bits(max_table_rows) < global_bits;
    const int bits = local ? key_bits(max_table_rows) : global_bits;

    char *ws = static_cast<char *>(workspace);
    int32_t *ka = reinterpret_cast<int32_t *>(ws + plan.off_ka);
    int32_t *va = reinterpret_cast<int32_t *>(ws + plan.off_va);
    int32_t *kb = reinterpret_cast<int32_t *>(ws + plan.off_kb);
    int32_t *vb = reinterpret_cast<int32_t *>(ws + plan.off_vb);
    int32_t *state = reinterpret_cast<int32_t *>(ws + plan.off_state);
    TileRec *recs = local ? reinterpret_cast<TileRec *>(ws + plan.off_recs) : nullptr;
    const int32_t sort_tiles = int32_t(plan.sort_tiles);
    const int32_t seg_tiles = int32_t(plan.seg_tiles);

    const SortDigits digits = sort_digits(plan, num_pairs, bits);
    const int passes = digits.passes, per_pass = digits.per_pass;
    int32_t *groups = reinterpret_cast<int32_t *>(ws + plan.off_counts + digits.counts_bytes);
    const int32_t num_segs = local ? num_tables : 1;
    const bool scan = scan_groups(plan.seg_tiles, num_segs);
    // behind the records: their area has room for one per 2048 pairs, twice the
    // tiles, and a scanned sort has 512 tiles or more
    static_assert(511 * sizeof(TileRec) >= (kMaxSegTables + 1) * sizeof(int32_t));
    int32_t *seg_first = scan && local ? reinterpret_cast<int32_t *>(recs + sort_tiles) : nullptr;
    const SortPrep prep{recs,   sort_tiles, groups,   int64_t(digits.group_words) * passes,
                        state,  plan.seg_tiles <= kOneLaunchTiles ? plan.seg_tiles + 1 : 0,
                        seg_first};
    if (fwd) {
        // the pair build's workgroups, then the forward's, in one launch
        const int64_t per_block = int64_t(kBlock / kWave) * (kWave / shape.lanes);
        const unsigned builders = build_grid(num_bags);
        const unsigned grid =
            builders + grid_for(num_bags, per_block, int64_t(device_cus()) * 32);
#define TC_FWD_BUILD(L, C)                                                                   \
    if (shape.lanes == L && shape.chunks == C)                                               \
        k_forward_build<L, C><<<grid, kBlock, 0, stream>>>(*fwd, num_tables, local, prep,     \
                                                           int32_t(builders), ka, va);
        TC_FWD_BUILD(1, 1)
        TC_FWD_BUILD(2, 1)
        TC_FWD_BUILD(4, 1)
        TC_FWD_BUILD(8, 1)
        TC_FWD_BUILD(16, 1)
        TC_FWD_BUILD(32, 1)
        TC_FWD_BUILD(64, 1)
        TC_FWD_BUILD(64, 2)
        TC_FWD_BUILD(64, 3)
        TC_FWD_BUILD(64, 4)
#undef TC_FWD_BUILD
        tc_status st = check_launch("k_forward_build");
        if (st != TC_OK) return st;
    } else {
        k_build_keys<<<build_grid(num_bags), kBlock, 0, stream>>>(
            indices, bag_offsets, table_row_offset, num_bags, bags_per_table, num_tables, local,
            positions, prep, ka, va);
        tc_status st = check_launch("k_build_keys");
        if (st != TC_OK) return st;
    }
    int32_t *kin = ka, *vin = va, *kout = kb, *vout = vb;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * per_pass;
        const int pb = (shift + per_pass <= bits) ? per_pass : bits - shift;
        const bool last = p == passes - 1;
        int32_t *vdst = last ? casted_src : vout;
        void *counts = digits.own_counts ? ws + plan.off_counts
                       : last            ? static_cast<void *>(vout)
                                         : static_cast<void *>(casted_src);
        tc_status st = launch_radix_pass(pb, kin, vin, kout, vdst, int32_t(num_pairs), shift,
                                         recs, static_cast<uint32_t *>(counts),
                                         groups + p * digits.group_words, sort_tiles, scan,
                                         seg_first, num_segs, last, stream);
        if (st != TC_OK) return st;
        // next pass reads what this one wrote
        int32_t *tk = kin, *tv = vin;
        kin = kout;
        vin = vout;
        kout = tk;
        vout = tv;
    }
    const int32_t *sorted_keys = kin;

    if (seg_tiles <= kOneLaunchTiles) {
        k_segments<<<seg_tiles, kSortThreads, 0, stream>>>(sorted_keys, num_pairs, seg_tiles,
                                                           state, unique_rows, seg_offsets,
                                                           casted_dst, num_unique);
        return check_launch("k_segments");
    }
    k_seg_count<<<tile_grid(seg_tiles), kSortThreads, 0, stream>>>(sorted_keys, num_pairs,
                                                                   seg_tiles, state);
    tc_status st = check_launch("k_seg_count");
    if (st != TC_OK) return st;
    k_seg_write<<<tile_grid(seg_tiles), kSortThreads, 0, stream>>>(
        sorted_keys, num_pairs, seg_tiles, state, unique_rows, seg_offsets, casted_dst,
        num_unique);
    return check_launch("k_seg_write");
}
}  // namespace

extern "C" tc_status tc_cast_index(const int64_t *table_row_offset, int32_t num_tables,
                                   int32_t bags_per_table, int64_t total_rows,
                                   int64_t max_table_rows, const int32_t *indices,
                                   const int32_t *bag_offsets, int64_t num_pairs,
                                   int32_t *unique_rows, int32_t *seg_offsets,
                                   int32_t *casted_src, int32_t *casted_dst, int32_t *num_unique,
                                   void *workspace, size_t workspace_bytes, hipStream_t stream) {
    clear_error();
    return cast_impl("tc_cast_index", false, table_row_offset, num_tables, bags_per_table,
                     total_rows, max_table_rows, indices, bag_offsets, num_pairs, unique_rows,
                     seg_offsets, casted_src, casted_dst, num_unique, workspace,
                     workspace_bytes, stream);
}

extern "C" tc_status tc_embed_forward_cast(
    const float *W, int64_t total_rows, int32_t dim, const int64_t *table_row_offset,
    int32_t num_tables, int32_t bags_per_table, int64_t max_table_rows, const int32_t *indices,
    const int32_t *bag_offsets, int64_t num_pairs, float *out, int32_t *unique_rows,
    int32_t *seg_offsets, int32_t *casted_src, int32_t *casted_dst, int32_t *num_unique,
    void *workspace, size_t workspace_bytes, hipStream_t stream) {
    clear_error();
    const char *what = "tc_embed_forward_cast";
    TC_REQUIRE(num_tables >= 0 && bags_per_table >= 0, TC_ERR_INVALID_ARG, "%s: negative size",
               what);
    TC_REQUIRE(dim > 0 && dim % 4 == 0 && dim <= kMaxDim, TC_ERR_UNSUPPORTED,
               "%s: dim %d must be a multiple of 4 in [4, %d]", what, dim, kMaxDim);
    const int64_t num_bags = int64_t(num_tables) * bags_per_table;
    if (num_bags > 0) {
        TC_REQUIRE(W && out && table_row_offset && bag_offsets, TC_ERR_INVALID_ARG,
                   "%s: null pointer", what);
        TC_REQUIRE(aligned16(W) && aligned16(out), TC_ERR_UNSUPPORTED,
                   "%s: W and out must be 16-byte aligned", what);
    }
    // the cast checks the rest before anything is launched
    const FwdSlice f{W, indices, bag_offsets, table_row_offset, out, 0, num_bags, dim,
                     bags_per_table};
    return cast_impl(what, false, table_row_offset, num_tables, bags_per_table, total_rows,
                     max_table_rows, indices, bag_offsets, num_pairs, unique_rows, seg_offsets,
                     casted_src, casted_dst, num_unique, workspace, workspace_bytes, stream,
                     num_bags > 0 ? &f : nullptr);
}

extern "C" tc_status tc_argsort_rows(const int64_t *table_row_offset, int32_t num_tables,
                                     int32_t bags_per_table, int64_t total_rows,
                                     int64_t max_table_rows, const int32_t *indices,
                                     const int32_t *bag_offsets, int64_t num_pairs,
                                     int32_t *unique_rows, int32_t *seg_offsets,
                                     int32_t *sorted_pos, int32_t *num_unique, void *workspace,
                                     size_t workspace_bytes, hipStream_t stream) {
    clear_error();
    return cast_impl("tc_argsort_rows", true, table_row_offset, num_tables, bags_per_table,
                     total_rows, max_table_rows, indices, bag_offsets, num_pairs, unique_rows,
                     seg_offsets, sorted_pos, nullptr, num_unique, workspace, workspace_bytes,
                     stream);
}
