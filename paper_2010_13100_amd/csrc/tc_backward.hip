// Backward: the casted gradient gather-reduce (Algorithm 3) on CDNA4.
//
// coal_grad[u] is the sum of grad_out rows casted_src[j] over the segment j
// in [seg_offsets[u], seg_offsets[u+1]). Segment lengths follow the index
// skew: under Zipf lookups a few table rows own tens of thousands of pairs.
// Short ones are summed by a lane group, long ones (kListLong pairs with a
// workspace, kLongSegment without) as chains of their own.
//
// With a workspace (two launches):
//  k_backward_list   scans the segment offsets and lists the long segments,
//                    and the pieces of the split ones.
//  k_backward_rows   its first workgroups run the listed chains, one per
//                    wavefront or, the longest and the pieces, per workgroup;
//                    the others run the short segments, a lane group each,
//                    exactly as the forward. The chains are bound by the
//                    latency of their gathers and the short segments by
//                    bandwidth, so they overlap.
// Without one, every segment is one chain of any length, and the longest
// sets the time:
//  k_backward_short  the short segments.
//  k_backward_long   workgroups scan ranges of segments for long ones and run
//                    each with four producer wavefronts that gather the rows
//                    into a ring of LDS buffers with 16-byte loads and one
//                    consumer wavefront (one column per lane) that runs the
//                    ordered adds out of LDS, so the chain never waits behind
//                    load issue.
//
// Summation order. Without a workspace every segment is one ordered chain
// from +0, the sequential definition bit for bit. With a workspace that
// covers them, segments of kSplitPairs pairs or more are cut into n =
// min(kMaxPieces, len / kPieceMin) pieces of consecutive pairs; each piece is
// an ordered chain from +0 of its own, whose last wavefront stores the piece
// sum, and the one that finishes a segment's last piece (an agent-scope
// counter per segment and part) adds the n piece sums in piece order from
// +0. The order is fixed by the segment's length alone, so results do not
// depend on scheduling and repeat bit for bit; the chain of the hottest row
// shrinks from len to len / n.
//
// Fused with the update (tc_embed_backward_update), the owner of coalesced
// row u applies the optimizer step to table row unique_rows[u] straight from
// its registers (tc_optim.h, the arithmetic of tc_sparse_update), so the
// coalesced rows need not go through HBM; unique rows are distinct, so every
// table row still has a single writer.
#include <type_traits>

#include "tc_group_sum.h"
#include "tc_optim.h"

namespace tc {
namespace {

// Without a workspace segments at least this long are long; also the fewest
// pairs that need one.
constexpr int kLongSegment = 80;
// With a workspace: a lane group takes 8 rows of a segment per round trip and
// holds up the wavefront's other groups meanwhile, a chain takes 40 at a time
// but costs a wavefront's start and end. Measured (us, k_backward_rows) at 80,
// 64, 48 and 41: 8 x 1M x 64 55.4, 51.5, 49.2, 49.4; 8 x 5M x 128 121.9, 118.8,
// 117.0, 117.1; 4 x 100k x 512 47.4, 46.8, 43.8, 42.5; 8 x 300k x 128 43.6,
// 42.0, 42.3, 43.4; 13 ragged x 16 19.6, 18.3, 16.1, 15.6.
constexpr int kListLong = 48;
static_assert(kListLong <= kLongSegment, "a workspace covers its long segments");
// A long-segment workgroup: one consumer and kProducers producer wavefronts.
constexpr int kProducers = 4;
constexpr int kLongThreads = (1 + kProducers) * kWave;
// Columns per workgroup (one per consumer lane) and rows per LDS buffer.
constexpr int kPartCols = kWave;
constexpr int kChunkRows = 64;
constexpr int kBuffers = 3;
// A producer load instruction brings kRowsPerLoad rows of the part: 16
// lanes x 16 bytes per row.
constexpr int kLanesPerRow = kPartCols / 4;
constexpr int kRowsPerLoad = kWave / kLanesPerRow;  // 4
constexpr int kLoadsPerChunk = kChunkRows / kRowsPerLoad;  // 16
// Chunks whose row loads (kAhead) and id loads (kIdAhead) a producer keeps in
// flight; the producer code is unrolled over kPeriod chunks so that every ring
// slot is a fixed register.
constexpr int kAhead = 3;
constexpr int kIdAhead = 6;
constexpr int kPeriod = 6;
static_assert(kPeriod % kAhead == 0 && kPeriod % kIdAhead == 0 && kPeriod % kBuffers == 0,
              "ring periods must divide kPeriod");
// Ranges of segments scanned by the blocks of the long kernel (per part).
constexpr int kLongRanges = 1024;
// Summing in pieces (with a workspace): segments of at least kSplitPairs
// pairs, pieces of at least kPieceMin pairs, at most kMaxPieces of them.
constexpr int32_t kSplitPairs = TC_BACKWARD_SPLIT_PAIRS;
constexpr int32_t kPieceMin = 1024;
constexpr int32_t kMaxPieces = 32;
// Long segments of at least kBigLong pairs, and pieces, are chains of a whole
// workgroup (about 5 ns per row), which end soon enough not to outlast the
// short segments; the shorter ones of a wavefront (17 ns), which holds a
// quarter of the workgroup's slots while the chain starts and ends.
constexpr int32_t kBigLong = 512;
static_assert(kPieceMin >= kBigLong && kBigLong > kListLong, "list entries");
static_assert(kSplitPairs >= 2 * kPieceMin && kPieceMin >= kLongSegment, "piece sizes");
// Workgroups of k_backward_list: kListBlocks, or kListBlocksSmall when the
// workspace is too small to hold more heads.
constexpr int kListBlocks = 256;
constexpr int kListBlocksSmall = 16;
// Cost of a segment outside the chains, in pairs of a chain (k_backward_rows).
constexpr float kSegmentCost = 12.f;
// Cost of a chain beyond its pairs.
constexpr float kChainCost = 64.f;

// The backward workspace, written by k_backward_list and read by
// k_backward_rows. A long segment [beg, beg + len) is covered when beg + len
// <= cap_pairs and split when also len >= kSplitPairs.
// Workgroup b of the list kernel scans a range of consecutive segments, that
// is the pairs [P0, P1), and keeps its entries in slots of its own, with no
// counter shared between workgroups to clear first: an entry of big[] stands
// for at least kBigLong pairs, so [P0 / kBigLong, P1 / kBigLong) holds all of
// them, and one of longs[] for at least kListLong.
//   heads[b]   {entries in big[], entries in longs[], P0, pairs of its long
//              segments}, zeros past the workgroups launched
//   big[k]     {u, q}: piece q of split segment u, or with q < 0 a segment of
//              at least kBigLong pairs that is not split
//   longs[k]   {u, beg}: a shorter long segment
// Split segments are disjoint intervals of at least kSplitPairs pairs, and
// pieces of at least kPieceMin pairs, so beg / kSplitPairs and (first pair of
// the piece) / kPieceMin name them without collisions:
//   seg_done[(beg / kSplitPairs) * parts + p]  pieces of part p finished
//   partial[(first pair / kPieceMin) * dim + c]  piece sums
struct SplitWs {
    int4 *heads;
    int2 *big;
    int2 *longs;
    int32_t *seg_done;
    float *partial;
    int64_t cap_pairs;  // 0: no workspace
    int32_t list_blocks;
    int32_t parts;
    int32_t *turns;  // kXcds counters, kTurnStride apart; null if there is no room
};
constexpr int kTurnStride = 8;  // 256 bytes in all

__device__ __forceinline__ int32_t num_pieces(int32_t len) {
    return len / kPieceMin < kMaxPieces ? len / kPieceMin : kMaxPieces;
}
// beg + floor(q * len / n), without the 64-bit division (about 170 instructions):
// with len = n * a + b, floor(q * len / n) = q * a + floor(q * b / n).
__device__ __forceinline__ int32_t piece_begin(int32_t beg, int32_t len, int32_t n, int32_t q) {
    const uint32_t a = uint32_t(len) / uint32_t(n), b = uint32_t(len) - a * uint32_t(n);
    return beg + int32_t(uint32_t(q) * a + uint32_t(q) * b / uint32_t(n));
}

// Buffer resource word 3 for gfx9-family buffers; out-of-range reads give 0.
constexpr int32_t kBufferWord3 = 0x00020000;
// A buffer offset past every resource here (resources span at most this):
// rows past the end of a segment load as +0.0, which leaves the sum unchanged
// (a sum started at +0.0 is never -0.0, and x + 0.0 == x for every other x).
constexpr int32_t kOutOfRange = 0x7ffff000;

// What becomes of a coalesced row: stored to coal (if not null) and/or
// applied to W[rows[u]] (if W is not null) with optimizer `kind`.
struct RowSink {
    float *coal;
    float *W;
    float *A;  // Adagrad / RMSprop accumulator
    const int32_t *rows;
    int32_t kind;  // TC_OPT_SGD, TC_OPT_ADAGRAD or TC_OPT_RMSPROP
    float lr, eps, gamma, omg;  // omg = 1 - gamma
};

// The table (and accumulator) value one lane's sink_value updates: column
// `col` of table row rows[u]. A consumer loads it before running the
// segment's chain, so that its two dependent loads overlap the chain.
struct SinkVal {
    int64_t at;
    float w, a;
};

__device__ __forceinline__ SinkVal sink_value_load(const RowSink &k, int64_t u, int32_t dim,
                                                   int32_t col) {
    SinkVal v{0, 0.f, 0.f};
    if (k.W && col < dim) {
        v.at = int64_t(k.rows[u]) * dim + col;
        v.w = stream_load(k.W + v.at);
        if (k.kind != TC_OPT_SGD) v.a = stream_load(k.A + v.at);
    }
    return v;
}

// One lane's column `col` of coalesced row u, with its table value in v.
__device__ __forceinline__ void sink_value(const RowSink &k, int64_t u, int32_t dim, int32_t col,
                                           float g, const SinkVal &v) {
    if (k.coal) k.coal[u * dim + col] = g;
    if (k.W) {
        float w = v.w;
        if (k.kind == TC_OPT_SGD) {
            w = sgd_step(w, g, k.lr);
        } else {
            float a = v.a;
            if (k.kind == TC_OPT_ADAGRAD)
                adagrad_step(w, a, g, k.lr, k.eps);
            else
                rmsprop_step(w, a, g, k.lr, k.eps, k.gamma, k.omg);
            stream_store(k.A + v.at, a);
        }
        stream_store(k.W + v.at, w);
    }
}

// A lane group's float4 chunks of coalesced row u, whose table row is r
// (rows[u], loaded by the caller together with the segment's offsets).
template <int LANES, int CHUNKS>
__device__ __forceinline__ void sink_group(const RowSink &k, int64_t u, int64_t r, int32_t dim,
                                           int sub, const float4 (&acc)[CHUNKS]) {
    if (k.coal) group_store<LANES, CHUNKS>(k.coal + u * dim, dim, sub, acc);
    if (k.W) {
        const int d4 = dim >> 2;
        float *wrow = k.W + r * dim;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const int col4 = sub + c * LANES;
            if (col4 >= d4) continue;
            const float4 g = acc[c];
            float4 w = stream_load4(wrow + 4 * col4);
            if (k.kind == TC_OPT_SGD) {
                w.x = sgd_step(w.x, g.x, k.lr);
                w.y = sgd_step(w.y, g.y, k.lr);
                w.z = sgd_step(w.z, g.z, k.lr);
                w.w = sgd_step(w.w, g.w, k.lr);
            } else {
                float *arow = k.A + r * dim;
                float4 a = stream_load4(arow + 4 * col4);
                if (k.kind == TC_OPT_ADAGRAD) {
                    adagrad_step(w.x, a.x, g.x, k.lr, k.eps);
                    adagrad_step(w.y, a.y, g.y, k.lr, k.eps);
                    adagrad_step(w.z, a.z, g.z, k.lr, k.eps);
                    adagrad_step(w.w, a.w, g.w, k.lr, k.eps);
                } else {
                    rmsprop_step(w.x, a.x, g.x, k.lr, k.eps, k.gamma, k.omg);
                    rmsprop_step(w.y, a.y, g.y, k.lr, k.eps, k.gamma, k.omg);
                    rmsprop_step(w.z, a.z, g.z, k.lr, k.eps, k.gamma, k.omg);
                    rmsprop_step(w.w, a.w, g.w, k.lr, k.eps, k.gamma, k.omg);
                }
                stream_store4(arow + 4 * col4, a);
            }
            stream_store4(wrow + 4 * col4, w);
        }
    }
}

// LDS buffer layout: column-major, so that one 16-byte read gives a consumer
// lane four consecutive rows of its column. Within column c, the group of
// rows 4k..4k+3 sits at group position k ^ swz(c); the swizzle spreads both
// the consumer's 16-byte reads (16 neighbouring columns, same k) and the
// producers' 4-byte writes (16 columns 4 apart, same k) over distinct banks.
struct LongLds {
    alignas(16) float cols[kBuffers][kPartCols][kChunkRows];
    int32_t offs[kProducers][kChunkRows];
};
__device__ __forceinline__ int32_t swz(int32_t c) { return (c & 15) ^ ((c >> 4) & 3); }
// byte offset of (row r, column c) within one buffer
__device__ __forceinline__ int32_t lds_pos(int32_t r, int32_t c) {
    return (c * kChunkRows + 4 * ((r >> 2) ^ swz(c)) + (r & 3)) * 4;
}
constexpr int32_t kBufferBytes = kPartCols * kChunkRows * 4;

// Workgroup barrier that orders LDS only: outstanding global loads stay in
// flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int K>
using Int = std::integral_constant<int, K>;

// Producer P of a long segment (rows ids[0..len) of grad, part columns at
// byte offset part_bytes). It gathers chunk c (rows 64c..64c+63) with the
// load instructions k = P, P + kProducers, ... of the chunk; instruction k brings rows
// 4k..4k+3, lane l reading 16 bytes of row 4k + l/16. Chunk c's loads are
// issued kAhead chunks before it is written to LDS buffer c % 3, two chunks
// ahead of the consumer; the chunk's ids are loaded kIdAhead chunks before
// that and turned into row offsets through a small per-producer LDS table.
// Executes exactly 1 + nchunks barriers, as the consumer does.
template <int P>
__device__ void long_producer(LongLds &lds, __amdgpu_buffer_rsrc_t id_rsrc, int32_t len,
                              int32_t first, int32_t row_bytes, int32_t part_bytes,
                              int32_t nchunks, __amdgpu_buffer_rsrc_t rsrc) {
    constexpr int L = (kLoadsPerChunk - P + kProducers - 1) / kProducers;
    const int lane = threadIdx.x & (kWave - 1);
    const int rsel = lane / kLanesPerRow;
    const int32_t col4 = (lane % kLanesPerRow) * 4;  // first of the lane's 4 columns
    const int32_t lane_bytes = part_bytes + col4 * 4;
    int32_t *offs = lds.offs[P];
    // ids of chunk c, one per lane. The whole byte offset goes in the
    // vector offset, which the buffer's range check covers (the scalar
    // offset is not checked): ids past the end of the segment read as 0
    // without touching memory, and such rows get kOutOfRange below.
    auto load_ids = [&](int32_t c) -> int32_t {
        return __builtin_amdgcn_raw_buffer_load_b32(id_rsrc, c * (kChunkRows * 4) + lane * 4, 0,
                                                    0);
    };
    int32_t iv[kIdAhead];
    float4 d[kAhead][L];
    auto issue = [&](auto ds, auto es, int32_t c) {
        constexpr int DS = decltype(ds)::value, ES = decltype(es)::value;
        offs[lane] = c * kChunkRows + lane < len ? (iv[ES] - first) * row_bytes : kOutOfRange;
        int32_t o[L];
#pragma unroll
        for (int t = 0; t < L; ++t) o[t] = offs[(P + kProducers * t) * kRowsPerLoad + rsel];
#pragma unroll
        for (int t = 0; t < L; ++t)
            d[DS][t] = __builtin_bit_cast(
                float4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, o[t] + lane_bytes, 0, 0));
        iv[ES] = load_ids(c + kIdAhead);
    };
    // byte offsets of this lane's four columns of row 4k + rsel, k = P + 3t
    int32_t wpos[L][4];
#pragma unroll
    for (int t = 0; t < L; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            wpos[t][e] = lds_pos((P + kProducers * t) * kRowsPerLoad + rsel, col4 + e);
    char *lds_cols = reinterpret_cast<char *>(&lds.cols[0][0][0]);
    auto write = [&](auto ds, auto bs) {
        constexpr int DS = decltype(ds)::value, B = decltype(bs)::value;
#pragma unroll
        for (int t = 0; t < L; ++t) {
            const float4 v = d[DS][t];
            *reinterpret_cast<float *>(lds_cols + B * kBufferBytes + wpos[t][0]) = v.x;
            *reinterpret_cast<float *>(lds_cols + B * kBufferBytes + wpos[t][1]) = v.y;
            *reinterpret_cast<float *>(lds_cols + B * kBufferBytes + wpos[t][2]) = v.z;
            *reinterpret_cast<float *>(lds_cols + B * kBufferBytes + wpos[t][3]) = v.w;
        }
    };
#pragma unroll
    for (int e = 0; e < kIdAhead; ++e) iv[e] = load_ids(e);
    static_assert(kAhead == 3, "the prologue issues kAhead chunks");
    static_assert(kIdAhead > 4, "the prologue uses the ids of chunks 0..4");
    issue(Int<0>{}, Int<0>{}, 0);
    issue(Int<1>{}, Int<1>{}, 1);
    issue(Int<2>{}, Int<2>{}, 2);
    write(Int<0>{}, Int<0>{});
    issue(Int<0>{}, Int<3>{}, 3);
    write(Int<1>{}, Int<1>{});
    issue(Int<1>{}, Int<4>{}, 4);
    lds_barrier();
    // Step i: write chunk i + 2, refill its registers with chunk i + 2 + kAhead.
    auto step = [&](auto ms, int32_t i) {
        constexpr int M = decltype(ms)::value;  // i % kPeriod
        write(Int<(M + 2) % kAhead>{}, Int<(M + 2) % kBuffers>{});
        issue(Int<(M + 2) % kAhead>{}, Int<(M + 2 + kAhead) % kIdAhead>{}, i + 2 + kAhead);
        lds_barrier();
    };
    // Whole periods in a loop with a single exit (a loop left from the middle
    // merges the load bookkeeping of every exit at its head, which costs a
    // full wait), then the remaining steps once.
    static_assert(kPeriod == 6, "the step loop is unrolled over 6 chunks");
    int32_t i = 0;
    const int32_t periods = nchunks / kPeriod;
    for (int32_t k = 0; k < periods; ++k, i += kPeriod) {
        step(Int<0>{}, i);
        step(Int<1>{}, i + 1);
        step(Int<2>{}, i + 2);
        step(Int<3>{}, i + 3);
        step(Int<4>{}, i + 4);
        step(Int<5>{}, i + 5);
    }
    const int32_t rem = nchunks - i;
    if (rem > 0) { step(Int<0>{}, i);
    if (rem > 1) { step(Int<1>{}, i + 1);
    if (rem > 2) { step(Int<2>{}, i + 2);
    if (rem > 3) { step(Int<3>{}, i + 3);
    if (rem > 4) { step(Int<4>{}, i + 4);
    }}}}}
}

// The consumer: lane l owns column l of the part and adds the rows of chunk
// i in order, 64 per step, four rows per 16-byte LDS read. Reads run kAheadG
// groups (4 rows each) ahead of the adds through a small register ring; chunk
// i + 1 is complete in LDS during step i (it was written one step ahead), so
// the read-ahead crosses into it freely and the chain never waits for LDS.
// Executes exactly 1 + nchunks barriers, as the producers do.
constexpr int kAheadG = 8;
__device__ float long_consumer(LongLds &lds, int32_t nchunks) {
    constexpr int G = kChunkRows / 4;
    static_assert(G % kAheadG == 0, "ring slots repeat every step");
    const int lane = threadIdx.x & (kWave - 1);
    const char *lds_cols = reinterpret_cast<const char *>(&lds.cols[0][0][0]);
    int32_t rpos[G];  // byte offset of rows 4k..4k+3 of this lane's column
#pragma unroll
    for (int k = 0; k < G; ++k) rpos[k] = lds_pos(4 * k, lane);
    auto read = [&](int b, int k) -> float4 {
        return *reinterpret_cast<const float4 *>(lds_cols + b * kBufferBytes + rpos[k]);
    };
    float acc = 0.f;
    lds_barrier();
    float4 ring[kAheadG];
#pragma unroll
    for (int k = 0; k < kAheadG; ++k) ring[k] = read(0, k);
    // step i: chunk i sits in buffer B = i % 3, chunk i + 1 in (B + 1) % 3
    auto step = [&](auto bs) {
        constexpr int B = decltype(bs)::value, BN = (B + 1) % kBuffers;
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const float4 x = ring[k % kAheadG];
            ring[k % kAheadG] = k + kAheadG < G ? read(B, k + kAheadG) : read(BN, k + kAheadG - G);
            acc = acc + x.x;
            acc = acc + x.y;
            acc = acc + x.z;
            acc = acc + x.w;
            __builtin_amdgcn_sched_barrier(0);
        }
        lds_barrier();
    };
    int32_t i = 0;
    for (;;) {
        if (i >= nchunks) break;
        step(Int<0>{});
        if (++i >= nchunks) break;
        step(Int<1>{});
        if (++i >= nchunks) break;
        step(Int<2>{});
        ++i;
    }
    return acc;
}

// The ordered chain over ids[beg, beg + len) for this block's part, run by
// all five wavefronts (each executes the same number of barriers). Returns
// the sum of column `col` in the consumer wavefront (w == 0), 0 elsewhere.
// grad_bytes: the size of the whole grad array when it is at most
// kOutOfRange (its rows are then addressed from its start), else 0 (the
// chain's rows are addressed from its first row).
__device__ __forceinline__ float run_chain(LongLds &lds, const float *__restrict__ grad,
                                           int32_t dim, const int32_t *__restrict__ ids,
                                           int32_t beg, int32_t len, int w, int32_t part,
                                           int32_t col, int32_t grad_bytes) {
    const int32_t row_bytes = dim * 4;
    const int32_t *sid = ids + beg;
    int32_t first = 0;
    uint64_t span = uint64_t(grad_bytes);
    if (grad_bytes == 0) {  // uniform
        // ids within a segment are non-decreasing (stable cast order)
        first = __builtin_amdgcn_readfirstlane(sid[0]);
        const int32_t last = __builtin_amdgcn_readfirstlane(sid[len - 1]);
        span = uint64_t(last - first + 1) * uint64_t(row_bytes);
    }
    if (span > uint64_t(kOutOfRange) || len >= (1 << 28)) {
        // rows spread over about 2 GiB or more, so that kOutOfRange would not
        // be past them (or a segment so long that the byte offsets of its ids
        // and of the id chunks read ahead would not stay below 2^31): the
        // consumer alone, with 64-bit addressed loads (no barriers on this
        // path)
        float acc = 0.f;
        if (w == 0) {
            const float *colp = grad + (col < dim ? col : dim - 1);
            for (int32_t k = 0; k < len; ++k) acc = acc + colp[int64_t(sid[k]) * dim];
        }
        return acc;
    }
    const int32_t nchunks = (len + kChunkRows - 1) / kChunkRows;
    const auto id_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(sid), 0, len * 4, kBufferWord3);
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(grad + int64_t(first) * dim), 0, int32_t(span), kBufferWord3);
    const int32_t part_bytes = part * kPartCols * 4;
    if (w == 0) return long_consumer(lds, nchunks);
    if (w == 1)
        long_producer<0>(lds, id_rsrc, len, first, row_bytes, part_bytes, nchunks, rsrc);
    else if (w == 2)
        long_producer<1>(lds, id_rsrc, len, first, row_bytes, part_bytes, nchunks, rsrc);
    else if (w == 3)
        long_producer<2>(lds, id_rsrc, len, first, row_bytes, part_bytes, nchunks, rsrc);
    else
        long_producer<3>(lds, id_rsrc, len, first, row_bytes, part_bytes, nchunks, rsrc);
    return 0.f;
}

// Wavefront that summed piece q of split segment u: store the piece sum,
// count the piece, and if it was the segment's last (for this part), add the
// n piece sums in piece order from +0 and hand the row to the sink. The piece
// sums and counts are agent-scope atomics throughout, so a wait between the
// store and the count orders them for every XCD; a fence at agent scope would
// write back and invalidate the whole L2 of the XCD for each piece. The n
// sums are loaded all at once: one after another they would end the call with
// up to 32 round trips.
__device__ __forceinline__ void finish_piece(const SplitWs &ws, const RowSink &sink, int32_t dim,
                                             int32_t part, int32_t col, int32_t u, int32_t beg,
                                             int32_t len, int32_t n, int32_t q, float acc) {
    const int lane = threadIdx.x & (kWave - 1);
    float *sums = ws.partial + (col < dim ? col : 0);
    if (col < dim)
        __hip_atomic_store(sums + int64_t(piece_begin(beg, len, n, q) / kPieceMin) * dim, acc,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // for the compiler
    __builtin_amdgcn_s_waitcnt(0);
    int32_t done = 0;
    if (lane == 0)
        done = __hip_atomic_fetch_add(&ws.seg_done[int64_t(beg / kSplitPairs) * ws.parts + part],
                                      1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    done = __builtin_amdgcn_readlane(done, 0);
    if (done != n - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const int32_t at = piece_begin(beg, len, n, min(lane, n - 1)) / kPieceMin;  // of piece `lane`
    float x[kMaxPieces];
#pragma unroll
    for (int k = 0; k < kMaxPieces; ++k)
        x[k] = __hip_atomic_load(sums + int64_t(__builtin_amdgcn_readlane(at, k)) * dim,
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    float tot = 0.f;
#pragma unroll
    for (int k = 0; k < kMaxPieces; ++k) tot = k < n ? tot + x[k] : tot;
    if (col < dim) sink_value(sink, u, dim, col, tot, sink_value_load(sink, u, dim, col));
}

// Long segments without a workspace. Each block (range x, part y) scans a
// contiguous range of segments and runs every long one it finds. All five
// wavefronts scan the same offsets, so they agree on every segment and on its
// number of chunks, which fixes the barrier count. A first pass reads every
// 64th offset: a batch of 64 segments spanning fewer than kLongSegment pairs
// cannot hold a long one.
__global__ __launch_bounds__(kLongThreads) void k_backward_long(
    const float *__restrict__ grad, int32_t dim, const int32_t *__restrict__ ids,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ num_out_dev,
    int64_t num_out_cap, RowSink sink, int32_t grad_bytes) {
    __shared__ LongLds lds;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int32_t part = blockIdx.y;
    const int32_t col = part * kPartCols + lane;
    const int64_t u_dev = *num_out_dev;
    const int64_t num = u_dev < num_out_cap ? u_dev : num_out_cap;
    if (w == 0) __builtin_amdgcn_s_setprio(3);
    const int32_t ranges = int32_t(gridDim.x);
    const int32_t range = int32_t(blockIdx.x);
    const int64_t per = (num + ranges - 1) / ranges;
    const int64_t r0 = int64_t(range) * per;
    const int64_t r1 = r0 + per < num ? r0 + per : num;
    for (int64_t c0 = r0; c0 < r1; c0 += int64_t(kWave) * kWave) {
        const int64_t s0 = c0 + int64_t(kWave) * lane;  // this lane's batch
        const int32_t os = offsets[s0 < r1 ? s0 : r1];
        const int64_t s1 = s0 + kWave < r1 ? s0 + kWave : r1;
        const int32_t oe = offsets[s1];
        uint64_t batches = __ballot(s0 < r1 && oe - os >= kLongSegment);
        while (batches) {
            const int i = __builtin_ctzll(batches);
            batches &= batches - 1;
            const int64_t u = c0 + int64_t(kWave) * i + lane;
            int32_t o0 = 0, o1 = 0;
            if (u < r1) {
                o0 = offsets[u];
                o1 = offsets[u + 1];
            }
            uint64_t longs = __ballot(u < r1 && o1 - o0 >= kLongSegment);
            while (longs) {
                const int j = __builtin_ctzll(longs);
                longs &= longs - 1;
                const int32_t beg = __builtin_amdgcn_readlane(o0, j);
                const int32_t len = __builtin_amdgcn_readlane(o1, j) - beg;
                const int64_t seg = c0 + int64_t(kWave) * i + j;
                SinkVal sv{0, 0.f, 0.f};
                if (w == 0) sv = sink_value_load(sink, seg, dim, col);
                const float acc =
                    run_chain(lds, grad, dim, ids, beg, len, w, part, col, grad_bytes);
                if (w == 0 && col < dim) sink_value(sink, seg, dim, col, acc, sv);
            }
        }
    }
}

// Lists the long segments inside the cover, in an order of no consequence. Any
// of the num segments may be one: those before it may be without pairs.
constexpr int kListThreads = 1024;
__global__ __launch_bounds__(kListThreads) void k_backward_list(
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ num_out_dev,
    int64_t num_out_cap, SplitWs ws) {
    __shared__ int32_t count[3];  // entries in big[], in longs[], pairs in both
    const int64_t u_dev = *num_out_dev;
    const int64_t num = u_dev < num_out_cap ? u_dev : num_out_cap;
    // Ranges of equal size. Nothing past offsets[num] is read: the capacities
    // say nothing of the array's length. (Loads by the capacity, beside num's
    // and not after it, were no faster: 24.2 us against 24.1 for the step of 1
    // table of 100k x 64, batch 256, and 16.5 against 16.1 for the backward of
    // 8 tables of 20k x 96, batch 500.)
    const int64_t per = (uint32_t(num) + gridDim.x - 1) / gridDim.x;  // num is below 2^31
    const int64_t s0 = min(int64_t(blockIdx.x) * per, num), s1 = min(s0 + per, num);
    int32_t p0 = s0 < s1 ? offsets[s0] : 0;
    if (threadIdx.x < 3) count[threadIdx.x] = 0;
    __syncthreads();
    const int32_t big0 = p0 / kBigLong, long0 = p0 / kListLong;
    auto list = [&](int64_t o, int32_t beg, int32_t len) {
        if (len < kListLong || int64_t(beg) + len > ws.cap_pairs) return;
        atomicAdd(&count[2], len);
        if (len < kBigLong) {
            ws.longs[long0 + atomicAdd(&count[1], 1)] = make_int2(int32_t(o), beg);
        } else if (len < kSplitPairs) {
            ws.big[big0 + atomicAdd(&count[0], 1)] = make_int2(int32_t(o), -1);
        } else {
            const int32_t n = num_pieces(len);
            int2 *at = ws.big + big0 + atomicAdd(&count[0], n);
            for (int32_t q = 0; q < n; ++q) at[q] = make_int2(int32_t(o), q);
            int32_t *done = ws.seg_done + int64_t(beg / kSplitPairs) * ws.parts;
            for (int32_t p = 0; p < ws.parts; ++p) done[p] = 0;
        }
    };
    if (per <= kListThreads) {  // uniform: a segment per thread at most
        const int64_t o = s0 + threadIdx.x;
        if (o < s1) {
            const int32_t beg = offsets[o], end = offsets[o + 1];
            list(o, beg, end - beg);
        }
    } else {
        // four segments per thread and trip, all their loads before any is used
        constexpr int kPer = 4;
        for (int64_t o0 = s0 + threadIdx.x; o0 < s1; o0 += kPer * kListThreads) {
            int32_t beg[kPer], end[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int64_t o = min(o0 + k * kListThreads, s1 - 1);
                beg[k] = offsets[o];
                end[k] = offsets[o + 1];
            }
#pragma unroll
            for (int k = 0; k < kPer; ++k)
                if (o0 + k * kListThreads < s1)
                    list(o0 + k * kListThreads, beg[k], end[k] - beg[k]);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) ws.heads[blockIdx.x] = make_int4(count[0], count[1], p0, count[2]);
    if (blockIdx.x == 0 && threadIdx.x < kXcds && ws.turns != nullptr)
        ws.turns[threadIdx.x * kTurnStride] = 0;
    if (blockIdx.x == 0 && gridDim.x + threadIdx.x < ws.list_blocks)
        ws.heads[gridDim.x + threadIdx.x] = make_int4(0, 0, 0, 0);
}

// The chain over ids sid[0..len) for one wavefront with 64-bit addresses, for
// segments whose rows no buffer window holds: kFarRows rows are on their way at
// once. Measured (us of the call; segments spread over 2.4 GB): 4000 of 48 to 79
// rows of 1024 floats 756 row after row, 214 with 32 at a time (184 if the lane
// groups of the short segments had them); of 80 to 200 1650 and 420; of 600 to
// 900 11800 and 2090. Ids are loaded by lane: loads of each by itself take a
// register more, which the widest rows spill.
constexpr int kFarRows = 32;
__device__ __forceinline__ float far_chain(const float *__restrict__ grad, int32_t dim,
                                           const int32_t *__restrict__ sid, int32_t len,
                                           int32_t col) {
    const float *colp = grad + min(col, dim - 1);
    const uint32_t lane = threadIdx.x & (kWave - 1);
    float acc = 0.f;
    for (uint32_t k = 0; k < uint32_t(len); k += kFarRows) {
        float row[kFarRows];
        const int32_t id = sid[min(k + lane, uint32_t(len) - 1)];
#pragma unroll
        for (uint32_t i = 0; i < kFarRows; ++i)
            row[i] = colp[int64_t(__builtin_amdgcn_readlane(id, i)) * dim];
#pragma unroll
        for (uint32_t i = 0; i < kFarRows; ++i) acc = k + i < uint32_t(len) ? acc + row[i] : acc;
    }
    return acc;
}

// The ordered chain over ids[beg, beg + len) for one wavefront, lane l owning
// column l of the part: kDepth row loads of 4 bytes per lane are in flight,
// one register each; each is added and replaced by the load of the row kDepth
// further on. Ids come kDepth at a time, one per lane, a round ahead, and are
// turned into byte offsets there; a row's offset is then one v_readlane into
// the load's scalar offset. Rows past the end are read as the last one again
// (a cache hit) and not added. `last()` is called when the last rows are on
// their way.
// What bounds it is the gathers' latency: about 700 ns / kDepth = 17 ns per
// row, with the chains of up to 32 wavefronts on a CU at once. 40 rows are
// what fits the 64 registers that the short segments' 8 wavefronts per SIMD
// allow (48 spill, and slow those down). Measured on chains alone (D = 128,
// 8192 of 100 rows over 16384 bags): 43 us, against 248 us with the chains one
// after another in five-wavefront workgroups like k_backward_long's, whose
// start-up each chain then pays by itself.
constexpr int kDepth = 40;
static_assert(kDepth % 8 == 0 && kDepth <= kWave && kListLong > kDepth, "chain rounds");
template <class Last>
__device__ __forceinline__ float wave_chain(const float *__restrict__ grad, int32_t dim,
                                            const int32_t *__restrict__ ids, int32_t beg,
                                            int32_t len, int32_t part, int32_t grad_bytes,
                                            Last &&last) {
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t col = part * kPartCols + lane;
    const int32_t row_bytes = dim * 4;
    const int32_t *sid = ids + beg;
    int32_t first = 0;
    uint64_t span = uint64_t(grad_bytes);
    if (grad_bytes == 0) {  // uniform
        // ids within a segment are non-decreasing (stable cast order)
        first = __builtin_amdgcn_readfirstlane(sid[0]);
        const int32_t end = __builtin_amdgcn_readfirstlane(sid[len - 1]);
        span = uint64_t(end - first + 1) * uint64_t(row_bytes);
    }
    if (span > uint64_t(kOutOfRange) || len >= (1 << 28)) {  // as in run_chain
        last();
        return far_chain(grad, dim, sid, len, col);
    }
    float acc = 0.f;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(grad + int64_t(first) * dim), 0, int32_t(span), kBufferWord3);
    // lanes past the row's columns read its last one (a row's offset, in the
    // scalar offset, is not range-checked)
    const int32_t lane_bytes = min(col, dim - 1) * 4;
    // ids of rows r + lane, rows past the end being the last one
    auto load_ids = [&](int32_t r) -> int32_t { return sid[min(r + lane, len - 1)]; };
    auto load = [&](int32_t offs) -> float {
        return __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, lane_bytes, offs, 0));
    };
    // The barriers hold the order of the instructions: an add, then the load
    // into the same register, so that kDepth registers do for the rows and
    // each add waits for its own row only.
    float row[kDepth];
    int32_t offs = load_ids(0), next_ids = load_ids(kDepth);
    __builtin_amdgcn_sched_barrier(0);
    offs = (offs - first) * row_bytes;
#pragma unroll
    for (int k = 0; k < kDepth; ++k) {
        row[k] = load(__builtin_amdgcn_readlane(offs, k));
        if (k % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
    int32_t r = kDepth;  // rows loaded; a chain has more
    do {
        offs = (next_ids - first) * row_bytes;
        r += kDepth;
        next_ids = load_ids(r);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < kDepth; k += 4) {
            int32_t o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_readlane(offs, k + i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc = acc + row[k + i];
                __builtin_amdgcn_sched_barrier(0);
                row[k + i] = load(o[i]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } while (r < len);
    last();
    const int32_t rem = len - (r - kDepth);  // rows of the last round
#pragma unroll
    for (int k = 0; k < kDepth; ++k) acc = k < rem ? acc + row[k] : acc;
    return acc;
}

// The ordered chain over ids[beg, beg + len) for a whole workgroup: its four
// wavefronts take groups of kGroupRows rows in turn, each holding the rows of
// its next group in registers while the others add theirs, and hand the sum
// on through LDS, one barrier per group. Only a group's adds and the hand-over
// are in the chain, about 5 ns per row (one chain of 2000 rows: 18 us for the
// call, 31 us in one wavefront); four groups are in flight. Returns the sum
// of column `part * kPartCols + lane` in the last wavefront. Every wavefront
// executes the same number of barriers. Rows past the end read as +0.0 from an
// out-of-range offset, as in run_chain.
constexpr int kGroupRows = 40;
constexpr int kWgWaves = kBlock / kWave;
static_assert(kGroupRows == 40 && kWgWaves == 4, "a group's loads are in three parts");
__device__ __forceinline__ float block_chain(float (&hand)[kWave], const float *__restrict__ grad,
                                             int32_t dim, const int32_t *__restrict__ ids,
                                             int32_t beg, int32_t len, int w, int32_t part,
                                             int32_t grad_bytes) {
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t col = part * kPartCols + lane;
    const int32_t row_bytes = dim * 4;
    const int32_t *sid = ids + beg;
    int32_t first = 0;
    uint64_t span = uint64_t(grad_bytes);
    if (grad_bytes == 0) {  // uniform
        first = __builtin_amdgcn_readfirstlane(sid[0]);
        const int32_t last = __builtin_amdgcn_readfirstlane(sid[len - 1]);
        span = uint64_t(last - first + 1) * uint64_t(row_bytes);
    }
    if (span > uint64_t(kOutOfRange) || len >= (1 << 28))
        // as in run_chain; one wavefront, no barriers
        return w == kWgWaves - 1 ? far_chain(grad, dim, sid, len, col) : 0.f;
    float acc = 0.f;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(grad + int64_t(first) * dim), 0, int32_t(span), kBufferWord3);
    const int32_t lane_bytes = min(col, dim - 1) * 4;
    const int32_t rounds = (len + kWgWaves * kGroupRows - 1) / (kWgWaves * kGroupRows);
    float row[kGroupRows];
    // ids of this wavefront's group of round r, one per lane
    auto load_id = [&](int32_t r) -> int32_t {
        return sid[min((r * kWgWaves + w) * kGroupRows + lane, len - 1)];
    };
    auto to_offs = [&](int32_t id, int32_t r) -> int32_t {
        return (r * kWgWaves + w) * kGroupRows + lane < len ? (id - first) * row_bytes
                                                            : kOutOfRange;
    };
    // the loads of rows K0 .. K0 + K - 1 of a group
    auto issue = [&](auto k0s, auto ks, int32_t offs) {
        constexpr int K0 = decltype(k0s)::value, K = decltype(ks)::value;
#pragma unroll
        for (int k = K0; k < K0 + K; k += 4) {
            int32_t o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_readlane(offs, k + i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                row[k + i] = __builtin_bit_cast(
                    float,
                    __builtin_amdgcn_raw_buffer_load_b32(rsrc, o[i] + lane_bytes, 0, 0));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (w == 0) hand[lane] = 0.f;
    int32_t id = load_id(0), next_id = load_id(1);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" : "+v"(next_id));  // waited for here, not behind the rows
    int32_t offs = to_offs(id, 0);
    issue(Int<0>{}, Int<kGroupRows>{}, offs);
    lds_barrier();
    for (int i = 0; i < w; ++i) lds_barrier();
    // (the loads issued in the last round are all past the end)
    for (int32_t r = 0; r < rounds; ++r) {
        acc = hand[lane];
#pragma unroll
        for (int k = 0; k < kGroupRows; ++k) acc = acc + row[k];
        hand[lane] = acc;
        lds_barrier();
        offs = to_offs(next_id, r + 1);
        next_id = load_id(r + 2);
        __builtin_amdgcn_sched_barrier(0);
        // a part of the next group's loads in each of the others' turns, so
        // that none of them waits at its barrier for all of the loads
        issue(Int<0>{}, Int<16>{}, offs);
        lds_barrier();
        issue(Int<16>{}, Int<12>{}, offs);
        lds_barrier();
        issue(Int<28>{}, Int<12>{}, offs);
        lds_barrier();
    }
    for (int i = w; i < kWgWaves - 1; ++i) lds_barrier();
    return acc;
}

// A list as k_backward_rows finds its way in it: before[b] entries come from
// the list kernel's workgroups before b, and b's own are in slots first[b] on.
struct ListIndex {
    int32_t before[kListBlocks], first[kListBlocks];
};
// Exclusive prefixes over the workgroup of N values per thread, and their sums.
template <int N>
__device__ __forceinline__ void block_prefix(int32_t (&v)[N], int32_t (&total)[N],
                                             int32_t (&wave_sum)[kBlock / kWave][N]) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int32_t p[N];
#pragma unroll
    for (int k = 0; k < N; ++k) p[k] = wave_prefix(v[k]);
    if (lane == kWave - 1)
#pragma unroll
        for (int k = 0; k < N; ++k) wave_sum[w][k] = p[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k) {
        v[k] = p[k] - v[k];
        int32_t tot = 0;
#pragma unroll
        for (int i = 0; i < kBlock / kWave; ++i) {
            if (i < w) v[k] += wave_sum[i][k];
            tot += wave_sum[i][k];
        }
        total[k] = __builtin_amdgcn_readfirstlane(tot);
    }
}
// The slot of entry i (below the list's length).
__device__ __forceinline__ int32_t list_slot(const ListIndex &x, int32_t i) {
    const int lane = threadIdx.x & (kWave - 1);
    // the last workgroup with before[b] <= i holds it: 64 of every fourth,
    // then the four
    int b = 4 * (63 - __builtin_clzll(__ballot(x.before[4 * lane] <= i)));
#pragma unroll
    for (int j = 3; j > 0; --j)
        if (x.before[b + j] <= i) {
            b += j;
            break;
        }
    return __builtin_amdgcn_readfirstlane(x.first[b] + i - x.before[b]);
}

// One chain, of list entry `slot` of big[] (a whole workgroup) or of longs[]
// (a wavefront), for the columns of one part.
__device__ __forceinline__ void run_big(float (&hand)[kWave], const float *__restrict__ grad,
                                        int32_t dim, const int32_t *__restrict__ ids,
                                        const int32_t *__restrict__ offsets, const RowSink &sink,
                                        const SplitWs &ws, int32_t slot, int w, int32_t part,
                                        int32_t grad_bytes) {
    const int2 e = ws.big[slot];
    const int32_t u = __builtin_amdgcn_readfirstlane(e.x);
    const int32_t q = __builtin_amdgcn_readfirstlane(e.y);
    const int32_t beg = __builtin_amdgcn_readfirstlane(offsets[u]);
    const int32_t len = __builtin_amdgcn_readfirstlane(offsets[u + 1]) - beg;
    const int32_t n = q < 0 ? 1 : num_pieces(len);
    const int32_t b = q < 0 ? beg : piece_begin(beg, len, n, q);
    const int32_t l = q < 0 ? len : piece_begin(beg, len, n, q + 1) - b;
    const float acc = block_chain(hand, grad, dim, ids, b, l, w, part, grad_bytes);
    if (w != kWgWaves - 1) return;
    const int32_t col = part * kPartCols + (threadIdx.x & (kWave - 1));
    if (q >= 0)
        finish_piece(ws, sink, dim, part, col, u, beg, len, n, q, acc);
    else if (col < dim)
        sink_value(sink, u, dim, col, acc, sink_value_load(sink, u, dim, col));
}
__device__ __forceinline__ void run_long(const float *__restrict__ grad, int32_t dim,
                                         const int32_t *__restrict__ ids,
                                         const int32_t *__restrict__ offsets, const RowSink &sink,
                                         const SplitWs &ws, int32_t slot, int32_t part,
                                         int32_t grad_bytes) {
    const int2 e = ws.longs[slot];
    const int32_t u = __builtin_amdgcn_readfirstlane(e.x);
    const int32_t beg = __builtin_amdgcn_readfirstlane(e.y);
    const int32_t len = __builtin_amdgcn_readfirstlane(offsets[u + 1]) - beg;
    const int32_t col = part * kPartCols + (threadIdx.x & (kWave - 1));
    // the table row's value, loaded before the chain's last rows are added
    SinkVal v{0, 0.f, 0.f};
    const float acc = wave_chain(grad, dim, ids, beg, len, part, grad_bytes,
                                 [&] { v = sink_value_load(sink, u, dim, col); });
    if (col < dim) sink_value(sink, u, dim, col, acc, v);
}

// Short segments o < num, from `start` on: one lane group per segment, as the
// forward; wavefront `wave` of `nwave`. Long ones are left to the chains: all of them without a
// workspace, the covered ones with one (uncovered ones are summed here).
template <int LANES, int CHUNKS>
__device__ __forceinline__ void short_segments(const float *__restrict__ grad, int32_t dim,
                                               const int32_t *__restrict__ ids,
                                               const int32_t *__restrict__ offsets, int64_t num,
                                               const RowSink &sink, int64_t cap_pairs,
                                               int64_t wave, int64_t nwave,
                                               int64_t start = 0) {
    constexpr int kGroups = kWave / LANES;
    const int lane = threadIdx.x & (kWave - 1);
    const int sub = lane & (LANES - 1);
    const int grp = lane / LANES;
    for (int64_t o0 = start + wave * kGroups; o0 < num; o0 += nwave * kGroups) {
        const int64_t o = o0 + grp;
        int32_t beg = 0, end = 0;
        bool mine = false;
        int64_t r = 0;  // the table row the sink updates
        if (o < num) {
            beg = offsets[o];
            end = offsets[o + 1];
            if (sink.W) r = sink.rows[o];
            mine = end - beg < (cap_pairs ? kListLong : kLongSegment) ||
                   (cap_pairs != 0 && end > cap_pairs);
            if (!mine) end = beg;
        }
        float4 acc[CHUNKS];
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        group_range_sum<LANES, CHUNKS>(grad, dim, ids, 0, beg, end, sub, acc);
        if (mine) sink_group<LANES, CHUNKS>(sink, o, r, dim, sub, acc);
    }
}

template <int LANES, int CHUNKS>
__global__ __launch_bounds__(kBlock) void k_backward_short(
    const float *__restrict__ grad, int32_t dim, const int32_t *__restrict__ ids,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ num_out_dev,
    int64_t num_out_cap, RowSink sink) {
    const int64_t u_dev = *num_out_dev;
    const int64_t num = u_dev < num_out_cap ? u_dev : num_out_cap;
    const int64_t wave = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwave = (int64_t(gridDim.x) * blockDim.x) / kWave;
    short_segments<LANES, CHUNKS>(grad, dim, ids, offsets, num, sink, 0, wave, nwave);
}

// All segments, with a workspace. The chains take the first workgroups
// (dispatched first, so that they start at once), big[] before longs[], the
// others the short segments. Chains of neighbouring segments (of one table,
// sharing its rows of grad) are put on one XCD, workgroups going round-robin
// over the XCDs, for the sake of its L2; any other mapping gives the same
// results. Up to 256 columns all workgroups are resident at once: more would
// sweep the short segments in uneven windows (32 tables of 1M x 256: 2.42 ms with
// half as many workgroups again, 2.14 ms with these). Of rows of 260 to 512
// columns 5 of 8 workgroups per CU are resident; the sweep takes no more where
// there are no chains (a million segments of 1 or 2 pairs, 320 columns 550 us and
// 601 with all, 512 columns 685 and 753), or few beside a sweep of kEvenWindows
// windows or more (a million segments of 1 to 3 pairs, 500 of them hot, 260 columns
// 568 and 622), but all where workgroups come free as chains end (100 thousand
// pairs of 30 tables of 2400 x 300, Zipf 1.2: 43.3 and 38.0 us). Chains are better
// off with all 8 (20 thousand segments of 1 to 90 pairs, 260 columns: 146 us, and
// 160 with 5), and wider rows, whose windows are few, too (50 thousand segments of
// 1 to 20 pairs, 1024 columns: 274 us, and 282 with the 3 that are resident).
// The chains' share of the workgroups is that of their pairs among all work,
// with kSegmentCost pairs for each segment and kChainCost for each chain (8 x
// 300k x 128, where many chains are short: 49.7 us without), so that both
// parts end together,
// but at least one workgroup per CU: few long chains are
// bound by their number of wavefronts. Measured (us, the kernel):
//   kSegmentCost        4    12    36      min per CU  1/2     1     2
//   8 x 1M x 64       57.9  55.5  55.6               55.7  55.5  59.3
//   8 x 5M x 128     134.7 123.3 135.4              121.9 123.3 123.2
//   1 x 50M x 128      386   385   384                385   385   394
//   8 x 300k x 128    45.9  44.0  44.2               47.8  44.0  43.2
// Against the short segments first and the chains after them, in a kernel of
// five-wavefront workgroups: 82, 178, 402 and 71 us.
//
// A sweep of kTurns * kTurnWindows windows or more is cut into kTurns parts. The
// workgroups take a share of the first part each, by position, and kTurns - 1
// times as many follow them, whose wavefronts take the shares of the others as
// they are next on their XCD's counter. Workgroups that start late, when another
// stream's kernels hold their places, then cost a part of the sweep, not the whole
// of it once more; and another stream's kernels find places when a part ends, not
// when the sweep does. Measured, 32 tables of 1M x 256 (steps/s, the next batch's
// cast on a side stream beside the backward, beside the whole step, and without
// a side stream): one sweep 235, 228 and 292; parts taken in turn by workgroups
// that stay 288.6, 293.1 and 297.8; by workgroups that end with their share
// 296.4, 296.1 and 299.0. Shorter sweeps end before another stream's kernels do,
// and would pay for the counters (0.5 us a share). A launch made for such a sweep
// whose batch turns out short takes 4 us for the workgroups it has no use for (a
// thousand segments in room for 5.2 million: 8.7 and 12.7 us).
constexpr int kTurns = 8;
constexpr int kTurnWindows = 32;
// Windows from which a sweep beside few chains keeps to the resident workgroups.
constexpr int kEvenWindows = 64;
// Workgroups on a CU (wavefronts on a SIMD) by float4 chunks per lane.
constexpr int rows_per_cu(int chunks) { return chunks == 1 ? 8 : 7 - chunks; }
// Whether the sweep of `num` segments by `blocks` workgroups is cut into parts.
template <int LANES>
constexpr bool sweep_in_parts(int64_t num, int32_t blocks) {
    const int64_t window = int64_t(blocks) * (kBlock / LANES);
    return (num + window - 1) / window >= kTurns * kTurnWindows && blocks % kXcds == 0;
}
template <int LANES, int CHUNKS>
__global__ __launch_bounds__(kBlock, rows_per_cu(CHUNKS)) void k_backward_rows(
    const float *__restrict__ grad, int32_t dim, const int32_t *__restrict__ ids,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ num_out_dev,
    int64_t num_out_cap, RowSink sink, SplitWs ws, int32_t grad_bytes, int32_t cus,
    int32_t blocks) {
    constexpr int kWaves = kBlock / kWave;
    static_assert(kBlock == kListBlocks, "one head per thread");
    __shared__ ListIndex big, longs;
    __shared__ int32_t wave_sum[kWaves][3];
    __shared__ float hand[kWave];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t u_dev = *num_out_dev;
    const int64_t num = u_dev < num_out_cap ? u_dev : num_out_cap;
    // the sweep in parts, if the launch has workgroups for the later ones
    const bool later = int32_t(blockIdx.x) >= blocks;
    const bool parts = int32_t(gridDim.x) > blocks && sweep_in_parts<LANES>(num, blocks);
    if (later && !parts) return;
    const int t = threadIdx.x;  // the lists' heads, one per thread
    const int4 h = t < ws.list_blocks ? ws.heads[t] : make_int4(0, 0, 0, 0);
    int32_t before[3] = {h.x, h.y, h.w}, total[3];
    block_prefix(before, total, wave_sum);
    const int32_t nbig = total[0], nlong = total[1], chain_pairs = total[2];
    big.before[t] = before[0];
    big.first[t] = h.z / kBigLong;
    longs.before[t] = before[1];
    longs.first[t] = h.z / kListLong;
    __syncthreads();
    // rounds of one workgroup per XCD: an (entry, part) item of big[] is a
    // workgroup's, one of longs[] a wavefront's
    const int64_t ibig = int64_t(nbig) * ws.parts, ilong = int64_t(nlong) * ws.parts;
    const int64_t rbig = (ibig + kXcds - 1) / kXcds;
    const int64_t rlong = (ilong + kXcds * kWaves - 1) / (kXcds * kWaves);
    const int64_t rounds = rbig + rlong;
    const float chains = float(chain_pairs) + kChainCost * float(nbig + nlong);
    const int32_t share =
        int32_t(float(blocks) * chains / (chains + kSegmentCost * float(num) + 1.f));
    const int32_t most = min(max(share, cus), blocks * 7 / 8) / kXcds;
    const int32_t chain_rounds = int32_t(rounds < most ? rounds : most);
    const int32_t chain_blocks = chain_rounds * kXcds;
    if (int32_t(blockIdx.x) >= chain_blocks) {
        int32_t short_blocks = blocks - chain_blocks;
        if (CHUNKS == 2 && !parts) {
            const int32_t resident = cus * rows_per_cu(CHUNKS);
            if (chain_blocks == 0 ||
                (chain_blocks <= resident / 2 && num >= int64_t(kEvenWindows) * blocks * kWaves))
                short_blocks = min(short_blocks, resident - chain_blocks);
            if (int32_t(blockIdx.x) >= chain_blocks + short_blocks) return;
        }
        const int32_t nwave = short_blocks * kWaves;
        int32_t wave = (int32_t(blockIdx.x) - chain_blocks) * kWaves + w;
        if (!parts) {
            short_segments<LANES, CHUNKS>(grad, dim, ids, offsets, num, sink, ws.cap_pairs, wave,
                                          nwave);
            return;
        }
        // part 0 is taken by position, of the others what is next on the XCD's
        // counter: each XCD has nwave / kXcds shares of a part, and wavefronts
        // for kTurns - 1 parts or more come later
        const int64_t window = int64_t(nwave) * (kWave / LANES);
        const int64_t per_turn = (num + window - 1) / window / kTurns * window;
        int32_t turn = 0;
        if (later) {
            const int32_t mates = nwave / kXcds;
            int32_t t = 0;
            if ((threadIdx.x & (kWave - 1)) == 0)
                t = __hip_atomic_fetch_add(ws.turns + blockIdx.x % kXcds * kTurnStride, 1,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            t = __builtin_amdgcn_readfirstlane(t);
            turn = 1 + t / mates;
            const int32_t mate = t % mates;
            wave = (mate / kWaves * kXcds + blockIdx.x % kXcds) * kWaves + mate % kWaves;
            if (turn >= kTurns) return;
        }
        short_segments<LANES, CHUNKS>(grad, dim, ids, offsets,
                                      turn < kTurns - 1 ? (turn + 1) * per_turn : num, sink,
                                      ws.cap_pairs, wave, nwave, turn * per_turn);
        return;
    }
    const int32_t xcd = blockIdx.x % kXcds;
    for (int64_t rd = blockIdx.x / kXcds; rd < rounds; rd += chain_rounds) {
        if (rd < rbig) {
            const int64_t item = xcd * rbig + rd;
            if (item < ibig)
                run_big(hand, grad, dim, ids, offsets, sink, ws,
                        list_slot(big, int32_t(item / ws.parts)), w, int32_t(item % ws.parts),
                        grad_bytes);
        } else {
            const int64_t item = (xcd * rlong + rd - rbig) * kWaves + w;
            if (item < ilong)
                run_long(grad, dim, ids, offsets, sink, ws,
                         list_slot(longs, int32_t(item / ws.parts)), int32_t(item % ws.parts),
                         grad_bytes);
        }
    }
}

// Gradient expand (the paper's baseline backward, Sec. II-B): every pair j of
// bag g gets a copy of grad_out[g]. One lane group per bag holds the row in
// registers and writes it once per pair of the bag.
template <int LANES, int CHUNKS>
__global__ __launch_bounds__(kBlock) void k_expand(const float *__restrict__ grad, int32_t dim,
                                                  const int32_t *__restrict__ bag_offsets,
                                                  int64_t num_bags, float *__restrict__ expanded) {
    constexpr int kGroups = kWave / LANES;
    const int lane = threadIdx.x & (kWave - 1);
    const int sub = lane & (LANES - 1);
    const int grp = lane / LANES;
    const int d4 = dim >> 2;
    const int64_t wave = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwave = (int64_t(gridDim.x) * blockDim.x) / kWave;
    for (int64_t g0 = wave * kGroups; g0 < num_bags; g0 += nwave * kGroups) {
        const int64_t g = g0 + grp;
        if (g >= num_bags) continue;
        const int32_t beg = bag_offsets[g], end = bag_offsets[g + 1];
        float4 v[CHUNKS];
        const float *row = grad + g * int64_t(dim);
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const int col4 = sub + c * LANES;
            v[c] = col4 < d4 ? *reinterpret_cast<const float4 *>(row + 4 * col4)
                             : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        for (int32_t j = beg; j < end; ++j)
            group_store<LANES, CHUNKS>(expanded + int64_t(j) * dim, dim, sub, v);
    }
}

tc_status launch_expand(const float *grad, int32_t dim, const int32_t *bag_offsets,
                        int64_t num_bags, float *expanded, hipStream_t stream) {
    const RowShape s = row_shape(dim);
    const int64_t rows_per_block = (kBlock / kWave) * (kWave / s.lanes);
    const unsigned grid = grid_for(num_bags, rows_per_block, int64_t(device_cus()) * 8);
#define TC_EXP_CASE(L, C)                                                                    \
    if (s.lanes == L && s.chunks == C) {                                                     \
        k_expand<L, C><<<grid, kBlock, 0, stream>>>(grad, dim, bag_offsets, num_bags,        \
                                                    expanded);                               \
        return check_launch("k_expand");                                                     \
    }
    TC_EXP_CASE(1, 1)
    TC_EXP_CASE(2, 1)
    TC_EXP_CASE(4, 1)
    TC_EXP_CASE(8, 1)
    TC_EXP_CASE(16, 1)
    TC_EXP_CASE(32, 1)
    TC_EXP_CASE(64, 1)
    TC_EXP_CASE(64, 2)
    TC_EXP_CASE(64, 3)
    TC_EXP_CASE(64, 4)
#undef TC_EXP_CASE
    set_error("no expand kernel for dim %d", dim);
    return TC_ERR_UNSUPPORTED;
}

// The backward workspace's layout for a cover of cap pairs. The heads of
// k_backward_list's workgroups are in the first area when there are few, and
// behind longs[] when that area (16 bytes for each kLongSegment pairs, 8 of
// which an entry takes for each kListLong) has room for kListBlocks: from
// about 125 thousand pairs on.
struct WsLayout {
    size_t heads, big, longs, seg_done, partial, total;
    int32_t list_blocks;
};
WsLayout ws_layout(int64_t cap, int32_t dim) {
    auto al = [](int64_t x) { return size_t((x + 255) & ~int64_t(255)); };
    const int64_t parts = (dim + kPartCols - 1) / kPartCols;
    // (an entry of big[], one for each kBigLong pairs at most, takes 8 bytes)
    const int64_t most_pieces = cap / kPieceMin + 1, area = cap / kLongSegment + 1;
    const int64_t most_long = cap / kListLong + 1;
    constexpr int64_t kHead = sizeof(int4);
    WsLayout l;
    l.heads = 0;
    l.big = l.heads + al(kListBlocksSmall * kHead);
    l.longs = l.big + al(most_pieces * 16);
    l.seg_done = l.longs + al(area * 16);
    l.partial = l.seg_done + al((cap / kSplitPairs + 1) * parts * 4);
    l.total = l.partial + al(most_pieces * dim * 4);
    l.list_blocks = kListBlocksSmall;
    if (al(most_long * 8) + kListBlocks * kHead <= al(area * 16)) {
        l.heads = l.longs + al(most_long * 8);
        l.list_blocks = kListBlocks;
    }
    return l;
}

// The workspace in `bytes` at `ws`: it covers the largest cap (below 2^31)
// whose layout fits; cap 0 (no workspace) if ws is null or not even
// kLongSegment pairs fit.
SplitWs make_split_ws(void *ws, size_t bytes, int32_t dim) {
    SplitWs s{nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0,
              (dim + kPartCols - 1) / kPartCols, nullptr};
    if (ws == nullptr || ws_layout(kLongSegment, dim).total > bytes) return s;
    int64_t lo = kLongSegment, hi = (int64_t(1) << 31) - 1;
    while (lo < hi) {  // largest cap whose layout fits
        const int64_t mid = lo + (hi - lo + 1) / 2;
        if (ws_layout(mid, dim).total <= bytes) lo = mid; else hi = mid - 1;
    }
    const WsLayout l = ws_layout(lo, dim);
    char *p = static_cast<char *>(ws);
    s.heads = reinterpret_cast<int4 *>(p + l.heads);
    s.big = reinterpret_cast<int2 *>(p + l.big);
    s.longs = reinterpret_cast<int2 *>(p + l.longs);
    s.seg_done = reinterpret_cast<int32_t *>(p + l.seg_done);
    s.partial = reinterpret_cast<float *>(p + l.partial);
    s.cap_pairs = lo;
    s.list_blocks = l.list_blocks;
    // the start of the workspace, where the heads are if there are few
    if (l.heads != 0) s.turns = reinterpret_cast<int32_t *>(p);
    return s;
}

tc_status launch_backward(const float *grad, int64_t grad_rows, int32_t dim,
                          const int32_t *ids, const int32_t *offsets,
                          const int32_t *num_out_dev, int64_t cap, const RowSink &out,
                          const SplitWs &ws, hipStream_t stream) {
    // the chains address rows from the start of grad when it fits in a
    // 32-bit buffer window with kOutOfRange past its end
    const int64_t gb = grad_rows * int64_t(dim) * 4;
    const int32_t grad_bytes = gb <= kOutOfRange ? int32_t(gb) : 0;
    const RowShape s = row_shape(dim);
    const int64_t rows_per_block = (kBlock / kWave) * (kWave / s.lanes);
    const unsigned grid = grid_for(cap, rows_per_block, int64_t(device_cus()) * 8);
    unsigned all_blocks = grid;
    if (ws.cap_pairs > 0) {
        k_backward_list<<<grid_for(cap, kListThreads, ws.list_blocks), kListThreads, 0, stream>>>(
            offsets, num_out_dev, cap, ws);
        const tc_status st = check_launch("k_backward_list");
        if (st != TC_OK) return st;
        // room for the most chains there can be, in whole rounds over the XCDs
        const int64_t most = (ws.cap_pairs / kListLong + 1) * ws.parts;
        const int64_t rounds = most / kXcds + 2;
        all_blocks = grid_for(grid + rounds * kXcds, 1, int64_t(device_cus()) * 8);
    }
    bool launched = false;
#define TC_BWD_CASE(L, C)                                                                    \
    if (!launched && s.lanes == L && s.chunks == C) {                                        \
        if (ws.cap_pairs > 0) {                                                              \
            const bool parts = ws.turns && sweep_in_parts<L>(cap, int32_t(all_blocks));      \
            k_backward_rows<L, C><<<parts ? kTurns * all_blocks : all_blocks, kBlock, 0,     \
                                    stream>>>(grad, dim, ids, offsets, num_out_dev, cap,     \
                                              out, ws, grad_bytes, device_cus(),             \
                                              int32_t(all_blocks));                          \
        } else                                                                               \
            k_backward_short<L, C><<<grid, kBlock, 0, stream>>>(grad, dim, ids, offsets,     \
                                                                num_out_dev, cap, out);      \
        launched = true;                                                                     \
    }
    TC_BWD_CASE(1, 1)
    TC_BWD_CASE(2, 1)
    TC_BWD_CASE(4, 1)
    TC_BWD_CASE(8, 1)
    TC_BWD_CASE(16, 1)
    TC_BWD_CASE(32, 1)
    TC_BWD_CASE(64, 1)
    TC_BWD_CASE(64, 2)
    TC_BWD_CASE(64, 3)
    TC_BWD_CASE(64, 4)
#undef TC_BWD_CASE
    if (!launched) {
        set_error("no backward kernel for dim %d", dim);
        return TC_ERR_UNSUPPORTED;
    }
    const tc_status st = check_launch(ws.cap_pairs > 0 ? "k_backward_rows" : "k_backward_short");
    if (st != TC_OK || ws.cap_pairs > 0) return st;
    const int parts = (dim + kPartCols - 1) / kPartCols;
    const int ranges = kLongRanges / parts > 64 ? kLongRanges / parts : 64;
    k_backward_long<<<dim3(ranges, parts), kLongThreads, 0, stream>>>(grad, dim, ids, offsets,
                                                                       num_out_dev, cap, out,
                                                                       grad_bytes);
    return check_launch("k_backward_long");
}

}  // namespace
}  // namespace tc

using namespace tc;

extern "C" tc_status tc_embed_backward(const float *grad_out, int32_t num_bags, int32_t dim,
                                       const int32_t *seg_offsets, const int32_t *casted_src,
                                       const int32_t *num_unique, int64_t max_unique,
                                       float *coal_grad, void *workspace,
                                       size_t workspace_bytes, hipStream_t stream) {
    clear_error();
    TC_REQUIRE(num_bags >= 0 && max_unique >= 0, TC_ERR_INVALID_ARG,
               "tc_embed_backward: negative size");
    TC_REQUIRE(max_unique < (int64_t(1) << 31), TC_ERR_INVALID_ARG,
               "tc_embed_backward: max_unique must be below 2^31");
    TC_REQUIRE(dim > 0 && dim % 4 == 0 && dim <= kMaxDim, TC_ERR_UNSUPPORTED,
               "tc_embed_backward: dim %d must be a multiple of 4 in [4, %d]", dim, kMaxDim);
    if (max_unique == 0) return TC_OK;
    TC_REQUIRE(grad_out && seg_offsets && casted_src && num_unique && coal_grad,
               TC_ERR_INVALID_ARG, "tc_embed_backward: null pointer");
    TC_REQUIRE(aligned16(grad_out) && aligned16(coal_grad), TC_ERR_UNSUPPORTED,
               "tc_embed_backward: grad_out and coal_grad must be 16-byte aligned");
    TC_REQUIRE(workspace_bytes == 0 || (workspace && aligned16(workspace)), TC_ERR_INVALID_ARG,
               "tc_embed_backward: workspace must be a 16-byte aligned pointer");
    const RowSink sink{coal_grad, nullptr, nullptr, nullptr, TC_OPT_SGD, 0.f, 0.f, 0.f, 1.f};
    return launch_backward(grad_out, num_bags, dim, casted_src, seg_offsets, num_unique,
                           max_unique, sink, make_split_ws(workspace, workspace_bytes, dim),
                           stream);
}

namespace tc {

// The no-allocation entry point's backward workspace: a fixed array in
// device memory, one copy per GPU, held until the process ends. Host code
// never passes `scratch` itself to a kernel (in host code the name is a
// stand-in, not a device address): it looks up the array's address on each
// device once and passes that.
constexpr size_t kScratchBytes = TC_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

// Argument checks shared by the two backward + update entry points (`what`
// names the caller in messages).
tc_status check_backward_update(const char *what, const float *grad_out, int32_t num_bags,
                                int32_t dim, const int32_t *seg_offsets,
                                const int32_t *casted_src, const int32_t *unique_rows,
                                const int32_t *num_unique, int64_t max_unique, const float *W,
                                const float *opt_state, int64_t total_rows, int32_t opt_kind,
                                float gamma, const float *coal_grad) {
    TC_REQUIRE(num_bags >= 0 && max_unique >= 0 && total_rows >= 0, TC_ERR_INVALID_ARG,
               "%s: negative size", what);
    TC_REQUIRE(max_unique < (int64_t(1) << 31) && total_rows < (int64_t(1) << 31),
               TC_ERR_INVALID_ARG, "%s: sizes must be below 2^31", what);
    TC_REQUIRE(dim > 0 && dim % 4 == 0 && dim <= kMaxDim, TC_ERR_UNSUPPORTED,
               "%s: dim %d must be a multiple of 4 in [4, %d]", what, dim, kMaxDim);
    TC_REQUIRE(opt_kind >= TC_OPT_SGD && opt_kind <= TC_OPT_ROWWISE_ADAGRAD, TC_ERR_INVALID_ARG,
               "%s: unknown optimizer %d", what, opt_kind);
    TC_REQUIRE(opt_kind != TC_OPT_ROWWISE_ADAGRAD, TC_ERR_UNSUPPORTED,
               "%s: row-wise Adagrad needs whole rows; use tc_embed_backward and "
               "tc_sparse_update", what);
    TC_REQUIRE((opt_kind == TC_OPT_SGD) == (opt_state == nullptr), TC_ERR_INVALID_ARG,
               "%s: opt_state must be NULL for SGD and given otherwise", what);
    TC_REQUIRE(opt_kind != TC_OPT_RMSPROP || (gamma >= 0.f && gamma <= 1.f), TC_ERR_INVALID_ARG,
               "%s: RMSprop gamma must lie in [0, 1]", what);
    if (max_unique == 0) return TC_OK;
    TC_REQUIRE(grad_out && seg_offsets && casted_src && unique_rows && num_unique && W,
               TC_ERR_INVALID_ARG, "%s: null pointer", what);
    TC_REQUIRE(aligned16(grad_out) && aligned16(W) && (!opt_state || aligned16(opt_state)) &&
                   (!coal_grad || aligned16(coal_grad)),
               TC_ERR_UNSUPPORTED, "%s: float pointers must be 16-byte aligned", what);
    return TC_OK;
}

// Address of `scratch` on the current device (hipGetSymbolAddress with that
// device current, looked up once per device), or nullptr with the error set.
void *scratch_address() {
    constexpr int kMaxDevices = 64;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_error("tc_embed_backward_update_noalloc: hipGetDevice: %s", hipGetErrorString(e));
        return nullptr;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        set_error("tc_embed_backward_update_noalloc: device %d beyond the %d supported", dev,
                  kMaxDevices);
        return nullptr;
    }
    void *p = __atomic_load_n(&addr[dev], __ATOMIC_ACQUIRE);
    if (p) return p;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) {
        set_error("tc_embed_backward_update_noalloc: hipGetSymbolAddress(scratch): %s",
                  hipGetErrorString(e));
        return nullptr;
    }
    __atomic_store_n(&addr[dev], p, __ATOMIC_RELEASE);
    return p;
}

}  // namespace
}  // namespace tc

extern "C" tc_status tc_embed_backward_update(
    const float *grad_out, int32_t num_bags, int32_t dim, const int32_t *seg_offsets,
    const int32_t *casted_src, const int32_t *unique_rows, const int32_t *num_unique,
    int64_t max_unique, float *W, float *opt_state, int64_t total_rows, int32_t opt_kind,
    float lr, float eps, float gamma, float *coal_grad, void *workspace, size_t workspace_bytes,
    hipStream_t stream) {
    clear_error();
    const tc_status st = check_backward_update(
        "tc_embed_backward_update", grad_out, num_bags, dim, seg_offsets, casted_src,
        unique_rows, num_unique, max_unique, W, opt_state, total_rows, opt_kind, gamma,
        coal_grad);
    if (st != TC_OK || max_unique == 0) return st;
    TC_REQUIRE(workspace_bytes == 0 || (workspace && aligned16(workspace)), TC_ERR_INVALID_ARG,
               "tc_embed_backward_update: workspace must be a 16-byte aligned pointer");
    const RowSink sink{coal_grad, W, opt_state, unique_rows, opt_kind, lr, eps, gamma,
                       1.0f - gamma};
    return launch_backward(grad_out, num_bags, dim, casted_src, seg_offsets, num_unique,
                           max_unique, sink, make_split_ws(workspace, workspace_bytes, dim),
                           stream);
}

extern "C" tc_status tc_embed_backward_update_noalloc(
    const float *grad_out, int32_t num_bags, int32_t dim, const int32_t *seg_offsets,
    const int32_t *casted_src, const int32_t *unique_rows, const int32_t *num_unique,
    int64_t max_unique, int64_t num_pairs, float *W, float *opt_state, int64_t total_rows,
    int32_t opt_kind, float lr, float eps, float gamma, float *coal_grad, hipStream_t stream) {
    clear_error();
    const tc_status st = check_backward_update(
        "tc_embed_backward_update_noalloc", grad_out, num_bags, dim, seg_offsets, casted_src,
        unique_rows, num_unique, max_unique, W, opt_state, total_rows, opt_kind, gamma,
        coal_grad);
    if (st != TC_OK) return st;
    TC_REQUIRE(num_pairs >= 0 && num_pairs < (int64_t(1) << 31), TC_ERR_INVALID_ARG,
               "tc_embed_backward_update_noalloc: num_pairs must lie in [0, 2^31)");
    const size_t need = num_pairs < kLongSegment ? 0 : ws_layout(num_pairs, dim).total;
    TC_REQUIRE(need <= kScratchBytes, TC_ERR_WORKSPACE,
               "tc_embed_backward_update_noalloc: %lld pairs of dim %d need %zu bytes of "
               "backward workspace, more than the %zu-byte scratch (TC_NOALLOC_SCRATCH_BYTES); "
               "use tc_embed_backward_update with a workspace",
               static_cast<long long>(num_pairs), dim, need, kScratchBytes);
    if (max_unique == 0) return TC_OK;
    void *ws = scratch_address();
    if (ws == nullptr) return TC_ERR_HIP;
    const RowSink sink{coal_grad, W, opt_state, unique_rows, opt_kind, lr, eps, gamma,
                       1.0f - gamma};
    return launch_backward(grad_out, num_bags, dim, casted_src, seg_offsets, num_unique,
                           max_unique, sink, make_split_ws(ws, kScratchBytes, dim), stream);
}

extern "C" tc_status tc_embed_expand(const float *grad_out, int32_t num_bags, int32_t dim,
                                     const int32_t *bag_offsets, int64_t num_pairs,
                                     float *expanded, hipStream_t stream) {
    clear_error();
    TC_REQUIRE(num_bags >= 0 && num_pairs >= 0, TC_ERR_INVALID_ARG,
               "tc_embed_expand: negative size");
    TC_REQUIRE(num_pairs < (int64_t(1) << 31), TC_ERR_INVALID_ARG,
               "tc_embed_expand: num_pairs must be below 2^31");
    TC_REQUIRE(dim > 0 && dim % 4 == 0 && dim <= kMaxDim, TC_ERR_UNSUPPORTED,
               "tc_embed_expand: dim %d must be a multiple of 4 in [4, %d]", dim, kMaxDim);
    if (num_bags == 0 || num_pairs == 0) return TC_OK;
    TC_REQUIRE(grad_out && bag_offsets && expanded, TC_ERR_INVALID_ARG,
               "tc_embed_expand: null pointer");
    TC_REQUIRE(aligned16(grad_out) && aligned16(expanded), TC_ERR_UNSUPPORTED,
               "tc_embed_expand: grad_out and expanded must be 16-byte aligned");
    return launch_expand(grad_out, dim, bag_offsets, num_bags, expanded, stream);
}

extern "C" tc_status tc_embed_coalesce(const float *expanded, int64_t num_pairs, int32_t dim,
                                       const int32_t *seg_offsets, const int32_t *sorted_pos,
                                       const int32_t *num_unique, int64_t max_unique,
                                       float *coal_grad, void *workspace,
                                       size_t workspace_bytes, hipStream_t stream) {
    clear_error();
    TC_REQUIRE(num_pairs >= 0 && max_unique >= 0, TC_ERR_INVALID_ARG,
               "tc_embed_coalesce: negative size");
    TC_REQUIRE(num_pairs < (int64_t(1) << 31) && max_unique < (int64_t(1) << 31),
               TC_ERR_INVALID_ARG, "tc_embed_coalesce: sizes must be below 2^31");
    TC_REQUIRE(dim > 0 && dim % 4 == 0 && dim <= kMaxDim, TC_ERR_UNSUPPORTED,
               "tc_embed_coalesce: dim %d must be a multiple of 4 in [4, %d]", dim, kMaxDim);
    if (max_unique == 0) return TC_OK;
    TC_REQUIRE(expanded && seg_offsets && sorted_pos && num_unique && coal_grad,
               TC_ERR_INVALID_ARG, "tc_embed_coalesce: null pointer");
    TC_REQUIRE(aligned16(expanded) && aligned16(coal_grad), TC_ERR_UNSUPPORTED,
               "tc_embed_coalesce: expanded and coal_grad must be 16-byte aligned");
    TC_REQUIRE(workspace_bytes == 0 || (workspace && aligned16(workspace)), TC_ERR_INVALID_ARG,
               "tc_embed_coalesce: workspace must be a 16-byte aligned pointer");
    // Algorithm 1's accumulate is the casted gather-reduce over the expanded
    // rows, in sorted order: the same kernels with sorted positions as ids.
    const RowSink sink{coal_grad, nullptr, nullptr, nullptr, TC_OPT_SGD, 0.f, 0.f, 0.f, 1.f};
    return launch_backward(expanded, num_pairs, dim, sorted_pos, seg_offsets, num_unique,
                           max_unique, sink, make_split_ws(workspace, workspace_bytes, dim),
                           stream);
}

extern "C" size_t tc_backward_workspace_bytes(int64_t num_pairs, int32_t dim) {
    if (num_pairs < kLongSegment || dim <= 0 || dim > kMaxDim ||
        num_pairs >= (int64_t(1) << 31))
        return 0;
    return ws_layout(num_pairs, dim).total;
}
