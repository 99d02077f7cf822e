// e2eg_normalize: d~_i = sum_j A~_ij and d~_i^-1/2 (paper: Section 3, "Notation"), and the
// schedule that the propagation kernels read (layout and the two forms of it: common.h).
//
// In both forms the kTopNodes nodes of highest degree, by descending degree (ties in node order), are
// "popular": every neighbour list starts with its popular entries, by popularity, and keeps the
// caller's order behind them.
//
// Large form: renumbered private copy.  The popular nodes get internal ids 0, 1, ...; all others follow
// in node order.  What this buys on a power-law user-item graph:
//   - the feature rows of the most popular nodes are one contiguous block (window 0);
//   - everything else keeps the caller's node order (users, then items), so at any time the
//     whole GPU gathers from the same side of the graph and the L2 caches hold one hot set.
// Because only kTopNodes nodes leave the node order, a row of the copy is a partition of the caller's
// row and an ordering of the popular part, not a sort of the whole: rows of up to kSegLen entries are
// a wavefront's work in registers, longer ones find their places from a bit per entry and a rank
// directory over those bits (running counts per tile and per 64 entries).  A row's popular part is
// ordered through a bitmap of kTopNodes bits in LDS: an entry's place is the number of bits below its
// own.  (The radix sort of (row, column) keys that this replaces moved 16 bytes per entry six times.)
//
// Small form (at most kSmallNnz stored entries: the subgraph of a mini-batch step, whose schedule
// serves one step): rows keep their node ids, four launches do everything.  What bounds it is the number of
// launches: a graph of 175 k nodes and 700 k entries took some 60 of them when it was made like a large
// one.
//
// Work lists: rows of at most kShortMax entries are listed ordered by length inside blocks of
// kSortBlock consecutive rows (the kernel sums several of them side by side, so neighbours in the list
// should be equally long, while the block-wise order keeps the users-then-items progression).
// Longer rows are cut into segments of kSegLen entries, the very longest ones of a large graph first
// at the boundaries of windows of kWindow internal ids; the segments of rows with several are
// ordered by the window of their first column, so that segments which read the same stretch of feature
// rows can be run at the same time on the same L2 (the list is dealt out to the XCDs in contiguous
// stretches of equal entry counts).
// All of it is integer work with results that do not depend on scheduling.  Nothing here depends on
// the feature width.  For a weighted graph (e2eg_normalize_weighted) d~ is the sum of the row's
// values and the values are carried into the schedule in the order of its column indices.
#include "entry_tiles.h"

namespace e2eg {
namespace {

constexpr int kThreads = kEntryThreads;
// The symmetry test of a large graph keeps a flag (asym[0]) and a count spread over kSymCounters
// addresses, one cache line each (asym[k * kSymStride], k = 1 .. kSymCounters).
constexpr int kSymCounters = 64;
constexpr int kSymStride = 32;
constexpr int kLengthCutCost = 6;   // in quarters: an entry of a segment cut by length only weighs 1.5 entries in the deal

inline dim3 grid_for(int64_t count) { return dim3((unsigned)ceil_div(count > 0 ? count : 1, kThreads)); }

// ---- row tiles ---------------------------------------------------------------------------------
// Row work goes by tiles of kSortBlock rows, one workgroup each; every workgroup adds up what the
// tiles before it counted, which saves the launches of a scan (a few thousand tiles at most).
// (Small form: tiles of a quarter of that, or a graph of 170 k nodes fills 43 compute units.)
template <bool SMALL>
constexpr int kTileRows = SMALL ? kSortBlock / 4 : kSortBlock;
constexpr int kTileThreads = 512;
constexpr int kTileWaves = kTileThreads / 64;
template <bool SMALL>
constexpr int kWaveRows = kTileRows<SMALL> / kTileWaves;   // consecutive rows of one wavefront
template <bool SMALL>
constexpr int kRowRounds = kWaveRows<SMALL> / 64;
constexpr int kTotals = 8;   // per tile: entries, short rows, one-segment rows, split rows, slots, chunks
enum { kTotEntries, kTotShort, kTotSingle, kTotMulti, kTotSlots, kTotChunks, kTotUsed };
constexpr int kChunk = 2048;   // large form: entries of a split row that one workgroup puts in place

// Sums of K values per thread over the workgroup, in every thread.
template <int K>
__device__ __forceinline__ void block_sums(int32_t (&v)[K], int32_t (*lds)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k)
        for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) lds[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int32_t t = 0;
#pragma unroll
        for (int w = 0; w < kTileWaves; ++w) t += lds[w][k];
        v[k] = t;
    }
}

// Row classes by length d:  short d <= kShortMax;  one segment up to kSegLen;  split beyond.  A split
// row is cut by length, or, wide (one of the first wide_rows internal rows, at least wide_min
// entries), at window boundaries first; wide rows get their slots later.
__device__ __forceinline__ void count_row(int32_t d, int64_t p, int32_t wide_rows, int32_t wide_min,
                                          int32_t (&tot)[kTotUsed]) {
    tot[kTotEntries] += d;
    tot[kTotShort] += d <= kShortMax ? 1 : 0;
    tot[kTotSingle] += d > kShortMax && d <= kSegLen ? 1 : 0;
    tot[kTotMulti] += d > kSegLen ? 1 : 0;
    if (d > kSegLen) {
        tot[kTotChunks] += (d + kChunk - 1) / kChunk;
        if (!(p < wide_rows && d >= wide_min)) tot[kTotSlots] += (d + kSegLen - 1) / kSegLen;
    }
}

// Classes of degrees for choosing the most popular nodes: exact up to 63, then 2^OCT to an octave.  Large
// graphs take 32 to an octave; small ones, which keep a histogram per tile, 8.
template <int OCT>
constexpr int kClasses = 64 + (25 << OCT);
constexpr int kLargeOct = 5, kSmallOct = 3;
template <int OCT>
__device__ __forceinline__ int degree_class(int32_t d) {
    if (d < 64) return d;
    const int e = 31 - __clz(d);
    return 64 + ((e - 6) << OCT) + ((d >> (e - OCT)) & ((1 << OCT) - 1));
}

// Per node: degree and d^-1/2, and the histogram of degree classes: of the whole graph, or (PER_TILE) of
// every tile, which needs no cleared memory and saves count_top.  Small form: also the tile's totals (the
// internal row is the node).
template <bool SMALL, bool PER_TILE, int OCT>
__global__ __launch_bounds__(kTileThreads) void row_stats(const int32_t* __restrict__ row_ptr, int64_t n,
                                                          int32_t* __restrict__ deg, float* __restrict__ dinv_sqrt,
                                                          int32_t* __restrict__ totals, int32_t* __restrict__ classes) {
    __shared__ int32_t red[kTileWaves][kTotUsed];
    __shared__ int32_t hist[kClasses<OCT>];
    for (int k = threadIdx.x; k < kClasses<OCT>; k += kTileThreads) hist[k] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    int32_t tot[kTotUsed] = {};
    const int64_t base = (int64_t)blockIdx.x * kTileRows<SMALL>;
#pragma unroll
    for (int r = 0; r < kTileRows<SMALL> / kTileThreads; ++r) {
        const int64_t i = base + r * kTileThreads + threadIdx.x;
        int c = -1;
        if (i < n) {
            const int32_t d = row_ptr[i + 1] - row_ptr[i];
            if (deg) deg[i] = d;
            dinv_sqrt[i] = d > 0 ? (float)(1.0 / sqrt((double)d)) : 0.0f;
            if (SMALL) count_row(d, i, 0, 0, tot);
            c = degree_class<OCT>(d);
        }
        // most rows of a sampled subgraph have the same one or two lengths: those are counted by ballot (64
        // atomics on one LDS word take their turns), the rest one by one
        uint64_t left = __ballot(c >= 0);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (left == 0) break;
            const int leader = __ffsll((unsigned long long)left) - 1;
            const int lc = __shfl(c, leader);
            const uint64_t same = __ballot(c == lc);
            if (lane == leader) atomicAdd(&hist[lc], __popcll(same));
            left &= ~same;
        }
        if ((left >> lane) & 1) atomicAdd(&hist[c], 1);
    }
    if (SMALL) {
        block_sums<kTotUsed>(tot, red);
        if (threadIdx.x == 0)
            for (int k = 0; k < kTotUsed; ++k) totals[(int64_t)blockIdx.x * kTotals + k] = tot[k];
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kClasses<OCT>; k += kTileThreads) {
        if (PER_TILE) classes[(int64_t)blockIdx.x * kClasses<OCT> + k] = hist[k];
        else if (hist[k] != 0) atomicAdd(classes + k, hist[k]);
    }
}

// Large form: the tile's totals over internal rows.
__global__ __launch_bounds__(kTileThreads) void row_totals(const int32_t* __restrict__ zdeg, int64_t n,
                                                           int32_t wide_rows, int32_t wide_min,
                                                           int32_t* __restrict__ totals) {
    __shared__ int32_t red[kTileWaves][kTotUsed];
    int32_t tot[kTotUsed] = {};
    const int64_t base = (int64_t)blockIdx.x * kTileRows<false>;
#pragma unroll
    for (int r = 0; r < kTileRows<false> / kTileThreads; ++r) {
        const int64_t p = base + r * kTileThreads + threadIdx.x;
        if (p < n) count_row(zdeg[p], p, wide_rows, wide_min, tot);
    }
    block_sums<kTotUsed>(tot, red);
    if (threadIdx.x == 0)
        for (int k = 0; k < kTotUsed; ++k) totals[(int64_t)blockIdx.x * kTotals + k] = tot[k];
}

// ---- the most popular nodes -------------------------------------------------------------------------
// Which nodes are popular follows from the histogram of degree classes: every node of a class above the
// threshold class, and, in node order, as many of the threshold class as there is room for.
struct Threshold {
    int32_t cls;     // the threshold class
    int32_t above;   // nodes of higher classes
};
// `classes` may be in LDS.
template <int OCT>
__device__ __forceinline__ Threshold find_threshold(const int32_t* classes, int32_t* lds) {
    __shared__ Threshold found;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    static_assert(kTileThreads * 2 >= kClasses<OCT>, "two classes per thread");
    // thread t: the classes 2 t and 2 t + 1 from the top, scanned over the workgroup
    const int hi = kClasses<OCT> - 1 - 2 * (int)threadIdx.x;
    const int32_t c0 = hi >= 0 ? classes[hi] : 0, c1 = hi >= 1 ? classes[hi - 1] : 0;
    int32_t inc = c0 + c1;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const int32_t t = __shfl_up(inc, dlt, 64);
        if (lane >= dlt) inc += t;
    }
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    int32_t all = 0;
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) {
        if (w < wave) inc += lds[w];
        all += lds[w];
    }
    const int32_t b0 = inc - c0 - c1, b1 = inc - c1;   // nodes above each of the two classes
    if (hi >= 0 && b0 < kTopNodes && b0 + c0 >= kTopNodes) found = Threshold{hi, b0};
    if (hi >= 1 && b1 < kTopNodes && b1 + c1 >= kTopNodes) found = Threshold{hi - 1, b1};
    if (threadIdx.x == 0 && all < kTopNodes) found = Threshold{-1, all};   // all of them are above
    __syncthreads();
    const Threshold t = found;
    __syncthreads();
    return t;
}

// Per tile of nodes: how many lie above the threshold class, how many in it.
template <bool SMALL, int OCT>
__global__ __launch_bounds__(kTileThreads) void count_top(const int32_t* __restrict__ row_ptr, int64_t n,
                                                          const int32_t* __restrict__ classes,
                                                          int32_t* __restrict__ top_totals) {
    __shared__ int32_t red[kTileWaves][2];
    __shared__ int32_t lds[kTileWaves];
    const Threshold th = find_threshold<OCT>(classes, lds);
    int32_t v[2] = {0, 0};
    const int64_t base = (int64_t)blockIdx.x * kTileRows<SMALL>;
#pragma unroll
    for (int r = 0; r < kTileRows<SMALL> / kTileThreads; ++r) {
        const int64_t i = base + r * kTileThreads + threadIdx.x;
        if (i < n) {
            const int c = degree_class<OCT>(row_ptr[i + 1] - row_ptr[i]);
            v[0] += c > th.cls ? 1 : 0;
            v[1] += c == th.cls ? 1 : 0;
        }
    }
    block_sums<2>(v, red);
    if (threadIdx.x == 0) {
        top_totals[2 * (int64_t)blockIdx.x] = v[0];
        top_totals[2 * (int64_t)blockIdx.x + 1] = v[1];
    }
}

// What the entry passes need of a column, in one 8-byte gather (two gathers, of position and scale, made
// order_rows 983 us on 101 M entries, 58 M of them in its rows).
struct alignas(8) NodeInfo {
    int32_t pos;   // large form: internal position (below kTopNodes: the rank of a popular node); small: rank, or kTopNodes
    float dinv;    // d~^-1/2
};
struct TopOut {
    int32_t* node;      // [kTopNodes] the popular nodes in node order
    int32_t* deg;       // [kTopNodes] and their degrees
    NodeInfo* info;     // [n]
    int32_t* zdeg;      // [n] large form: row lengths by internal row
    uint64_t* is_top;   // large form: a bit per node
};

// One tile of nodes; before[0], before[1]: nodes above the threshold class and in it in earlier tiles.
// Large form: internal positions of the nodes that are not popular (behind the popular ones, in node order).
template <bool SMALL>
__device__ __forceinline__ void number_tile(const int32_t* __restrict__ row_ptr, const float* __restrict__ dinv_sqrt,
                                            int64_t n, const Threshold th,
                                            int32_t (&before)[2], const SchedView& s, const TopOut& out,
                                            int32_t (*red)[2]) {
    const int32_t room = kTopNodes - th.above;   // popular nodes of the threshold class
    const int32_t n_top = n < kTopNodes ? (int32_t)n : kTopNodes;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t base = (int64_t)blockIdx.x * kTileRows<SMALL> + wave * kWaveRows<SMALL>;
    int32_t d[kRowRounds<SMALL>];
    uint64_t above[kRowRounds<SMALL>], tied[kRowRounds<SMALL>];
    int32_t run[2] = {0, 0};
#pragma unroll
    for (int r = 0; r < kRowRounds<SMALL>; ++r) {
        const int64_t i = base + r * 64 + lane;
        d[r] = i < n ? row_ptr[i + 1] - row_ptr[i] : 0;
        const int c = i < n ? degree_class<SMALL ? kSmallOct : kLargeOct>(d[r]) : -2;
        above[r] = __ballot(c > th.cls);
        tied[r] = __ballot(c == th.cls);
        run[0] += __popcll(above[r]);
        run[1] += __popcll(tied[r]);
    }
    __syncthreads();
    if (lane == 0) {
        red[wave][0] = run[0];
        red[wave][1] = run[1];
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w)
        if (w < wave) {
            before[0] += red[w][0];
            before[1] += red[w][1];
        }
#pragma unroll
    for (int r = 0; r < kRowRounds<SMALL>; ++r) {
        const int64_t i = base + r * 64 + lane;
        const int32_t a = before[0] + __popcll(above[r] & lt_mask), t = before[1] + __popcll(tied[r] & lt_mask);
        const int32_t top_before = a + (t < room ? t : room);
        const bool top = ((above[r] >> lane) & 1) || (((tied[r] >> lane) & 1) && t < room);
        const uint64_t bits = __ballot(top);
        if (i < n) {
            if (!SMALL && lane == 0) out.is_top[i >> 6] = bits;
            if (top) {
                out.node[top_before] = (int32_t)i;
                out.deg[top_before] = d[r];
            } else if (SMALL) {
                out.info[i] = NodeInfo{kTopNodes, dinv_sqrt[i]};
            } else {
                const int32_t p = n_top + (int32_t)i - top_before;
                s.orig[p] = (int32_t)i;
                out.info[i] = NodeInfo{p, dinv_sqrt[i]};
                out.zdeg[p] = d[r];
            }
        }
        before[0] += __popcll(above[r]);
        before[1] += __popcll(tied[r]);
    }
}

template <bool SMALL, int OCT>
__global__ __launch_bounds__(kTileThreads) void number_nodes(const int32_t* __restrict__ row_ptr,
                                                             const float* __restrict__ dinv_sqrt, int64_t n,
                                                             const int32_t* __restrict__ classes,
                                                             const int32_t* __restrict__ top_totals, SchedView s, TopOut out) {
    __shared__ int32_t red[kTileWaves][2];
    __shared__ int32_t lds[kTileWaves];
    const Threshold th = find_threshold<OCT>(classes, lds);
    int32_t before[2] = {0, 0};
    for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kTileThreads) {
        before[0] += top_totals[2 * t];
        before[1] += top_totals[2 * t + 1];
    }
    block_sums<2>(before, red);
    number_tile<SMALL>(row_ptr, dinv_sqrt, n, th, before, s, out, red);
}

// A popular node's rank is the number of popular nodes of larger degree, or of equal degree and before it:
// kRankLanes lanes count for one node, over all degrees held in LDS.
constexpr int kRankLanes = 16;
constexpr int kRankThreads = 512;
template <bool SMALL>
__global__ __launch_bounds__(kRankThreads) void rank_top(int32_t n_top, const float* __restrict__ dinv_sqrt, SchedView s, TopOut out) {
    __shared__ __attribute__((aligned(16))) int32_t deg[kTopNodes];
    constexpr int kLoads = kTopNodes / 4 / kRankThreads;
#pragma unroll
    for (int r = 0; r < kLoads; ++r) {
        const int k = 4 * (r * kRankThreads + (int)threadIdx.x);
        int4 v = make_int4(-1, -1, -1, -1);   // past the end: of no larger degree than anybody
        if (k + 3 < n_top) {
            v = *reinterpret_cast<const int4*>(out.deg + k);
        } else {
            if (k < n_top) v.x = out.deg[k];
            if (k + 1 < n_top) v.y = out.deg[k + 1];
            if (k + 2 < n_top) v.z = out.deg[k + 2];
        }
        *reinterpret_cast<int4*>(deg + k) = v;
    }
    __syncthreads();
    const int c = blockIdx.x * (kRankThreads / kRankLanes) + (int)threadIdx.x / kRankLanes;
    const int32_t d = c < n_top ? deg[c] : 0;
    int32_t rank = 0;
    // One comparison each: node k comes before node c iff deg[k] + (k < c) > d, and k < c is the same for a whole
    // group of four but the one that holds c.
    const int c4 = c & ~3;
#pragma unroll 8
    for (int k = 4 * (threadIdx.x % kRankLanes); k < n_top; k += 4 * kRankLanes) {
        const int4 v = *reinterpret_cast<const int4*>(deg + k);
        const int32_t bar = k < c4 ? d - 1 : d;
        rank += (v.x > bar ? 1 : 0) + (v.y > bar ? 1 : 0) + (v.z > bar ? 1 : 0) + (v.w > bar ? 1 : 0);
    }
    if (threadIdx.x % kRankLanes == 0 && c < n_top)
        for (int k = c4; k < c; ++k) rank += deg[k] == d ? 1 : 0;
#pragma unroll
    for (int off = kRankLanes / 2; off > 0; off >>= 1) rank += __shfl_xor(rank, off);
    if (c < n_top && threadIdx.x % kRankLanes == 0) {
        const int32_t i = out.node[c];
        out.info[i] = NodeInfo{rank, dinv_sqrt[i]};
        if (!SMALL) {
            s.orig[rank] = i;
            out.zdeg[rank] = d;
        }
    }
}

// ---- work lists --------------------------------------------------------------------------------
// Large form: the split rows in pieces of kChunk entries.
struct Chunks {
    int32_t* split;   // [max_chunks] split row (its number) of every piece
    int32_t* first;   // [max_multi] first piece of every split row
    int32_t* tops;    // [max_chunks] popular entries in every piece (count_chunks)
    int64_t max_chunks;
};

// The tile's work lists.  Rows are ranked by a stable counting sort over 131 digits: the lengths of
// the short rows, then one digit for rows of one segment and one for split rows, which come out in row
// order.  Large form: also zrow_ptr (the small form has the caller's).  Split rows cut by length get
// their slots and segments here: in the small form the final list, in the large one seg_tmp, to be
// ordered by window once the columns are in place.  The last workgroup writes the header.
template <bool SMALL, bool NUMBER>
__global__ __launch_bounds__(kTileThreads) void emit_rows(const int32_t* __restrict__ row_ptr,
                                                          const int32_t* __restrict__ zdeg,
                                                          const float* __restrict__ dinv_sqrt, int64_t n, int64_t nnz,
                                                          int32_t wide_rows, int32_t wide_min,
                                                          const int32_t* __restrict__ totals, SchedView s,
                                                          Segment* __restrict__ seg_out, Chunks chunks,
                                                          const int32_t* __restrict__ classes, TopOut out) {
    constexpr int kDigits = 136;   // 0 .. 128 short lengths, 129 one segment, 130 split; 135: past the end
    __shared__ int32_t red[kTileWaves][2 * kTotUsed];
    __shared__ int32_t wave_cnt[kTileWaves][kDigits];
    __shared__ int32_t first[kDigits];     // place of the digit's first row in the tile
    __shared__ uint16_t sorted[kTileRows<SMALL>]; // rows of the tile in digit order
    __shared__ int32_t beg[kTileRows<SMALL>];     // first entry of every row of the tile
    __shared__ int32_t slot0[SMALL ? kTileRows<SMALL> : 1];   // split rows: first slot
    __shared__ int32_t wave_chunks[kTileWaves];
    constexpr int kThreadSegs = 8;
    __shared__ int32_t wave_tot[kTileWaves];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t base = (int64_t)blockIdx.x * kTileRows<SMALL>;
    const int rows = n - base < kTileRows<SMALL> ? (int)(n - base) : kTileRows<SMALL>;

    int32_t before[kTotUsed] = {};
    for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kTileThreads)
#pragma unroll
        for (int k = 0; k < kTotUsed; ++k) before[k] += totals[t * kTotals + k];
    block_sums<kTotUsed>(before, reinterpret_cast<int32_t(*)[kTotUsed]>(red));
    int32_t own[kTotUsed];
#pragma unroll
    for (int k = 0; k < kTotUsed; ++k) own[k] = totals[(int64_t)blockIdx.x * kTotals + k];

    for (int k = threadIdx.x; k < kTileWaves * kDigits; k += kTileThreads) (&wave_cnt[0][0])[k] = 0;
    __syncthreads();
    int32_t len[kRowRounds<SMALL>], rank[kRowRounds<SMALL>];
    int digit[kRowRounds<SMALL>];
#pragma unroll
    for (int r = 0; r < kRowRounds<SMALL>; ++r) {
        const int at = wave * kWaveRows<SMALL> + r * 64 + lane;
        const bool valid = at < rows;
        int32_t d = 0;
        if (valid) {
            if (SMALL) {
                const int32_t b = row_ptr[base + at];
                beg[at] = b;
                d = row_ptr[base + at + 1] - b;
            } else {
                d = zdeg[base + at];
            }
        }
        len[r] = d;
        const int g = !valid ? kDigits - 1 : d <= kShortMax ? d : d <= kSegLen ? kShortMax + 1 : kShortMax + 2;
        digit[r] = g;
        const uint64_t peers = lanes_of_digit<8>(g, 8, ~0ull);
        const int pre = wave_cnt[wave][g];
        const int below = __popcll(peers & lt_mask);
        rank[r] = pre + below;
        if (below == 0) wave_cnt[wave][g] = pre + __popcll(peers);
    }
    __syncthreads();
    if (threadIdx.x < 192) {   // exclusive scan over the digits (three wavefronts cover them)
        const int g = threadIdx.x;
        int mine = 0;
        if (g < kDigits)
#pragma unroll
            for (int w = 0; w < kTileWaves; ++w) mine += wave_cnt[w][g];
        int inc = mine;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const int t = __shfl_up(inc, dlt, 64);
            if (lane >= dlt) inc += t;
        }
        if (lane == 63) wave_tot[wave] = inc;
        if (g < kDigits) first[g] = inc - mine;
    }
    __syncthreads();
    if (threadIdx.x < kDigits) {
        const int g = threadIdx.x;
        int at = first[g];
        if (wave > 0) at += wave_tot[0];
        if (wave > 1) at += wave_tot[1];
        first[g] = at;
#pragma unroll
        for (int w = 0; w < kTileWaves; ++w) {
            const int c = wave_cnt[w][g];
            wave_cnt[w][g] = at;
            at += c;
        }
    }
    if (!SMALL) {   // zrow_ptr: a wavefront's rows are consecutive, 64 a round
        int32_t run = 0;
        int32_t inc[kRowRounds<SMALL>];
#pragma unroll
        for (int r = 0; r < kRowRounds<SMALL>; ++r) {
            int32_t v = len[r];
#pragma unroll
            for (int dlt = 1; dlt < 64; dlt <<= 1) {
                const int32_t t = __shfl_up(v, dlt, 64);
                if (lane >= dlt) v += t;
            }
            inc[r] = run + v - len[r];
            run += __shfl(v, 63);
        }
        __syncthreads();   // wave_tot has been read
        if (lane == 0) wave_tot[wave] = run;
        __syncthreads();
        int32_t off = before[kTotEntries];
#pragma unroll
        for (int w = 0; w < kTileWaves; ++w)
            if (w < wave) off += wave_tot[w];
#pragma unroll
        for (int r = 0; r < kRowRounds<SMALL>; ++r) {
            const int at = wave * kWaveRows<SMALL> + r * 64 + lane;
            if (at < rows) {
                beg[at] = off + inc[r];
                s.zrow_ptr[base + at] = off + inc[r];
            }
        }
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) s.zrow_ptr[n] = (int32_t)nnz;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRowRounds<SMALL>; ++r) {
        const int at = wave * kWaveRows<SMALL> + r * 64 + lane;
        if (at < rows) sorted[wave_cnt[wave][digit[r]] + rank[r]] = (uint16_t)at;
    }
    __syncthreads();
    const int n_short = own[kTotShort], n_single = own[kTotSingle], n_multi = own[kTotMulti];
    auto row_end = [&](int at) {   // one past the row's last entry
        if (SMALL) return row_ptr[base + at + 1];
        return at + 1 < rows ? beg[at + 1] : before[kTotEntries] + own[kTotEntries];
    };
    for (int k = threadIdx.x; k < n_short; k += kTileThreads) {
        const int at = sorted[k];
        const int32_t row = (int32_t)(base + at);
        s.short_rows[before[kTotShort] + k] = ShortRow{row, beg[at], row_end(at) - beg[at], SMALL ? row : s.orig[row]};
    }
    for (int k = threadIdx.x; k < n_single; k += kTileThreads) {
        const int at = sorted[n_short + k];
        s.singles[before[kTotSingle] + k] = Segment{(int32_t)(base + at), beg[at], row_end(at), -1};
    }
    if (n_multi > 0) {
        const uint16_t* multi = sorted + n_short + n_single;
        int32_t carry = 0;
        uint32_t carry_chunks = 0;
        for (int k0 = 0; k0 < n_multi; k0 += kTileThreads) {   // slots of the rows cut by length: a scan in row order
            const int k = k0 + threadIdx.x;
            int32_t cnt = 0, pieces = 0;
            if (k < n_multi) {
                const int at = multi[k];
                const int32_t d = row_end(at) - beg[at];
                pieces = (d + kChunk - 1) / kChunk;
                if (!(base + at < wide_rows && d >= wide_min)) cnt = (d + kSegLen - 1) / kSegLen;
            }
            int32_t v = cnt, pv = pieces;
#pragma unroll
            for (int dlt = 1; dlt < 64; dlt <<= 1) {
                const int32_t t = __shfl_up(v, dlt, 64), pt = __shfl_up(pv, dlt, 64);
                if (lane >= dlt) {
                    v += t;
                    pv += pt;
                }
            }
            __syncthreads();
            if (lane == 63) {
                wave_tot[wave] = v;
                wave_chunks[wave] = pv;
            }
            __syncthreads();
            int32_t off = carry + v - cnt, poff = carry_chunks + pv - pieces;
#pragma unroll
            for (int w = 0; w < kTileWaves; ++w) {
                if (w < wave) {
                    off += wave_tot[w];
                    poff += wave_chunks[w];
                }
                carry += wave_tot[w];
                carry_chunks += wave_chunks[w];
            }
            if (k < n_multi) {
                const int at = multi[k];
                const int32_t m = before[kTotMulti] + k, t0 = before[kTotSlots] + off;
                if (SMALL) slot0[k] = t0;
                s.multi_row[m] = (int32_t)(base + at);
                if (cnt > 0) {
                    s.slot_base[m] = t0;
                    s.slot_cnt[m] = cnt;
                }
                if (SMALL && cnt <= kThreadSegs) {   // few segments: by this thread
                    const int32_t b = beg[at], e = row_end(at);
                    for (int32_t q = 0; q < cnt; ++q) {
                        const int32_t sb = b + q * kSegLen;
                        seg_out[t0 + q] = Segment{(int32_t)(base + at), sb, sb + kSegLen < e ? sb + kSegLen : e, t0 + q};
                    }
                }
                if (!SMALL) chunks.first[m] = before[kTotChunks] + poff;
            }
        }
        __syncthreads();
        if (SMALL)
            for (int k = wave; k < n_multi; k += kTileWaves) {   // many: a wavefront per row, a lane per segment
                const int at = multi[k];
                const int32_t b = beg[at], e = row_end(at);
                if (e - b <= kThreadSegs * kSegLen) continue;
                for (int32_t q = lane; b + q * kSegLen < e; q += 64) {
                    const int32_t sb = b + q * kSegLen;
                    seg_out[slot0[k] + q] = Segment{(int32_t)(base + at), sb, sb + kSegLen < e ? sb + kSegLen : e, slot0[k] + q};
                }
            }
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        SchedHeader h = {};
        h.n_short = before[kTotShort] + n_short;
        h.n_single = before[kTotSingle] + n_single;
        h.n_multi = before[kTotMulti] + n_multi;
        h.n_slot = h.n_slot_plain = before[kTotSlots] + own[kTotSlots];   // large form: deal_segments adds the wide rows'
        h.n_chunks = before[kTotChunks] + own[kTotChunks];
        h.n = (int32_t)n;
        h.nnz = (int32_t)nnz;
        for (int x = 0; x <= kXcds; ++x) h.xcd_first[x] = (int32_t)((int64_t)h.n_slot * x / kXcds);
        *s.header = h;
    }
    if (NUMBER) {
        constexpr int kC = kClasses<kSmallOct>;
        static_assert(kC % 4 == 0, "read four at a time");
        constexpr int kParts = kTileThreads / (kC / 4);   // threads of one part sum every kParts-th tile
        __shared__ int32_t class_all[kC], class_before[kC];
        __shared__ int32_t red2[kTileWaves][2];
        for (int c = threadIdx.x; c < kC; c += kTileThreads) class_all[c] = class_before[c] = 0;
        __syncthreads();
        const int part = threadIdx.x / (kC / 4), c4 = 4 * (threadIdx.x % (kC / 4));
        if (part < kParts) {
            int4 all = make_int4(0, 0, 0, 0), bef = make_int4(0, 0, 0, 0);
#pragma unroll 8
            for (int t = part; t < (int)gridDim.x; t += kParts) {
                const int4 v = *reinterpret_cast<const int4*>(classes + (int64_t)t * kC + c4);
                const int m = t < (int)blockIdx.x ? 1 : 0;
                all.x += v.x; all.y += v.y; all.z += v.z; all.w += v.w;
                bef.x += m * v.x; bef.y += m * v.y; bef.z += m * v.z; bef.w += m * v.w;
            }
            const int32_t a4[4] = {all.x, all.y, all.z, all.w}, b4[4] = {bef.x, bef.y, bef.z, bef.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (a4[k] != 0) atomicAdd(&class_all[c4 + k], a4[k]);
                if (b4[k] != 0) atomicAdd(&class_before[c4 + k], b4[k]);
            }
        }
        __syncthreads();
        const Threshold th = find_threshold<kSmallOct>(class_all, wave_tot);
        int32_t counts[2] = {0, 0};
        for (int c = threadIdx.x; c < kC; c += kTileThreads) {
            counts[0] += c > th.cls ? class_before[c] : 0;
            counts[1] += c == th.cls ? class_before[c] : 0;
        }
        block_sums<2>(counts, red2);
        number_tile<true>(row_ptr, dinv_sqrt, n, th, counts, s, out, red2);
    }
}

// Large form: the pieces of the split rows, and the segments of those cut by length only, a wavefront per row (in
// emit_rows they are all one workgroup's, that of the popular nodes: 104 us instead of 20 on 101 M entries).
__global__ __launch_bounds__(kThreads) void emit_split(SchedView s, int32_t wide_rows, int32_t wide_min,
                                                       Segment* __restrict__ seg_out, Chunks chunks) {
    const int lane = threadIdx.x & 63;
    const int32_t n_multi = s.header->n_multi;
    const int32_t stride = gridDim.x * (kThreads / 64);
    for (int32_t m = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); m < n_multi; m += stride) {
        const int32_t p = s.multi_row[m], first = chunks.first[m];
        const int32_t b = s.zrow_ptr[p], e = s.zrow_ptr[p + 1];
        for (int32_t q = lane; b + q * kChunk < e; q += 64) chunks.split[first + q] = m;
        if (p < wide_rows && e - b >= wide_min) continue;
        const int32_t t0 = s.slot_base[m];
        for (int32_t q = lane; b + q * kSegLen < e; q += 64) {
            const int32_t sb = b + q * kSegLen;
            seg_out[t0 + q] = Segment{p, sb, sb + kSegLen < e ? sb + kSegLen : e, t0 + q};
        }
    }
}

// ---- entries ------------------------------------------------------------------------------------
// Where a row's popular entries go: a bitmap of their ranks; an entry's place is the number of bits below
// its own.
constexpr int kTopWords = kTopNodes / 32;
struct TopBitmap {
    uint32_t word[kTopWords];
    uint16_t below[kTopWords];   // bits set in the words before
    __device__ __forceinline__ void set(int32_t rank) { atomicOr(&word[rank >> 5], 1u << (rank & 31)); }
    __device__ __forceinline__ int32_t place(int32_t rank) const {
        return below[rank >> 5] + __popc(word[rank >> 5] & ((1u << (rank & 31)) - 1u));
    }
    // by one wavefront: -> the number of bits set
    __device__ __forceinline__ int32_t count(int lane) {
        constexpr int kPer = kTopWords / 64;
        int32_t c[kPer], mine = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            c[k] = mine;
            mine += __popc(word[lane * kPer + k]);
        }
        int32_t inc = mine;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const int32_t t = __shfl_up(inc, dlt, 64);
            if (lane >= dlt) inc += t;
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) below[lane * kPer + k] = (uint16_t)(inc - mine + c[k]);
        return __shfl(inc, 63);
    }
};

// Beside every column of the ordered lists go its node id and that node's d~^-1/2 (times the entry's
// value on a weighted graph): the first layer of a propagation reads these and gathers the caller's feature
// rows directly, which saves the pass that would pre-scale them.
template <bool SMALL>
__device__ __forceinline__ void put_entry(const SchedView& s, int32_t at, int32_t node, int32_t pos, float dinv, float v) {
    if (!SMALL) s.zcol[at] = pos;
    s.znode[at] = node;
    if (s.zval) s.zval[at] = v;
    s.zs[at] = s.zval ? v * dinv : dinv;
}

// Small form.  Workgroups below `tile_blocks`: the rows of up to kShortMax entries that begin in one tile of
// entries, a thread to every few entries; all keys of the tile stand in LDS (popular: the rank; others: in
// the caller's order behind them) and an entry's place in its row is the number of smaller ones.  The other
// workgroups take longer rows, one at a time: twice through the row, bitmap and counts, then places.  A
// row that lists a popular column twice has fewer bits than popular entries and keeps the caller's order
// among them.
constexpr int kSmallTile = 1024;
constexpr int kSmallRounds = (kSmallTile + kShortMax + kThreads - 1) / kThreads;
__global__ __launch_bounds__(kThreads) void order_small(const int32_t* __restrict__ row_ptr,
                                                        const int32_t* __restrict__ col, const float* __restrict__ val,
                                                        const NodeInfo* __restrict__ info, int64_t n, int64_t nnz,
                                                        int tile, int64_t tile_blocks, SchedView s) {
    __shared__ int32_t rows[kTileRowsMax + 1];
    __shared__ int32_t keys[kSmallRounds * kThreads];
    __shared__ TopBitmap map;
    __shared__ int32_t round_tops[8][kThreads / 64];
    __shared__ int32_t shared_count[2];   // popular entries of a long row, bits set in its map
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int64_t)blockIdx.x < tile_blocks) {
        const int64_t first = (int64_t)blockIdx.x * tile;
        const int64_t last = (first + tile < nnz ? first + tile : nnz) - 1;
        int64_t range[2];
        rows_of_tile(row_ptr, n, first > 0 ? first - 1 : 0, last, range);
        for (int64_t r0 = first > 0 ? range[0] + 1 : 0; r0 <= range[1]; r0 += kTileRowsMax) {
            const int count = range[1] - r0 + 1 < kTileRowsMax ? (int)(range[1] - r0 + 1) : kTileRowsMax;
            for (int k = threadIdx.x; k <= count; k += kThreads) rows[k] = row_ptr[r0 + k];
            __syncthreads();
            const int32_t e0 = rows[0];
            // the last row may reach past the tile, and past what keys[] holds if it is a long one
            const int32_t e1 = rows[count] - rows[count - 1] <= kShortMax ? rows[count] : rows[count - 1];
            int32_t j[kSmallRounds];
            float di[kSmallRounds];
#pragma unroll
            for (int r = 0; r < kSmallRounds; ++r) {
                const int32_t e = e0 + r * kThreads + (int32_t)threadIdx.x;
                j[r] = e < e1 ? col[e] : -1;
            }
#pragma unroll
            for (int r = 0; r < kSmallRounds; ++r) {
                const int32_t x = r * kThreads + (int32_t)threadIdx.x;
                di[r] = 0.0f;
                if (j[r] >= 0) {
                    const NodeInfo t = info[j[r]];
                    di[r] = t.dinv;
                    keys[x] = t.pos == kTopNodes ? kTopNodes + x : t.pos;
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kSmallRounds; ++r) {
                if (j[r] < 0) continue;
                const int32_t e = e0 + r * kThreads + (int32_t)threadIdx.x;
                const int64_t k = row_of_entry(rows, e, 0, count - 1);
                const int32_t b = rows[k], end = rows[k + 1];
                if (end - b > kShortMax) continue;
                const int32_t mine = keys[e - e0];
                int32_t at = b;
                for (int32_t q = b; q < end; ++q) {
                    const int32_t other = keys[q - e0];
                    at += (other < mine || (other == mine && q < e)) ? 1 : 0;
                }
                put_entry<true>(s, at, j[r], j[r], di[r], val ? val[e] : 0.0f);
            }
            __syncthreads();
        }
        return;
    }
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t n_single = s.header->n_single, n_long = n_single + s.header->n_multi;
    for (int64_t m = (int64_t)blockIdx.x - tile_blocks; m < n_long; m += gridDim.x - tile_blocks) {
        const int32_t i = m < n_single ? s.singles[m].row : s.multi_row[m - n_single];
        const int32_t b = row_ptr[i], L = row_ptr[i + 1] - b;
        constexpr int kRounds = 8;
        for (int k = threadIdx.x; k < kTopWords; k += kThreads) map.word[k] = 0;
        if (threadIdx.x == 0) shared_count[0] = 0;
        __syncthreads();
        int32_t tops = 0;
#pragma unroll 8
        for (int32_t idx = threadIdx.x; idx < L; idx += kThreads) {
            const int32_t r = info[col[b + idx]].pos;
            if (r != kTopNodes) {
                map.set(r);
                ++tops;
            }
        }
        for (int off = 32; off > 0; off >>= 1) tops += __shfl_xor(tops, off);
        if (lane == 0 && tops > 0) atomicAdd(&shared_count[0], tops);
        __syncthreads();
        tops = shared_count[0];
        if (wave == 0) {
            const int32_t bits = map.count(lane);
            if (lane == 0) shared_count[1] = bits;
        }
        __syncthreads();
        const bool distinct = shared_count[1] == tops;
        int32_t run = 0;   // popular entries in earlier chunks
        for (int32_t c0 = 0; c0 < L; c0 += kRounds * kThreads) {
            int32_t j[kRounds], rank[kRounds];
            float di[kRounds];
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const int32_t idx = c0 + r * kThreads + (int32_t)threadIdx.x;
                j[r] = idx < L ? col[b + idx] : -1;
            }
            uint64_t bal[kRounds];
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const NodeInfo t = j[r] >= 0 ? info[j[r]] : NodeInfo{kTopNodes, 0.0f};
                di[r] = t.dinv;
                rank[r] = t.pos == kTopNodes ? -1 : t.pos;
                bal[r] = __ballot(rank[r] >= 0);
                if (lane == 0) round_tops[r][wave] = __popcll(bal[r]);
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                int32_t t = run + __popcll(bal[r] & lt_mask);
#pragma unroll
                for (int v = 0; v < kThreads / 64; ++v) {
                    if (v < wave) t += round_tops[r][v];
                    run += round_tops[r][v];
                }
                if (j[r] >= 0) {
                    const int32_t idx = c0 + r * kThreads + (int32_t)threadIdx.x;
                    const int32_t at = rank[r] < 0 ? tops + idx - t : distinct ? map.place(rank[r]) : t;
                    put_entry<true>(s, b + at, j[r], j[r], di[r], val ? val[b + idx] : 0.0f);
                }
            }
            __syncthreads();
        }
    }
}

// Large form, rows of up to kSegLen entries.  A wavefront takes kRowsPerWave consecutive rows.  Those of up
// to kShortMax entries are read together, all loads of one kind in flight at once (one row after the
// other was bound by the latency of its three dependent loads); then the longer ones one by one, ROUNDS
// rounds of 64 entries in registers.
constexpr int kRowsPerWave = 4;
constexpr int kOrderWaves = kThreads / 64;

// One row, its entries in registers (entry r * 64 + lane in round r; node -1 past the end).
template <int ROUNDS>
__device__ __forceinline__ void order_row(const SchedView& s, TopBitmap& map, int lane, int32_t dest,
                                          const int32_t (&node)[ROUNDS], const int32_t (&pos)[ROUNDS],
                                          const float (&dinv)[ROUNDS], const float (&v)[ROUNDS]) {
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint64_t bal[ROUNDS];
    int32_t tops = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        bal[r] = __ballot(node[r] >= 0 && pos[r] < kTopNodes);
        tops += __popcll(bal[r]);
    }
    bool distinct = true;
    if (tops > 1) {
#pragma unroll
        for (int k = 0; k < kTopWords / 64; ++k) map.word[k * 64 + lane] = 0;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            if ((bal[r] >> lane) & 1) map.set(pos[r]);
        __builtin_amdgcn_wave_barrier();
        distinct = map.count(lane) == tops;
        __builtin_amdgcn_wave_barrier();
    }
    int32_t before = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int32_t t = before + __popcll(bal[r] & lt_mask);   // popular entries of the row before this one
        before += __popcll(bal[r]);
        if (node[r] >= 0) {
            const bool top = (bal[r] >> lane) & 1;
            const int32_t at = !top ? tops + r * 64 + lane - t : (distinct && tops > 1) ? map.place(pos[r]) : t;
            put_entry<false>(s, dest + at, node[r], pos[r], dinv[r], v[r]);
        }
    }
    __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(kThreads) void order_rows(const int32_t* __restrict__ row_ptr,
                                                       const int32_t* __restrict__ col, const float* __restrict__ val,
                                                       const NodeInfo* __restrict__ info, int64_t n, SchedView s) {
    __shared__ TopBitmap maps[kOrderWaves];
    constexpr int kShortRounds = kShortMax / 64;
    constexpr int kLongRounds = kSegLen / 64;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = ((int64_t)blockIdx.x * kOrderWaves + wave) * kRowsPerWave;
    if (row0 >= n) return;
    const int q0 = lane < kRowsPerWave && row0 + lane < n ? lane : 0;
    const int32_t my_beg = row_ptr[row0 + q0];
    int32_t my_len = row_ptr[row0 + q0 + 1] - my_beg;
    const int32_t my_dest = s.zrow_ptr[info[row0 + q0].pos];
    if (row0 + lane >= n) my_len = 0;
    int32_t beg[kRowsPerWave], len[kRowsPerWave], dest[kRowsPerWave];
#pragma unroll
    for (int q = 0; q < kRowsPerWave; ++q) {
        beg[q] = __builtin_amdgcn_readlane(my_beg, q);
        len[q] = __builtin_amdgcn_readlane(my_len, q);
        dest[q] = __builtin_amdgcn_readlane(my_dest, q);
    }
    TopBitmap& map = maps[wave];
    {
        int32_t node[kRowsPerWave][kShortRounds], pos[kRowsPerWave][kShortRounds];
        float dinv[kRowsPerWave][kShortRounds], v[kRowsPerWave][kShortRounds];
#pragma unroll
        for (int q = 0; q < kRowsPerWave; ++q)
#pragma unroll
            for (int r = 0; r < kShortRounds; ++r) {
                const int32_t idx = r * 64 + lane;
                const bool have = len[q] <= kShortMax && idx < len[q];
                node[q][r] = have ? col[beg[q] + idx] : -1;
                v[q][r] = have && val ? val[beg[q] + idx] : 0.0f;
            }
#pragma unroll
        for (int q = 0; q < kRowsPerWave; ++q)
#pragma unroll
            for (int r = 0; r < kShortRounds; ++r) {
                pos[q][r] = 0;
                dinv[q][r] = 0.0f;
                if (node[q][r] >= 0) {
                    const NodeInfo t = info[node[q][r]];
                    pos[q][r] = t.pos;
                    dinv[q][r] = t.dinv;
                }
            }
#pragma unroll
        for (int q = 0; q < kRowsPerWave; ++q)
            if (len[q] > 0 && len[q] <= kShortMax) order_row<kShortRounds>(s, map, lane, dest[q], node[q], pos[q], dinv[q], v[q]);
    }
#pragma unroll 1
    for (int q = 0; q < kRowsPerWave; ++q) {
        const int32_t L = __builtin_amdgcn_readlane(my_len, q);
        if (L <= kShortMax || L > kSegLen) continue;
        const int32_t b = __builtin_amdgcn_readlane(my_beg, q);
        int32_t node[kLongRounds], pos[kLongRounds];
        float dinv[kLongRounds], v[kLongRounds];
#pragma unroll
        for (int r = 0; r < kLongRounds; ++r) {
            const int32_t idx = r * 64 + lane;
            node[r] = idx < L ? col[b + idx] : -1;
            v[r] = idx < L && val ? val[b + idx] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < kLongRounds; ++r) {
            pos[r] = 0;
            dinv[r] = 0.0f;
            if (node[r] >= 0) {
                const NodeInfo t = info[node[r]];
                pos[r] = t.pos;
                dinv[r] = t.dinv;
            }
        }
        order_row<kLongRounds>(s, map, lane, __builtin_amdgcn_readlane(my_dest, q), node, pos, dinv, v);
    }
}

// Large form, split rows, a workgroup per piece of kChunk entries (of one row, so that nothing has to be
// searched for): how many of the piece's entries are popular, then every entry to its place, the popular
// ones in the caller's order, for order_split_rows to put right.  A row of one piece (most of them) is put in
// order at once.
constexpr int kChunkRounds = kChunk / kThreads;
__global__ __launch_bounds__(kThreads) void count_chunks(const int32_t* __restrict__ row_ptr,
                                                         const int32_t* __restrict__ col,
                                                         const uint64_t* __restrict__ is_top, SchedView s, Chunks chunks) {
    __shared__ int32_t red[kThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t n_chunks = s.header->n_chunks;
    for (int64_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        const int32_t m = chunks.split[c];
        const int32_t i = s.orig[s.multi_row[m]];
        const int32_t beg = row_ptr[i], end = row_ptr[i + 1];
        if (end - beg <= kChunk) continue;
        const int32_t e0 = beg + (int32_t)(c - chunks.first[m]) * kChunk;
        int32_t j[kChunkRounds], tops = 0;
#pragma unroll
        for (int r = 0; r < kChunkRounds; ++r) {
            const int32_t e = e0 + r * kThreads + (int32_t)threadIdx.x;
            j[r] = e < end ? col[e] : -1;
        }
#pragma unroll
        for (int r = 0; r < kChunkRounds; ++r)
            tops += __popcll(__ballot(j[r] >= 0 && ((is_top[j[r] >> 6] >> (j[r] & 63)) & 1)));
        if (lane == 0) red[wave] = tops;
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t t = 0;
#pragma unroll
            for (int w = 0; w < kThreads / 64; ++w) t += red[w];
            chunks.tops[c] = t;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kThreads) void place_chunks(const int32_t* __restrict__ row_ptr,
                                                         const int32_t* __restrict__ col, const float* __restrict__ val,
                                                         const NodeInfo* __restrict__ info, SchedView s, Chunks chunks) {
    __shared__ int32_t red[kThreads / 64][2];
    __shared__ int32_t round_tops[kChunkRounds][kThreads / 64];
    __shared__ TopBitmap map;
    __shared__ int32_t map_bits;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int32_t n_chunks = s.header->n_chunks;
    for (int64_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        const int32_t m = chunks.split[c], first = chunks.first[m];
        const int32_t p = s.multi_row[m];
        const int32_t i = s.orig[p], dest = s.zrow_ptr[p];
        const int32_t beg = row_ptr[i], end = row_ptr[i + 1];
        const int32_t e0 = beg + (int32_t)(c - first) * kChunk;
        int32_t j[kChunkRounds], pos[kChunkRounds];
        float di[kChunkRounds], v[kChunkRounds];
        uint64_t bal[kChunkRounds];
#pragma unroll
        for (int r = 0; r < kChunkRounds; ++r) {
            const int32_t e = e0 + r * kThreads + (int32_t)threadIdx.x;
            j[r] = e < end ? col[e] : -1;
            v[r] = val && e < end ? val[e] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < kChunkRounds; ++r) {
            pos[r] = kTopNodes;
            di[r] = 0.0f;
            if (j[r] >= 0) {
                const NodeInfo t = info[j[r]];
                pos[r] = t.pos;
                di[r] = t.dinv;
            }
        }
        // the row's popular entries in pieces before this one, and in all
        int32_t before = 0, tops = 0;
        const int32_t pieces = (end - beg + kChunk - 1) / kChunk;
        const bool whole = pieces == 1;   // the piece is the row
        if (whole)
            for (int k = threadIdx.x; k < kTopWords; k += kThreads) map.word[k] = 0;
        else for (int32_t q = threadIdx.x; q < pieces; q += kThreads) {
            const int32_t t = chunks.tops[first + q];
            tops += t;
            if (first + q < c) before += t;
        }
        for (int off = 32; off > 0; off >>= 1) {
            tops += __shfl_xor(tops, off);
            before += __shfl_xor(before, off);
        }
        if (whole) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kChunkRounds; ++r) {
                if (pos[r] < kTopNodes) map.set(pos[r]);
                tops += __popcll(__ballot(pos[r] < kTopNodes));   // of the wavefront, summed below
            }
        }
#pragma unroll
        for (int r = 0; r < kChunkRounds; ++r) {
            bal[r] = __ballot(pos[r] < kTopNodes);
            if (lane == 0) round_tops[r][wave] = __popcll(bal[r]);
        }
        if (lane == 0) {
            red[wave][0] = before;
            red[wave][1] = tops;
        }
        __syncthreads();
        before = tops = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            before += red[w][0];
            tops += red[w][1];
        }
        if (whole) {
            if (wave == 0) {
                const int32_t bits = map.count(lane);
                if (lane == 0) map_bits = bits;
            }
            __syncthreads();
        }
        const bool placed = whole && map_bits == tops;   // else in the caller's order: to be put right, or a column is listed twice
#pragma unroll
        for (int r = 0; r < kChunkRounds; ++r) {
            int32_t t = before + __popcll(bal[r] & lt_mask);
#pragma unroll
            for (int w = 0; w < kThreads / 64; ++w) {
                if (w < wave) t += round_tops[r][w];
                before += round_tops[r][w];
            }
            if (j[r] >= 0) {
                const int32_t idx = e0 - beg + r * kThreads + (int32_t)threadIdx.x;
                put_entry<false>(s, dest + (pos[r] >= kTopNodes ? tops + idx - t : placed ? map.place(pos[r]) : t), j[r], pos[r], di[r], v[r]);
            }
        }
        __syncthreads();
    }
}

// The popular entries of the split rows, which stand at the front of each in the caller's order, by rank:
// one workgroup per row, kTopNodes / kSplitThreads entries in a thread's registers.
constexpr int kSplitThreads = 1024;
__global__ __launch_bounds__(kSplitThreads) void order_split_rows(SchedView s) {
    __shared__ TopBitmap map;
    __shared__ int32_t shared_count[2];
    constexpr int kRounds = kTopNodes / kSplitThreads;
    const int lane = threadIdx.x & 63;
    const int32_t n_multi = s.header->n_multi;
    for (int64_t m = blockIdx.x; m < n_multi; m += gridDim.x) {
        const int32_t p = s.multi_row[m];
        const int32_t beg = s.zrow_ptr[p];
        if (s.zrow_ptr[p + 1] - beg <= kChunk) continue;   // in order already
        const int32_t L = s.zrow_ptr[p + 1] - beg < kTopNodes ? s.zrow_ptr[p + 1] - beg : kTopNodes;
        for (int k = threadIdx.x; k < kTopWords; k += kSplitThreads) map.word[k] = 0;
        if (threadIdx.x < 2) shared_count[threadIdx.x] = 0;
        __syncthreads();
        int32_t c[kRounds], tops = 0;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int32_t idx = r * kSplitThreads + (int32_t)threadIdx.x;
            c[r] = idx < L ? s.zcol[beg + idx] : kTopNodes;
            if (c[r] < kTopNodes) {
                map.set(c[r]);
                ++tops;
            }
        }
        for (int off = 32; off > 0; off >>= 1) tops += __shfl_xor(tops, off);
        if (lane == 0 && tops > 0) atomicAdd(&shared_count[0], tops);
        __syncthreads();
        if (threadIdx.x < 64) {
            const int32_t bits = map.count(lane);
            if (lane == 0) shared_count[1] = bits;
        }
        __syncthreads();
        if (shared_count[0] == shared_count[1]) {   // else a column is listed twice: the order stays
            int32_t node[kRounds];
            float sc[kRounds], v[kRounds];
#pragma unroll
            for (int r = 0; r < kRounds; ++r)
                if (c[r] < kTopNodes) {
                    const int64_t e = (int64_t)beg + r * kSplitThreads + threadIdx.x;
                    node[r] = s.znode[e];
                    sc[r] = s.zs[e];
                    if (s.zval) v[r] = s.zval[e];
                }
            __syncthreads();   // all of the row's popular entries have been read
#pragma unroll
            for (int r = 0; r < kRounds; ++r)
                if (c[r] < kTopNodes) {
                    const int64_t e = (int64_t)beg + map.place(c[r]);
                    s.zcol[e] = c[r];
                    s.znode[e] = node[r];
                    s.zs[e] = sc[r];
                    if (s.zval) s.zval[e] = v[r];
                }
        }
        __syncthreads();
    }
}

// The symmetry test (the transposed entry points run on the schedule only if it passes).  It is left out
// where the structure is symmetric by construction (e2eg_normalize_built).
// Of the two entries of a symmetric pair exactly one "looks": the one whose own row is the longer (ties:
// the larger row id).  It searches for its mirror in the other, shorter row (so no search walks a popular
// node's row); weighted: the mirror must carry the same value bit for bit, else the transposed entry points
// would apply another operator than the transpose.  The structure is symmetric iff every looking entry
// finds its mirror and there are as many looking as not-looking entries (the mirrors found are distinct
// not-looking entries; equal counts leave none without a partner).  ALL (small form): every entry looks,
// which needs no count and so no pass behind this one to judge it.
// kMirrorLooks searches of a thread run in step, their probes in flight together: the pass is bound by the
// latency of dependent probes.  The caller's columns ascend; should they not, a search can miss what is
// there, so before a miss counts the row is read from end to end.
constexpr int kMirrorLooks = 8;
template <bool ALL>
__global__ __launch_bounds__(kThreads) void check_mirrors(const int32_t* __restrict__ row_ptr,
                                                          const int32_t* __restrict__ col, const float* __restrict__ val,
                                                          int64_t n, int64_t nnz, int32_t* flags, int32_t* __restrict__ counters) {
    static_assert(kMirrorLooks * kThreads == kEntryTile, "one batch of searches per tile");
    __shared__ int32_t rows[kTileRowsMax + 1];
    __shared__ int32_t balance;
    if (threadIdx.x == 0) balance = 0;
    const EntryTile tile(row_ptr, n, nnz, rows);
    int32_t mine = 0;   // looking minus not-looking entries
    int32_t i[kMirrorLooks], at[kMirrorLooks], left[kMirrorLooks], beg[kMirrorLooks], end[kMirrorLooks];
#pragma unroll
    for (int u = 0; u < kMirrorLooks; ++u) {
        const int64_t e = tile.first + u * kThreads + threadIdx.x;
        left[u] = 0;
        beg[u] = end[u] = at[u] = 0;
        i[u] = -1;
        if (e > tile.last) continue;
        const int64_t k = tile.row(e);
        const int32_t own = tile.row_begin(k + 1) - tile.row_begin(k);
        i[u] = (int32_t)(tile.row0 + k);
        const int32_t j = col[e];
        if (i[u] == j) {
            i[u] = -1;
            continue;
        }
        beg[u] = row_ptr[j];
        end[u] = row_ptr[j + 1];
        const int32_t other = end[u] - beg[u];
        const bool looks = ALL || own > other || (own == other && i[u] > j);
        mine += looks ? 1 : -1;
        if (!looks) {
            i[u] = -1;
            continue;
        }
        at[u] = beg[u];
        left[u] = other;   // the mirror is among the `left` entries from `at` on, or nowhere
    }
    for (;;) {
        bool more = false;
        int32_t probe[kMirrorLooks];
#pragma unroll
        for (int u = 0; u < kMirrorLooks; ++u) probe[u] = left[u] > 1 ? col[at[u] + left[u] / 2] : 0;
#pragma unroll
        for (int u = 0; u < kMirrorLooks; ++u) {
            if (left[u] > 1) {
                const int32_t half = left[u] / 2;
                if (probe[u] <= i[u]) {
                    at[u] += half;
                    left[u] -= half;
                } else {
                    left[u] = half;
                }
                more |= left[u] > 1;
            }
        }
        if (!more) break;
    }
#pragma unroll
    for (int u = 0; u < kMirrorLooks; ++u) {
        if (i[u] < 0) continue;
        bool found = left[u] == 1 && col[at[u]] == i[u];
        if (!found) {
            if (__hip_atomic_load(flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kSchedNotSymmetric) continue;
            for (at[u] = beg[u]; at[u] < end[u] && col[at[u]] != i[u]; ++at[u]) {}
            found = at[u] < end[u];
        }
        if (!found) atomicOr(flags, kSchedNotSymmetric);
        else if (val && __float_as_uint(val[at[u]]) != __float_as_uint(val[tile.first + u * kThreads + threadIdx.x]))
            atomicOr(flags, kSchedValuesNotSymmetric);
    }
    if (ALL) return;
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_down(mine, off);
    if ((threadIdx.x & 63) == 0 && mine != 0) atomicAdd(&balance, mine);
    __syncthreads();
    if (threadIdx.x == 0 && balance != 0)
        atomicAdd(counters + (1 + blockIdx.x % kSymCounters) * kSymStride, balance);
}

// ---- weighted degrees --------------------------------------------------------------------------
// d~_i = sum of the stored values of row i (the diagonal entry carries the 1 of D~ = D + I), added in
// double in a fixed order.  Workgroups below `short_blocks`: kDegLanes lanes to a row of at most
// kSegLen entries; the others: one workgroup to a split row (a row of a million entries would otherwise be
// one wavefront's loop), striding over them.
constexpr int kDegLanes = 16;
__global__ __launch_bounds__(kThreads) void weighted_degrees(const int32_t* __restrict__ row_ptr,
                                                             const float* __restrict__ val, int64_t n, int64_t short_blocks,
                                                             SchedView s, float* __restrict__ deg_w,
                                                             float* __restrict__ dinv_sqrt, NodeInfo* __restrict__ info) {
    __shared__ double red[kThreads];
    auto finish = [&](int64_t row, double sum) {
        if (deg_w) deg_w[row] = (float)sum;
        const float dinv = sum > 0.0 ? (float)(1.0 / sqrt(sum)) : 0.0f;
        dinv_sqrt[row] = dinv;
        info[row].dinv = dinv;   // over the one of the row's length
    };
    if ((int64_t)blockIdx.x < short_blocks) {
        const int64_t row = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kDegLanes;
        const int l = threadIdx.x % kDegLanes;
        double sum = 0.0;
        bool mine = false;
        if (row < n) {
            const int32_t beg = row_ptr[row], end = row_ptr[row + 1];
            mine = end - beg <= kSegLen;
            if (mine)
#pragma unroll 4
                for (int32_t p = beg + l; p < end; p += kDegLanes) sum += (double)val[p];
        }
#pragma unroll
        for (int off = kDegLanes / 2; off > 0; off >>= 1) sum += __shfl_down(sum, off, kDegLanes);
        if (mine && l == 0) finish(row, sum);
        return;
    }
    const int32_t n_multi = s.header->n_multi;
    for (int64_t m = (int64_t)blockIdx.x - short_blocks; m < n_multi; m += gridDim.x - short_blocks) {
        const int32_t p = s.multi_row[m];
        const int32_t row = s.orig ? s.orig[p] : p;
        const int32_t beg = row_ptr[row], end = row_ptr[row + 1];
        double sum = 0.0;
#pragma unroll 8
        for (int32_t q = beg + (int32_t)threadIdx.x; q < end; q += kThreads) sum += (double)val[q];
        __syncthreads();
        red[threadIdx.x] = sum;
        __syncthreads();
        for (int half = kThreads / 2; half > 0; half >>= 1) {   // fixed pairing: the same tree every run
            if ((int)threadIdx.x < half) red[threadIdx.x] += red[threadIdx.x + half];
            __syncthreads();
        }
        if (threadIdx.x == 0) finish(row, red[0]);
    }
}
constexpr int64_t kDegBlocks = 2048;     // workgroups for the split rows
constexpr int64_t kChunkBlocks = 16384;  // workgroups for their pieces, which stride over the real ones

// ---- large form: segments ------------------------------------------------------------------------
// Wide rows, one workgroup each: where every window's run of entries begins (bounds, nwin + 1 per row)
// and the number of segments in the windows before it (win_seg); the row's total goes to row_slots.
// The popular columns come first in a row and the others ascend, so a binary search finds the
// boundary; the running maximum keeps the runs a partition of the row whatever the caller's order was.
__global__ __launch_bounds__(kThreads) void wide_bounds(SchedView s, int32_t nwin, int32_t wide_min,
                                                        int32_t* __restrict__ bounds, int32_t* __restrict__ win_seg,
                                                        int32_t* __restrict__ row_slots) {
    __shared__ int32_t tot[kThreads / 64];
    const int64_t p = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t beg = s.zrow_ptr[p], end = s.zrow_ptr[p + 1];
    if (end - beg < wide_min) {
        if (threadIdx.x == 0) row_slots[p] = 0;
        return;
    }
    bounds += p * (nwin + 1);
    win_seg += p * nwin;
    int32_t carry_pos = beg, carry_seg = 0;
    if (threadIdx.x == 0) bounds[0] = beg;
    for (int32_t w0 = 0; w0 < nwin; w0 += kThreads) {
        const int32_t w = w0 + (int32_t)threadIdx.x;
        int32_t pos = 0;   // end of window w's run
        if (w < nwin) {
            if (w + 1 == nwin) pos = end;
            else {
                const int32_t key = (w + 1) * kWindow;
                int32_t lo = beg, hi = end;
                while (lo < hi) {
                    const int32_t mid = lo + ((hi - lo) >> 1);
                    if (s.zcol[mid] < key) lo = mid + 1; else hi = mid;
                }
                pos = lo;
            }
        }
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const int32_t t = __shfl_up(pos, dlt, 64);
            if (lane >= dlt && t > pos) pos = t;
        }
        if (lane == 63) tot[wave] = pos;
        __syncthreads();
        int32_t base = carry_pos;
#pragma unroll
        for (int v = 0; v < kThreads / 64; ++v) {
            if (v < wave && tot[v] > base) base = tot[v];
            if (tot[v] > carry_pos) carry_pos = tot[v];
        }
        if (pos < base) pos = base;
        int32_t prev = __shfl_up(pos, 1, 64);
        if (lane == 0) prev = base;
        const int32_t cnt = w < nwin ? (pos - prev + kSegLen - 1) / kSegLen : 0;
        int32_t inc = cnt;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const int32_t t = __shfl_up(inc, dlt, 64);
            if (lane >= dlt) inc += t;
        }
        __syncthreads();
        if (lane == 63) tot[wave] = inc;
        __syncthreads();
        int32_t off = carry_seg + inc - cnt;
#pragma unroll
        for (int v = 0; v < kThreads / 64; ++v) {
            if (v < wave) off += tot[v];
            carry_seg += tot[v];
        }
        if (w < nwin) {
            bounds[w + 1] = pos;
            win_seg[w] = off;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) row_slots[p] = carry_seg;
}

// Sort key of a slotted segment: its first column's window, or nwin for the padding behind the real
// segments (sorts last); the lower half is the segment's number t, which is also its slot and its place
// in the key array, so that the stable sort keeps segments of one window in order of t.
__device__ __forceinline__ uint64_t segment_key(int32_t window, int64_t t) {
    return ((uint64_t)(uint32_t)window << 32) | (uint32_t)t;
}

// Workgroups below wide_rows: the segments of one wide row, behind those of the rows cut by length.
// The others, one thread per t: the keys of the segments cut by length, and the padding.
__global__ __launch_bounds__(kThreads) void key_segments(SchedView s, int32_t wide_rows, int32_t nwin, int32_t wide_min,
                                                         const int32_t* __restrict__ bounds,
                                                         const int32_t* __restrict__ win_seg,
                                                         const int32_t* __restrict__ row_slots,
                                                         Segment* __restrict__ seg_tmp, uint64_t* __restrict__ keys) {
    __shared__ int32_t red[kThreads / 64];
    const int64_t n_plain = s.header->n_slot_plain;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool wide_block = (int64_t)blockIdx.x < wide_rows;
    // slots of the wide rows before this one, or of all of them
    int32_t sum = 0;
    const int32_t upto = wide_block ? (int32_t)blockIdx.x : wide_rows;
    for (int32_t q = threadIdx.x; q < upto; q += kThreads) sum += row_slots[q];
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    sum = 0;
#pragma unroll
    for (int v = 0; v < kThreads / 64; ++v) sum += red[v];
    if (wide_block) {
        const int64_t p = blockIdx.x;
        const int32_t cnt = row_slots[p];
        if (cnt == 0) return;
        const int32_t t0 = (int32_t)n_plain + sum;
        if (threadIdx.x == 0) {   // rows are in order of degree, so the p-th row is the p-th split row
            s.slot_base[p] = t0;
            s.slot_cnt[p] = cnt;
        }
        for (int32_t w = threadIdx.x; w < nwin; w += kThreads) {
            const int32_t e = bounds[p * (nwin + 1) + w + 1];
            int32_t t = t0 + win_seg[p * nwin + w];
            for (int32_t b = bounds[p * (nwin + 1) + w]; b < e; b += kSegLen, ++t) {
                seg_tmp[t] = Segment{(int32_t)p, b, b + kSegLen < e ? b + kSegLen : e, t};
                keys[t] = segment_key(s.zcol[b] / kWindow, t);
            }
        }
        return;
    }
    const int64_t t = ((int64_t)blockIdx.x - wide_rows) * kThreads + threadIdx.x;
    if (t >= s.max_slot) return;
    if (t < n_plain) keys[t] = segment_key(s.zcol[seg_tmp[t].beg] / kWindow, t);
    else if (t >= n_plain + sum) keys[t] = segment_key(nwin, t);
}

// Sorted keys -> the ordered segment list, and each segment's length for the deal.
// (A segment cut by length only reaches across many windows and mostly misses in L2, so its
// entries count kLengthCutCost / 4 times in the deal; such segments have the lowest first columns
// and would otherwise make the first XCD's stretch the slowest.)
__global__ void place_segments(const uint64_t* __restrict__ keys, const Segment* __restrict__ seg_tmp, int32_t nwin,
                               SchedView s, uint64_t* __restrict__ seg_len) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p > s.max_slot) return;
    uint64_t len = 0;
    if (p < s.max_slot) {
        const uint64_t key = keys[p];
        if ((int32_t)(key >> 32) < nwin) {
            const Segment g = seg_tmp[(uint32_t)key];
            s.segs[p] = g;
            const bool by_length = g.slot < s.header->n_slot_plain;
            len = by_length ? (uint64_t)(g.end - g.beg) * kLengthCutCost / 4 : (uint64_t)(g.end - g.beg);
        }
    }
    seg_len[p] = len;
}

// len_off = exclusive scan of seg_len (max_slot + 1 entries; the last is the total; 64-bit, since
// the weighted counts of a graph near the int32 limit of nnz pass 2^31).  XCD x gets the slotted
// segments whose running entry count starts in [x, x+1) eighths of the total.  Thread 0 completes the
// header: the number of slots and the verdict of the symmetry test.
__global__ __launch_bounds__(kThreads) void deal_segments(const uint64_t* __restrict__ len_off,
                                                          const int32_t* __restrict__ row_slots, int32_t wide_rows,
                                                          const int32_t* __restrict__ asym, SchedView s) {
    __shared__ int32_t red[kThreads / 64];
    int32_t sum = 0;
    for (int32_t q = threadIdx.x; q < wide_rows; q += kThreads) sum += row_slots[q];
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    sum = 0;
#pragma unroll
    for (int v = 0; v < kThreads / 64; ++v) sum += red[v];
    const int32_t n_slot = s.header->n_slot_plain + sum;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p == 0) {
        uint32_t balance = 0;
        for (int k = 1; k <= kSymCounters; ++k) balance += (uint32_t)asym[k * kSymStride];
        s.header->flags = asym[0] | (balance != 0 ? kSchedNotSymmetric : 0);
        s.header->n_slot = n_slot;
        s.header->xcd_first[kXcds] = n_slot;
        if (n_slot == 0)
            for (int x = 0; x < kXcds; ++x) s.header->xcd_first[x] = 0;
    }
    if (p >= n_slot) return;
    const int64_t total = (int64_t)len_off[s.max_slot];
    const int64_t here = (int64_t)len_off[p], prev = p > 0 ? (int64_t)len_off[p - 1] : -1;
    const int64_t next = (int64_t)len_off[p + 1];
    for (int x = 0; x < kXcds; ++x) {
        const int64_t mark = total * x / kXcds;   // first segment whose start count is >= mark
        if (here >= mark && prev < mark) s.header->xcd_first[x] = (int32_t)p;
        // the mark lies inside the last segment: nothing starts behind it
        if (p == n_slot - 1 && here < mark && mark <= next) s.header->xcd_first[x] = n_slot;
    }
}

__global__ void fill_words(int32_t* __restrict__ p, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0;
}

struct NormWs {
    int32_t* totals;       // [row tiles][kTotals]
    int32_t* zeroed;       // degree classes, then the symmetry flag and counters
    int32_t* top_totals;   // [row tiles][2]
    TopOut top;
    // small form only
    int32_t* tile_classes; // [row tiles][classes], for up to kFewTiles of them
    // large form only
    Chunks chunks;
    int32_t* bounds;       // [wide rows][windows + 1]
    int32_t* win_seg;      // [wide rows][windows]
    int32_t* row_slots;    // [wide rows]
    Segment* seg_tmp;      // [max_slot]
    uint64_t* keys_a;      // [max_slot]
    uint64_t* keys_b;
    uint64_t* seg_len;     // [max_slot + 1]
    void* scan_ws;
    void* sort_ws;
    size_t bytes;
};
constexpr int64_t kFewTiles = 256;   // up to here a workgroup reads all tiles' class histograms (0.27 MB)
constexpr int kAsymAt = (kClasses<kLargeOct> + 63) / 64 * 64;
constexpr int kZeroed = kAsymAt + (kSymCounters + 1) * kSymStride;

NormWs carve_norm(void* base, int64_t n, int64_t nnz) {
    Carver c(base);
    NormWs w = {};
    const int64_t tiles = ceil_div(n > 0 ? n : 1, sched_is_small(nnz) ? kTileRows<true> : kTileRows<false>);
    w.totals = c.take<int32_t>(tiles * kTotals);
    w.zeroed = c.take<int32_t>(kZeroed);
    w.top_totals = c.take<int32_t>(2 * tiles);
    w.top.node = c.take<int32_t>(kTopNodes);
    w.top.deg = c.take<int32_t>(kTopNodes);
    w.top.info = c.take<NodeInfo>(n > 0 ? n : 1);
    if (sched_is_small(nnz)) {
        if (tiles <= kFewTiles) w.tile_classes = c.take<int32_t>(tiles * kClasses<kSmallOct>);
    } else {
        const int64_t wide = sched_max_wide_rows(n, nnz), nwin = sched_windows(n), slots = sched_max_slot(n, nnz);
        w.top.zdeg = c.take<int32_t>(n > 0 ? n : 1);
        w.top.is_top = c.take<uint64_t>(n / 64 + 1);
        w.chunks.max_chunks = nnz / kChunk + sched_max_multi(nnz);
        w.chunks.split = c.take<int32_t>(w.chunks.max_chunks);
        w.chunks.first = c.take<int32_t>(sched_max_multi(nnz));
        w.chunks.tops = c.take<int32_t>(w.chunks.max_chunks);
        w.bounds = c.take<int32_t>(wide * (nwin + 1) + 1);
        w.win_seg = c.take<int32_t>(wide * nwin + 1);
        w.row_slots = c.take<int32_t>(wide + 1);
        w.seg_tmp = c.take<Segment>(slots);
        w.keys_a = c.take<uint64_t>(slots);
        w.keys_b = c.take<uint64_t>(slots);
        w.seg_len = c.take<uint64_t>(slots + 1);
        w.scan_ws = c.take<char>(scan_u64_workspace_bytes(slots + 1));
        w.sort_ws = c.take<char>(radix_sort_workspace_bytes(slots));
    }
    w.bytes = c.size();
    return w;
}

int32_t run_weighted_degrees(int64_t n, int64_t nnz, const int32_t* row_ptr, const float* val, const SchedView& view,
                             float* deg_w, float* dinv, NodeInfo* info, hipStream_t stream) {
    const int64_t short_blocks = ceil_div(n * kDegLanes, kThreads);
    const int64_t split = nnz <= kSegLen ? 0 : view.max_multi < kDegBlocks ? view.max_multi : kDegBlocks;
    weighted_degrees<<<dim3((unsigned)(short_blocks + split)), dim3(kThreads), 0, stream>>>(row_ptr, val, n, short_blocks,
                                                                                          view, deg_w, dinv, info);
    E2EG_LAUNCH_CHECK("weighted_degrees");
    return E2EG_OK;
}

int32_t normalize_small(int32_t n, int64_t nnz, const int32_t* row_ptr, const int32_t* col, const float* val, int32_t* deg,
                        float* deg_w, float* dinv, const SchedView& view, const NormWs& w, bool test, hipStream_t stream) {
    const dim3 tiles((unsigned)ceil_div(n > 0 ? n : 1, kTileRows<true>)), tile_blk(kTileThreads), blk(kThreads);
    if (w.tile_classes) {
        row_stats<true, true, kSmallOct><<<tiles, tile_blk, 0, stream>>>(row_ptr, n, deg, dinv, w.totals, w.tile_classes);
        E2EG_LAUNCH_CHECK("row_stats");
        emit_rows<true, true><<<tiles, tile_blk, 0, stream>>>(row_ptr, nullptr, dinv, n, nnz, 0, 0, w.totals, view, view.segs,
                                                             w.chunks, w.tile_classes, w.top);
        E2EG_LAUNCH_CHECK("emit_rows");
    } else {
        fill_words<<<grid_for(kClasses<kSmallOct>), blk, 0, stream>>>(w.zeroed, kClasses<kSmallOct>);
        E2EG_LAUNCH_CHECK("fill_words");
        row_stats<true, false, kSmallOct><<<tiles, tile_blk, 0, stream>>>(row_ptr, n, deg, dinv, w.totals, w.zeroed);
        E2EG_LAUNCH_CHECK("row_stats");
        emit_rows<true, false><<<tiles, tile_blk, 0, stream>>>(row_ptr, nullptr, nullptr, n, nnz, 0, 0, w.totals, view, view.segs,
                                                              w.chunks, nullptr, w.top);
        E2EG_LAUNCH_CHECK("emit_rows");
        count_top<true, kSmallOct><<<tiles, tile_blk, 0, stream>>>(row_ptr, n, w.zeroed, w.top_totals);
        E2EG_LAUNCH_CHECK("count_top");
        number_nodes<true, kSmallOct><<<tiles, tile_blk, 0, stream>>>(row_ptr, dinv, n, w.zeroed, w.top_totals, view, w.top);
        E2EG_LAUNCH_CHECK("number_nodes");
    }
    if (val && n > 0) {
        const int32_t st = run_weighted_degrees(n, nnz, row_ptr, val, view, deg_w, dinv, w.top.info, stream);
        if (st != E2EG_OK) return st;
    }
    if (nnz == 0) return E2EG_OK;
    const int32_t n_top = n < kTopNodes ? n : kTopNodes;
    rank_top<true><<<dim3((unsigned)ceil_div(n_top, kRankThreads / kRankLanes)), dim3(kRankThreads), 0, stream>>>(n_top, dinv, view, w.top);
    E2EG_LAUNCH_CHECK("rank_top");
    // tiles small enough that the pass has a workgroup for every compute unit
    int tile = kSmallTile;
    while (tile > kThreads && ceil_div(nnz, tile) < 512) tile /= 2;
    const int64_t tile_blocks = ceil_div(nnz, tile);
    const int64_t long_blocks = nnz <= kShortMax ? 0 : view.max_plain < 1024 ? view.max_plain : 1024;
    order_small<<<dim3((unsigned)(tile_blocks + long_blocks)), blk, 0, stream>>>(row_ptr, col, val, w.top.info, n, nnz,
                                                                              tile, tile_blocks, view);
    E2EG_LAUNCH_CHECK("order_small");
    if (test) {
        check_mirrors<true><<<dim3((unsigned)ceil_div(nnz, kEntryTile)), blk, 0, stream>>>(row_ptr, col, val, n, nnz,
                                                                                         &view.header->flags, nullptr);
        E2EG_LAUNCH_CHECK("check_mirrors");
    }
    return E2EG_OK;
}

int32_t normalize_large(int32_t n, int64_t nnz, const int32_t* row_ptr, const int32_t* col, const float* val, int32_t* deg,
                        float* deg_w, float* dinv, const SchedView& view, const NormWs& w, bool test, hipStream_t stream) {
    const dim3 blk(kThreads), tile_blk(kTileThreads);
    const dim3 tiles((unsigned)ceil_div(n > 0 ? n : 1, kTileRows<false>));
    const int32_t wide_rows = (int32_t)sched_max_wide_rows(n, nnz);
    const int32_t wide_min = (int32_t)sched_wide_threshold(n);
    const int32_t nwin = (int32_t)sched_windows(n);
    int32_t* classes = w.zeroed;
    int32_t* asym = w.zeroed + kAsymAt;

    // 1. degrees, d^-1/2, internal numbering
    fill_words<<<grid_for(kZeroed), blk, 0, stream>>>(w.zeroed, kZeroed);
    E2EG_LAUNCH_CHECK("fill_words");
    row_stats<false, false, kLargeOct><<<tiles, tile_blk, 0, stream>>>(row_ptr, n, deg, dinv, nullptr, classes);
    E2EG_LAUNCH_CHECK("row_stats");
    count_top<false, kLargeOct><<<tiles, tile_blk, 0, stream>>>(row_ptr, n, classes, w.top_totals);
    E2EG_LAUNCH_CHECK("count_top");
    number_nodes<false, kLargeOct><<<tiles, tile_blk, 0, stream>>>(row_ptr, dinv, n, classes, w.top_totals, view, w.top);
    E2EG_LAUNCH_CHECK("number_nodes");
    const int32_t n_top = n < kTopNodes ? n : kTopNodes;
    rank_top<false><<<dim3((unsigned)ceil_div(n_top, kRankThreads / kRankLanes)), dim3(kRankThreads), 0, stream>>>(n_top, dinv, view, w.top);
    E2EG_LAUNCH_CHECK("rank_top");

    // 2. row pointers and work lists
    row_totals<<<tiles, tile_blk, 0, stream>>>(w.top.zdeg, n, wide_rows, wide_min, w.totals);
    E2EG_LAUNCH_CHECK("row_totals");
    emit_rows<false, false><<<tiles, tile_blk, 0, stream>>>(nullptr, w.top.zdeg, nullptr, n, nnz, wide_rows, wide_min, w.totals, view,
                                                           w.seg_tmp, w.chunks, nullptr, w.top);
    E2EG_LAUNCH_CHECK("emit_rows");
    const int64_t split_waves = view.max_multi < 16384 ? view.max_multi : 16384;
    emit_split<<<dim3((unsigned)ceil_div(split_waves, kThreads / 64)), blk, 0, stream>>>(view, wide_rows, wide_min, w.seg_tmp, w.chunks);
    E2EG_LAUNCH_CHECK("emit_split");
    if (val) {
        const int32_t st = run_weighted_degrees(n, nnz, row_ptr, val, view, deg_w, dinv, w.top.info, stream);
        if (st != E2EG_OK) return st;
    }

    // 3. the CSR in internal ids, and the symmetry test
    order_rows<<<dim3((unsigned)ceil_div(n, kOrderWaves * kRowsPerWave)), blk, 0, stream>>>(row_ptr, col, val, w.top.info, n, view);
    E2EG_LAUNCH_CHECK("order_rows");
    const dim3 chunk_blocks((unsigned)(w.chunks.max_chunks < kChunkBlocks ? w.chunks.max_chunks : kChunkBlocks));
    count_chunks<<<chunk_blocks, blk, 0, stream>>>(row_ptr, col, w.top.is_top, view, w.chunks);
    E2EG_LAUNCH_CHECK("count_chunks");
    place_chunks<<<chunk_blocks, blk, 0, stream>>>(row_ptr, col, val, w.top.info, view, w.chunks);
    E2EG_LAUNCH_CHECK("place_chunks");
    const int64_t split_blocks = view.max_multi < 4096 ? view.max_multi : 4096;
    order_split_rows<<<dim3((unsigned)split_blocks), dim3(kSplitThreads), 0, stream>>>(view);
    E2EG_LAUNCH_CHECK("order_split_rows");
    if (test) {
        check_mirrors<false><<<dim3((unsigned)ceil_div(nnz, kEntryTile)), blk, 0, stream>>>(row_ptr, col, val, n, nnz, asym, asym);
        E2EG_LAUNCH_CHECK("check_mirrors");
    }

    // 4. slotted segments: wide rows by window then length, the other split rows by length; ordered and dealt
    wide_bounds<<<dim3((unsigned)wide_rows), blk, 0, stream>>>(view, nwin, wide_min, w.bounds, w.win_seg, w.row_slots);
    E2EG_LAUNCH_CHECK("wide_bounds");
    key_segments<<<dim3((unsigned)(wide_rows + ceil_div(view.max_slot, kThreads))), blk, 0, stream>>>(
        view, wide_rows, nwin, wide_min, w.bounds, w.win_seg, w.row_slots, w.seg_tmp, w.keys_a);
    E2EG_LAUNCH_CHECK("key_segments");
    uint64_t* src = w.keys_a;
    uint64_t* dst = w.keys_b;
    const int32_t st = radix_sort_u64(&src, &dst, view.max_slot, 32, bits_for((int64_t)nwin + 1), w.sort_ws, stream);
    if (st != E2EG_OK) return st;
    place_segments<<<grid_for(view.max_slot + 1), blk, 0, stream>>>(src, w.seg_tmp, nwin, view, w.seg_len);
    E2EG_LAUNCH_CHECK("place_segments");
    E2EG_HIP_TRY(exclusive_scan_u64(w.seg_len, w.seg_len, view.max_slot + 1, nullptr, w.scan_ws, stream));
    deal_segments<<<grid_for(view.max_slot + 1), blk, 0, stream>>>(w.seg_len, w.row_slots, wide_rows, asym, view);
    E2EG_LAUNCH_CHECK("deal_segments");
    return E2EG_OK;
}

}  // namespace
}  // namespace e2eg

using namespace e2eg;

extern "C" size_t e2eg_sched_bytes(int32_t n, int64_t nnz) {
    if (n < 0 || nnz < 0) return 0;
    return sched_carve(nullptr, n, nnz, nullptr, false, nullptr);
}

extern "C" size_t e2eg_sched_weighted_bytes(int32_t n, int64_t nnz) {
    if (n < 0 || nnz < 0) return 0;
    return sched_carve(nullptr, n, nnz, nullptr, true, nullptr);
}

extern "C" size_t e2eg_normalize_workspace_bytes(int32_t n, int64_t nnz) {
    if (n < 0 || nnz < 0) return 0;
    // The size is part of the interface: it has always held two arrays of 8-byte keys per entry, and a caller's
    // buffer for one size may serve smaller ones.  What is used of it now is less.
    const size_t used = carve_norm(nullptr, n, nnz).bytes, promised = 16 * (size_t)nnz;
    return used > promised ? used : promised;
}

namespace {
// `test`: look whether the structure (and the values) are symmetric.  d_val == nullptr: the unweighted
// call.  Otherwise d~ and d~^-1/2 come from the values (d_deg_w may be null), d_deg receives the row
// lengths, and the schedule also receives the values in internal order.
int32_t normalize_impl(bool test, int32_t n, int64_t nnz, const int32_t* d_row_ptr, const int32_t* d_col_idx,
                       const float* d_val, int32_t* d_deg, float* d_deg_w, float* d_dinv_sqrt, void* d_sched,
                       size_t sched_bytes, void* ws, size_t ws_bytes, void* stream_) {
    const bool weighted = d_val != nullptr;
    if (n < 0 || nnz < 0) return fail(E2EG_ERR_INVALID_ARG, "normalize: negative size");
    if (nnz > (int64_t)INT32_MAX || n == INT32_MAX)
        return fail(E2EG_ERR_OVERFLOW, "normalize: nnz=%lld exceeds int32", (long long)nnz);
    if (!d_row_ptr || !d_dinv_sqrt || !d_sched || (nnz > 0 && !d_col_idx))
        return fail(E2EG_ERR_NULL_PTR, "normalize: null pointer");
    const size_t sched_need = sched_carve(nullptr, n, nnz, nullptr, weighted, nullptr);
    if (!aligned_to(d_sched, kAlign) || sched_bytes < sched_need)
        return fail(E2EG_ERR_CAPACITY, "normalize: d_sched needs %zu bytes, 256-byte aligned", sched_need);
    const size_t need = e2eg_normalize_workspace_bytes(n, nnz);
    if (!ws || !aligned_to(ws, kAlign) || ws_bytes < need)
        return fail(E2EG_ERR_WORKSPACE, "normalize: workspace needs %zu bytes, 256-byte aligned", need);
    if (n == 0 && nnz > 0) return fail(E2EG_ERR_INVALID_ARG, "normalize: entries given but no nodes");

    hipStream_t stream = static_cast<hipStream_t>(stream_);
    const NormWs w = carve_norm(ws, n, nnz);
    SchedView view;
    sched_carve(d_sched, n, nnz, &view, weighted, d_row_ptr);
    if (sched_is_small(nnz))
        return normalize_small(n, nnz, d_row_ptr, d_col_idx, d_val, d_deg, d_deg_w, d_dinv_sqrt, view, w, test, stream);
    return normalize_large(n, nnz, d_row_ptr, d_col_idx, d_val, d_deg, d_deg_w, d_dinv_sqrt, view, w, test, stream);
}
}  // namespace

extern "C" int32_t e2eg_normalize(int32_t n, int64_t nnz, const int32_t* d_row_ptr,
                                  const int32_t* d_col_idx, int32_t* d_deg, float* d_dinv_sqrt,
                                  void* d_sched, size_t sched_bytes, void* ws, size_t ws_bytes,
                                  void* stream) {
    return normalize_impl(true, n, nnz, d_row_ptr, d_col_idx, nullptr, d_deg, nullptr, d_dinv_sqrt, d_sched, sched_bytes, ws,
                          ws_bytes, stream);
}

extern "C" int32_t e2eg_normalize_built(int32_t n, int64_t nnz, const int32_t* d_row_ptr, const int32_t* d_col_idx,
                                        const float* d_val, int32_t* d_deg, float* d_deg_w, float* d_dinv_sqrt,
                                        void* d_sched, size_t sched_bytes, void* ws, size_t ws_bytes, void* stream) {
    return normalize_impl(false, n, nnz, d_row_ptr, d_col_idx, d_val, d_deg, d_deg_w, d_dinv_sqrt, d_sched, sched_bytes, ws,
                          ws_bytes, stream);
}

extern "C" int32_t e2eg_normalize_weighted(int32_t n, int64_t nnz, const int32_t* d_row_ptr,
                                           const int32_t* d_col_idx, const float* d_val, int32_t* d_deg,
                                           float* d_deg_w, float* d_dinv_sqrt, void* d_sched, size_t sched_bytes,
                                           void* ws, size_t ws_bytes, void* stream) {
    if (!d_val && nnz > 0) return fail(E2EG_ERR_NULL_PTR, "normalize_weighted: d_val is null");
    static const float kOne = 1.0f;  // nnz == 0: any non-null pointer selects the weighted layout
    return normalize_impl(true, n, nnz, d_row_ptr, d_col_idx, d_val ? d_val : &kOne, d_deg, d_deg_w, d_dinv_sqrt, d_sched,
                          sched_bytes, ws, ws_bytes, stream);
}

extern "C" int32_t e2eg_sched_check_symmetric(const void* d_sched, void* stream_) {
    if (!d_sched) return fail(E2EG_ERR_NULL_PTR, "sched_check_symmetric: d_sched is null");
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    SchedHeader h;   // the schedule starts with its header
    E2EG_HIP_TRY(hipMemcpyAsync(&h, d_sched, sizeof(h), hipMemcpyDeviceToHost, stream));
    E2EG_HIP_TRY(hipStreamSynchronize(stream));
    if (h.flags & kSchedNotSymmetric)
        return fail(E2EG_ERR_INVALID_ARG, "sched_check_symmetric: the structure holds an entry (i, j) without (j, i); "
                                          "the transposed entry points cannot run on it");
    if (h.flags & kSchedValuesNotSymmetric)
        return fail(E2EG_ERR_INVALID_ARG, "sched_check_symmetric: the values of (i, j) and (j, i) differ somewhere; "
                                          "the transposed entry points cannot run on it");
    return E2EG_OK;
}
