// e2eg_build_csr: (user, item) pairs -> CSR structure of A~ = A + I (paper: Section 3,
// "Notation"; A_ij > 0 iff (i,j) in E, so repeated pairs are one edge).
//
// Design for the GPU: everything is integer work and deterministic.
//   1. LSD radix sort of the keys (user, item), packed into as few bits as the id ranges need; the
//      first pass reads the caller's pairs and checks the id ranges;
//   2. drop repeats (heads counted per tile, then compacted) -> distinct pairs; the same pass writes the
//      user rows (a user's items are a contiguous, ascending run), notes where each user's run starts and
//      ends, and turns the keys round to (item, user);
//   3. stable radix sort by item; the last pass writes the item rows and counts them;
//   4. row_ptr from a prefix sum of the counts, the diagonal beside it.
// The number of distinct pairs is known on the device only; launches are sized by the number of pairs
// given, and the host waits once, at the end.
// Large graphs: the same steps with 32-bit keys where the ids allow it ("long lists" below).
// Small graphs are bound by the number of launches (17 of the above) and take another way, "buckets" below:
// five launches.
#include "entry_tiles.h"
#include "radix.h"

namespace e2eg {
namespace {

constexpr int kThreads = 256;

inline unsigned blocks_for(int64_t count, int per_block) {
    return (unsigned)ceil_div(count > 0 ? count : 1, per_block);
}

__global__ void zero_i32(int32_t* p, int64_t count) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0;
}

// The caller's pairs as keys (user << item_bits | item); ids out of range are reported (once, by the first
// pass's histogram) and read as 0.
struct PairsIn {
    const int32_t* users;
    const int32_t* items;
    int32_t n_users, n_items;
    int item_bits;
    int32_t* bad;
    __device__ __forceinline__ bool ok(int32_t u, int32_t i) const {
        return (uint32_t)u < (uint32_t)n_users && (uint32_t)i < (uint32_t)n_items;
    }
    using Key = uint64_t;
    struct raw {
        int32_t user, item;
    };
    __device__ __forceinline__ PairsIn from(int64_t base) const {
        return PairsIn{users + base, items + base, n_users, n_items, item_bits, bad};
    }
    __device__ __forceinline__ raw load(uint32_t e) const { return raw{users[e], items[e]}; }
    __device__ __forceinline__ raw none() const { return raw{0, 0}; }
    __device__ __forceinline__ bool ok(raw r) const { return ok(r.user, r.item); }
    __device__ __forceinline__ uint64_t key(raw r) const {
        const uint32_t u = (uint32_t)r.user < (uint32_t)n_users ? (uint32_t)r.user : 0u;
        const uint32_t i = (uint32_t)r.item < (uint32_t)n_items ? (uint32_t)r.item : 0u;
        return ((uint64_t)u << item_bits) | i;
    }
    __device__ __forceinline__ void report() const { atomicOr(bad, 1); }
};

// Their users alone, for digits of the user.
struct UsersIn {
    const int32_t* users;
    int32_t n_users;
    int item_bits;
    using Key = uint64_t;
    using raw = int32_t;
    __device__ __forceinline__ UsersIn from(int64_t base) const { return UsersIn{users + base, n_users, item_bits}; }
    __device__ __forceinline__ raw load(uint32_t e) const { return users[e]; }
    __device__ __forceinline__ raw none() const { return 0; }
    __device__ __forceinline__ bool ok(raw) const { return true; }
    __device__ __forceinline__ uint64_t key(raw r) const {
        return (uint64_t)((uint32_t)r < (uint32_t)n_users ? (uint32_t)r : 0u) << item_bits;
    }
    __device__ __forceinline__ void report() const {}
};

// Sorted (item, user) keys -> item rows: key k of the list lands behind the user rows and the earlier
// items' diagonal entries.
struct ItemRowsOut {
    static constexpr bool kRuns = true, kChecks = false;
    int32_t* col_idx;
    const int32_t* pairs;   // number of distinct pairs
    int32_t* counts;        // per item, cleared
    int64_t n_users;
    int32_t self;
    int user_bits;
    __device__ __forceinline__ int32_t group(uint64_t key, int) const { return (int32_t)(key >> user_bits); }
    __device__ __forceinline__ void store(uint32_t at, uint64_t key, int segment) const {
        const int64_t row0 = *pairs + (n_users + group(key, segment)) * self;
        col_idx[row0 + at] = (int32_t)(key & ((1ull << user_bits) - 1));
    }
};

// The same for keys that have lost the leading digit of the item, which is the segment.
struct ItemSegmentsOut {
    static constexpr bool kRuns = true, kChecks = false;
    int32_t* col_idx;
    const int32_t* pairs;
    int32_t* counts;
    int64_t n_users;
    int32_t self;
    int user_bits, item_low;
    __device__ __forceinline__ int32_t group(uint32_t key, int segment) const {
        return (segment << item_low) | (int32_t)(key >> user_bits);
    }
    __device__ __forceinline__ void store(uint32_t at, uint32_t key, int segment) const {
        const int64_t row0 = *pairs + (n_users + group(key, segment)) * self;
        col_idx[row0 + at] = (int32_t)(key & ((1u << user_bits) - 1));
    }
};

// ---- repeats -------------------------------------------------------------------------------------
constexpr int kHeadThreads = 512;
constexpr int kHeadRounds = 8;
constexpr int kHeadTile = kHeadThreads * kHeadRounds;
constexpr int kHeadWaves = kHeadThreads / 64;
constexpr int64_t kHeadFew = 1024;   // up to this many tiles every workgroup adds up the counts before it

// Keys that differ from their predecessor, per tile.
__global__ __launch_bounds__(kHeadThreads) void count_heads(const uint64_t* __restrict__ keys, int64_t count,
                                                            int32_t* __restrict__ tile_cnt) {
    __shared__ int32_t red[kHeadWaves];
    const int64_t base = (int64_t)blockIdx.x * kHeadTile;
    int32_t heads = 0;
#pragma unroll
    for (int r = 0; r < kHeadRounds; ++r) {
        const int64_t k = base + r * kHeadThreads + threadIdx.x;
        heads += __popcll(__ballot(k < count && (k == 0 || keys[k] != keys[k - 1])));
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = heads;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int w = 0; w < kHeadWaves; ++w) t += red[w];
        tile_cnt[blockIdx.x] = t;
    }
}

// The distinct pairs: turned round for the second sort, and as user rows (pair k lands behind its user's
// diagonal entry).  SCANNED: tile_cnt holds the counts before each tile, else the tiles' own.
template <bool SCANNED>
__global__ __launch_bounds__(kHeadThreads) void emit_pairs(const uint64_t* __restrict__ keys, int64_t count,
                                                           const int32_t* __restrict__ tile_cnt, int user_bits,
                                                           int item_bits, int32_t n_users, int32_t self,
                                                           uint64_t* __restrict__ turned, int32_t* __restrict__ col_idx,
                                                           int32_t* __restrict__ run_start, int32_t* __restrict__ run_end,
                                                           int32_t* __restrict__ n_pairs) {
    __shared__ int32_t red[kHeadWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int32_t before = 0;
    if (SCANNED) {
        before = tile_cnt[blockIdx.x];
    } else {
        for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kHeadThreads) before += tile_cnt[t];
        for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off);
        if (lane == 0) red[wave] = before;
        __syncthreads();
        before = 0;
#pragma unroll
        for (int w = 0; w < kHeadWaves; ++w) before += red[w];
        __syncthreads();
    }
    const int64_t base = (int64_t)blockIdx.x * kHeadTile + (int64_t)wave * (64 * kHeadRounds);
    uint64_t key[kHeadRounds], bal[kHeadRounds];
    bool first_of_user[kHeadRounds], last_of_user[kHeadRounds];
    int32_t mine = 0;
#pragma unroll
    for (int r = 0; r < kHeadRounds; ++r) {
        const int64_t k = base + r * 64 + lane;
        key[r] = k < count ? keys[k] : 0ull;
        const uint64_t prev = k > 0 && k < count ? keys[k - 1] : 0ull;
        const uint64_t next = k + 1 < count ? keys[k + 1] : 0ull;
        bal[r] = __ballot(k < count && (k == 0 || key[r] != prev));
        first_of_user[r] = k < count && (k == 0 || (prev >> item_bits) != (key[r] >> item_bits));
        last_of_user[r] = k < count && (k + 1 == count || (next >> item_bits) != (key[r] >> item_bits));
        mine += __popcll(bal[r]);
    }
    if (lane == 0) red[wave] = mine;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kHeadWaves; ++w)
        if (w < wave) before += red[w];
#pragma unroll
    for (int r = 0; r < kHeadRounds; ++r) {
        const int64_t k = base + r * 64 + lane;
        const int32_t pos = before + __popcll(bal[r] & lt_mask);
        const bool head = (bal[r] >> lane) & 1;
        before += __popcll(bal[r]);
        const uint32_t u = (uint32_t)(key[r] >> item_bits);
        const uint32_t i = (uint32_t)(key[r] & ((1ull << item_bits) - 1));
        if (head) {
            turned[pos] = ((uint64_t)i << user_bits) | u;
            col_idx[pos + (int64_t)(u + 1) * self] = n_users + (int32_t)i;
        }
        if (first_of_user[r]) run_start[u] = pos;
        if (last_of_user[r]) run_end[u] = pos + (head ? 1 : 0);
        if (k == count - 1) *n_pairs = pos + (head ? 1 : 0);
    }
}

// ---- long lists: 32-bit keys ------------------------------------------------------------------------
// A pass over a list of tens of millions moves its keys twice through memory, so they are made half as
// large: the first pass takes the leading digit of the user off, and what is left of user and item, up to 32 bits,
// is sorted segment by segment (Segmented).  The distinct pairs go to segments of the item's leading
// digit in the kernel that writes the user rows; there only the rest of the item is left to sort by, since
// the users of an item arrive in order.  50 M pairs of 20 + 19 bits: 2830 us with 64-bit keys throughout (eight passes
// of about 300, repeats counted and dropped in 320), 1910 us so (a pass: histogram 48, offsets 17, scatter 136).
// The scatter is bound by the ranking of the keys (103 us of vector instructions), not by its 400 MB any more.
struct ListSort {
    static constexpr int kThreads = 512, kItems = 16, kBits = 8, kCopies = 16, kTile = kThreads * kItems;
};

// Where the segments begin: `offs` is the scanned table [segments][tiles] of the pass that made them,
// d_count (or count) the number of keys.
__global__ __launch_bounds__(kMaxSegments) void plan_segments(const int32_t* __restrict__ offs, int32_t tiles, int32_t n,
                                                              int64_t count, const int32_t* __restrict__ d_count, Segments* s) {
    __shared__ int32_t first[kMaxSegments + 1];
    __shared__ int32_t red[kMaxSegments / 64];
    const int g = threadIdx.x, lane = g & 63, wave = g >> 6;
    if (g < n) first[g] = offs[(int64_t)g * tiles];
    if (g == 0) first[n] = d_count ? *d_count : (int32_t)count;
    __syncthreads();
    const int32_t mine = g < n ? (first[g + 1] - first[g] + ListSort::kTile - 1) / ListSort::kTile : 0;
    int32_t inc = mine;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const int32_t t = __shfl_up(inc, dlt, 64);
        if (lane >= dlt) inc += t;
    }
    if (lane == 63) red[wave] = inc;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kMaxSegments / 64; ++w)
        if (w < wave) inc += red[w];
    if (g < n) {
        s->first[g] = first[g];
        s->tile[g] = inc - mine;
        if (g == n - 1) {
            s->first[n] = first[n];
            s->tile[n] = inc;
        }
    }
}

// The sorted list, its repeats skipped: distinct pairs of every tile, and their counts by the item's leading
// digit, [digits][tiles].
__global__ __launch_bounds__(ListSort::kThreads) void count_distinct(const uint32_t* __restrict__ keys, Segmented tiling,
                                                                     int item_bits, int item_low, int bins,
                                                                     int32_t* __restrict__ tile_cnt, int32_t* __restrict__ hist) {
    using S = ListSort;
    __shared__ int h[kMaxSegments * S::kCopies];
    __shared__ int32_t red[S::kThreads / 64];
    const Place at = tiling.place<S>(bins);
    for (int k = threadIdx.x; k < kMaxSegments * S::kCopies; k += S::kThreads) h[k] = 0;
    __syncthreads();
    int* mine = h + threadIdx.x % S::kCopies;
    // indexes inside the tile: its keys, and whether there is one before them in the segment
    const int left = (int)(at.end - at.base);
    const bool starts = left <= 0 || at.base == tiling.s->first[at.segment];
    const uint32_t* tile_keys = keys + at.base;
    const uint32_t item_mask = (1u << item_bits) - 1;
    uint32_t key[S::kItems], prev[S::kItems];
#pragma unroll
    for (int k = 0; k < S::kItems; ++k) {
        const int i = k * S::kThreads + (int)threadIdx.x;
        key[k] = i < left ? tile_keys[i] : 0u;
        prev[k] = i < left && (i > 0 || !starts) ? tile_keys[i - 1] : 0u;
    }
    int32_t heads = 0;
#pragma unroll
    for (int k = 0; k < S::kItems; ++k) {
        const int i = k * S::kThreads + (int)threadIdx.x;
        const bool head = i < left && ((i == 0 && starts) || key[k] != prev[k]);
        if (head) atomicAdd(&mine[((key[k] & item_mask) >> item_low) * S::kCopies], 1);
        heads += __popcll(__ballot(head));
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = heads;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
#pragma unroll
        for (int w = 0; w < S::kThreads / 64; ++w) t += red[w];
        tile_cnt[blockIdx.x] = t;
    }
    for (int d = threadIdx.x; d < bins; d += S::kThreads) {
        int t = 0;
#pragma unroll
        for (int c = 0; c < S::kCopies; ++c) t += h[d * S::kCopies + ((c + d) % S::kCopies)];
        hist[(int64_t)d * gridDim.x + blockIdx.x] = t;
    }
}

// The lanes of a wavefront whose key (round r of its consecutive keys) is no repeat: the lane before's key comes by
// wave_shr:1, which leaves lane 0 its first operand, the last key of the round before.
template <int ITEMS>
__device__ __forceinline__ uint32_t key_before(const uint32_t (&key)[ITEMS], int r, uint32_t before_all) {
    const uint32_t edge = r == 0 ? before_all : (uint32_t)__builtin_amdgcn_readlane((int)key[r > 0 ? r - 1 : 0], 63);
    return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)key[r], 0x138, 0xf, 0xf, false);
}

// The distinct pairs as user rows: pair k lands behind its user's diagonal entry.  tile_cnt: the distinct pairs
// before every tile.  (In one kernel with spread_distinct, which reads the same keys, the two took 320 us, its
// registers leaving room for one workgroup on a compute unit; apart they take 132 + 159.)
constexpr int kUserRounds = 8;
constexpr int kUserThreads = ListSort::kTile / kUserRounds;
__global__ __launch_bounds__(kUserThreads) void write_user_rows(const uint32_t* __restrict__ keys, Segmented tiling, int64_t count,
                                                                int user_low, int item_bits, int32_t n_users, int32_t self,
                                                                const int32_t* __restrict__ tile_cnt,
                                                                int32_t* __restrict__ col_idx, int32_t* __restrict__ run_start,
                                                                int32_t* __restrict__ run_end, int32_t* __restrict__ n_pairs) {
    constexpr int kWaves = kUserThreads / 64;
    __shared__ int32_t red[kWaves];
    const Place at = tiling.place<ListSort>(1);
    if (at.base >= at.end) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // indexes inside the tile: of its keys, of the segment's first and last, of the list's last
    const int left = (int)(at.end - at.base), chunk = wave * (64 * kUserRounds);
    const int first = at.base == tiling.s->first[at.segment] ? 0 : -1;
    const int last = at.end == tiling.s->first[at.segment + 1] ? left - 1 : left;
    const int list_last = at.end == count ? left - 1 : left;
    const uint32_t* tile_keys = keys + at.base;
    const uint32_t item_mask = (1u << item_bits) - 1;
    uint32_t key[kUserRounds];
#pragma unroll
    for (int r = 0; r < kUserRounds; ++r) {
        const int i = chunk + r * 64 + lane;
        key[r] = i < left ? tile_keys[i] : 0u;
    }
    // the keys before and behind the wavefront's (a tile that is not full ends with its segment)
    const int behind_at = chunk + 64 * kUserRounds;
    const uint32_t before_all = chunk > first && chunk < left ? tile_keys[chunk - 1] : 0u;
    const uint32_t behind_all = behind_at <= last ? tile_keys[behind_at] : 0u;
    // which keys are no repeats, which are the first of their user's
    uint64_t head[kUserRounds], lead[kUserRounds + 1];
    int32_t heads = 0;
#pragma unroll
    for (int r = 0; r < kUserRounds; ++r) {
        const int i = chunk + r * 64 + lane;
        const uint32_t prev = key_before(key, r, before_all);
        head[r] = __ballot(i < left && (i == first || key[r] != prev));
        lead[r] = __ballot(i < left && (i == first || (prev >> item_bits) != (key[r] >> item_bits)));
        heads += __popcll(head[r]);
    }
    const uint32_t last_key = (uint32_t)__builtin_amdgcn_readlane((int)key[kUserRounds - 1], 63);
    lead[kUserRounds] = (behind_all >> item_bits) != (last_key >> item_bits) ? 1 : 0;
    if (lane == 0) red[wave] = heads;
    __syncthreads();
    int32_t pos0 = tile_cnt[blockIdx.x];
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
        if (w < wave) pos0 += red[w];
#pragma unroll
    for (int r = 0; r < kUserRounds; ++r) {
        const int i = chunk + r * 64 + lane;
        const bool mine = (head[r] >> lane) & 1;
        const int32_t pos = pos0 + __popcll(head[r] & lt_mask);
        pos0 += __popcll(head[r]);
        const int32_t u = (int32_t)(((uint32_t)at.segment << user_low) | (key[r] >> item_bits));
        if (mine) col_idx[pos + (int64_t)(u + 1) * self] = n_users + (int32_t)(key[r] & item_mask);
        if (i >= left) continue;
        if ((lead[r] >> lane) & 1) run_start[u] = pos;
        // the last of its user's: the next key leads, or there is none
        const uint64_t ends = (lead[r] >> 1) | (lead[r + 1] << 63);
        if (i == last || ((ends >> lane) & 1)) run_end[u] = pos + (mine ? 1 : 0);
        if (i == list_last) *n_pairs = pos + (mine ? 1 : 0);
    }
}

// The distinct pairs by the leading digit of the item, in order, as keys (rest of the item, user).  offs: the
// counts of count_distinct, scanned.
__global__ __launch_bounds__(ListSort::kThreads) __attribute__((amdgpu_waves_per_eu(4))) void spread_distinct(const uint32_t* __restrict__ keys, Segmented tiling,
                                                                      int user_low, int user_bits, int item_bits, int item_low,
                                                                      int digit_bits, const int32_t* __restrict__ offs,
                                                                      uint32_t* __restrict__ by_item) {
    using S = ListSort;
    constexpr int kWaves = S::kThreads / 64;
    static_assert(S::kThreads >= kMaxSegments && kMaxSegments == 256, "a thread per digit, digits in bytes");
    __shared__ uint16_t wave_cnt[kWaves][kMaxSegments];
    __shared__ int32_t shift_by[kMaxSegments];
    __shared__ int32_t red[kWaves];
    __shared__ uint32_t tile[S::kTile];
    __shared__ uint8_t tile_digit[S::kTile];
    const Place at = tiling.place<S>(1);
    if (at.base >= at.end) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int left = (int)(at.end - at.base), chunk = wave * (64 * S::kItems);
    const int first = at.base == tiling.s->first[at.segment] ? 0 : -1;   // the segment's first key, seen from the tile
    const uint32_t* tile_keys = keys + at.base;
    const uint32_t item_mask = (1u << item_bits) - 1, low_mask = (1u << item_low) - 1;
    const int32_t base = (int)threadIdx.x < 1 << digit_bits ? offs[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] : 0;
    uint32_t key[S::kItems];
#pragma unroll
    for (int r = 0; r < S::kItems; ++r) {
        const int i = chunk + r * 64 + lane;
        key[r] = i < left ? tile_keys[i] : 0u;
    }
    const uint32_t before_all = chunk > first && chunk < left ? tile_keys[chunk - 1] : 0u;
    for (int k = threadIdx.x; k < kWaves * kMaxSegments / 2; k += S::kThreads) reinterpret_cast<uint32_t*>(&wave_cnt[0][0])[k] = 0;
    __syncthreads();
    uint64_t head[S::kItems];
    uint16_t rank[S::kItems];
#pragma unroll
    for (int r = 0; r < S::kItems; ++r) {
        const int i = chunk + r * 64 + lane;
        const uint32_t prev = key_before(key, r, before_all);
        const bool mine = i < left && (i == first || key[r] != prev);
        head[r] = __ballot(mine);
        const int d = (int)((key[r] & item_mask) >> item_low);
        const uint64_t peers = lanes_of_digit<8>(d, digit_bits, head[r]);
        const int pre = wave_cnt[wave][d];
        const int below = __popcll(peers & lt_mask);
        rank[r] = (uint16_t)(pre + below);
        if (mine && below == 0) wave_cnt[wave][d] = (uint16_t)(pre + __popcll(peers));
    }
    __syncthreads();
    {   // digit t of thread t: its place in the tile, where the tile's keys of it go, and every wavefront's first place
        int32_t mine = 0;
        if (threadIdx.x < kMaxSegments)
#pragma unroll
            for (int w = 0; w < kWaves; ++w) mine += wave_cnt[w][threadIdx.x];
        int32_t inc = mine;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const int32_t t = __shfl_up(inc, dlt, 64);
            if (lane >= dlt) inc += t;
        }
        if (lane == 63) red[wave] = inc;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            if (w < wave) inc += red[w];
        if (threadIdx.x < kMaxSegments) {
            int32_t place = inc - mine;
            shift_by[threadIdx.x] = base - place;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const int c = wave_cnt[w][threadIdx.x];
                wave_cnt[w][threadIdx.x] = (uint16_t)place;
                place += c;
            }
        }
    }
    __syncthreads();
    int32_t all = 0;   // red[] holds inclusive sums over the digits; those of the first wavefronts cover them all
#pragma unroll
    for (int w = 0; w < kMaxSegments / 64; ++w) all += red[w];
#pragma unroll
    for (int r = 0; r < S::kItems; ++r) {
        if ((head[r] >> lane) & 1) {
            const uint32_t item = key[r] & item_mask;
            const int d = (int)(item >> item_low);
            const uint32_t u = ((uint32_t)at.segment << user_low) | (key[r] >> item_bits);
            const int place = wave_cnt[wave][d] + rank[r];
            tile[place] = ((item & low_mask) << user_bits) | u;
            tile_digit[place] = (uint8_t)d;
        }
    }
    __syncthreads();
#pragma unroll 4
    for (int p = threadIdx.x; p < all; p += S::kThreads) by_item[(uint32_t)(shift_by[tile_digit[p]] + p)] = tile[p];
}

// ---- row pointers ----------------------------------------------------------------------------------
// Row v holds run_end[v] - run_start[v] entries (items: the count is in run_end, run_start is 0) and the
// diagonal.  Tiles of kRowTile rows; SCANNED as above.
constexpr int kRowThreads = 256;
constexpr int kRowItems = 8;
constexpr int kRowTile = kRowThreads * kRowItems;
constexpr int64_t kRowFew = 2048;

__global__ __launch_bounds__(kRowThreads) void row_sums(const int32_t* __restrict__ start, const int32_t* __restrict__ end,
                                                        int64_t n, int32_t self, int32_t* __restrict__ tile_sum) {
    __shared__ int32_t red[kRowThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kRowTile;
    int32_t sum = 0;
#pragma unroll
    for (int r = 0; r < kRowItems; ++r) {
        const int64_t v = base + r * kRowThreads + threadIdx.x;
        if (v < n) sum += end[v] - start[v] + self;
    }
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int w = 0; w < kRowThreads / 64; ++w) t += red[w];
        tile_sum[blockIdx.x] = t;
    }
}

template <bool SCANNED>
__global__ __launch_bounds__(kRowThreads) void row_pointers(const int32_t* __restrict__ start, const int32_t* __restrict__ end,
                                                            int64_t n, int32_t n_users, int32_t self,
                                                            const int32_t* __restrict__ tile_sum, int32_t* __restrict__ row_ptr,
                                                            int32_t* __restrict__ col_idx) {
    constexpr int kWaves = kRowThreads / 64;
    __shared__ int32_t red[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t before = 0;
    if (SCANNED) {
        before = tile_sum[blockIdx.x];
    } else {
        for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kRowThreads) before += tile_sum[t];
        for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off);
        if (lane == 0) red[wave] = before;
        __syncthreads();
        before = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) before += red[w];
        __syncthreads();
    }
    const int64_t base = (int64_t)blockIdx.x * kRowTile + (int64_t)wave * (64 * kRowItems);
    int32_t cnt[kRowItems], inc[kRowItems], run = 0;
#pragma unroll
    for (int r = 0; r < kRowItems; ++r) {
        const int64_t v = base + r * 64 + lane;
        cnt[r] = v < n ? end[v] - start[v] + self : 0;
    }
#pragma unroll
    for (int r = 0; r < kRowItems; ++r) {
        int32_t t = cnt[r];
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const int32_t o = __shfl_up(t, dlt, 64);
            if (lane >= dlt) t += o;
        }
        inc[r] = run + t;
        run += __shfl(t, 63);
    }
    if (lane == 0) red[wave] = run;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
        if (w < wave) before += red[w];
#pragma unroll
    for (int r = 0; r < kRowItems; ++r) {
        const int64_t v = base + r * 64 + lane;
        if (v >= n) continue;
        const int32_t last = before + inc[r], first = last - cnt[r];
        row_ptr[v + 1] = last;
        if (v == 0) row_ptr[0] = 0;
        // user row: itself first (items have larger ids); item row: itself last
        if (self) col_idx[v < n_users ? first : last - 1] = (int32_t)v;
    }
}

// ---- small graphs: buckets ----------------------------------------------------------------------------
// The pairs are split once into at most 256 ranges of users; a workgroup sorts its range in LDS, drops
// repeats and counts how its pairs spread over 256 ranges of items; the distinct pairs go to their ranges
// of items in order, while the same kernel writes the user rows; a workgroup puts its range of items in
// order, a range of any length, since the users of an item arrive sorted.  Row pointers and the diagonal
// fall out of the per-range counts.  A range of users with more pairs than fit in LDS (ids in order of activity,
// say) raises a flag, and the host, which waits at the end anyhow, then takes the general way.
// Sampled subgraph of 291 k pairs, 173 k nodes: 215 us the general way, launch gaps included.
constexpr int64_t kBucketMaxPairs = 1 << 20;
constexpr int kBucketBits = 8;
constexpr int kBuckets = 1 << kBucketBits;
constexpr int kBucketThreads = 1024;
constexpr int kBucketWaves = kBucketThreads / 64;
constexpr int kBucketRounds = 8;
constexpr int kBucketCap = kBucketThreads * kBucketRounds;   // pairs of one range of users
constexpr int kLowBitsMax = 12;                              // ids of one range
constexpr int kItemThreads = 512;
constexpr int kItemWaves = kItemThreads / 64;

struct BucketPlan {
    int user_bits, item_bits;
    int user_low, item_low;     // bits of an id inside its range
    int n_user_ranges, n_item_ranges;
};

bool plan_buckets(int32_t n_users, int32_t n_items, int64_t n_edges, BucketPlan* p) {
    p->user_bits = bits_for(n_users);
    p->item_bits = bits_for(n_items);
    p->user_low = p->user_bits > kBucketBits ? p->user_bits - kBucketBits : 0;
    p->item_low = p->item_bits > kBucketBits ? p->item_bits - kBucketBits : 0;
    p->n_user_ranges = 1 << (p->user_bits - p->user_low);
    p->n_item_ranges = 1 << (p->item_bits - p->item_low);
    return n_edges > 0 && n_edges <= kBucketMaxPairs && p->user_low <= kLowBitsMax && p->item_low <= kLowBitsMax &&
           p->user_low + p->item_bits <= 32;
}

struct BucketWs {
    int32_t* user_hist;   // [tiles of pairs][kBuckets]
    int32_t* tile_bad;    // [tiles of pairs] an id out of range
    int32_t* item_hist;   // [user ranges][kBuckets]
    int32_t* range_first; // [user ranges] first pair of every range of users
    int32_t* distinct;    // [user ranges] distinct pairs
    int32_t* overflow;    // [user ranges]
    int32_t* item_first;  // [item ranges + 1] first pair of every range of items
    int32_t* result;      // [4] distinct pairs, bad ids, overflow
};

BucketWs carve_buckets(Carver& c, int64_t n_edges) {
    BucketWs w = {};
    if (n_edges > kBucketMaxPairs) return w;
    const int64_t tiles = ceil_div(n_edges > 0 ? n_edges : 1, SplitSort::kTile);
    w.user_hist = c.take<int32_t>(tiles * kBuckets);
    w.tile_bad = c.take<int32_t>(tiles);
    w.item_hist = c.take<int32_t>(kBuckets * kBuckets);
    w.range_first = c.take<int32_t>(kBuckets);
    w.distinct = c.take<int32_t>(kBuckets);
    w.overflow = c.take<int32_t>(kBuckets);
    w.item_first = c.take<int32_t>(kBuckets + 1);
    w.result = c.take<int32_t>(4);
    return w;
}

// Pairs per range of users, in every tile.
__global__ __launch_bounds__(SplitSort::kThreads) void count_ranges(PairsIn in, int64_t count, int shift, int bins,
                                                                    BucketWs w) {
    __shared__ int h[kBuckets];
    __shared__ int bad;
    for (int k = threadIdx.x; k < kBuckets; k += SplitSort::kThreads) h[k] = 0;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * SplitSort::kTile;
    int32_t u[SplitSort::kItems], i[SplitSort::kItems];
#pragma unroll
    for (int k = 0; k < SplitSort::kItems; ++k) {
        const int64_t e = base + k * SplitSort::kThreads + threadIdx.x;
        u[k] = e < count ? in.users[e] : 0;
        i[k] = e < count ? in.items[e] : 0;
    }
#pragma unroll
    for (int k = 0; k < SplitSort::kItems; ++k) {
        const int64_t e = base + k * SplitSort::kThreads + threadIdx.x;
        if (e < count) {
            const bool ok = in.ok(u[k], i[k]);
            if (!ok) bad = 1;
            atomicAdd(&h[(int)(in.key(PairsIn::raw{u[k], i[k]}) >> shift)], 1);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < bins; k += SplitSort::kThreads) w.user_hist[(int64_t)blockIdx.x * bins + k] = h[k];
    if (threadIdx.x == 0) w.tile_bad[blockIdx.x] = bad;
}

// Exclusive scan of one value per thread over a workgroup of WAVES wavefronts.
template <int WAVES>
__device__ __forceinline__ int32_t scan_block(int32_t v, int32_t* lds, int32_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t inc = v;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const int32_t t = __shfl_up(inc, dlt, 64);
        if (lane >= dlt) inc += t;
    }
    __syncthreads();
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    int32_t before = inc - v, all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        if (w < wave) before += lds[w];
        all += lds[w];
    }
    *total = all;
    return before;
}

// Ranks of a wavefront's keys by digit, in input order: the running per-wavefront counts are in `cnt`.
template <int BITS>
__device__ __forceinline__ int rank_digit(int d, bool valid, int nbits, uint64_t lt_mask, uint16_t* cnt) {
    const uint64_t peers = lanes_of_digit<BITS>(d, nbits, __ballot(valid));
    const int below = __popcll(peers & lt_mask);
    const int pre = cnt[d];
    if (valid && below == 0) cnt[d] = (uint16_t)(pre + __popcll(peers));
    return pre + below;
}

// One range of users: sorted by (user, item) in LDS, repeats dropped, turned round to (item, user).
__global__ __launch_bounds__(kBucketThreads) void sort_ranges(const uint64_t* __restrict__ pairs, int32_t tiles,
                                                              BucketPlan p, uint64_t* __restrict__ turned, BucketWs w) {
    __shared__ uint32_t keys[2][kBucketCap];
    __shared__ uint16_t cnt[kBucketWaves][256];
    __shared__ int32_t hist[kBuckets];
    __shared__ int32_t part[kBucketThreads / kBuckets][kBuckets];
    __shared__ int32_t lds[kBucketWaves];
    __shared__ int32_t span[2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int r = blockIdx.x;
    {   // where the range's pairs are: totals of all ranges, scanned
        const int d = threadIdx.x % kBuckets, q = threadIdx.x / kBuckets;
        int32_t t = 0;
        if (d < p.n_user_ranges)
#pragma unroll 8
            for (int b = q; b < tiles; b += kBucketThreads / kBuckets) t += w.user_hist[(int64_t)b * p.n_user_ranges + d];
        part[q][d] = t;
        __syncthreads();
        t = 0;
        if (threadIdx.x < kBuckets)
#pragma unroll
            for (int k = 0; k < kBucketThreads / kBuckets; ++k) t += part[k][threadIdx.x];
        int32_t all;
        const int32_t before = scan_block<kBucketWaves>(t, lds, &all);
        if ((int)threadIdx.x == r) {
            span[0] = before;
            span[1] = t;
        }
        if (threadIdx.x < kBuckets) hist[threadIdx.x] = 0;
        __syncthreads();
    }
    const int32_t first = span[0], n = span[1];
    if (threadIdx.x == 0) {
        w.range_first[r] = first;
        w.overflow[r] = n > kBucketCap ? 1 : 0;
    }
    if (n > kBucketCap) {
        if (threadIdx.x == 0) w.distinct[r] = 0;
        if ((int)threadIdx.x < p.n_item_ranges) w.item_hist[r * p.n_item_ranges + threadIdx.x] = 0;
        return;
    }
    const int key_bits = p.user_low + p.item_bits;
    const uint64_t key_mask = (1ull << key_bits) - 1;
    for (int k = threadIdx.x; k < n; k += kBucketThreads) keys[0][k] = (uint32_t)(pairs[first + k] & key_mask);
    const int rounds = (n + kBucketThreads - 1) / kBucketThreads;   // a wavefront's keys: 64 * rounds consecutive ones
    const int chunk = wave * 64 * rounds;
    const int passes = (key_bits + 7) / 8;
    int cur = 0;
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = key_bits * pass / passes, nbits = key_bits * (pass + 1) / passes - shift;
        const int bins = 1 << nbits;
        for (int k = threadIdx.x; k < kBucketWaves * 128; k += kBucketThreads) reinterpret_cast<uint32_t*>(&cnt[0][0])[k] = 0;
        __syncthreads();
        uint32_t key[kBucketRounds];
        int rank[kBucketRounds];
#pragma unroll
        for (int q = 0; q < kBucketRounds; ++q) {
            if (q >= rounds) break;
            const int at = chunk + q * 64 + lane;
            key[q] = at < n ? keys[cur][at] : 0u;
            rank[q] = rank_digit<8>((int)(key[q] >> shift) & (bins - 1), at < n, nbits, lt_mask, cnt[wave]);
        }
        __syncthreads();
        {   // digit t of thread t < 256: counts of the wavefronts become first places
            int32_t mine = 0;
            if (threadIdx.x < 256)
#pragma unroll
                for (int v = 0; v < kBucketWaves; ++v) mine += cnt[v][threadIdx.x];
            int32_t all;
            int32_t at = scan_block<kBucketWaves>(mine, lds, &all);
            if (threadIdx.x < 256)
#pragma unroll
                for (int v = 0; v < kBucketWaves; ++v) {
                    const int c = cnt[v][threadIdx.x];
                    cnt[v][threadIdx.x] = (uint16_t)at;
                    at += c;
                }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kBucketRounds; ++q) {
            if (q >= rounds) break;
            if (chunk + q * 64 + lane < n) keys[1 - cur][cnt[wave][(int)(key[q] >> shift) & (bins - 1)] + rank[q]] = key[q];
        }
        cur = 1 - cur;
        __syncthreads();
    }
    // repeats
    int32_t heads = 0;
    uint64_t bal[kBucketRounds];
#pragma unroll
    for (int q = 0; q < kBucketRounds; ++q) {
        bal[q] = 0;
        if (q >= rounds) break;
        const int at = chunk + q * 64 + lane;
        bal[q] = __ballot(at < n && (at == 0 || keys[cur][at] != keys[cur][at - 1]));
        heads += __popcll(bal[q]);
    }
    if (lane == 0) lds[wave] = heads;
    __syncthreads();
    int32_t before = 0, all = 0;
#pragma unroll
    for (int v = 0; v < kBucketWaves; ++v) {
        if (v < wave) before += lds[v];
        all += lds[v];
    }
#pragma unroll
    for (int q = 0; q < kBucketRounds; ++q) {
        if (q >= rounds) break;
        if ((bal[q] >> lane) & 1) {
            const uint32_t key = keys[cur][chunk + q * 64 + lane];
            const uint32_t item = key & (uint32_t)((1ull << p.item_bits) - 1);
            const uint32_t user = ((uint32_t)r << p.user_low) | (uint32_t)((uint64_t)key >> p.item_bits);
            turned[first + before + __popcll(bal[q] & lt_mask)] = ((uint64_t)item << p.user_bits) | user;
            atomicAdd(&hist[item >> p.item_low], 1);
        }
        before += __popcll(bal[q]);
    }
    __syncthreads();
    if ((int)threadIdx.x < p.n_item_ranges) w.item_hist[r * p.n_item_ranges + threadIdx.x] = hist[threadIdx.x];
    if (threadIdx.x == 0) w.distinct[r] = all;
}

// One range of users: its rows, row pointers and diagonal entries, and its pairs to their ranges of items.
__global__ __launch_bounds__(kBucketThreads) void spread_ranges(const uint64_t* __restrict__ turned, BucketPlan p,
                                                                int32_t n_users, int32_t self, uint64_t* __restrict__ by_item,
                                                                int32_t* __restrict__ row_ptr, int32_t* __restrict__ col_idx,
                                                                BucketWs w) {
    constexpr int kLow = 1 << kLowBitsMax;
    constexpr int kPer = kLow / kBucketThreads;
    __shared__ uint16_t cnt[kBucketWaves][256];
    __shared__ int32_t users[kLow];
    __shared__ int32_t part[2][kBucketThreads / kBuckets][kBuckets];
    __shared__ int32_t base[kBuckets];
    __shared__ int32_t lds[kBucketWaves];
    __shared__ int32_t pairs_before;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int r = blockIdx.x;
    const int32_t n = w.distinct[r], first = w.range_first[r];
    const int rounds = (n + kBucketThreads - 1) / kBucketThreads;
    const int chunk = wave * 64 * rounds;
    uint64_t key[kBucketRounds];
#pragma unroll
    for (int q = 0; q < kBucketRounds; ++q) {
        const int at = chunk + q * 64 + lane;
        key[q] = q < rounds && at < n ? turned[first + at] : 0ull;
    }
    for (int k = threadIdx.x; k < kBucketWaves * 128; k += kBucketThreads) reinterpret_cast<uint32_t*>(&cnt[0][0])[k] = 0;
    for (int k = threadIdx.x; k < kLow; k += kBucketThreads) users[k] = 0;
    {   // where this range's pairs go in every range of items
        const int d = threadIdx.x % kBuckets, q = threadIdx.x / kBuckets;
        int32_t before = 0, total = 0;
        if (d < p.n_item_ranges)
#pragma unroll 16
            for (int b = q; b < p.n_user_ranges; b += kBucketThreads / kBuckets) {
                const int32_t c = w.item_hist[b * p.n_item_ranges + d];
                if (b < r) before += c;
                total += c;
            }
        part[0][q][d] = before;
        part[1][q][d] = total;
        __syncthreads();
        before = total = 0;
        if (threadIdx.x < kBuckets)
#pragma unroll
            for (int k = 0; k < kBucketThreads / kBuckets; ++k) {
                before += part[0][k][threadIdx.x];
                total += part[1][k][threadIdx.x];
            }
        int32_t all;
        const int32_t lower = scan_block<kBucketWaves>(total, lds, &all);
        if (threadIdx.x < kBuckets) base[threadIdx.x] = lower + before;
        if (r == 0 && threadIdx.x < kBuckets) {
            if ((int)threadIdx.x < p.n_item_ranges) w.item_first[threadIdx.x] = lower;
            if (threadIdx.x == 0) w.item_first[p.n_item_ranges] = all;
        }
        const int32_t dist = (int)threadIdx.x < p.n_user_ranges ? w.distinct[threadIdx.x] : 0;
        const int32_t earlier = scan_block<kBucketWaves>(dist, lds, &all);
        if ((int)threadIdx.x == r) pairs_before = earlier;
        __syncthreads();
    }
    const uint64_t user_mask = (1ull << p.user_bits) - 1;
    const uint32_t low_mask = (1u << p.user_low) - 1;
    const int shift = p.user_bits + p.item_low, nbits = p.item_bits - p.item_low;
    int rank[kBucketRounds];
#pragma unroll
    for (int q = 0; q < kBucketRounds; ++q) {
        if (q >= rounds) break;
        const int at = chunk + q * 64 + lane;
        const bool valid = at < n;
        rank[q] = rank_digit<kBucketBits>((int)(key[q] >> shift), valid, nbits, lt_mask, cnt[wave]);
        if (valid) {
            const uint32_t user = (uint32_t)(key[q] & user_mask);
            const int32_t item = (int32_t)(key[q] >> p.user_bits);
            atomicAdd(&users[user & low_mask], 1);
            col_idx[(int64_t)pairs_before + at + (int64_t)(user + 1) * self] = n_users + item;
        }
    }
    __syncthreads();
    if (threadIdx.x < kBuckets) {
        int run = 0;
#pragma unroll
        for (int v = 0; v < kBucketWaves; ++v) {
            const int c = cnt[v][threadIdx.x];
            cnt[v][threadIdx.x] = (uint16_t)run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kBucketRounds; ++q) {
        if (q >= rounds) break;
        if (chunk + q * 64 + lane < n) {
            const int d = (int)(key[q] >> shift);
            by_item[base[d] + cnt[wave][d] + rank[q]] = key[q];
        }
    }
    // row pointers of the range's users
    int32_t mine[kPer], sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        mine[k] = users[threadIdx.x * kPer + k];
        sum += mine[k];
    }
    int32_t all;
    int32_t at = scan_block<kBucketWaves>(sum, lds, &all) + pairs_before;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t low = threadIdx.x * kPer + k;
        const int64_t u = ((int64_t)r << p.user_low) + low;
        if (low <= low_mask && u < n_users) {
            const int32_t row = at + (int32_t)u * self;
            row_ptr[u] = row;
            if (self) col_idx[row] = (int32_t)u;   // user row: itself first (items have larger ids)
        }
        at += mine[k];
    }
}

// One range of items: its rows, row pointers and diagonal entries.  Any number of pairs: a tile of them at a
// time, each item's place moving on from tile to tile.  Workgroup 0 also writes the result for the host.
__global__ __launch_bounds__(kItemThreads) void item_ranges(const uint64_t* __restrict__ by_item, BucketPlan p,
                                                            int32_t n_users, int32_t n_items, int32_t self, int32_t tiles,
                                                            int32_t* __restrict__ row_ptr, int32_t* __restrict__ col_idx,
                                                            BucketWs w) {
    constexpr int kLow = 1 << kLowBitsMax;
    constexpr int kPer = kLow / kItemThreads;
    constexpr int kRounds = 4;
    __shared__ uint16_t cnt[kItemWaves][kLow];
    __shared__ int32_t place[kLow];   // where the item's next user goes in col_idx
    __shared__ int32_t lds[kItemWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int r = blockIdx.x;
    const int32_t first = w.item_first[r], end = w.item_first[r + 1], pairs = w.item_first[p.n_item_ranges];
    const int ids = 1 << p.item_low;
    if (r == 0) {
        int32_t bad = 0, over = 0, all;
        for (int t = threadIdx.x; t < tiles; t += kItemThreads) bad |= w.tile_bad[t];
        for (int t = threadIdx.x; t < p.n_user_ranges; t += kItemThreads) over |= w.overflow[t];
        scan_block<kItemWaves>(bad, lds, &all);
        if (threadIdx.x == 0) w.result[1] = all;
        scan_block<kItemWaves>(over, lds, &all);
        if (threadIdx.x == 0) {
            w.result[0] = pairs;
            w.result[2] = all;
            row_ptr[n_users + n_items] = 2 * pairs + (n_users + n_items) * self;
        }
    }
    for (int k = threadIdx.x; k < ids; k += kItemThreads) place[k] = 0;
    __syncthreads();
    const uint32_t low_mask = (uint32_t)ids - 1;
#pragma unroll 4
    for (int32_t k = first + (int32_t)threadIdx.x; k < end; k += kItemThreads)
        atomicAdd(&place[(uint32_t)(by_item[k] >> p.user_bits) & low_mask], 1);
    __syncthreads();
    {
        int32_t mine[kPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int id = threadIdx.x * kPer + k;
            mine[k] = id < ids ? place[id] : 0;
            sum += mine[k];
        }
        int32_t all;
        int32_t at = scan_block<kItemWaves>(sum, lds, &all) + pairs + n_users * self + first;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int id = threadIdx.x * kPer + k;
            const int64_t i = ((int64_t)r << p.item_low) + id;
            if (id < ids && i < n_items) {
                const int32_t row = at + (int32_t)i * self;
                row_ptr[n_users + i] = row;
                place[id] = row;
                if (self) col_idx[row + mine[k]] = n_users + (int32_t)i;   // item row: itself last
            }
            at += mine[k];
        }
    }
    __syncthreads();
    const uint64_t user_mask = (1ull << p.user_bits) - 1;
    for (int32_t t0 = first; t0 < end; t0 += kRounds * kItemThreads) {
        for (int k = threadIdx.x; k < ids; k += kItemThreads)
#pragma unroll
            for (int v = 0; v < kItemWaves; ++v) cnt[v][k] = 0;
        __syncthreads();
        uint64_t key[kRounds];
        int rank[kRounds];
#pragma unroll
        for (int q = 0; q < kRounds; ++q) {
            const int32_t k = t0 + wave * 64 * kRounds + q * 64 + lane;
            key[q] = k < end ? by_item[k] : 0ull;
        }
#pragma unroll
        for (int q = 0; q < kRounds; ++q) {
            const int32_t k = t0 + wave * 64 * kRounds + q * 64 + lane;
            rank[q] = rank_digit<kLowBitsMax>((int)((uint32_t)(key[q] >> p.user_bits) & low_mask), k < end, p.item_low,
                                              lt_mask, cnt[wave]);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kRounds; ++q) {
            const int32_t k = t0 + wave * 64 * kRounds + q * 64 + lane;
            if (k < end) {
                const int d = (int)((uint32_t)(key[q] >> p.user_bits) & low_mask);
                int32_t at = place[d] + rank[q];
#pragma unroll
                for (int v = 0; v < kItemWaves; ++v)
                    if (v < wave) at += cnt[v][d];
                col_idx[at] = (int32_t)(key[q] & user_mask);
            }
        }
        __syncthreads();
        if (t0 + kRounds * kItemThreads < end)
            for (int k = threadIdx.x; k < ids; k += kItemThreads) {
                int32_t sum = 0;
#pragma unroll
                for (int v = 0; v < kItemWaves; ++v) sum += cnt[v][k];
                place[k] += sum;
            }
        __syncthreads();
    }
}

// Weighted graphs (Section 3, "Notation": A_ij > 0 marks an edge, so its size is free to carry
// a strength).  Stored values of A~: 1 on the diagonal, 0 until a listed pair brings its weight.
// Of the two entries of a pair the one on the side with more nodes, whose rows are the shorter on average, takes
// the weights; the other then copies its value.  So nothing is searched for in a popular node's row, and half
// of the entries see no atomics.  Both passes are bound by the number of scattered reads (some 130 G a second
// in all), so a search ends in one read of the last few entries.  2 M pairs: 325 us with every pair
// searched for in both rows and every entry's row in all of row_ptr, 200 so.
// Where column c stands among the ascending columns [lo, hi), or -1.
__device__ __forceinline__ int32_t find_column(const int32_t* __restrict__ col, int32_t lo, int32_t hi, int32_t c, int64_t nnz) {
    constexpr int kTail = 8;
    while (hi - lo > kTail) {   // the answer, if there is one, is in [lo, hi)
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (col[mid] <= c) lo = mid; else hi = mid;
    }
    if (lo + kTail <= nnz) {
        typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));
        const i32x4 a = *reinterpret_cast<const i32x4*>(col + lo), b = *reinterpret_cast<const i32x4*>(col + lo + 4);
        int32_t at = -1;
#pragma unroll
        for (int k = kTail - 1; k >= 0; --k)
            if ((k < 4 ? a[k & 3] : b[k & 3]) == c) at = lo + k;
        return at < hi ? at : -1;
    }
    for (; lo < hi; ++lo)
        if (col[lo] == c) return lo;
    return -1;
}

__global__ void zero_values(float* __restrict__ val, int64_t nnz) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < nnz) val[e] = 0.0f;
}

// One thread per pair.  A pair listed several times keeps its largest weight: positive floats order like their
// bit patterns read as integers, which makes the maximum an integer atomic and the result independent of the
// order of arrival.
__global__ void apply_weights(const int32_t* __restrict__ users, const int32_t* __restrict__ items,
                              const float* __restrict__ weights, int64_t n_edges, int32_t n_users,
                              int32_t n_items, int64_t nnz, bool by_user, const int32_t* __restrict__ row_ptr,
                              const int32_t* __restrict__ col_idx, float* val) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_edges) return;
    const int32_t u = users[e], i = items[e];
    const float w = weights[e];
    if (u < 0 || u >= n_users || i < 0 || i >= n_items || !(w > 0.0f)) return;
    const int32_t row = by_user ? u : n_users + i, c = by_user ? n_users + i : u;
    int32_t r[2];
    __builtin_memcpy(r, row_ptr + row, sizeof(r));
    const int32_t at = find_column(col_idx, r[0], r[1], c, nnz);
    if (at >= 0) atomicMax(reinterpret_cast<int*>(val) + at, __float_as_int(w));
}

// The other entry of every pair, and the diagonal, by tiles of entries.
__global__ __launch_bounds__(kEntryThreads) void mirror_weights(const int32_t* __restrict__ row_ptr,
                                                                const int32_t* __restrict__ col_idx, int64_t n, int64_t nnz,
                                                                int32_t n_users, bool by_user, float* val) {
    __shared__ int32_t rows[kTileRowsMax + 1];
    const EntryTile tile(row_ptr, n, nnz, rows);
    // entries before `split` are in rows of users
    const int64_t split = row_ptr[n_users];
    int32_t c[kEntryRounds], far[kEntryRounds][2];
#pragma unroll
    for (int r = 0; r < kEntryRounds; ++r) {
        const int64_t e = tile.first + r * kEntryThreads + threadIdx.x;
        c[r] = e <= tile.last ? col_idx[e] : -1;
    }
#pragma unroll
    for (int r = 0; r < kEntryRounds; ++r) {
        const int64_t e = tile.first + r * kEntryThreads + threadIdx.x;
        far[r][0] = far[r][1] = 0;
        if (c[r] >= 0 && (e < split) != by_user) __builtin_memcpy(far[r], row_ptr + c[r], sizeof(far[r]));
    }
#pragma unroll
    for (int r = 0; r < kEntryRounds; ++r) {
        if (c[r] < 0) continue;
        const int64_t e = tile.first + r * kEntryThreads + threadIdx.x;
        const int32_t i = (int32_t)(tile.row0 + tile.row(e));
        if (c[r] == i) {
            val[e] = 1.0f;
        } else if (far[r][1] > far[r][0]) {
            const int32_t at = find_column(col_idx, far[r][0], far[r][1], i, nnz);
            if (at >= 0) val[e] = val[at];
        }
    }
}

struct BuildWs {
    uint64_t* buf_a;
    uint64_t* buf_b;
    int32_t* tile_cnt;
    void* sort_ws;
    int32_t* zeroed;     // small[64], run_start[n + 1], run_end[n + 1]
    int32_t* small;      // [0] distinct-pair count, [1] bad-id flag
    int32_t* run_start;
    int32_t* run_end;
    int64_t zero_count;
    void* scan_ws;
    Segments* segments;  // [2] of the users, of the items
    int32_t* cells;      // digit counts of the segments' tiles
    BucketWs buckets;
    size_t bytes;
};

// The widths of the 32-bit way; tiles 0 where it is not taken: short lists, whose passes are bound by launches,
// and id ranges of more than 40 bits together.
struct ListPlan {
    int user_bits, item_bits;
    int user_low, item_low;   // bits behind the leading digit
    int64_t tiles;            // upper bound
};
ListPlan plan_lists(int32_t n_users, int32_t n_items, int64_t n_edges) {
    ListPlan p = {bits_for(n_users), bits_for(n_items), 0, 0, 0};
    p.user_low = p.user_bits > 8 ? p.user_bits - 8 : 0;
    p.item_low = p.item_bits > 9 ? p.item_bits - 8 : 1;   // something is left for the pass that writes the item rows
    if (sorts_large(n_edges) && p.user_low + p.item_bits <= 32 && p.item_low + p.user_bits <= 32)
        p.tiles = ceil_div(n_edges, ListSort::kTile) + kMaxSegments;
    return p;
}

BuildWs carve_build(void* base, int32_t n_users, int32_t n_items, int64_t n_edges) {
    const int64_t n = (int64_t)n_users + n_items;
    const int64_t e = n_edges > 0 ? n_edges : 1;
    Carver c(base);
    BuildWs w;
    w.buf_a = c.take<uint64_t>(e);
    w.buf_b = c.take<uint64_t>(e);
    const int64_t head_tiles = ceil_div(e, kHeadTile), row_tiles = ceil_div(n > 0 ? n : 1, kRowTile);
    const int64_t tiles = head_tiles > row_tiles ? head_tiles : row_tiles;
    const int64_t cells = plan_lists(n_users, n_items, n_edges).tiles * kMaxSegments;
    w.tile_cnt = c.take<int32_t>(tiles);
    w.sort_ws = c.take<char>(radix_sort_workspace_bytes(e));
    w.zero_count = 64 + 2 * (n + 1);
    w.zeroed = c.take<int32_t>(w.zero_count);
    w.small = w.zeroed;
    w.run_start = w.zeroed ? w.zeroed + 64 : nullptr;
    w.run_end = w.zeroed ? w.run_start + (n + 1) : nullptr;
    w.scan_ws = c.take<char>(scan_workspace_bytes(tiles > cells ? tiles : cells));
    w.segments = c.take<Segments>(2);
    w.cells = c.take<int32_t>(cells > 0 ? cells : 1);
    w.buckets = carve_buckets(c, n_edges);
    w.bytes = c.size();
    return w;
}

// The sort of all pairs by (user, item), the distinct ones as user rows, and their sort by item as item rows.
int32_t sort_pairs(const BuildWs& w, int32_t n_users, int32_t n_items, int64_t n_edges, const int32_t* users,
                   const int32_t* items, int32_t self, int32_t* col_idx, hipStream_t stream) {
    const int user_bits = bits_for(n_users), item_bits = bits_for(n_items);
    uint64_t* src = w.buf_a;
    uint64_t* dst = w.buf_b;
    int passes = sort_passes(n_edges, user_bits + item_bits);
    for (int p = 0, shift = 0; p < passes; ++p) {
        const int width = sort_width(user_bits + item_bits, passes, p);
        const int32_t st = p == 0 ? radix_pass(PairsIn{users, items, n_users, n_items, item_bits, w.small + 1}, KeysOut{dst},
                                               n_edges, nullptr, shift, width, w.sort_ws, stream)
                                  : radix_pass(KeysIn{src}, KeysOut{dst}, n_edges, nullptr, shift, width, w.sort_ws, stream);
        if (st != E2EG_OK) return st;
        shift += width;
        uint64_t* t = src;
        src = dst;
        dst = t;
    }
    const int64_t tiles = ceil_div(n_edges, kHeadTile);
    const dim3 grid((unsigned)tiles), blk(kHeadThreads);
    count_heads<<<grid, blk, 0, stream>>>(src, n_edges, w.tile_cnt);
    E2EG_LAUNCH_CHECK("count_heads");
    if (tiles > kHeadFew) {
        E2EG_HIP_TRY(exclusive_scan_i32(w.tile_cnt, w.tile_cnt, tiles, nullptr, w.scan_ws, stream));
        emit_pairs<true><<<grid, blk, 0, stream>>>(src, n_edges, w.tile_cnt, user_bits, item_bits, n_users, self, dst, col_idx,
                                                  w.run_start, w.run_end, w.small);
    } else {
        emit_pairs<false><<<grid, blk, 0, stream>>>(src, n_edges, w.tile_cnt, user_bits, item_bits, n_users, self, dst, col_idx,
                                                   w.run_start, w.run_end, w.small);
    }
    E2EG_LAUNCH_CHECK("emit_pairs");
    uint64_t* t = src;
    src = dst;
    dst = t;
    passes = sort_passes(n_edges, item_bits);
    for (int p = 0, shift = user_bits; p < passes; ++p) {
        const int width = sort_width(item_bits, passes, p);
        const int32_t st =
            p + 1 < passes ? radix_pass(KeysIn{src}, KeysOut{dst}, n_edges, w.small, shift, width, w.sort_ws, stream)
                           : radix_pass(KeysIn{src}, ItemRowsOut{col_idx, w.small, w.run_end + n_users, n_users, self, user_bits},
                                        n_edges, w.small, shift, width, w.sort_ws, stream);
        if (st != E2EG_OK) return st;
        shift += width;
        t = src;
        src = dst;
        dst = t;
    }
    return E2EG_OK;
}

// One pass over the segments' keys.
template <typename Out>
int32_t segment_pass(const BuildWs& w, const ListPlan& p, const Segments* s, int n, const uint32_t* keys, Out out, int shift,
                     int nbits, hipStream_t stream) {
    const ArrayIn<uint32_t> in{keys};
    const Segmented tiling{s, n};
    const dim3 grid((unsigned)p.tiles), blk(ListSort::kThreads);
    sort_histogram<ListSort, ArrayIn<uint32_t>, Segmented, false><<<grid, blk, 0, stream>>>(in, tiling, shift, nbits, w.cells);
    E2EG_LAUNCH_CHECK("sort_histogram");
    E2EG_HIP_TRY(exclusive_scan_i32(w.cells, w.cells, p.tiles << nbits, nullptr, w.scan_ws, stream));
    sort_scatter<ListSort, ArrayIn<uint32_t>, Out, Segmented, false><<<grid, blk, 0, stream>>>(in, out, tiling, shift, nbits, w.cells);
    E2EG_LAUNCH_CHECK("sort_scatter");
    return E2EG_OK;
}

// As sort_pairs, with 32-bit keys.
int32_t sort_lists(const BuildWs& w, const ListPlan& p, int32_t n_users, int32_t n_items, int64_t n_edges, const int32_t* users,
                   const int32_t* items, int32_t self, int32_t* col_idx, hipStream_t stream) {
    uint32_t* src = reinterpret_cast<uint32_t*>(w.buf_a);
    uint32_t* dst = reinterpret_cast<uint32_t*>(w.buf_b);
    const auto swap = [&] { uint32_t* t = src; src = dst; dst = t; };
    const dim3 blk(ListSort::kThreads);
    const int32_t whole_tiles = (int32_t)ceil_div(n_edges, ListSort::kTile);
    const int user_digit = p.user_bits - p.user_low, item_digit = p.item_bits - p.item_low;
    const int rest = p.user_low + p.item_bits;   // bits of a user segment's keys
    {   // segments of the user's leading digit
        const Whole whole{n_edges, nullptr, whole_tiles};
        sort_histogram<ListSort, UsersIn, Whole, false><<<dim3((unsigned)whole_tiles), blk, 0, stream>>>(
            UsersIn{users, n_users, p.item_bits}, whole, rest, user_digit, w.cells);
        E2EG_LAUNCH_CHECK("sort_histogram");
        E2EG_HIP_TRY(exclusive_scan_i32(w.cells, w.cells, (int64_t)whole_tiles << user_digit, nullptr, w.scan_ws, stream));
        sort_scatter<ListSort, PairsIn, LowBitsOut, Whole, false><<<dim3((unsigned)whole_tiles), blk, 0, stream>>>(
            PairsIn{users, items, n_users, n_items, p.item_bits, w.small + 1},
            LowBitsOut{src, (uint32_t)((1ull << rest) - 1)}, whole, rest, user_digit, w.cells);
        E2EG_LAUNCH_CHECK("sort_scatter");
        plan_segments<<<dim3(1), dim3(kMaxSegments), 0, stream>>>(w.cells, whole_tiles, 1 << user_digit, n_edges, nullptr, w.segments);
        E2EG_LAUNCH_CHECK("plan_segments");
    }
    const int passes = (rest + ListSort::kBits - 1) / ListSort::kBits;
    for (int q = 0, shift = 0; q < passes; ++q) {
        const int width = sort_width(rest, passes, q);
        const int32_t st = segment_pass(w, p, w.segments, 1 << user_digit, src, ArrayOut<uint32_t>{dst}, shift, width, stream);
        if (st != E2EG_OK) return st;
        shift += width;
        swap();
    }
    const dim3 grid((unsigned)p.tiles);
    const Segmented tiling{w.segments, 1 << user_digit};
    count_distinct<<<grid, blk, 0, stream>>>(src, tiling, p.item_bits, p.item_low, 1 << item_digit, w.tile_cnt, w.cells);
    E2EG_LAUNCH_CHECK("count_distinct");
    E2EG_HIP_TRY(exclusive_scan_i32(w.tile_cnt, w.tile_cnt, p.tiles, nullptr, w.scan_ws, stream));
    E2EG_HIP_TRY(exclusive_scan_i32(w.cells, w.cells, p.tiles << item_digit, nullptr, w.scan_ws, stream));
    write_user_rows<<<grid, dim3(kUserThreads), 0, stream>>>(src, tiling, n_edges, p.user_low, p.item_bits, n_users, self, w.tile_cnt,
                                                            col_idx, w.run_start, w.run_end, w.small);
    E2EG_LAUNCH_CHECK("write_user_rows");
    spread_distinct<<<grid, blk, 0, stream>>>(src, tiling, p.user_low, p.user_bits, p.item_bits, p.item_low, item_digit, w.cells, dst);
    E2EG_LAUNCH_CHECK("spread_distinct");
    plan_segments<<<dim3(1), dim3(kMaxSegments), 0, stream>>>(w.cells, (int32_t)p.tiles, 1 << item_digit, 0, w.small,
                                                             w.segments + 1);
    E2EG_LAUNCH_CHECK("plan_segments");
    swap();
    const int item_passes = (p.item_low + ListSort::kBits - 1) / ListSort::kBits;
    for (int q = 0, shift = p.user_bits; q < item_passes; ++q) {
        const int width = sort_width(p.item_low, item_passes, q);
        const int32_t st =
            q + 1 < item_passes
                ? segment_pass(w, p, w.segments + 1, 1 << item_digit, src, ArrayOut<uint32_t>{dst}, shift, width, stream)
                : segment_pass(w, p, w.segments + 1, 1 << item_digit, src,
                               ItemSegmentsOut{col_idx, w.small, w.run_end + n_users, n_users, self, p.user_bits, p.item_low},
                               shift, width, stream);
        if (st != E2EG_OK) return st;
        shift += width;
        swap();
    }
    return E2EG_OK;
}

// The general way.
int32_t build_sorted(const BuildWs& w, int32_t n_users, int32_t n_items, int64_t n_edges, const int32_t* users,
                     const int32_t* items, int32_t self, int32_t* row_ptr, int32_t* col_idx, hipStream_t stream) {
    const int64_t n = (int64_t)n_users + n_items;
    zero_i32<<<dim3(blocks_for(w.zero_count, kThreads)), dim3(kThreads), 0, stream>>>(w.zeroed, w.zero_count);
    E2EG_LAUNCH_CHECK("zero_i32");
    if (n_edges > 0) {
        const ListPlan p = plan_lists(n_users, n_items, n_edges);
        const int32_t st = p.tiles > 0 ? sort_lists(w, p, n_users, n_items, n_edges, users, items, self, col_idx, stream)
                                       : sort_pairs(w, n_users, n_items, n_edges, users, items, self, col_idx, stream);
        if (st != E2EG_OK) return st;
    }
    if (n == 0) {
        zero_i32<<<dim3(1), dim3(64), 0, stream>>>(row_ptr, 1);
        E2EG_LAUNCH_CHECK("zero_i32");
        return E2EG_OK;
    }
    const int64_t tiles = ceil_div(n, kRowTile);
    const dim3 grid((unsigned)tiles), blk(kRowThreads);
    row_sums<<<grid, blk, 0, stream>>>(w.run_start, w.run_end, n, self, w.tile_cnt);
    E2EG_LAUNCH_CHECK("row_sums");
    if (tiles > kRowFew) {
        E2EG_HIP_TRY(exclusive_scan_i32(w.tile_cnt, w.tile_cnt, tiles, nullptr, w.scan_ws, stream));
        row_pointers<true><<<grid, blk, 0, stream>>>(w.run_start, w.run_end, n, n_users, self, w.tile_cnt, row_ptr, col_idx);
    } else {
        row_pointers<false><<<grid, blk, 0, stream>>>(w.run_start, w.run_end, n, n_users, self, w.tile_cnt, row_ptr, col_idx);
    }
    E2EG_LAUNCH_CHECK("row_pointers");
    return E2EG_OK;
}

int32_t build_bucketed(const BuildWs& w, const BucketPlan& p, int32_t n_users, int32_t n_items, int64_t n_edges,
                       const int32_t* users, const int32_t* items, int32_t self, int32_t* row_ptr, int32_t* col_idx,
                       hipStream_t stream) {
    const PairsIn in{users, items, n_users, n_items, p.item_bits, nullptr};
    const int32_t tiles = (int32_t)ceil_div(n_edges, SplitSort::kTile);
    const int shift = p.item_bits + p.user_low;
    const dim3 split_grid((unsigned)tiles), split_blk(SplitSort::kThreads);
    const dim3 user_grid((unsigned)p.n_user_ranges), user_blk(kBucketThreads);
    count_ranges<<<split_grid, split_blk, 0, stream>>>(in, n_edges, shift, p.n_user_ranges, w.buckets);
    E2EG_LAUNCH_CHECK("count_ranges");
    sort_scatter<SplitSort, PairsIn, KeysOut, Whole, true><<<split_grid, split_blk, 0, stream>>>(
        in, KeysOut{w.buf_a}, Whole{n_edges, nullptr, tiles}, shift, p.user_bits - p.user_low, w.buckets.user_hist);
    E2EG_LAUNCH_CHECK("sort_scatter");
    sort_ranges<<<user_grid, user_blk, 0, stream>>>(w.buf_a, tiles, p, w.buf_b, w.buckets);
    E2EG_LAUNCH_CHECK("sort_ranges");
    spread_ranges<<<user_grid, user_blk, 0, stream>>>(w.buf_b, p, n_users, self, w.buf_a, row_ptr, col_idx, w.buckets);
    E2EG_LAUNCH_CHECK("spread_ranges");
    item_ranges<<<dim3((unsigned)p.n_item_ranges), dim3(kItemThreads), 0, stream>>>(w.buf_a, p, n_users, n_items, self, tiles,
                                                                                 row_ptr, col_idx, w.buckets);
    E2EG_LAUNCH_CHECK("item_ranges");
    return E2EG_OK;
}

}  // namespace
}  // namespace e2eg

using namespace e2eg;

extern "C" size_t e2eg_build_csr_workspace_bytes(int32_t n_users, int32_t n_items,
                                                 int64_t n_edges) {
    if (n_users < 0 || n_items < 0 || n_edges < 0) return 0;
    return carve_build(nullptr, n_users, n_items, n_edges).bytes;
}

extern "C" int32_t e2eg_build_csr(int32_t n_users, int32_t n_items, int64_t n_edges,
                                  const int32_t* d_user_ids, const int32_t* d_item_ids,
                                  int32_t flags, int32_t* d_row_ptr, int32_t* d_col_idx,
                                  int64_t col_capacity, int64_t* h_nnz_out, void* ws,
                                  size_t ws_bytes, void* stream_) {
    if (n_users < 0 || n_items < 0 || n_edges < 0)
        return fail(E2EG_ERR_INVALID_ARG, "build_csr: negative size");
    if (flags & ~E2EG_ADD_SELF_LOOPS) return fail(E2EG_ERR_INVALID_ARG, "build_csr: unknown flag bits 0x%x", flags);
    const int64_t n = (int64_t)n_users + n_items;
    const int32_t self = (flags & E2EG_ADD_SELF_LOOPS) ? 1 : 0;
    if (n > INT32_MAX - 1 || n_edges > (int64_t)INT32_MAX || 2 * n_edges + n > (int64_t)INT32_MAX)
        return fail(E2EG_ERR_OVERFLOW, "build_csr: n=%lld, 2*n_edges+n=%lld exceed int32",
                    (long long)n, (long long)(2 * n_edges + n));
    if (!d_row_ptr || !h_nnz_out || (n_edges > 0 && (!d_user_ids || !d_item_ids)))
        return fail(E2EG_ERR_NULL_PTR, "build_csr: null pointer");
    if ((2 * n_edges + n * self) > 0 && !d_col_idx)
        return fail(E2EG_ERR_NULL_PTR, "build_csr: d_col_idx is null");
    if (col_capacity < 2 * n_edges + n * self)
        return fail(E2EG_ERR_CAPACITY, "build_csr: col_capacity %lld < 2*n_edges+n = %lld",
                    (long long)col_capacity, (long long)(2 * n_edges + n * self));
    if (n_edges > 0 && (n_users == 0 || n_items == 0))
        return fail(E2EG_ERR_INVALID_ARG, "build_csr: edges given but no users or no items");
    const size_t need = e2eg_build_csr_workspace_bytes(n_users, n_items, n_edges);
    if (!ws || !aligned_to(ws, kAlign) || ws_bytes < need)
        return fail(E2EG_ERR_WORKSPACE, "build_csr: workspace needs %zu bytes, 256-byte aligned", need);

    hipStream_t stream = static_cast<hipStream_t>(stream_);
    BuildWs w = carve_build(ws, n_users, n_items, n_edges);
    // The one wait is at the end: the pair count is the caller's to know.
    int32_t host_small[3] = {0, 0, 0};   // distinct pairs, bad ids, buckets overflowed
    BucketPlan plan;
    const bool bucketed = plan_buckets(n_users, n_items, n_edges, &plan);
    if (bucketed) {
        int32_t st = build_bucketed(w, plan, n_users, n_items, n_edges, d_user_ids, d_item_ids, self, d_row_ptr, d_col_idx, stream);
        if (st != E2EG_OK) return st;
        if ((st = read_back(w.buckets.result, 3, host_small, stream)) != E2EG_OK) return st;
    }
    if (!bucketed || (host_small[1] == 0 && host_small[2] != 0)) {
        int32_t st = build_sorted(w, n_users, n_items, n_edges, d_user_ids, d_item_ids, self, d_row_ptr, d_col_idx, stream);
        if (st != E2EG_OK) return st;
        if (n_edges > 0) {
            if ((st = read_back(w.small, 2, host_small, stream)) != E2EG_OK) return st;
        } else {
            E2EG_HIP_TRY(hipStreamSynchronize(stream));
        }
    }
    if (host_small[1] != 0) return fail(E2EG_ERR_BAD_INDEX, "build_csr: a user or item id is out of range");
    *h_nnz_out = 2 * (int64_t)host_small[0] + n * self;
    return E2EG_OK;
}

extern "C" int32_t e2eg_edge_weights(int32_t n_users, int32_t n_items, int64_t n_edges,
                                     const int32_t* d_user_ids, const int32_t* d_item_ids,
                                     const float* d_weights, int64_t nnz, const int32_t* d_row_ptr,
                                     const int32_t* d_col_idx, float* d_val, void* stream_) {
    if (n_users < 0 || n_items < 0 || n_edges < 0 || nnz < 0)
        return fail(E2EG_ERR_INVALID_ARG, "edge_weights: negative size");
    const int64_t n = (int64_t)n_users + n_items;
    if (n > INT32_MAX - 1 || n_edges > (int64_t)INT32_MAX || nnz > (int64_t)INT32_MAX)
        return fail(E2EG_ERR_OVERFLOW, "edge_weights: n=%lld, nnz=%lld exceed int32", (long long)n, (long long)nnz);
    if (!d_row_ptr || (n_edges > 0 && (!d_user_ids || !d_item_ids || !d_weights)) || (nnz > 0 && (!d_col_idx || !d_val)))
        return fail(E2EG_ERR_NULL_PTR, "edge_weights: null pointer");
    if (nnz > 0 && n == 0) return fail(E2EG_ERR_INVALID_ARG, "edge_weights: entries given but no nodes");
    if (nnz == 0) return E2EG_OK;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    const dim3 blk(kThreads);
    const bool by_user = n_users >= n_items;
    zero_values<<<dim3(blocks_for(nnz, kThreads)), blk, 0, stream>>>(d_val, nnz);
    E2EG_LAUNCH_CHECK("zero_values");
    if (n_edges > 0) {
        apply_weights<<<dim3(blocks_for(n_edges, kThreads)), blk, 0, stream>>>(
            d_user_ids, d_item_ids, d_weights, n_edges, n_users, n_items, nnz, by_user, d_row_ptr, d_col_idx, d_val);
        E2EG_LAUNCH_CHECK("apply_weights");
    }
    mirror_weights<<<dim3((unsigned)ceil_div(nnz, kEntryTile)), dim3(kEntryThreads), 0, stream>>>(d_row_ptr, d_col_idx, n, nnz,
                                                                                                n_users, by_user, d_val);
    E2EG_LAUNCH_CHECK("mirror_weights");
    return E2EG_OK;
}
