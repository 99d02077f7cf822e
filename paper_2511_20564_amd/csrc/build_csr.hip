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
// Bound by HBM for large graphs (8 sort passes of 16 bytes read and 8 written per pair), by the number
// of launches for small ones.
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
    __device__ __forceinline__ uint64_t load(int64_t e) const {
        const int32_t u = users[e], i = items[e];
        return ok(u, i) ? ((uint64_t)(uint32_t)u << item_bits) | (uint32_t)i : 0ull;
    }
    __device__ __forceinline__ void check(int64_t e) const {
        if (!ok(users[e], items[e])) atomicOr(bad, 1);
    }
};

// Sorted (item, user) keys -> item rows: key k of the list lands behind the user rows and the earlier
// items' diagonal entries.
struct ItemRowsOut {
    static constexpr bool kRuns = true;
    int32_t* col_idx;
    const int32_t* pairs;   // number of distinct pairs
    int32_t* counts;        // per item, cleared
    int64_t n_users;
    int32_t self;
    int user_bits;
    __device__ __forceinline__ int32_t group(uint64_t key) const { return (int32_t)(key >> user_bits); }
    __device__ __forceinline__ void store(int64_t at, uint64_t key) const {
        const int64_t row0 = *pairs + (n_users + group(key)) * self;
        col_idx[row0 + at] = (int32_t)(key & ((1ull << user_bits) - 1));
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

// Weighted graphs (Section 3, "Notation": A_ij > 0 marks an edge, so its size is free to carry
// a strength).  Stored values of A~: 1 on the diagonal, 0 until a listed pair brings its weight.
__global__ void init_values(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                            int64_t n, int64_t nnz, float* __restrict__ val) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    int64_t lo = 0, hi = n - 1;  // the row of entry e: last i with row_ptr[i] <= e
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (row_ptr[mid] <= e) lo = mid; else hi = mid - 1;
    }
    val[e] = col_idx[e] == (int32_t)lo ? 1.0f : 0.0f;
}

// One thread per (pair, direction): the entry is found by binary search in its (ascending) row; a
// pair listed several times keeps its largest weight.  Positive floats order like their bit
// patterns read as integers, which makes the maximum an integer atomic and the result independent
// of the order of arrival.
__global__ void apply_weights(const int32_t* __restrict__ users, const int32_t* __restrict__ items,
                              const float* __restrict__ weights, int64_t n_edges, int32_t n_users,
                              int32_t n_items, const int32_t* __restrict__ row_ptr,
                              const int32_t* __restrict__ col_idx, float* val) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * n_edges) return;
    const int64_t e = t >> 1;
    const int32_t u = users[e], i = items[e];
    const float w = weights[e];
    if (u < 0 || u >= n_users || i < 0 || i >= n_items || !(w > 0.0f)) return;
    const int32_t r = (t & 1) ? n_users + i : u;
    const int32_t c = (t & 1) ? u : n_users + i;
    const int32_t end = row_ptr[r + 1];
    int32_t lo = row_ptr[r], hi = end;  // first position with col_idx >= c
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (col_idx[mid] < c) lo = mid + 1; else hi = mid;
    }
    if (lo < end && col_idx[lo] == c) atomicMax(reinterpret_cast<int*>(val) + lo, __float_as_int(w));
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
    size_t bytes;
};

BuildWs carve_build(void* base, int32_t n_users, int32_t n_items, int64_t n_edges) {
    const int64_t n = (int64_t)n_users + n_items;
    const int64_t e = n_edges > 0 ? n_edges : 1;
    Carver c(base);
    BuildWs w;
    w.buf_a = c.take<uint64_t>(e);
    w.buf_b = c.take<uint64_t>(e);
    const int64_t head_tiles = ceil_div(e, kHeadTile), row_tiles = ceil_div(n > 0 ? n : 1, kRowTile);
    const int64_t tiles = head_tiles > row_tiles ? head_tiles : row_tiles;
    w.tile_cnt = c.take<int32_t>(tiles);
    w.sort_ws = c.take<char>(radix_sort_workspace_bytes(e));
    w.zero_count = 64 + 2 * (n + 1);
    w.zeroed = c.take<int32_t>(w.zero_count);
    w.small = w.zeroed;
    w.run_start = w.zeroed ? w.zeroed + 64 : nullptr;
    w.run_end = w.zeroed ? w.run_start + (n + 1) : nullptr;
    w.scan_ws = c.take<char>(scan_workspace_bytes(tiles));
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
    zero_i32<<<dim3(blocks_for(w.zero_count, kThreads)), dim3(kThreads), 0, stream>>>(w.zeroed, w.zero_count);
    E2EG_LAUNCH_CHECK("zero_i32");
    if (n_edges > 0) {
        const int32_t st = sort_pairs(w, n_users, n_items, n_edges, d_user_ids, d_item_ids, self, d_col_idx, stream);
        if (st != E2EG_OK) return st;
    }
    if (n > 0) {
        const int64_t tiles = ceil_div(n, kRowTile);
        const dim3 grid((unsigned)tiles), blk(kRowThreads);
        row_sums<<<grid, blk, 0, stream>>>(w.run_start, w.run_end, n, self, w.tile_cnt);
        E2EG_LAUNCH_CHECK("row_sums");
        if (tiles > kRowFew) {
            E2EG_HIP_TRY(exclusive_scan_i32(w.tile_cnt, w.tile_cnt, tiles, nullptr, w.scan_ws, stream));
            row_pointers<true><<<grid, blk, 0, stream>>>(w.run_start, w.run_end, n, n_users, self, w.tile_cnt, d_row_ptr, d_col_idx);
        } else {
            row_pointers<false><<<grid, blk, 0, stream>>>(w.run_start, w.run_end, n, n_users, self, w.tile_cnt, d_row_ptr, d_col_idx);
        }
        E2EG_LAUNCH_CHECK("row_pointers");
    } else {
        zero_i32<<<dim3(1), dim3(64), 0, stream>>>(d_row_ptr, 1);
        E2EG_LAUNCH_CHECK("zero_i32");
    }
    int32_t host_small[2] = {0, 0};
    if (n_edges > 0)
        E2EG_HIP_TRY(hipMemcpyAsync(host_small, w.small, sizeof(host_small), hipMemcpyDeviceToHost, stream));
    E2EG_HIP_TRY(hipStreamSynchronize(stream));  // the one wait: the pair count is the caller's to know
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
    init_values<<<dim3(blocks_for(nnz, kThreads)), blk, 0, stream>>>(d_row_ptr, d_col_idx, n, nnz, d_val);
    E2EG_LAUNCH_CHECK("init_values");
    if (n_edges > 0) {
        apply_weights<<<dim3(blocks_for(2 * n_edges, kThreads)), blk, 0, stream>>>(
            d_user_ids, d_item_ids, d_weights, n_edges, n_users, n_items, d_row_ptr, d_col_idx, d_val);
        E2EG_LAUNCH_CHECK("apply_weights");
    }
    return E2EG_OK;
}
