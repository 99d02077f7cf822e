// Importance sampling of a multi-hop subgraph (paper: Section 4.1, the sampling probability
// p(u->v) = w_uv^beta / sum_k w_uk^beta with at most k neighbours per node and depth L; Section 5,
// "Subgraph Sampling": fan-outs per hop).
//
// Design for the GPU: every decision is integer arithmetic, so the result is a function of the
// inputs and the seed alone.
//   * e2eg_sampler_prepare turns each row's weights into integers (2^24 at the row maximum, the
//     division decided in fp32 with IEEE rounding) and prefix-sums them over the whole CSR: the
//     table holds cum[e] = sum of the integer weights before entry e, nnz + 1 values of 64 bits.
//     By entries throughout, so that a row of a million entries is no wavefront's loop.
//   * a draw is one thread: 64 random bits from the counter-based generator Philox4x32-10 (Salmon,
//     Moraes, Dror, Shaw, SC 2011; counter = (draw, node, hop, 0), key = the seed), scaled to the
//     row total by a 64x64->128-bit multiply, then a search in the row's slice of the table.
//   * the nodes reached at each hop are marked with plain byte stores (all writers write the same value);
//     bitmaps are made of the marks, and frontiers, the node list and the edge list are compacted with prefix
//     sums, so their order is ascending node id / draw order and does not depend on scheduling.  A node's local
//     id is its rank in the bitmap of all nodes.
//   * launch sizes come from upper bounds (seeds x fan-outs); the real frontier sizes stay on the
//     device.  The one wait is at the end, for the three counts handed to the host.
// A two-hop sample is bound by the number of launches and by the latency of the draws' dependent reads.
// 4096 seeds, fan-outs 25 and 10, graph of 1.5 M nodes: 23 launches and 178 us with flags and scans over all
// nodes for every hop; 11 launches now.  (Marking by atomic OR into the bitmaps themselves: the 280 k draws
// of the second hop meet on 190 KB of them and took 52 us.)
#include "entry_tiles.h"

namespace e2eg {
namespace {

constexpr int kThreads = kEntryThreads;
constexpr int kMaxHops = 8;
constexpr int kMaxFanout = 1 << 16;

inline dim3 grid_for(int64_t count) { return dim3((unsigned)ceil_div(count > 0 ? count : 1, kThreads)); }

__device__ __forceinline__ bool usable(float p) { return p > 0.0f && p <= 3.402823466e38f; }

__global__ void pow_weights(const float* __restrict__ val, int64_t nnz, float beta, float* __restrict__ p) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    const float v = val[e];
    float r = 0.0f;
    if (v > 0.0f) r = beta == 1.0f ? v : beta == 0.0f ? 1.0f : powf(v, beta);
    p[e] = r;
}

// The largest usable weight off the diagonal of every row, as the bit pattern of a positive float (which
// orders like an integer); row_max_bits is cleared.  The entries of a row are neighbours: a wavefront takes the
// maximum of each run of equal rows among its lanes, the first lane of a run goes to the row's word in LDS, and a
// tile goes to memory once per row.  Four million entries: 24 us (tiles of 256 entries, each searching all rows
// for its own: 56).
__global__ __launch_bounds__(kThreads) void row_max(const int32_t* __restrict__ row_ptr,
                                                    const int32_t* __restrict__ col_idx, const float* __restrict__ p,
                                                    int64_t n, int64_t nnz, int32_t* row_max_bits) {
    __shared__ int32_t rows[kTileRowsMax + 1];
    __shared__ int32_t best[kTileRowsMax];
    for (int k = threadIdx.x; k < kTileRowsMax; k += kThreads) best[k] = 0;
    const EntryTile tile(row_ptr, n, nnz, rows);
    const int lane = threadIdx.x & 63;
    float v[kEntryRounds];
    int32_t c[kEntryRounds];
#pragma unroll
    for (int r = 0; r < kEntryRounds; ++r) {
        const int64_t e = tile.first + r * kThreads + threadIdx.x;
        v[r] = e <= tile.last ? p[e] : 0.0f;
        c[r] = e <= tile.last ? col_idx[e] : -1;
    }
#pragma unroll
    for (int r = 0; r < kEntryRounds; ++r) {
        const int64_t e = tile.first + r * kThreads + threadIdx.x;
        const int32_t k = e <= tile.last ? (int32_t)tile.row(e) : -1;
        int32_t bits = 0;
        if (k >= 0 && c[r] != (int32_t)(tile.row0 + k) && usable(v[r])) bits = __float_as_int(v[r]);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t other = __shfl_down(bits, d, 64);
            const int32_t other_row = __shfl_down(k, d, 64);
            if (lane + d < 64 && other_row == k && other > bits) bits = other;
        }
        const int32_t before = __shfl_up(k, 1, 64);
        if (k >= 0 && (lane == 0 || before != k) && bits > 0) {
            if (tile.cached) atomicMax(&best[k], bits);
            else atomicMax(row_max_bits + tile.row0 + k, bits);
        }
    }
    __syncthreads();
    if (tile.cached)
        for (int64_t k = threadIdx.x; k < tile.count; k += kThreads)
            if (best[k] > 0) atomicMax(row_max_bits + tile.row0 + k, best[k]);
}

// Every entry's integer weight.  The entry past the end gets the 0 that closes the scan.
__global__ __launch_bounds__(kThreads) void quantise_entries(const int32_t* __restrict__ row_ptr,
                                                             const int32_t* __restrict__ col_idx,
                                                             const float* __restrict__ p, int64_t n, int64_t nnz,
                                                             const int32_t* __restrict__ row_max_bits,
                                                             uint64_t* __restrict__ q) {
    __shared__ int32_t rows[kTileRowsMax + 1];
    __shared__ float best[kTileRowsMax];
    if (blockIdx.x == 0 && threadIdx.x == 0) q[nnz] = 0;
    if (nnz == 0) return;
    const EntryTile tile(row_ptr, n, nnz, rows);
    float v[kEntryRounds];
    int32_t c[kEntryRounds];
#pragma unroll
    for (int r = 0; r < kEntryRounds; ++r) {
        const int64_t e = tile.first + r * kThreads + threadIdx.x;
        v[r] = e <= tile.last ? p[e] : 0.0f;
        c[r] = e <= tile.last ? col_idx[e] : -1;
    }
    if (tile.cached)
        for (int64_t k = threadIdx.x; k < tile.count; k += kThreads) best[k] = __int_as_float(row_max_bits[tile.row0 + k]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kEntryRounds; ++r) {
        const int64_t e = tile.first + r * kThreads + threadIdx.x;
        if (e > tile.last) continue;
        const int64_t k = tile.row(e);
        uint64_t w = 0;
        if (c[r] != (int32_t)(tile.row0 + k) && usable(v[r])) {
            const float pmax = tile.cached ? best[k] : __int_as_float(row_max_bits[tile.row0 + k]);
            const float scaled = floorf(__fmul_rn(__fdiv_rn(v[r], pmax), 16777216.0f));
            w = scaled >= 1.0f ? (uint64_t)scaled : 1u;
        }
        q[e] = w;
    }
}

__global__ void fill_i32(int32_t* __restrict__ p, int64_t count, int32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

__global__ void zero16(uint4* __restrict__ p, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// ---- node sets -----------------------------------------------------------------------------------------
// marks[h * stride + v]: h = 0 the seeds, h > 0 the nodes picked at hop h - 1, whether or not they were reached
// before.
// One 64-node word a thread.  Small workgroups: list_set walks a wavefront's words one after the other, and 1.5 M
// nodes in workgroups of 1024 were 23 of them (13.2 us then, 10.2 in 183).
constexpr int kSetThreads = 128;
constexpr int64_t kSetFew = 2048;   // up to this many tiles of words a workgroup adds up the counts before its own

struct Marks {
    uint8_t* marks;
    int64_t stride;
    __device__ __forceinline__ void add(int h, int32_t v) const { marks[h * stride + v] = 1; }
    // level h of word w as bits
    __device__ __forceinline__ uint64_t word(int h, int64_t w) const {
        const uint4* p = reinterpret_cast<const uint4*>(marks + h * stride + w * 64);
        uint64_t bits = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 v = p[q];
            // four 0/1 bytes -> four bits: the products land on bits 24 .. 27 without carries
            const uint32_t b = ((v.x * 0x01020408u) >> 24 & 15u) | ((v.y * 0x01020408u) >> 24 & 15u) << 4 |
                               ((v.z * 0x01020408u) >> 24 & 15u) << 8 | ((v.w * 0x01020408u) >> 24 & 15u) << 12;
            bits |= (uint64_t)b << (16 * q);
        }
        return bits;
    }
};

__global__ void mark_seeds(const int32_t* __restrict__ seeds, int32_t n_seeds, int32_t n, Marks marks,
                           int32_t* __restrict__ bad) {
    const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_seeds) return;
    const int32_t v = seeds[s];
    if (v < 0 || v >= n) {
        atomicOr(bad, 1);
        return;
    }
    marks.add(0, v);
}

// The nodes first reached at `level`, or (ALL) those of levels 0 .. level, as a bitmap; and their number per tile.
template <bool ALL>
__global__ __launch_bounds__(kSetThreads) void make_set(Marks marks, int level, int64_t words, uint64_t* __restrict__ set,
                                                        int32_t* __restrict__ tile_cnt) {
    __shared__ int32_t lds[kSetThreads / 64];
    const int64_t w = (int64_t)blockIdx.x * kSetThreads + threadIdx.x;
    uint64_t v = 0;
    if (w < words) {
        v = marks.word(level, w);
        for (int k = 0; k < level; ++k) {
            const uint64_t o = marks.word(k, w);
            v = ALL ? v | o : v & ~o;
        }
        set[w] = v;
    }
    int32_t c = __popcll(v);
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int k = 0; k < kSetThreads / 64; ++k) t += lds[k];
        tile_cnt[blockIdx.x] = t;
    }
}

// The set as an ascending list, and its size in *total.  rank (may be null): nodes before every word, and
// *boundary = the rank of node n_users.  SCANNED: tile_cnt holds the number of nodes before each tile, else the tiles' own.
template <bool SCANNED>
__global__ __launch_bounds__(kSetThreads) void list_set(const uint64_t* __restrict__ set, int64_t words,
                                                        const int32_t* __restrict__ tile_cnt, int32_t* __restrict__ out,
                                                        int64_t capacity, int32_t* __restrict__ total,
                                                        int32_t* __restrict__ rank, int32_t n_users,
                                                        int32_t* __restrict__ boundary) {
    constexpr int kWaves = kSetThreads / 64;
    __shared__ int32_t lds[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t w = (int64_t)blockIdx.x * kSetThreads + threadIdx.x;
    const uint64_t bits = w < words ? set[w] : 0ull;
    int32_t at = 0;
    if (SCANNED) {
        at = tile_cnt[blockIdx.x];
    } else {
#pragma unroll 4
        for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kSetThreads) at += tile_cnt[t];
        for (int off = 32; off > 0; off >>= 1) at += __shfl_xor(at, off);
        if (lane == 0) lds[wave] = at;
        __syncthreads();
        at = 0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) at += lds[k];
        __syncthreads();
    }
    const int32_t c = __popcll(bits);
    int32_t inc = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t t = __shfl_up(inc, d, 64);
        if (lane >= d) inc += t;
    }
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    at += inc - c;
#pragma unroll
    for (int k = 0; k < kWaves; ++k)
        if (k < wave) at += lds[k];
    if (w < words) {
        if (rank) {
            rank[w] = at;
            if (w == n_users >> 6) *boundary = at + __popcll(bits & ((1ull << (n_users & 63)) - 1));
        }
        if (w == words - 1) *total = at + c;
    }
    // a word at a time, a lane per node, so that ids leave side by side; the word comes by readlane, which needs no
    // trip through LDS
    uint64_t some = __ballot(c > 0);
    const int32_t word0 = (int32_t)((int64_t)blockIdx.x * kSetThreads + wave * 64);
    while (some) {
        const int k = __ffsll((unsigned long long)some) - 1;
        some &= some - 1;
        const uint64_t v = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, k) |
                           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(bits >> 32), k) << 32;
        const int32_t pos = __builtin_amdgcn_readlane(at, k) + __popcll(v & lt_mask);
        if (((v >> lane) & 1) && pos < capacity) out[pos] = (word0 + k) * 64 + lane;
    }
}

struct Philox {
    uint32_t c[4];
};

__device__ __forceinline__ Philox philox4x32_10(Philox x, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, x.c[0]), lo0 = 0xD2511F53u * x.c[0];
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, x.c[2]), lo1 = 0xCD9E8D57u * x.c[2];
        Philox y;
        y.c[0] = hi1 ^ x.c[1] ^ k0;
        y.c[1] = lo1;
        y.c[2] = hi0 ^ x.c[3] ^ k1;
        y.c[3] = lo0;
        x = y;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return x;
}

// Smallest e in [beg, end) with cum[e + 1] - base > r, which is known to exist.  Seven pivots a step, their
// loads in flight together: a step costs the latency of one read, and a row of 2000 takes four of them
// instead of eleven.
__device__ __forceinline__ int32_t pick_entry(const uint64_t* __restrict__ cum, int32_t beg, int32_t end, uint64_t base,
                                              uint64_t r) {
    int32_t lo = beg, hi = end - 1;
    while (hi - lo >= 8) {
        const int32_t step = (int32_t)(((int64_t)hi - lo + 1) >> 3);
        int below = 0;
#pragma unroll
        for (int k = 1; k < 8; ++k) below += cum[lo + k * step] - base > r ? 0 : 1;
        if (below < 7) hi = lo + (below + 1) * step - 1;
        lo += below * step;
    }
    int below = 0;
#pragma unroll
    for (int k = 1; k < 8; ++k)
        if (lo + k <= hi) below += cum[lo + k] - base > r ? 0 : 1;
    return lo + below;
}

// One thread per (frontier position f, draw t) of hop `hop`, for the upper bound of the frontier's size that
// sized the launch; the real size is *front_count.  Every slot of a tile that has any is written: the source
// node, the picked neighbour (or -1: no pick) and the index of the stored entry; and the tile's number of picks.
constexpr int kDrawThreads = 512;   // slots per tile
__global__ __launch_bounds__(kDrawThreads) void draw_picks(const int32_t* __restrict__ row_ptr,
                                                           const int32_t* __restrict__ col_idx,
                                                           const uint64_t* __restrict__ cum,
                                                           const int32_t* __restrict__ frontier,
                                                           const int32_t* __restrict__ front_count, int32_t k, int32_t hop,
                                                           uint32_t seed_lo, uint32_t seed_hi, Marks marks,
                                                           int32_t* __restrict__ slot_src, int32_t* __restrict__ slot_dst,
                                                           int32_t* __restrict__ slot_ent, int32_t* __restrict__ tile_cnt) {
    __shared__ int32_t picks;
    const int64_t s = (int64_t)blockIdx.x * kDrawThreads + threadIdx.x;
    const int64_t slots = (int64_t)*front_count * k;
    if ((int64_t)blockIdx.x * kDrawThreads >= slots) {
        if (threadIdx.x == 0) tile_cnt[blockIdx.x] = 0;
        return;
    }
    if (threadIdx.x == 0) picks = 0;
    __syncthreads();
    int32_t u = -1, v = -1, ent = -1;
    if (s < slots) {
        const int64_t f = s / k;
        const int32_t t = (int32_t)(s - f * k);
        u = frontier[f];
        const int32_t beg = row_ptr[u], end = row_ptr[u + 1];
        // A node with at most k neighbours keeps every one that can be drawn at all.  Its row may
        // also hold the node itself (the diagonal entry, never drawn), so a row of k + 1 entries
        // qualifies when one of them is the diagonal: slot t then takes the t-th entry beside it.
        int32_t diag = -1;   // where the diagonal entry sits, looked for only where it decides
        if (end - beg == k + 1) {
            int32_t lo = beg, hi = end;   // first entry with column >= u (columns ascend)
            while (lo < hi) {
                const int32_t mid = lo + ((hi - lo) >> 1);
                if (col_idx[mid] < u) lo = mid + 1; else hi = mid;
            }
            if (lo < end && col_idx[lo] == u) diag = lo;
        }
        if (end - beg <= k) {
            if (t < end - beg && cum[beg + t + 1] > cum[beg + t]) ent = beg + t;
        } else if (diag >= 0) {
            const int32_t e = beg + t + (beg + t >= diag ? 1 : 0);
            if (cum[e + 1] > cum[e]) ent = e;
        } else {
            const uint64_t base = cum[beg], total = cum[end] - base;
            if (total > 0) {
                Philox x;
                x.c[0] = (uint32_t)t;
                x.c[1] = (uint32_t)u;
                x.c[2] = (uint32_t)hop;
                x.c[3] = 0u;
                x = philox4x32_10(x, seed_lo, seed_hi);
                const uint64_t bits = (uint64_t)x.c[0] | ((uint64_t)x.c[1] << 32);
                ent = pick_entry(cum, beg, end, base, __umul64hi(bits, total));  // uniform on [0, total)
            }
        }
        if (ent >= 0) {
            v = col_idx[ent];
            marks.add(hop + 1, v);
        }
    }
    slot_src[s] = u;
    slot_dst[s] = v;
    slot_ent[s] = ent;
    const int32_t c = __popcll(__ballot(v >= 0));
    if ((threadIdx.x & 63) == 0 && c > 0) atomicAdd(&picks, c);
    __syncthreads();
    if (threadIdx.x == 0) tile_cnt[blockIdx.x] = picks;
}

// Picks in slot order -> (local user, local item[, weight]); an entry that joins two nodes of the
// same side is reported through counts[3].  Local ids are ranks in the set of all nodes.  SCANNED: tile_cnt holds the
// number of picks before each tile, else the tiles' own.
struct Ranks {
    const uint64_t* set;
    const int32_t* rank;
    __device__ __forceinline__ int32_t of(int32_t v) const {
        return rank[v >> 6] + __popcll(set[v >> 6] & ((1ull << (v & 63)) - 1));
    }
};
template <bool SCANNED>
__global__ __launch_bounds__(kDrawThreads) void emit_edges(const int32_t* __restrict__ slot_src,
                                                           const int32_t* __restrict__ slot_dst,
                                                           const int32_t* __restrict__ slot_ent,
                                                           const int32_t* __restrict__ tile_cnt, Ranks ranks,
                                                           int32_t n_users, const float* __restrict__ val,
                                                           int32_t* __restrict__ edge_users, int32_t* __restrict__ edge_items,
                                                           float* __restrict__ edge_w, int32_t* __restrict__ n_edges,
                                                           const int32_t* __restrict__ boundary, int32_t* __restrict__ bad) {
    __shared__ int32_t lds[kDrawThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t own = SCANNED ? tile_cnt[blockIdx.x + 1] - tile_cnt[blockIdx.x] : tile_cnt[blockIdx.x];
    const bool last = blockIdx.x == gridDim.x - 1;
    if (own == 0 && !last) return;
    int32_t at = 0;
    if (SCANNED) {
        at = tile_cnt[blockIdx.x];
    } else {
#pragma unroll 4
        for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kDrawThreads) at += tile_cnt[t];
        for (int off = 32; off > 0; off >>= 1) at += __shfl_xor(at, off);
        if (lane == 0) lds[wave] = at;
        __syncthreads();
        at = 0;
#pragma unroll
        for (int w = 0; w < kDrawThreads / 64; ++w) at += lds[w];
        __syncthreads();
    }
    if (last && threadIdx.x == 0) *n_edges = at + own;
    if (own == 0) return;
    const int64_t s = (int64_t)blockIdx.x * kDrawThreads + threadIdx.x;
    const int32_t a = slot_src[s], b = slot_dst[s];
    const uint64_t bal = __ballot(b >= 0);
    if (lane == 0) lds[wave] = __popcll(bal);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kDrawThreads / 64; ++w)
        if (w < wave) at += lds[w];
    if (b < 0) return;
    at += __popcll(bal & ((1ull << lane) - 1));
    const int32_t user = a < b ? a : b, item = a < b ? b : a;
    if (user >= n_users || item < n_users) {
        atomicOr(bad, 2);
        edge_users[at] = 0;
        edge_items[at] = 0;
    } else {
        edge_users[at] = ranks.of(user);
        edge_items[at] = ranks.of(item) - *boundary;
    }
    if (edge_w) edge_w[at] = val[slot_ent[s]];
}

// Upper bounds that size the launches: cap_front[h] >= size of the frontier of hop h, slots[h] =
// cap_front[h] * fanout[h]; returns the total number of slots, or -1 when it does not fit int32.
int64_t plan(int64_t n, int64_t n_seeds, int32_t L, const int32_t* fanout, int64_t* cap_front, int64_t* slot_base) {
    int64_t total = 0, width = n_seeds < n ? n_seeds : n;
    for (int32_t h = 0; h < L; ++h) {
        cap_front[h] = width;
        slot_base[h] = total;
        const int64_t slots = width * fanout[h];
        total += slots;
        if (total > (int64_t)INT32_MAX - 1) return -1;
        width = slots < n ? slots : n;
    }
    return total;
}

int32_t check_plan(const char* who, int32_t n, int32_t n_seeds, int32_t L, const int32_t* h_fanout) {
    if (n < 0 || n_seeds < 0) return fail(E2EG_ERR_INVALID_ARG, "%s: negative size", who);
    if (L < 1 || L > kMaxHops) return fail(E2EG_ERR_INVALID_ARG, "%s: depth L=%d must be in [1, %d]", who, L, kMaxHops);
    if (!h_fanout) return fail(E2EG_ERR_NULL_PTR, "%s: h_fanout is null", who);
    for (int32_t h = 0; h < L; ++h)
        if (h_fanout[h] < 1 || h_fanout[h] > kMaxFanout)
            return fail(E2EG_ERR_INVALID_ARG, "%s: fan-out %d of hop %d must be in [1, %d]", who, h_fanout[h], h, kMaxFanout);
    return E2EG_OK;
}

struct SampleWs {
    int32_t* small;     // [64]: [0] local users, [1] nodes, [2] edges, [3] bad; [8 ..] frontier sizes
    uint8_t* marks;     // [L + 1][64 * words], behind `small` so that one launch clears both
    int64_t words;
    int64_t zero_count; // in int32
    uint64_t* set;      // [words] the set in hand, in the end all nodes
    int32_t* rank;      // [words]
    int32_t* frontier;  // [max cap_front]
    int32_t* slot_src;  // [slot tiles * kDrawThreads]
    int32_t* slot_dst;
    int32_t* slot_ent;
    int32_t* tile_cnt;  // [slot tiles + 1]
    int32_t* set_cnt;   // [tiles of words]
    void* scan_ws;
    size_t bytes;
};

constexpr int64_t kDrawFew = 4096;   // up to this many slot tiles emit_edges adds up the counts before its own

int64_t slot_tiles(int32_t L, const int64_t* cap_front, const int32_t* fanout, int64_t* tile_base) {
    int64_t tiles = 0;
    for (int32_t h = 0; h < L; ++h) {
        tile_base[h] = tiles;
        tiles += ceil_div(cap_front[h] * fanout[h], kDrawThreads);
    }
    return tiles;
}

SampleWs carve_sample(void* base, int64_t n, int32_t L, int64_t max_front, int64_t tiles) {
    Carver c(base);
    SampleWs w;
    w.words = n / 64 + 1;   // one bit past the last node, whose rank is asked for
    char* zeroed = c.take<char>(64 * sizeof(int32_t) + (size_t)(L + 1) * (size_t)w.words * 64);
    w.small = reinterpret_cast<int32_t*>(zeroed);
    w.marks = zeroed ? reinterpret_cast<uint8_t*>(zeroed + 64 * sizeof(int32_t)) : nullptr;
    w.zero_count = 64 + 16 * (int64_t)(L + 1) * w.words;
    w.set = c.take<uint64_t>(w.words);
    w.rank = c.take<int32_t>(w.words);
    w.frontier = c.take<int32_t>(max_front > 0 ? max_front : 1);
    w.slot_src = c.take<int32_t>(tiles * kDrawThreads + 1);
    w.slot_dst = c.take<int32_t>(tiles * kDrawThreads + 1);
    w.slot_ent = c.take<int32_t>(tiles * kDrawThreads + 1);
    w.tile_cnt = c.take<int32_t>(tiles + 1);
    const int64_t set_tiles = ceil_div(w.words, kSetThreads);
    w.set_cnt = c.take<int32_t>(set_tiles);
    const int64_t longest = set_tiles > tiles + 1 ? set_tiles : tiles + 1;
    w.scan_ws = c.take<char>(scan_workspace_bytes(longest));
    w.bytes = c.size();
    return w;
}

// The nodes of one level (or of all levels up to it: `all`, with their ranks) as a list.
int32_t run_list(const SampleWs& w, const Marks& marks, int level, bool all, int32_t* out, int64_t capacity, int32_t* total,
                 int32_t n_users, hipStream_t stream) {
    const int64_t tiles = ceil_div(w.words, kSetThreads);
    const dim3 grid((unsigned)tiles), blk(kSetThreads);
    if (all) make_set<true><<<grid, blk, 0, stream>>>(marks, level, w.words, w.set, w.set_cnt);
    else make_set<false><<<grid, blk, 0, stream>>>(marks, level, w.words, w.set, w.set_cnt);
    E2EG_LAUNCH_CHECK("make_set");
    int32_t* rank = all ? w.rank : nullptr;
    if (tiles > kSetFew) {
        E2EG_HIP_TRY(exclusive_scan_i32(w.set_cnt, w.set_cnt, tiles, nullptr, w.scan_ws, stream));
        list_set<true><<<grid, blk, 0, stream>>>(w.set, w.words, w.set_cnt, out, capacity, total, rank, n_users, w.small);
    } else {
        list_set<false><<<grid, blk, 0, stream>>>(w.set, w.words, w.set_cnt, out, capacity, total, rank, n_users, w.small);
    }
    E2EG_LAUNCH_CHECK("list_set");
    return E2EG_OK;
}

}  // namespace
}  // namespace e2eg

using namespace e2eg;

extern "C" int32_t e2eg_sampling_weights(int64_t nnz, const float* d_val, float beta, float* d_p, void* stream_) {
    if (nnz < 0) return fail(E2EG_ERR_INVALID_ARG, "sampling_weights: negative size");
    if (!(beta >= 0.0f)) return fail(E2EG_ERR_INVALID_ARG, "sampling_weights: beta must be >= 0");
    if (nnz > 0 && (!d_val || !d_p)) return fail(E2EG_ERR_NULL_PTR, "sampling_weights: null pointer");
    if (nnz == 0) return E2EG_OK;
    pow_weights<<<grid_for(nnz), dim3(kThreads), 0, static_cast<hipStream_t>(stream_)>>>(d_val, nnz, beta, d_p);
    E2EG_LAUNCH_CHECK("pow_weights");
    return E2EG_OK;
}

extern "C" size_t e2eg_sampler_table_bytes(int64_t nnz) {
    if (nnz < 0) return 0;
    return align_up((size_t)(nnz + 1) * sizeof(uint64_t));
}

extern "C" size_t e2eg_sampler_prepare_workspace_bytes(int32_t n, int64_t nnz) {
    if (n < 0 || nnz < 0) return 0;
    return align_up((size_t)(n > 0 ? n : 1) * sizeof(int32_t)) + scan_u64_workspace_bytes(nnz + 1);   // row maxima, scan
}

extern "C" int32_t e2eg_sampler_prepare(int32_t n, int64_t nnz, const int32_t* d_row_ptr, const int32_t* d_col_idx,
                                        const float* d_p, void* d_table, size_t table_bytes, void* ws,
                                        size_t ws_bytes, void* stream_) {
    if (n < 0 || nnz < 0) return fail(E2EG_ERR_INVALID_ARG, "sampler_prepare: negative size");
    if (nnz > (int64_t)INT32_MAX || n == INT32_MAX)
        return fail(E2EG_ERR_OVERFLOW, "sampler_prepare: nnz=%lld exceeds int32", (long long)nnz);
    if (!d_row_ptr || !d_table || (nnz > 0 && (!d_col_idx || !d_p)))
        return fail(E2EG_ERR_NULL_PTR, "sampler_prepare: null pointer");
    if (nnz > 0 && n == 0) return fail(E2EG_ERR_INVALID_ARG, "sampler_prepare: entries given but no nodes");
    if (!aligned_to(d_table, kAlign) || table_bytes < e2eg_sampler_table_bytes(nnz))
        return fail(E2EG_ERR_CAPACITY, "sampler_prepare: d_table needs %zu bytes, 256-byte aligned",
                    e2eg_sampler_table_bytes(nnz));
    const size_t need = e2eg_sampler_prepare_workspace_bytes(n, nnz);
    if (!ws || !aligned_to(ws, kAlign) || ws_bytes < need)
        return fail(E2EG_ERR_WORKSPACE, "sampler_prepare: workspace needs %zu bytes, 256-byte aligned", need);
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    uint64_t* q = static_cast<uint64_t*>(d_table);
    int32_t* row_max_bits = static_cast<int32_t*>(ws);
    void* scan_ws = static_cast<char*>(ws) + align_up((size_t)(n > 0 ? n : 1) * sizeof(int32_t));
    const dim3 blk(kThreads);
    if (n > 0) {
        fill_i32<<<grid_for(n), blk, 0, stream>>>(row_max_bits, n, 0);
        E2EG_LAUNCH_CHECK("fill_i32");
    }
    if (nnz > 0) {
        row_max<<<dim3((unsigned)ceil_div(nnz, kEntryTile)), blk, 0, stream>>>(d_row_ptr, d_col_idx, d_p, n, nnz, row_max_bits);
        E2EG_LAUNCH_CHECK("row_max");
    }
    quantise_entries<<<dim3((unsigned)ceil_div(nnz > 0 ? nnz : 1, kEntryTile)), blk, 0, stream>>>(d_row_ptr, d_col_idx, d_p, n, nnz, row_max_bits, q);
    E2EG_LAUNCH_CHECK("quantise_entries");
    E2EG_HIP_TRY(exclusive_scan_u64(q, q, nnz + 1, nullptr, scan_ws, stream));
    return E2EG_OK;
}

extern "C" int64_t e2eg_sample_capacity(int32_t n, int32_t n_seeds, int32_t L, const int32_t* h_fanout) {
    if (check_plan("sample_capacity", n, n_seeds, L, h_fanout) != E2EG_OK) return -1;
    int64_t cap_front[kMaxHops], slot_base[kMaxHops];
    const int64_t slots = plan(n, n_seeds, L, h_fanout, cap_front, slot_base);
    if (slots < 0) fail(E2EG_ERR_OVERFLOW, "sample_capacity: seeds x fan-outs exceed int32");
    return slots;
}

extern "C" size_t e2eg_sample_subgraph_workspace_bytes(int32_t n, int32_t n_seeds, int32_t L,
                                                       const int32_t* h_fanout) {
    if (check_plan("sample_subgraph_workspace_bytes", n, n_seeds, L, h_fanout) != E2EG_OK) return 0;
    int64_t cap_front[kMaxHops], slot_base[kMaxHops];
    const int64_t slots = plan(n, n_seeds, L, h_fanout, cap_front, slot_base);
    if (slots < 0) return 0;
    int64_t max_front = 0;
    for (int32_t h = 0; h < L; ++h) max_front = cap_front[h] > max_front ? cap_front[h] : max_front;
    int64_t tile_base[kMaxHops];
    return carve_sample(nullptr, n, L, max_front, slot_tiles(L, cap_front, h_fanout, tile_base)).bytes;
}

extern "C" int32_t e2eg_sample_subgraph(int32_t n_users, int32_t n, int64_t nnz, const int32_t* d_row_ptr,
                                        const int32_t* d_col_idx, const void* d_table, const float* d_val,
                                        int32_t n_seeds, const int32_t* d_seeds, int32_t L, const int32_t* h_fanout,
                                        uint64_t seed, int32_t* d_nodes, int64_t node_capacity,
                                        int32_t* d_edge_users, int32_t* d_edge_items, float* d_edge_w,
                                        int64_t edge_capacity, int32_t* h_counts, void* ws, size_t ws_bytes,
                                        void* stream_) {
    const char* who = "sample_subgraph";
    int32_t st = check_plan(who, n, n_seeds, L, h_fanout);
    if (st != E2EG_OK) return st;
    if (nnz < 0 || n_users < 0 || n_users > n) return fail(E2EG_ERR_INVALID_ARG, "%s: bad n_users or nnz", who);
    if (nnz > (int64_t)INT32_MAX || n == INT32_MAX)
        return fail(E2EG_ERR_OVERFLOW, "%s: nnz=%lld exceeds int32", who, (long long)nnz);
    if (!h_counts || !d_row_ptr || !d_table || (nnz > 0 && !d_col_idx) || (n_seeds > 0 && !d_seeds))
        return fail(E2EG_ERR_NULL_PTR, "%s: null pointer", who);
    if (d_edge_w && !d_val) return fail(E2EG_ERR_NULL_PTR, "%s: d_edge_w asks for weights but d_val is null", who);
    int64_t cap_front[kMaxHops], slot_base[kMaxHops];
    const int64_t slots = plan(n, n_seeds, L, h_fanout, cap_front, slot_base);
    if (slots < 0) return fail(E2EG_ERR_OVERFLOW, "%s: seeds x fan-outs exceed int32", who);
    const int64_t max_nodes = (int64_t)n_seeds + slots < n ? (int64_t)n_seeds + slots : n;
    if (node_capacity < max_nodes || edge_capacity < slots)
        return fail(E2EG_ERR_CAPACITY, "%s: needs room for %lld nodes and %lld edges", who, (long long)max_nodes,
                    (long long)slots);
    if ((max_nodes > 0 && !d_nodes) || (slots > 0 && (!d_edge_users || !d_edge_items)))
        return fail(E2EG_ERR_NULL_PTR, "%s: null output pointer", who);
    int64_t max_front = 0;
    for (int32_t h = 0; h < L; ++h) max_front = cap_front[h] > max_front ? cap_front[h] : max_front;
    int64_t tile_base[kMaxHops];
    const int64_t tiles = slot_tiles(L, cap_front, h_fanout, tile_base);
    const size_t need = carve_sample(nullptr, n, L, max_front, tiles).bytes;
    if (!ws || !aligned_to(ws, kAlign) || ws_bytes < need)
        return fail(E2EG_ERR_WORKSPACE, "%s: workspace needs %zu bytes, 256-byte aligned", who, need);
    h_counts[0] = h_counts[1] = h_counts[2] = 0;
    if (n == 0 || n_seeds == 0) return E2EG_OK;

    hipStream_t stream = static_cast<hipStream_t>(stream_);
    const SampleWs w = carve_sample(ws, n, L, max_front, tiles);
    const uint64_t* cum = static_cast<const uint64_t*>(d_table);
    const dim3 blk(kThreads);
    const Marks marks{w.marks, w.words * 64};
    zero16<<<grid_for(w.zero_count / 4), blk, 0, stream>>>(reinterpret_cast<uint4*>(w.small), w.zero_count / 4);
    E2EG_LAUNCH_CHECK("zero16");
    mark_seeds<<<grid_for(n_seeds), blk, 0, stream>>>(d_seeds, n_seeds, n, marks, w.small + 3);
    E2EG_LAUNCH_CHECK("mark_seeds");
    for (int32_t h = 0; h < L; ++h) {
        // the frontier of hop h, ascending: nodes first reached at level h
        int32_t* size = w.small + 8 + h;
        if ((st = run_list(w, marks, h, false, w.frontier, cap_front[h], size, n_users, stream)) != E2EG_OK) return st;
        const int64_t at = tile_base[h] * kDrawThreads;
        draw_picks<<<dim3((unsigned)ceil_div(cap_front[h] * h_fanout[h], kDrawThreads)), dim3(kDrawThreads), 0, stream>>>(
            d_row_ptr, d_col_idx, cum, w.frontier, size, h_fanout[h], h, (uint32_t)seed, (uint32_t)(seed >> 32), marks,
            w.slot_src + at, w.slot_dst + at, w.slot_ent + at, w.tile_cnt + tile_base[h]);
        E2EG_LAUNCH_CHECK("draw_picks");
    }
    // local numbering: all nodes in ascending order (users first, as in the parent)
    if ((st = run_list(w, marks, L, true, d_nodes, node_capacity, w.small + 1, n_users, stream)) != E2EG_OK) return st;
    // the picks, without the empty slots, in slot order
    const dim3 edge_grid((unsigned)tiles), edge_blk(kDrawThreads);
    const Ranks ranks{w.set, w.rank};
    if (tiles > kDrawFew) {
        fill_i32<<<dim3(1), dim3(64), 0, stream>>>(w.tile_cnt + tiles, 1, 0);
        E2EG_LAUNCH_CHECK("fill_i32");
        E2EG_HIP_TRY(exclusive_scan_i32(w.tile_cnt, w.tile_cnt, tiles + 1, nullptr, w.scan_ws, stream));
        emit_edges<true><<<edge_grid, edge_blk, 0, stream>>>(w.slot_src, w.slot_dst, w.slot_ent, w.tile_cnt, ranks, n_users, d_val,
                                                            d_edge_users, d_edge_items, d_edge_w, w.small + 2, w.small, w.small + 3);
    } else {
        emit_edges<false><<<edge_grid, edge_blk, 0, stream>>>(w.slot_src, w.slot_dst, w.slot_ent, w.tile_cnt, ranks, n_users, d_val,
                                                             d_edge_users, d_edge_items, d_edge_w, w.small + 2, w.small, w.small + 3);
    }
    E2EG_LAUNCH_CHECK("emit_edges");
    int32_t host[4] = {0, 0, 0, 0};
    if ((st = read_back(w.small, 4, host, stream)) != E2EG_OK) return st;  // the one wait: the counts size what the caller does next
    if (host[3] & 1) return fail(E2EG_ERR_BAD_INDEX, "%s: a seed is out of range", who);
    if (host[3] & 2) return fail(E2EG_ERR_BAD_INDEX, "%s: a stored entry joins two users or two items", who);
    h_counts[0] = host[0];
    h_counts[1] = host[1] - host[0];
    h_counts[2] = host[2];
    return E2EG_OK;
}
