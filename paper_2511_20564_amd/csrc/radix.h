// One pass of a stable LSD radix sort of 64-bit keys, as kernel templates: where the keys come from
// (an array, or the caller's pairs) and what the sorted keys become (an array, or entries of a CSR) are
// template parameters, so that the first pass needs no packing pass before it and the last no unpacking
// pass behind it.  Integer work only; the result does not depend on scheduling.
#pragma once
#include "common.h"

namespace e2eg {

// Shapes.  Large sorts: tiles of 8192 keys and digits of up to 8 bits, so that a tile's keys of one digit
// leave as a run of some 32 keys = 256 bytes (tiles of 2048: 64-byte runs; 50 M keys, histogram + offsets +
// scatter: 470 us a pass then, 330 now) and the table of digit counts stays small.  Small sorts are bound by the number
// of launches: digits of up to 11 bits (two launches a pass while the table is so small that every workgroup
// adds up its own offsets).
struct LargeSort {
    static constexpr int kThreads = 512, kItems = 16, kBits = 8, kCopies = 4, kTile = kThreads * kItems;
};
struct SmallSort {
    static constexpr int kThreads = 1024, kItems = 8, kBits = 11, kCopies = 1, kTile = kThreads * kItems;
};
// One 8-bit digit of a small list (the bucketed CSR build): more, smaller tiles.
struct SplitSort {
    static constexpr int kThreads = 512, kItems = 8, kBits = 8, kCopies = 1, kTile = kThreads * kItems;
};
constexpr int64_t kLargeSortMin = 4 << 20;
constexpr int kFusedTiles = 64;   // up to this many tiles the scatter adds up its offsets itself

struct KeysIn {
    const uint64_t* keys;
    using raw = uint64_t;   // what is loaded, and the key of it
    __device__ __forceinline__ raw load(int64_t i) const { return keys[i]; }
    __device__ __forceinline__ raw none() const { return 0ull; }
    __device__ __forceinline__ uint64_t key(raw r) const { return r; }
    __device__ __forceinline__ bool ok(raw) const { return true; }
    __device__ __forceinline__ void report() const {}
};
struct KeysOut {
    static constexpr bool kRuns = false;
    uint64_t* keys;
    __device__ __forceinline__ void store(int64_t at, uint64_t key) const { keys[at] = key; }
};

// Digit counts of every tile.  The table is digit-major [bins][tiles] for a scan, or (TILE_MAJOR)
// [tiles][bins] for a scatter that adds up its offsets itself.  d_count (may be null): the number of keys,
// known on the device only; `count` is then its upper bound, which sized the launch.
template <typename S, typename In, bool TILE_MAJOR>
__global__ __launch_bounds__(S::kThreads) void sort_histogram(In in, int64_t count, const int32_t* __restrict__ d_count,
                                                              int shift, int nbits, int32_t* __restrict__ hist,
                                                              int32_t tiles) {
    __shared__ int h[S::kCopies][1 << S::kBits];   // copies: fewer lanes meet on one word
    const int bins = 1 << nbits;
    for (int k = threadIdx.x; k < S::kCopies << S::kBits; k += S::kThreads) (&h[0][0])[k] = 0;
    __syncthreads();
    if (d_count) count = *d_count;
    const int64_t base = (int64_t)blockIdx.x * S::kTile;
    int* mine = h[(threadIdx.x >> 6) % S::kCopies];
    typename In::raw raw[S::kItems];
#pragma unroll
    for (int k = 0; k < S::kItems; ++k) {
        const int64_t i = base + k * S::kThreads + threadIdx.x;
        raw[k] = i < count ? in.load(i) : in.none();
    }
    bool ok = true;
#pragma unroll
    for (int k = 0; k < S::kItems; ++k) {
        const int64_t i = base + k * S::kThreads + threadIdx.x;
        if (i < count) {
            ok = ok && in.ok(raw[k]);
            atomicAdd(&mine[(int)(in.key(raw[k]) >> shift) & (bins - 1)], 1);
        }
    }
    if (!ok) in.report();
    __syncthreads();
    for (int d = threadIdx.x; d < bins; d += S::kThreads) {
        int t = 0;
#pragma unroll
        for (int c = 0; c < S::kCopies; ++c) t += h[c][d];
        if (TILE_MAJOR) hist[(int64_t)blockIdx.x * bins + d] = t;
        else hist[(int64_t)d * tiles + blockIdx.x] = t;
    }
}

// Stable scatter.  A tile is split into one contiguous chunk per wavefront; a wavefront walks its chunk 64
// keys at a time, ranking equal digits by lane order plus a running per-wavefront digit count, so ranks
// follow input order.  The keys are then put in digit order inside the tile (in LDS) and written out
// from there, consecutive threads writing consecutive keys: keys of one digit leave as one contiguous run.
// `offs` is the digit-major table of scanned offsets, or, with COUNTS, the raw tile-major histogram, from
// which every workgroup then adds up its own offsets (few tiles: a short loop of coalesced reads that
// saves the launches of a scan).
template <typename S, typename In, typename Out, bool COUNTS>
__global__ __launch_bounds__(S::kThreads) void sort_scatter(In in, Out out, int64_t count,
                                                            const int32_t* __restrict__ d_count, int shift, int nbits,
                                                            const int32_t* __restrict__ offs, int32_t tiles) {
    constexpr int kBins = 1 << S::kBits;
    constexpr int kWaves = S::kThreads / 64;
    constexpr int kPer = kBins > S::kThreads ? kBins / S::kThreads : 1;   // digits of one thread, consecutive
    __shared__ uint16_t wave_cnt[kWaves][kBins];   // keys of digit d in wavefront w, then their first place in the tile
    __shared__ int wave_tot[kWaves];
    __shared__ int shift_by[kBins];                // where the tile's keys of digit d go, less their first place in the tile
    __shared__ uint64_t tile[S::kTile];
    const int bins = 1 << nbits;
    if (d_count) count = *d_count;
    const int64_t tile_base = (int64_t)blockIdx.x * S::kTile;
    if (tile_base >= count) return;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t chunk = tile_base + (int64_t)wave * (64 * S::kItems);
    uint64_t key[S::kItems];
    uint16_t rank[S::kItems];
    {
        typename In::raw raw[S::kItems];
#pragma unroll
        for (int r = 0; r < S::kItems; ++r) {
            const int64_t i = chunk + r * 64 + lane;
            raw[r] = i < count ? in.load(i) : in.none();
        }
#pragma unroll
        for (int r = 0; r < S::kItems; ++r) key[r] = in.key(raw[r]);
    }
    for (int k = threadIdx.x; k < kWaves * kBins / 2; k += S::kThreads) reinterpret_cast<uint32_t*>(&wave_cnt[0][0])[k] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < S::kItems; ++r) {
        const bool valid = chunk + r * 64 + lane < count;
        const int d = (int)(key[r] >> shift) & (bins - 1);
        const uint64_t peers = lanes_of_digit<S::kBits>(d, nbits, __ballot(valid));
        const int pre = wave_cnt[wave][d];
        const int below = __popcll(peers & lt_mask);
        rank[r] = (uint16_t)(pre + below);
        if (valid && below == 0) wave_cnt[wave][d] = (uint16_t)(pre + __popcll(peers));
    }
    __syncthreads();
    {
        // this thread's digits: their keys in the tile (all wavefronts), the first place of each in the tile
        // (exclusive scan over the digits), and where they go
        const int d0 = threadIdx.x * kPer;
        int mine[kPer], sum = 0;
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            mine[p] = 0;
            if (d0 + p < kBins)
#pragma unroll
                for (int w = 0; w < kWaves; ++w) mine[p] += wave_cnt[w][d0 + p];
            sum += mine[p];
        }
        auto scan = [&](int v) {   // exclusive over the workgroup
            int inc = v;
#pragma unroll
            for (int dlt = 1; dlt < 64; dlt <<= 1) {
                const int t = __shfl_up(inc, dlt, 64);
                if (lane >= dlt) inc += t;
            }
            if (lane == 63) wave_tot[wave] = inc;
            __syncthreads();
            int before = inc - v;
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
                if (w < wave) before += wave_tot[w];
            __syncthreads();
            return before;
        };
        int first = scan(sum);
        int base[kPer];
        if (COUNTS) {
            // keys with a smaller digit anywhere, plus keys with this digit in earlier tiles
            int before[kPer], total[kPer], all = 0;
#pragma unroll
            for (int p = 0; p < kPer; ++p) before[p] = total[p] = 0;
            // with more threads than digits, kParts threads share a digit's tiles
            constexpr int kParts = S::kThreads / kBins > 1 ? S::kThreads / kBins : 1;
            __shared__ int part_sum[kParts > 1 ? kParts : 1][2][kParts > 1 ? kBins : 1];
            const int dd = kParts > 1 ? threadIdx.x % kBins : d0, part = kParts > 1 ? threadIdx.x / kBins : 0;
            if (dd < bins) {
#pragma unroll 16
                for (int b = part; b < tiles; b += kParts)
#pragma unroll
                    for (int p = 0; p < kPer; ++p) {
                        const int c = dd + p < bins ? offs[(int64_t)b * bins + dd + p] : 0;
                        if (b < (int)blockIdx.x) before[p] += c;
                        total[p] += c;
                    }
            }
            if constexpr (kParts > 1) {
                part_sum[part][0][dd] = before[0];
                part_sum[part][1][dd] = total[0];
                __syncthreads();
                before[0] = total[0] = 0;
                if (d0 < kBins)
#pragma unroll
                    for (int q = 0; q < kParts; ++q) {
                        before[0] += part_sum[q][0][d0];
                        total[0] += part_sum[q][1][d0];
                    }
            }
#pragma unroll
            for (int p = 0; p < kPer; ++p) all += total[p];
            int lower = scan(all);
#pragma unroll
            for (int p = 0; p < kPer; ++p) {
                base[p] = lower + before[p];
                lower += total[p];
            }
        } else {
#pragma unroll
            for (int p = 0; p < kPer; ++p) base[p] = d0 + p < bins ? offs[(int64_t)(d0 + p) * tiles + blockIdx.x] : 0;
        }
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            if (d0 + p < kBins) {
                shift_by[d0 + p] = base[p] - first;
                int at = first;   // wave_cnt[w][d] becomes the first tile place of wavefront w's keys of digit d
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    const int c = wave_cnt[w][d0 + p];
                    wave_cnt[w][d0 + p] = (uint16_t)at;
                    at += c;
                }
            }
            first += mine[p];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < S::kItems; ++r) {
        if (chunk + r * 64 + lane < count) {
            const int d = (int)(key[r] >> shift) & (bins - 1);
            tile[wave_cnt[wave][d] + rank[r]] = key[r];
        }
    }
    __syncthreads();
    const int64_t left = count - tile_base;
    const int valid_keys = left < S::kTile ? (int)left : S::kTile;
#pragma unroll 4
    for (int p = threadIdx.x; p < valid_keys; p += S::kThreads) {
        const uint64_t k = tile[p];
        const int d = (int)(k >> shift) & (bins - 1);
        out.store((int64_t)shift_by[d] + p, k);
        if constexpr (Out::kRuns) {
            // the last pass leaves equal groups next to each other in the tile: a group's number of keys is
            // one past its last place less its first
            const int32_t g = out.group(k);
            const bool head = p == 0 || out.group(tile[p - 1]) != g;
            const bool tail = p == valid_keys - 1 || out.group(tile[p + 1]) != g;
            const int delta = (tail ? p + 1 : 0) - (head ? p : 0);
            if (delta != 0) atomicAdd(out.counts + g, delta);
        }
    }
}

// One digit of nbits (at most S::kBits) from bit `shift`.  `ws` as for radix_sort_workspace_bytes(count).
template <typename S, typename In, typename Out>
int32_t radix_pass_as(In in, Out out, int64_t count, const int32_t* d_count, int shift, int nbits, void* ws,
                      hipStream_t stream) {
    const int32_t tiles = (int32_t)ceil_div(count, S::kTile);
    const dim3 grid((unsigned)tiles), blk(S::kThreads);
    int32_t* hist = static_cast<int32_t*>(ws);
    if (tiles <= kFusedTiles) {
        sort_histogram<S, In, true><<<grid, blk, 0, stream>>>(in, count, d_count, shift, nbits, hist, tiles);
        E2EG_LAUNCH_CHECK("sort_histogram");
        sort_scatter<S, In, Out, true><<<grid, blk, 0, stream>>>(in, out, count, d_count, shift, nbits, hist, tiles);
    } else {
        const int64_t cells = (int64_t)tiles << nbits;
        void* scan_ws = static_cast<char*>(ws) + align_up((size_t)cells * sizeof(int32_t));
        sort_histogram<S, In, false><<<grid, blk, 0, stream>>>(in, count, d_count, shift, nbits, hist, tiles);
        E2EG_LAUNCH_CHECK("sort_histogram");
        E2EG_HIP_TRY(exclusive_scan_i32(hist, hist, cells, nullptr, scan_ws, stream));
        sort_scatter<S, In, Out, false><<<grid, blk, 0, stream>>>(in, out, count, d_count, shift, nbits, hist, tiles);
    }
    E2EG_LAUNCH_CHECK("sort_scatter");
    return E2EG_OK;
}

inline bool sorts_large(int64_t count) { return count >= kLargeSortMin; }
// Digits of a sort by nbits bits: `passes` of them, the widths as even as they come.
inline int sort_passes(int64_t count, int nbits) {
    const int most = sorts_large(count) ? LargeSort::kBits : SmallSort::kBits;
    return (nbits + most - 1) / most;
}
inline int sort_width(int nbits, int passes, int pass) { return nbits * (pass + 1) / passes - nbits * pass / passes; }

template <typename In, typename Out>
int32_t radix_pass(In in, Out out, int64_t count, const int32_t* d_count, int shift, int nbits, void* ws, hipStream_t stream) {
    if (sorts_large(count)) return radix_pass_as<LargeSort>(in, out, count, d_count, shift, nbits, ws, stream);
    return radix_pass_as<SmallSort>(in, out, count, d_count, shift, nbits, ws, stream);
}

}  // namespace e2eg
