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
    static constexpr int kThreads = 512, kItems = 16, kBits = 8, kCopies = 16, kTile = kThreads * kItems;
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

// Keys come as K: 64-bit, or 32-bit once the leading digit has been taken off (Segmented).
template <typename K>
struct ArrayIn {
    const K* keys;
    using Key = K;
    using raw = K;   // what is loaded, and the key of it
    __device__ __forceinline__ ArrayIn from(int64_t base) const { return ArrayIn{keys + base}; }   // as of key `base`
    __device__ __forceinline__ raw load(uint32_t i) const { return keys[i]; }
    __device__ __forceinline__ raw none() const { return 0; }
    __device__ __forceinline__ K key(raw r) const { return r; }
    __device__ __forceinline__ bool ok(raw) const { return true; }
    __device__ __forceinline__ void report() const {}
};
template <typename K>
struct ArrayOut {
    static constexpr bool kRuns = false, kChecks = false;
    K* keys;
    __device__ __forceinline__ void store(uint32_t at, K key, int) const { keys[at] = key; }
};
using KeysIn = ArrayIn<uint64_t>;
using KeysOut = ArrayOut<uint64_t>;
// 64-bit keys in, their low bits out (kChecks: the scatter reports bad input, its histogram having seen less).
struct LowBitsOut {
    static constexpr bool kRuns = false, kChecks = true;
    uint32_t* keys;
    uint32_t mask;
    __device__ __forceinline__ void store(uint32_t at, uint64_t key, int) const { keys[at] = (uint32_t)key & mask; }
};

// How a list is cut into tiles, one workgroup each.
// Whole: tiles of consecutive keys; the table of digit counts is digit-major [bins][tiles] for a scan, or
// tile-major [tiles][bins] for a scatter that adds up its offsets itself.  d_count (may be null): the
// number of keys, known on the device only; `count` is then its upper bound, which sized the launch.
struct Place {
    int64_t base, end;   // keys of the tile (base >= end: none)
    int64_t cell;        // its count of digit d is at cell + d * step
    int32_t step;
    int segment;
};
struct Whole {
    int64_t count;
    const int32_t* d_count;
    int32_t tiles;
    template <typename S>
    __device__ __forceinline__ Place place(int) const {
        const int64_t n = d_count ? *d_count : count, base = (int64_t)blockIdx.x * S::kTile;
        return Place{base, base + S::kTile < n ? base + S::kTile : n, (int64_t)blockIdx.x, tiles, 0};
    }
};
// Segmented: every segment (the keys of one value of a leading digit) is sorted by itself and has its own
// tiles; the table is [segments][bins][tiles of the segment], so that one scan of it gives the places in
// the whole list.
constexpr int kMaxSegments = 256;
struct Segments {
    int32_t first[kMaxSegments + 1];   // first key of every segment
    int32_t tile[kMaxSegments + 1];    // first tile
};
struct Segmented {
    const Segments* s;
    int32_t n;   // segments
    template <typename S>
    __device__ __forceinline__ Place place(int bins) const {
        // the segment whose tiles these are: the last one that begins at or before this tile (empty ones begin there too)
        const int g = __syncthreads_count((int)threadIdx.x < n && s->tile[threadIdx.x] <= (int)blockIdx.x) - 1;
        const int32_t t0 = s->tile[g], t1 = s->tile[g + 1];
        const int64_t end = s->first[g + 1];
        if ((int)blockIdx.x >= t1) return Place{end, end, 0, 0, g};   // the launch is sized for an upper bound
        const int64_t base = s->first[g] + (int64_t)((int)blockIdx.x - t0) * S::kTile;
        return Place{base, base + S::kTile < end ? base + S::kTile : end, (int64_t)t0 * bins + ((int)blockIdx.x - t0), t1 - t0, g};
    }
};

// Digit counts of every tile.
template <typename S, typename In, typename Tiling, bool TILE_MAJOR>
__global__ __launch_bounds__(S::kThreads) void sort_histogram(In in, Tiling tiling, int shift, int nbits,
                                                              int32_t* __restrict__ hist) {
    // [digit][copy], a copy for every kCopies-th lane: with few digits, or popular ones, the lanes of a wavefront
    // would meet on one word and take turns
    __shared__ int h[S::kCopies << S::kBits];
    const int bins = 1 << nbits;
    for (int k = threadIdx.x; k < S::kCopies << S::kBits; k += S::kThreads) h[k] = 0;
    __syncthreads();
    const Place at = tiling.template place<S>(bins);
    int* mine = h + threadIdx.x % S::kCopies;
    const int left = (int)(at.end - at.base);   // 32-bit indexes inside the tile: the passes are bound by VALU work
    const In tile_in = in.from(at.base);
    typename In::raw raw[S::kItems];
#pragma unroll
    for (int k = 0; k < S::kItems; ++k) {
        const int i = k * S::kThreads + (int)threadIdx.x;
        raw[k] = i < left ? tile_in.load(i) : in.none();
    }
    bool ok = true;
#pragma unroll
    for (int k = 0; k < S::kItems; ++k) {
        const int i = k * S::kThreads + (int)threadIdx.x;
        if (i < left) {
            ok = ok && in.ok(raw[k]);
            atomicAdd(&mine[((int)(in.key(raw[k]) >> shift) & (bins - 1)) * S::kCopies], 1);
        }
    }
    if (!ok) in.report();
    __syncthreads();
    for (int d = threadIdx.x; d < bins; d += S::kThreads) {
        int t = 0;
#pragma unroll
        for (int c = 0; c < S::kCopies; ++c) t += h[d * S::kCopies + ((c + d) % S::kCopies)];
        if (TILE_MAJOR) hist[(int64_t)blockIdx.x * bins + d] = t;
        else if (at.step > 0) hist[at.cell + (int64_t)d * at.step] = t;
    }
}

// Stable scatter.  A tile is split into one contiguous chunk per wavefront; a wavefront walks its chunk 64
// keys at a time, ranking equal digits by lane order plus a running per-wavefront digit count, so ranks
// follow input order.  The keys are then put in digit order inside the tile (in LDS) and written out
// from there, consecutive threads writing consecutive keys: keys of one digit leave as one contiguous run.
// `offs` is the digit-major table of scanned offsets, or, with COUNTS, the raw tile-major histogram, from
// which every workgroup then adds up its own offsets (few tiles: a short loop of coalesced reads that
// saves the launches of a scan).
template <typename S, typename In, typename Out, typename Tiling, bool COUNTS>
__global__ __launch_bounds__(S::kThreads) void sort_scatter(In in, Out out, Tiling tiling, int shift, int nbits,
                                                            const int32_t* __restrict__ offs) {
    using Key = typename In::Key;
    constexpr int kBins = 1 << S::kBits;
    constexpr int kWaves = S::kThreads / 64;
    constexpr int kPer = kBins > S::kThreads ? kBins / S::kThreads : 1;   // digits of one thread, consecutive
    __shared__ uint16_t wave_cnt[kWaves][kBins];   // keys of digit d in wavefront w, then their first place in the tile
    __shared__ int wave_tot[kWaves];
    __shared__ int shift_by[kBins];                // where the tile's keys of digit d go, less their first place in the tile
    __shared__ Key tile[S::kTile];
    const int bins = 1 << nbits;
    const Place place = tiling.template place<S>(bins);
    if (place.base >= place.end) return;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int left = (int)(place.end - place.base), chunk = wave * (64 * S::kItems);   // indexes inside the tile
    const In tile_in = in.from(place.base);
    Key key[S::kItems];
    uint16_t rank[S::kItems];
    {
        typename In::raw raw[S::kItems];
#pragma unroll
        for (int r = 0; r < S::kItems; ++r) {
            const int i = chunk + r * 64 + lane;
            raw[r] = i < left ? tile_in.load(i) : in.none();
        }
#pragma unroll
        for (int r = 0; r < S::kItems; ++r) key[r] = in.key(raw[r]);
        if constexpr (Out::kChecks) {
            bool ok = true;
#pragma unroll
            for (int r = 0; r < S::kItems; ++r) ok = ok && (chunk + r * 64 + lane >= left || in.ok(raw[r]));
            if (!ok) in.report();
        }
    }
    for (int k = threadIdx.x; k < kWaves * kBins / 2; k += S::kThreads) reinterpret_cast<uint32_t*>(&wave_cnt[0][0])[k] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < S::kItems; ++r) {
        const bool valid = chunk + r * 64 + lane < left;
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
        if constexpr (COUNTS) {
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
                for (int b = part; b < tiling.tiles; b += kParts)
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
            for (int p = 0; p < kPer; ++p) base[p] = d0 + p < bins ? offs[place.cell + (int64_t)(d0 + p) * place.step] : 0;
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
        if (chunk + r * 64 + lane < left) {
            const int d = (int)(key[r] >> shift) & (bins - 1);
            tile[wave_cnt[wave][d] + rank[r]] = key[r];
        }
    }
    __syncthreads();
#pragma unroll 4
    for (int p = threadIdx.x; p < left; p += S::kThreads) {
        const Key k = tile[p];
        const int d = (int)(k >> shift) & (bins - 1);
        out.store((uint32_t)(shift_by[d] + p), k, place.segment);
        if constexpr (Out::kRuns) {
            // the last pass leaves equal groups next to each other in the tile: a group's number of keys is
            // one past its last place less its first
            const int32_t g = out.group(k, place.segment);
            const bool head = p == 0 || out.group(tile[p - 1], place.segment) != g;
            const bool tail = p == left - 1 || out.group(tile[p + 1], place.segment) != g;
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
    const Whole whole{count, d_count, tiles};
    if (tiles <= kFusedTiles) {
        sort_histogram<S, In, Whole, true><<<grid, blk, 0, stream>>>(in, whole, shift, nbits, hist);
        E2EG_LAUNCH_CHECK("sort_histogram");
        sort_scatter<S, In, Out, Whole, true><<<grid, blk, 0, stream>>>(in, out, whole, shift, nbits, hist);
    } else {
        const int64_t cells = (int64_t)tiles << nbits;
        void* scan_ws = static_cast<char*>(ws) + align_up((size_t)cells * sizeof(int32_t));
        sort_histogram<S, In, Whole, false><<<grid, blk, 0, stream>>>(in, whole, shift, nbits, hist);
        E2EG_LAUNCH_CHECK("sort_histogram");
        E2EG_HIP_TRY(exclusive_scan_i32(hist, hist, cells, nullptr, scan_ws, stream));
        sort_scatter<S, In, Out, Whole, false><<<grid, blk, 0, stream>>>(in, out, whole, shift, nbits, hist);
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
