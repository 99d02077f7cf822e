// Entry work goes by tiles of consecutive CSR entries, one workgroup of kEntryThreads each: the rows of a tile
// are found by all threads together, kEntryThreads probes a round, and kept in LDS, where every entry finds its own
// (one search of the whole of row_ptr per entry costs 17 dependent loads on a graph of 150 k nodes).
#pragma once
#include "common.h"

namespace e2eg {

constexpr int kEntryThreads = 256;
constexpr int kEntryTile = 2048;
constexpr int kEntryRounds = kEntryTile / kEntryThreads;
constexpr int kTileRowsMax = 1024;   // rows of a tile held in LDS (a tile of mostly empty rows has more: then global memory)

// -> range[0], range[1]: the last i in [0, n) with row_ptr[i] <= first, and <= last.
__device__ __forceinline__ void rows_of_tile(const int32_t* __restrict__ row_ptr, int64_t n, int64_t first, int64_t last,
                                             int64_t (&range)[2]) {
    int64_t lo[2] = {0, 0}, hi[2] = {n, n};
    while (hi[0] - lo[0] > 1 || hi[1] - lo[1] > 1) {
        const int64_t want[2] = {first, last};
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int64_t step = (hi[k] - lo[k] + kEntryThreads - 1) / kEntryThreads;
            const int64_t at = lo[k] + step * threadIdx.x;
            const int cnt = __syncthreads_count(at < hi[k] && row_ptr[at] <= want[k]);   // a prefix of the threads, at least thread 0
            lo[k] += step * (cnt - 1);
            if (hi[k] - lo[k] > step) hi[k] = lo[k] + step;
        }
    }
    range[0] = lo[0];
    range[1] = lo[1];
}

// The row of entry e: the last i in [lo, hi] with row_ptr[i] <= e.
__device__ __forceinline__ int64_t row_of_entry(const int32_t* __restrict__ row_ptr, int64_t e, int64_t lo, int64_t hi) {
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (row_ptr[mid] <= e) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The rows of this workgroup's tile.  rows: LDS, kTileRowsMax + 1.
struct EntryTile {
    int64_t first, last;    // entries of the tile
    int64_t row0, count;    // its rows
    bool cached;
    const int32_t* rows;
    const int32_t* row_ptr;
    __device__ __forceinline__ EntryTile(const int32_t* __restrict__ row_ptr_, int64_t n, int64_t nnz, int32_t* lds) {
        first = (int64_t)blockIdx.x * kEntryTile;
        last = (first + kEntryTile < nnz ? first + kEntryTile : nnz) - 1;
        int64_t range[2];
        rows_of_tile(row_ptr_, n, first, last, range);
        row0 = range[0];
        count = range[1] - range[0] + 1;
        cached = count <= kTileRowsMax;
        if (cached)
            for (int64_t k = threadIdx.x; k <= count; k += kEntryThreads) lds[k] = row_ptr_[row0 + k];
        rows = lds;
        row_ptr = row_ptr_;
        __syncthreads();
    }
    // Entry e's row less row0.
    __device__ __forceinline__ int64_t row(int64_t e) const {
        return cached ? row_of_entry(rows, e, 0, count - 1) : row_of_entry(row_ptr, e, row0, row0 + count - 1) - row0;
    }
    __device__ __forceinline__ int32_t row_begin(int64_t k) const { return cached ? rows[k] : row_ptr[row0 + k]; }
};

}  // namespace e2eg
