// LSD radix sort of 64-bit keys over a chosen bit range, stable (passes: radix.h).  Orders the row
// segments of the schedule; the CSR build runs its passes itself.
#include "radix.h"

namespace e2eg {

size_t radix_sort_workspace_bytes(int64_t count) {
    if (count < 1) count = 1;
    const int64_t cells = sorts_large(count) ? ceil_div(count, LargeSort::kTile) << LargeSort::kBits
                                             : ceil_div(count, SmallSort::kTile) << SmallSort::kBits;
    return align_up((size_t)cells * sizeof(int32_t)) + scan_workspace_bytes(cells);
}

int32_t radix_sort_u64(uint64_t** src, uint64_t** dst, int64_t count, int lo, int nbits, void* ws,
                       hipStream_t stream) {
    if (count <= 0) return E2EG_OK;
    const int passes = sort_passes(count, nbits);
    for (int p = 0, shift = lo; p < passes; ++p) {
        const int width = sort_width(nbits, passes, p);
        const int32_t st = radix_pass(KeysIn{*src}, KeysOut{*dst}, count, nullptr, shift, width, ws, stream);
        if (st != E2EG_OK) return st;
        shift += width;
        uint64_t* t = *src;
        *src = *dst;
        *dst = t;
    }
    return E2EG_OK;
}

int bits_for(int64_t count) {
    int b = 1;
    while (b < 31 && ((int64_t)1 << b) < count) ++b;
    return b;
}

}  // namespace e2eg
