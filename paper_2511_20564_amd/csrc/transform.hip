// e2eg_layer_transform: the dense per-layer update H' = relu(P W) and its backward (paper: the
// update function psi of the generic message-passing layer in Section 3, with the W and sigma of
// the GraphSAGE layer in Section 3.1).
//
// This is the one real contraction on the path, so it runs on the matrix cores: bf16 operands,
// fp32 accumulation, v_mfma_f32_32x32x16_bf16 (wave64; each lane feeds 8 consecutive k of one
// row / column).  The products are computed transposed, D[out column][row], so that a lane ends
// up holding runs of 4 consecutive output columns of ONE row and can store them as 8 bytes.
//   forward : H  = relu(P W)        rows = nodes, k = Fin,  weight tile W^T staged in LDS
//   backward: dP = dZ W^T, dW = P^T dZ with dZ = gH * [H > 0], in one kernel that reads gH, H and P once:
//             rows = nodes, k = Fout for dP; k = nodes for dW, each workgroup adding up its share of the
//             nodes into an fp32 partial [Fin][Fout]; partials are added in block order by a second kernel
//             (no atomics, reproducible).
#include "common.h"

#include <mutex>

namespace e2eg {
namespace {

constexpr int kReduceThreads = 256;
constexpr int kMaxF = 256;
constexpr int kPad = 8;                      // LDS row padding (elements) against bank conflicts

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma(const uint4 a, const uint4 b, const f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Two floats -> packed bf16, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Keep the bf16 halves of g where the matching half of h is > 0.
__device__ __forceinline__ uint32_t mask_pair(uint32_t g, uint32_t h) {
    uint32_t m = 0;
    if (__uint_as_float(h << 16) > 0.0f) m |= 0x0000ffffu;
    if (__uint_as_float(h & 0xffff0000u) > 0.0f) m |= 0xffff0000u;
    return g & m;
}
__device__ __forceinline__ uint4 mask_vec(uint4 g, uint4 h) {
    return make_uint4(mask_pair(g.x, h.x), mask_pair(g.y, h.y), mask_pair(g.z, h.z), mask_pair(g.w, h.w));
}

// ---- forward ----------------------------------------------------------------------------------------
// out[r][c] = relu( sum_k A[r][k] W[k][c] ).  KB, NB: the most blocks of 32 input and output columns; EXACT: exactly
// that many.  W^T is staged in LDS once per workgroup, all of it, so that A is read once.  A tile of R rows at a
// time, taken in turn across the grid (at any moment the workgroups in flight read and write one moving stretch
// of the tables): the rows stand in LDS, each wavefront forms one block of 32 x 32 results, and these leave
// through LDS as whole rows.  The rows of the next two tiles are in flight in registers meanwhile.
// Bound by HBM.  Measured, 3 M rows of 256 x 128: 702 us when each of two groups of 64 columns read A again,
// 411 now; 200 k of 128 x 128: 22.9 -> 20.2 us (a copy of the bytes: 16.4).
constexpr int kTileThreads = 1024;   // one workgroup per compute unit
constexpr int kTileGroups = 256;

template <int KB, int NB>
struct ForwardTile {
    static constexpr int kRows = KB * NB <= 16 ? 128 : KB * NB <= 32 ? 64 : 32;
    static constexpr int kLdA = KB * 32 + kPad;
    static constexpr int kLdO = NB * 32 + kPad;
    static constexpr bool kShared = KB * NB > 32;   // results take the place of the rows: there is no room for both
    static constexpr int kPassesA = kRows * KB * 4 / kTileThreads;   // 16-byte pieces of a tile per thread
    static constexpr int kPassesO = kRows * NB * 4 / kTileThreads;
    static constexpr int kOut = kRows * kLdO, kIn = kRows * kLdA;
};

template <bool RELU, int KB, int NB, bool EXACT>
__global__ __launch_bounds__(kTileThreads) void dense_forward(const uint16_t* __restrict__ a_rows,
                                                              const uint16_t* __restrict__ w, uint16_t* __restrict__ out,
                                                              int32_t n, int32_t kdim_, int32_t ndim_, int32_t stream_out) {
    using T = ForwardTile<KB, NB>;
    constexpr int R = T::kRows;
    __shared__ __attribute__((aligned(16))) uint16_t wt[NB * 32 * T::kLdA];   // [ndim][kdim]
    __shared__ __attribute__((aligned(16))) uint16_t at[T::kShared ? (T::kIn > T::kOut ? T::kIn : T::kOut) : T::kIn];
    __shared__ __attribute__((aligned(16))) uint16_t ot_[T::kShared ? 8 : T::kOut];
    uint16_t* ot = T::kShared ? at : ot_;
    const int kdim = EXACT ? KB * 32 : kdim_, ndim = EXACT ? NB * 32 : ndim_;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31;
    const int khalf = lane >> 5;
    const int kvecs = kdim / 8, nvecs = ndim / 8;
    int arow[T::kPassesA], acol[T::kPassesA], orow[T::kPassesO], ocol[T::kPassesO];   // this thread's pieces of a tile
#pragma unroll
    for (int i = 0; i < T::kPassesA; ++i) {
        const int e = i * kTileThreads + threadIdx.x;
        arow[i] = e / kvecs;
        acol[i] = (e - arow[i] * kvecs) * 8;
    }
#pragma unroll
    for (int i = 0; i < T::kPassesO; ++i) {
        const int e = i * kTileThreads + threadIdx.x;
        orow[i] = e / nvecs;
        ocol[i] = (e - orow[i] * nvecs) * 8;
    }
    struct Rows {
        uint4 v[T::kPassesA];
    };
    auto load_tile = [&](Rows& q, int64_t r0) {   // rows past the end: zeros
#pragma unroll
        for (int i = 0; i < T::kPassesA; ++i) {
            q.v[i] = make_uint4(0u, 0u, 0u, 0u);
            if ((EXACT || arow[i] < R) && r0 + arow[i] < n)
                q.v[i] = *reinterpret_cast<const uint4*>(a_rows + (r0 + arow[i]) * kdim + acol[i]);
        }
    };
    const int64_t step = (int64_t)gridDim.x * R;
    int64_t r0 = (int64_t)blockIdx.x * R;
    Rows qa, qb;
    load_tile(qa, r0);
    load_tile(qb, r0 + step);
    {
        // W^T: a thread takes the same 8 columns of two consecutive rows of W (k = 2 kp, 2 kp + 1), 16 bytes each, and
        // writes, for each of the 8 columns, the pair as one 4-byte word into that column's row of the tile.
        // Consecutive lanes hold consecutive kp: a store instruction fills consecutive banks.
        const int kpairs = kdim / 2;
        uint32_t* wt32 = reinterpret_cast<uint32_t*>(wt);
        constexpr int ldw = T::kLdA / 2;
        for (int e = threadIdx.x; e < kpairs * nvecs; e += kTileThreads) {
            const int ch = e / kpairs, kp = e - ch * kpairs;
            const uint16_t* src = w + (int64_t)(2 * kp) * ndim + ch * 8;
            const uint4 q0 = *reinterpret_cast<const uint4*>(src);
            const uint4 q1 = *reinterpret_cast<const uint4*>(src + ndim);
            const uint32_t w0[4] = {q0.x, q0.y, q0.z, q0.w};
            const uint32_t w1[4] = {q1.x, q1.y, q1.z, q1.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = ch * 8 + 2 * j;
                wt32[c * ldw + kp] = (w0[j] & 0xffffu) | (w1[j] << 16);
                wt32[(c + 1) * ldw + kp] = (w0[j] >> 16) | (w1[j] & 0xffff0000u);
            }
        }
    }
    const int rb = wave % (R / 32), cb = wave / (R / 32);   // this wavefront's block of a tile
    const bool live = cb < NB && (EXACT || cb * 32 < ndim);
    const uint16_t* wb = wt + (cb * 32 + l32) * T::kLdA + khalf * 8;
    const uint16_t* ab = at + (rb * 32 + l32) * T::kLdA + khalf * 8;
    auto do_tile = [&](Rows& q) {
#pragma unroll
        for (int i = 0; i < T::kPassesA; ++i)
            if (EXACT || arow[i] < R) *reinterpret_cast<uint4*>(at + arow[i] * T::kLdA + acol[i]) = q.v[i];
        __syncthreads();
        if (r0 + 2 * step < n) load_tile(q, r0 + 2 * step);
        f32x16 d;
        if (live) {
#pragma unroll
            for (int i = 0; i < 16; ++i) d[i] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KB * 2; ++ks)
                if (EXACT || ks * 16 < kdim)
                    d = mfma(*reinterpret_cast<const uint4*>(wb + ks * 16), *reinterpret_cast<const uint4*>(ab + ks * 16), d);  // D[c][r]
        }
        if (T::kShared) __syncthreads();
        if (live) {
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = d[g4 * 4 + i];
                    if (RELU && !(v[i] > 0.0f)) v[i] = 0.0f;
                }
                *reinterpret_cast<uint2*>(ot + (rb * 32 + l32) * T::kLdO + cb * 32 + g4 * 8 + khalf * 4) =
                    make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < T::kPassesO; ++i) {
            if ((EXACT || orow[i] < R) && r0 + orow[i] < n) {
                const uint4 v = *reinterpret_cast<const uint4*>(ot + orow[i] * T::kLdO + ocol[i]);
                uint16_t* dst = out + (r0 + orow[i]) * ndim + ocol[i];
                if (stream_out) {   // tables far larger than the caches: do not let the results displace the inputs
                    const u32x4 w4 = {v.x, v.y, v.z, v.w};
                    __builtin_nontemporal_store(w4, reinterpret_cast<u32x4*>(dst));
                } else {
                    *reinterpret_cast<uint4*>(dst) = v;
                }
            }
        }
        if (T::kShared) __syncthreads();
        r0 += step;
    };
#pragma unroll 1
    while (r0 < n) {
        do_tile(qa);
        if (r0 < n) do_tile(qb);
    }
}

// ---- backward ---------------------------------------------------------------------------------------
// Four 16-bit values of one matrix column, from four consecutive rows of a row-major LDS tile: in every group
// of 16 lanes, lanes 4 k .. 4 k + 3 name the 16 columns of row k (8 bytes each), and lane m gets column m of
// the four rows.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 read_transposed(const uint16_t* p) {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(const_cast<uint16_t*>(p))));
}

// dP[r][c] = sum_o dZ[r][o] W[c][o] and partial[blockIdx.x][c][o] = sum over this workgroup's rows of
// P[r][c] dZ[r][o], with dZ = gH, or gH where H > 0 (MASKED).  FINB, FOUTB: the most blocks of 32 columns of P (of
// one group, grid.y) and of dZ; EXACT: exactly that many.
// A tile of R rows at a time, taken in turn across the grid; gH, H and P are read once and stand in LDS row by
// row.  For dP the contraction runs along a row, for dW down the rows: there the matrix cores' operands come
// from the same tiles through transposing LDS reads.  Sixteen wavefronts, each with one block of 32 x 32 of dP per
// tile and one or two of dW for the whole kernel; the next tile's rows are in flight in registers during
// the products.  (Row pitches: dZ is read both ways; a pitch of 20 banks beyond a multiple of 64 serves rows
// without conflicts and columns nearly so; P is read down the columns only: 16 banks.)
// Bound by HBM: 2 x (2 Fout + 2 Fin) bytes a row.  Measured with the reduction behind it: 200 k rows of 128 x 128
// 69 us when dP and dW were two kernels that both read gH and H, 41 now (a copy of the bytes: 33); 3 M rows of
// 256 x 128 1722 and 862 us (738).
constexpr int kBackWaves = kTileThreads / 64;

template <int FINB, int FOUTB>
struct BackTile {
    static constexpr int kRows = FINB * FOUTB == 16 ? 128 : 64;
    static constexpr int kLdW = FOUTB * 32 + kPad;
    static constexpr int kLdZ = FOUTB * 32 + (FINB == 8 ? 8 : 40);
    static constexpr int kLdP = FINB * 32 + 32;
    static constexpr int kLdO = FINB * 32 + kPad;
    static constexpr int kPassesZ = kRows * FOUTB * 4 / kTileThreads;   // 16-byte pieces of a tile per thread
    static constexpr int kPassesP = kRows * FINB * 4 / kTileThreads;
    static constexpr int kAccs = FINB * FOUTB / kBackWaves;             // blocks of dW per wavefront
};

template <bool MASKED, int FINB, int FOUTB, bool EXACT>
__global__ __launch_bounds__(kTileThreads) void dense_backward(const uint16_t* __restrict__ p_rows,
                                                               const uint16_t* __restrict__ w,
                                                               const uint16_t* __restrict__ h_rows,
                                                               const uint16_t* __restrict__ gh_rows,
                                                               uint16_t* __restrict__ gp, float* __restrict__ partial,
                                                               int32_t n, int32_t fin_, int32_t fout_, int32_t stream_out) {
    using T = BackTile<FINB, FOUTB>;
    constexpr int R = T::kRows;
    __shared__ __attribute__((aligned(16))) uint16_t wt[FINB * 32 * T::kLdW];   // [c][o]
    __shared__ __attribute__((aligned(16))) uint16_t zt[R * T::kLdZ];           // [r][o]
    __shared__ __attribute__((aligned(16))) uint16_t pt[R * T::kLdP];           // [r][c]
    __shared__ __attribute__((aligned(16))) uint16_t ot[R * T::kLdO];           // [r][c]
    const int fin = EXACT ? FINB * 32 : fin_, fout = EXACT ? FOUTB * 32 : fout_;
    const int c0 = EXACT ? 0 : blockIdx.y * (FINB * 32);
    const int cg = EXACT ? FINB * 32 : (fin - c0 < FINB * 32 ? fin - c0 : FINB * 32);   // columns of P in this group
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31;
    const int khalf = lane >> 5;
    // a thread's pieces of a tile: row and first column, the same in every tile
    const int zvecs = fout / 8, pvecs = cg / 8;
    int zrow[T::kPassesZ], zcol[T::kPassesZ], prow[T::kPassesP], pcol[T::kPassesP];
#pragma unroll
    for (int i = 0; i < T::kPassesZ; ++i) {
        const int e = i * kTileThreads + threadIdx.x;
        zrow[i] = e / zvecs;
        zcol[i] = (e - zrow[i] * zvecs) * 8;
    }
#pragma unroll
    for (int i = 0; i < T::kPassesP; ++i) {
        const int e = i * kTileThreads + threadIdx.x;
        prow[i] = e / pvecs;
        pcol[i] = (e - prow[i] * pvecs) * 8;
    }
    uint4 qz[T::kPassesZ], qh[MASKED ? T::kPassesZ : 1], qp[T::kPassesP];
    auto load_tile = [&](int64_t r0) {   // rows past the end: zeros
        const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int i = 0; i < T::kPassesZ; ++i) {
            qz[i] = zero;
            if (MASKED) qh[i] = zero;
            if ((EXACT || zrow[i] < R) && r0 + zrow[i] < n) {
                const int64_t at = (r0 + zrow[i]) * fout + zcol[i];
                qz[i] = *reinterpret_cast<const uint4*>(gh_rows + at);
                if (MASKED) qh[i] = *reinterpret_cast<const uint4*>(h_rows + at);
            }
        }
#pragma unroll
        for (int i = 0; i < T::kPassesP; ++i) {
            qp[i] = zero;
            if ((EXACT || prow[i] < R) && r0 + prow[i] < n)
                qp[i] = *reinterpret_cast<const uint4*>(p_rows + (r0 + prow[i]) * fin + c0 + pcol[i]);
        }
    };
    const int64_t step = (int64_t)gridDim.x * R;
    int64_t r0 = (int64_t)blockIdx.x * R;
    load_tile(r0);
    for (int e = threadIdx.x; e < cg * zvecs; e += kTileThreads) {
        const int c = e / zvecs, v = e - c * zvecs;
        *reinterpret_cast<uint4*>(wt + c * T::kLdW + v * 8) = *reinterpret_cast<const uint4*>(w + (int64_t)(c0 + c) * fout + v * 8);
    }
    // this wavefront's block of dP in every tile, and its blocks of dW
    constexpr int kRowBlocks = R / 32;
    const int prb = wave % kRowBlocks, pcb = wave / kRowBlocks;
    const bool p_live = gp && pcb < FINB && (EXACT || pcb * 32 < cg);
    const int wcb = wave * T::kAccs / FOUTB, wob = wave * T::kAccs % FOUTB;   // blocks (wcb, wob), (wcb, wob + 1)
    const bool w_live = partial && (EXACT || wcb * 32 < cg);
    const int obs = fout / 32;
    // offset of this lane in a transposing read of 16 rows x 32 columns (see read_transposed)
    const int tr_row = khalf * 8 + ((lane & 15) >> 2), tr_col = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    f32x16 acc[T::kAccs];
#pragma unroll
    for (int u = 0; u < T::kAccs; ++u)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[u][i] = 0.0f;

#pragma unroll 1
    for (; r0 < n; r0 += step) {
#pragma unroll
        for (int i = 0; i < T::kPassesZ; ++i)
            if (EXACT || zrow[i] < R)
                *reinterpret_cast<uint4*>(zt + zrow[i] * T::kLdZ + zcol[i]) = MASKED ? mask_vec(qz[i], qh[i]) : qz[i];
#pragma unroll
        for (int i = 0; i < T::kPassesP; ++i)
            if (EXACT || prow[i] < R) *reinterpret_cast<uint4*>(pt + prow[i] * T::kLdP + pcol[i]) = qp[i];
        __syncthreads();
        if (r0 + step < n) load_tile(r0 + step);
        if (p_live) {
            f32x16 d;
#pragma unroll
            for (int i = 0; i < 16; ++i) d[i] = 0.0f;
            const uint16_t* wb = wt + (pcb * 32 + l32) * T::kLdW + khalf * 8;
            const uint16_t* zb = zt + (prb * 32 + l32) * T::kLdZ + khalf * 8;
#pragma unroll
            for (int ks = 0; ks < FOUTB * 2; ++ks) {
                if (EXACT || ks * 16 < fout)
                    d = mfma(*reinterpret_cast<const uint4*>(wb + ks * 16), *reinterpret_cast<const uint4*>(zb + ks * 16), d);  // D[c][r]
            }
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                *reinterpret_cast<uint2*>(ot + (prb * 32 + l32) * T::kLdO + pcb * 32 + g4 * 8 + khalf * 4) =
                    make_uint2(pack_bf16(d[g4 * 4], d[g4 * 4 + 1]), pack_bf16(d[g4 * 4 + 2], d[g4 * 4 + 3]));
        }
        if (w_live) {
            const uint16_t* pb = pt + tr_row * T::kLdP + wcb * 32 + tr_col;
            const uint16_t* zb = zt + tr_row * T::kLdZ + wob * 32 + tr_col;
#pragma unroll
            for (int ks = 0; ks < R / 16; ++ks) {
                const uint2 a0 = read_transposed(pb + ks * 16 * T::kLdP), a1 = read_transposed(pb + (ks * 16 + 4) * T::kLdP);
                const uint4 a = make_uint4(a0.x, a0.y, a1.x, a1.y);
#pragma unroll
                for (int u = 0; u < T::kAccs; ++u) {
                    if (EXACT || wob + u < obs) {
                        const uint16_t* zu = zb + u * 32;
                        const uint2 b0 = read_transposed(zu + ks * 16 * T::kLdZ), b1 = read_transposed(zu + (ks * 16 + 4) * T::kLdZ);
                        acc[u] = mfma(a, make_uint4(b0.x, b0.y, b1.x, b1.y), acc[u]);  // D[c][o]
                    }
                }
            }
        }
        __syncthreads();
        if (gp) {
#pragma unroll
            for (int i = 0; i < T::kPassesP; ++i) {
                if ((EXACT || prow[i] < R) && r0 + prow[i] < n) {
                    const uint4 v = *reinterpret_cast<const uint4*>(ot + prow[i] * T::kLdO + pcol[i]);
                    uint16_t* dst = gp + (r0 + prow[i]) * fin + c0 + pcol[i];
                    if (stream_out) {
                        const u32x4 w4 = {v.x, v.y, v.z, v.w};
                        __builtin_nontemporal_store(w4, reinterpret_cast<u32x4*>(dst));
                    } else {
                        *reinterpret_cast<uint4*>(dst) = v;
                    }
                }
            }
        }
    }
    if (!w_live) return;
    float* dst = partial + (int64_t)blockIdx.x * fin * fout;
#pragma unroll
    for (int u = 0; u < T::kAccs; ++u) {
        if (EXACT || wob + u < obs) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int c = c0 + wcb * 32 + (i / 4) * 8 + khalf * 4 + (i % 4);
                dst[(int64_t)c * fout + (wob + u) * 32 + l32] = acc[u][i];
            }
        }
    }
}

// gw[e] = sum over blocks of partial[b][e], in double and in a fixed order: thread (q, j) of a
// workgroup adds blocks q, q + 8, q + 16, ... for element e0 + j; the eight sums of an element are
// then added in q order.
constexpr int kReduceElems = 32;   // elements per workgroup (one 128-byte line of every partial matrix)
constexpr int kReduceSlices = kReduceThreads / kReduceElems;

__global__ __launch_bounds__(kReduceThreads) void weight_grad_reduce(const float* __restrict__ partial, int32_t nblocks,
                                                               int32_t count, float* __restrict__ gw) {
    __shared__ double red[kReduceSlices][kReduceElems];
    const int j = threadIdx.x % kReduceElems, q = threadIdx.x / kReduceElems;
    const int e = blockIdx.x * kReduceElems + j;
    double s = 0.0;
    if (e < count) {
#pragma unroll 16
        for (int32_t b = q; b < nblocks; b += kReduceSlices) s += (double)partial[(int64_t)b * count + e];
    }
    red[q][j] = s;
    __syncthreads();
    if (q == 0 && e < count) {
        double t = red[0][j];
#pragma unroll
        for (int k = 1; k < kReduceSlices; ++k) t += red[k][j];
        gw[e] = (float)t;
    }
}

// Partial matrices the workspace query promises: at most 256, each of a multiple of 64 rows, at least 128.
int64_t promised_partials(int64_t n) {
    int64_t rows = ceil_div(ceil_div(n > 0 ? n : 1, 256), 64) * 64;
    if (rows < 128) rows = 128;
    return ceil_div(n > 0 ? n : 1, rows);
}

// Workgroups of dense_backward per group of columns of P, and so partial matrices: one per compute unit, fewer
// where there are fewer than 128 rows for each, or where only the promised number fits in the static array.
int32_t back_groups(int32_t n, int32_t fin, int32_t fout) {
    const int64_t column_groups = fout > 128 ? ceil_div(fin, 128) : 1;
    const int64_t most = kTileGroups / column_groups;
    const int64_t want = ceil_div(n > 0 ? n : 1, 128);
    const int64_t groups = want < most ? want : most;
    const int64_t fit = E2EG_TRANSFORM_STATIC_SCRATCH_BYTES / ((int64_t)fin * fout * (int64_t)sizeof(float));
    const int64_t promised = promised_partials(n);
    return (int32_t)(groups > fit && promised <= fit ? promised : groups);
}

// Streaming stores once the result is far larger than the caches (5 % at 4 M rows); below that the next
// kernel of a mini-batch step finds the rows in the caches if they are written normally.
int32_t streams_out(int64_t n, int32_t cols) { return n * cols * 2 > (64ll << 20) ? 1 : 0; }

template <bool RELU, int KB, int NB>
void launch_forward_as(const uint16_t* a, const uint16_t* w, uint16_t* out, int32_t n, int32_t kdim, int32_t ndim, hipStream_t stream) {
    const int64_t tiles = ceil_div(n, ForwardTile<KB, NB>::kRows);
    const dim3 grid((unsigned)(tiles < kTileGroups ? tiles : kTileGroups)), blk(kTileThreads);
    const int32_t so = streams_out(n, ndim);
    if (kdim == KB * 32 && ndim == NB * 32)
        dense_forward<RELU, KB, NB, true><<<grid, blk, 0, stream>>>(a, w, out, n, kdim, ndim, so);
    else
        dense_forward<RELU, KB, NB, false><<<grid, blk, 0, stream>>>(a, w, out, n, kdim, ndim, so);
}

template <bool RELU>
void launch_forward(const void* a_, const void* w_, void* out_, int32_t n, int32_t kdim, int32_t ndim, hipStream_t stream) {
    const uint16_t* a = static_cast<const uint16_t*>(a_);
    const uint16_t* w = static_cast<const uint16_t*>(w_);
    uint16_t* out = static_cast<uint16_t*>(out_);
    if (kdim <= 128 && ndim <= 128) launch_forward_as<RELU, 4, 4>(a, w, out, n, kdim, ndim, stream);
    else if (kdim <= 128) launch_forward_as<RELU, 4, 8>(a, w, out, n, kdim, ndim, stream);
    else if (ndim <= 128) launch_forward_as<RELU, 8, 4>(a, w, out, n, kdim, ndim, stream);
    else launch_forward_as<RELU, 8, 8>(a, w, out, n, kdim, ndim, stream);
}

template <bool MASKED, int FINB, int FOUTB>
void launch_back_as(const uint16_t* p, const uint16_t* w, const uint16_t* h, const uint16_t* gh, uint16_t* gp, float* partial,
                    int32_t n, int32_t fin, int32_t fout, hipStream_t stream) {
    const dim3 grid((unsigned)back_groups(n, fin, fout), (unsigned)ceil_div(fin, FINB * 32)), blk(kTileThreads);
    const int32_t so = streams_out(n, fin);
    if (fin == FINB * 32 && fout == FOUTB * 32)
        dense_backward<MASKED, FINB, FOUTB, true><<<grid, blk, 0, stream>>>(p, w, h, gh, gp, partial, n, fin, fout, so);
    else
        dense_backward<MASKED, FINB, FOUTB, false><<<grid, blk, 0, stream>>>(p, w, h, gh, gp, partial, n, fin, fout, so);
}

template <bool MASKED>
void launch_back(const void* p_, const void* w_, const void* h_, const void* gh_, void* gp_, float* partial, int32_t n,
                 int32_t fin, int32_t fout, hipStream_t stream) {
    const uint16_t* p = static_cast<const uint16_t*>(p_);
    const uint16_t* w = static_cast<const uint16_t*>(w_);
    const uint16_t* h = static_cast<const uint16_t*>(h_);
    const uint16_t* gh = static_cast<const uint16_t*>(gh_);
    uint16_t* gp = static_cast<uint16_t*>(gp_);
    // wide gradients: groups of 128 columns of P, or W and the tiles do not fit in LDS together
    if (fout > 128) launch_back_as<MASKED, 4, 8>(p, w, h, gh, gp, partial, n, fin, fout, stream);
    else if (fin > 128) launch_back_as<MASKED, 8, 4>(p, w, h, gh, gp, partial, n, fin, fout, stream);
    else launch_back_as<MASKED, 4, 4>(p, w, h, gh, gp, partial, n, fin, fout, stream);
}

}  // namespace
}  // namespace e2eg

using namespace e2eg;

extern "C" size_t e2eg_layer_transform_workspace_bytes(int32_t mode, int32_t n, int32_t Fin,
                                                       int32_t Fout, int32_t dtype) {
    if (n < 0 || Fin <= 0 || Fout <= 0 || dtype != E2EG_BF16) return 0;
    if (mode != E2EG_TRANSFORM_BWD) return kAlign;
    const int64_t used = back_groups(n, Fin, Fout), promised = promised_partials(n);
    const int64_t blocks = used > promised ? used : promised;
    return align_up((size_t)blocks * (size_t)Fin * (size_t)Fout * sizeof(float));
}

// ---- the same call for callers that cannot allocate ------------------------------------------
// The partial weight-gradient matrices live in a device array that is part of the library's code
// object, so no workspace has to come from anywhere.  Each GPU holds its own copy of the array at
// its own address; host code never uses the array's name as an address, only the pointer
// hipGetSymbolAddress returns for the current device, looked up once per device and kept.
static __device__ __align__(256) float scratch[E2EG_TRANSFORM_STATIC_SCRATCH_BYTES / sizeof(float)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kMaxDevices];   // address of `scratch` on each device, null until looked up

int32_t static_scratch_of_current_device(float** out) {
    int dev = -1;
    E2EG_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(E2EG_ERR_HIP, "layer_transform_noalloc: device index %d", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        float* p = nullptr;
        E2EG_HIP_TRY(hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch)));
        if (!p) return fail(E2EG_ERR_HIP, "layer_transform_noalloc: the scratch array has no address on device %d", dev);
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return E2EG_OK;
}
}  // namespace

namespace {
// Shared by the two entry points: `ws` is the caller's workspace, or the library's static scratch
// array (static_scratch: looked up here once the arguments have passed; a need beyond its size is a
// CAPACITY error).
int32_t transform_impl(const char* who, bool static_scratch, int32_t mode, int32_t n, int32_t Fin, int32_t Fout,
                       int32_t dtype, int32_t relu, const void* d_P, const void* d_W, void* d_H, const void* d_gH,
                       void* d_gP, float* d_gW, void* ws, size_t ws_bytes, void* stream_) {
    if (mode != E2EG_TRANSFORM_FWD && mode != E2EG_TRANSFORM_BWD)
        return fail(E2EG_ERR_INVALID_ARG, "%s: mode %d", who, mode);
    if (dtype != E2EG_BF16)
        return fail(E2EG_ERR_BAD_DTYPE, "%s: only E2EG_BF16 is supported (got %d)", who, dtype);
    if (n < 0) return fail(E2EG_ERR_INVALID_ARG, "%s: negative n", who);
    if (Fin <= 0 || Fout <= 0 || Fin % 32 || Fout % 32 || Fin > kMaxF || Fout > kMaxF)
        return fail(E2EG_ERR_INVALID_ARG, "%s: Fin=%d, Fout=%d must be multiples of 32 in [32, %d]", who, Fin,
                    Fout, kMaxF);
    if (!d_P || !d_W || !d_H) return fail(E2EG_ERR_NULL_PTR, "%s: d_P, d_W or d_H is null", who);
    if (mode == E2EG_TRANSFORM_BWD && !d_gH) return fail(E2EG_ERR_NULL_PTR, "%s: d_gH is null", who);
    const void* ptrs[] = {d_P, d_W, d_H, d_gH, d_gP, d_gW};
    for (const void* q : ptrs)
        if (q && !aligned_to(q, 16)) return fail(E2EG_ERR_INVALID_ARG, "%s: a pointer is not 16-byte aligned", who);
    const size_t need = e2eg_layer_transform_workspace_bytes(mode, n, Fin, Fout, dtype);
    if (static_scratch && E2EG_TRANSFORM_STATIC_SCRATCH_BYTES < need)
        return fail(E2EG_ERR_CAPACITY, "%s: n=%d, Fin=%d, Fout=%d need %zu bytes of scratch memory, the static array "
                                       "holds %zu; use e2eg_layer_transform with a workspace", who, n, Fin, Fout, need,
                    (size_t)E2EG_TRANSFORM_STATIC_SCRATCH_BYTES);
    if (static_scratch) {   // arguments are fine: now the array's address on this device
        float* ptr = nullptr;
        const int32_t st = static_scratch_of_current_device(&ptr);
        if (st != E2EG_OK) return st;
        ws = ptr;
        ws_bytes = E2EG_TRANSFORM_STATIC_SCRATCH_BYTES;
    }
    if (!ws || !aligned_to(ws, kAlign) || ws_bytes < need)
        return fail(E2EG_ERR_WORKSPACE, "%s: workspace needs %zu bytes, 256-byte aligned", who, need);
    hipStream_t stream = static_cast<hipStream_t>(stream_);

    if (mode == E2EG_TRANSFORM_FWD) {
        if (n == 0) return E2EG_OK;
        if (relu) launch_forward<true>(d_P, d_W, d_H, n, Fin, Fout, stream);
        else launch_forward<false>(d_P, d_W, d_H, n, Fin, Fout, stream);
        E2EG_LAUNCH_CHECK("dense_forward");
        return E2EG_OK;
    }
    float* partial = d_gW ? static_cast<float*>(ws) : nullptr;
    if (n > 0 && (d_gP || d_gW)) {
        if (relu) launch_back<true>(d_P, d_W, d_H, d_gH, d_gP, partial, n, Fin, Fout, stream);
        else launch_back<false>(d_P, d_W, d_H, d_gH, d_gP, partial, n, Fin, Fout, stream);
        E2EG_LAUNCH_CHECK("dense_backward");
    }
    if (d_gW) {
        const int32_t count = Fin * Fout;
        weight_grad_reduce<<<dim3((unsigned)ceil_div(count, kReduceElems)), dim3(kReduceThreads), 0, stream>>>(
            partial, n > 0 ? back_groups(n, Fin, Fout) : 0, count, d_gW);
        E2EG_LAUNCH_CHECK("weight_grad_reduce");
    }
    return E2EG_OK;
}
}  // namespace

extern "C" int32_t e2eg_layer_transform(int32_t mode, int32_t n, int32_t Fin, int32_t Fout,
                                        int32_t dtype, int32_t relu, const void* d_P,
                                        const void* d_W, void* d_H, const void* d_gH, void* d_gP,
                                        float* d_gW, void* ws, size_t ws_bytes, void* stream) {
    return transform_impl("layer_transform", false, mode, n, Fin, Fout, dtype, relu, d_P, d_W, d_H, d_gH, d_gP, d_gW, ws,
                          ws_bytes, stream);
}

extern "C" int32_t e2eg_layer_transform_noalloc(int32_t mode, int32_t n, int32_t Fin, int32_t Fout, int32_t dtype,
                                                int32_t relu, const void* d_P, const void* d_W, void* d_H,
                                                const void* d_gH, void* d_gP, float* d_gW, void* stream) {
    // every partial matrix the reduction reads is written in full by the kernel before it, so the
    // array's old contents (the previous call's) never show and nothing has to be cleared
    return transform_impl("layer_transform_noalloc", true, mode, n, Fin, Fout, dtype, relu, d_P, d_W, d_H, d_gH, d_gP,
                          d_gW, nullptr, 0, stream);
}
