// Device-side helpers shared by the HIP sources of libgroot (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>

#include "groot_internal.h"

namespace groot {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kBlock = 256;                  // threads per workgroup (4 wavefronts)
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kLdTileRows = 64;              // consecutive rows per wavefront tile
constexpr int kLdTileCap = 512;              // non-zeros of a tile that are staged in LDS
constexpr int kXcds = 8;                     // workgroups are dealt round-robin over 8 XCDs

// Each XCD has its own L2.  Consecutive hardware workgroup ids land on
// different XCDs, so the logical block index is transposed: XCD x walks the
// x-th contiguous eighth of the tiles in ascending order.
__device__ __forceinline__ int64_t logical_block(int64_t blocks_per_xcd, int remap)
{
    int64_t b = blockIdx.x;
    return remap ? (b % kXcds) * blocks_per_xcd + b / kXcds : b;
}

// Weight of the entries of a row: kExplicit reads val[]; kMean and kOnes are
// the row-uniform weights of graphs built from an AIG and need no weight array
// (1/row length is recomputed in registers, correctly rounded, from the row
// pointer; this saves 4 bytes of HBM traffic per non-zero).
enum : int { kOnes = (int)WeightMode::Ones, kMean = (int)WeightMode::Mean, kExplicit = (int)WeightMode::Explicit };

template <int W>
__device__ __forceinline__ float row_weight(int64_t row_nnz)
{
    return W == kMean ? (row_nnz > 0 ? 1.0f / (float)row_nnz : 0.0f) : 1.0f;
}

// Sum of one row for one float4 slice: the feature slices of up to D neighbours are gathered
// before the first add (kStaged: indices/weights come from the tile's copy in LDS, else from
// global memory), accumulated in registers in CSR order, and scaled by the row weight.
template <int W, bool kStaged, int D = 8>
__device__ __forceinline__ v4f ld_row_sum(int64_t s, int64_t e, const int32_t *__restrict__ cols,
                                          const float *__restrict__ vals, const v4f *__restrict__ X,
                                          int32_t F4, int32_t ff)
{
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    for (int64_t p = s; p < e; p += D) {
        v4f x[D];
        float w[D];
#pragma unroll
        for (int k = 0; k < D; ++k) {
            if (p + k < e) {
                int32_t c = kStaged ? cols[p + k] : __builtin_nontemporal_load(&cols[p + k]);
                if (W == kExplicit) w[k] = kStaged ? vals[p + k] : __builtin_nontemporal_load(&vals[p + k]);
                x[k] = X[(int64_t)c * F4 + ff];
            }
        }
#pragma unroll
        for (int k = 0; k < D; ++k)
            if (p + k < e) {
                if (W == kExplicit) acc += w[k] * x[k];
                else acc += x[k];
            }
    }
    if (W != kExplicit) acc *= row_weight<W>(e - s);
    return acc;
}

// Rows before `row` in the ascending list of high-degree rows, found by the whole wavefront: 64 samples of what is left of
// the list per step, so two or three loads one after the other where a binary search has a dozen (at about 0.8 us each).
__device__ __forceinline__ int32_t hd_place(const int32_t *__restrict__ hd_rows, int32_t n_hd, int64_t row)
{
    const int lane = threadIdx.x % kWave;
    int32_t place = 0;
    for (int32_t len = n_hd; len > 0;) {                 // the answer lies in [place, place + len]
        const int32_t step = (len + kWave - 1) / kWave, at = lane * step;
        const int below = __popcll(__ballot(at < len && hd_rows[place + (at < len ? at : 0)] < row));
        if (below == 0) break;
        const int32_t cut = (below - 1) * step + 1;
        place += cut;
        len = step - 1 < len - cut ? step - 1 : len - cut;
    }
    return place;
}

// Sum of one row for one float4 slice with row-uniform weights, in CSR order, eight gathers in flight without a branch between
// them (an entry past the row's end reads the row of zeros).  Xf: the lane's slice of row 0; zero_off: byte distance to its
// slice of the row of zeros.
template <int W>
__device__ __forceinline__ v4f row_sum_ahead(int64_t s, int64_t e, const int32_t *__restrict__ cols, const char *__restrict__ Xf,
                                             int row_shift, int64_t zero_off)
{
    v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int64_t p = s; p < e; p += 8) {
        int64_t c[8];
        v4f x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = cols[p + k < e ? p + k : e - 1];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = *(const v4f *)(Xf + (p + k < e ? c[k] << row_shift : zero_off));
#pragma unroll
        for (int k = 0; k < 8; ++k) acc += x[k];
    }
    if (W == kMean) acc *= row_weight<kMean>(e - s);
    return acc;
}

// ---------------------------------------------------------------------------
// HD part.  One workgroup per piece of a high-degree row (the plan cuts a row
// into balanced pieces).  The 256/L lane groups of the workgroup stride over
// the piece's non-zeros, each keeping a register accumulator for its float4
// slice; the group sums meet in LDS and are added by a tree.  The result goes
// to Y (single-piece rows) or to the row's slot of partial sums.
// ---------------------------------------------------------------------------
template <int L, int W>
__device__ __forceinline__ void hd_piece(char *smem, const HdChunk ch, const int32_t *__restrict__ col,
                                         const float *__restrict__ val, const v4f *__restrict__ X,
                                         v4f *__restrict__ Y, v4f *__restrict__ partials, int32_t F4,
                                         const int64_t *__restrict__ out_ids)
{
    constexpr int G = kBlock / L;
    v4f(*s_red)[L] = (v4f(*)[L])smem;                    // [G][L]
    const int g = threadIdx.x / L, f = threadIdx.x % L;
    const int64_t end = ch.begin + ch.len;
    const float rw = row_weight<W>(ch.row_nnz);

    for (int32_t fb = 0; fb < F4; fb += L) {
        const int32_t ff = fb + f;
        const bool live = ff < F4;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        if (live) {
            int64_t p = ch.begin + g;
            for (; p + 3 * G < end; p += 4 * G) {
                int32_t c0 = col[p], c1 = col[p + G], c2 = col[p + 2 * G], c3 = col[p + 3 * G];
                v4f x0 = X[(int64_t)c0 * F4 + ff], x1 = X[(int64_t)c1 * F4 + ff];
                v4f x2 = X[(int64_t)c2 * F4 + ff], x3 = X[(int64_t)c3 * F4 + ff];
                if (W == kExplicit) {
                    acc += val[p] * x0;
                    acc += val[p + G] * x1;
                    acc += val[p + 2 * G] * x2;
                    acc += val[p + 3 * G] * x3;
                } else {
                    acc += (x0 + x1) + (x2 + x3);
                }
            }
            for (; p < end; p += G) {
                v4f x = X[(int64_t)col[p] * F4 + ff];
                if (W == kExplicit) acc += val[p] * x;
                else acc += x;
            }
            if (W != kExplicit) acc *= rw;
        }
        s_red[g][f] = acc;
        __syncthreads();
#pragma unroll
        for (int stride = G / 2; stride > 0; stride /= 2) {
            if (g < stride) s_red[g][f] += s_red[g + stride][f];
            __syncthreads();
        }
        if (g == 0 && live) {
            v4f sum = s_red[0][f];
            if (ch.slot < 0) Y[(out_ids ? out_ids[ch.row] : (int64_t)ch.row) * F4 + ff] = sum;
            else partials[(int64_t)ch.slot * F4 + ff] = sum;
        }
        __syncthreads();
    }
}

#define GROOT_DISPATCH_L(L, CALL)        \
    switch (L) {                         \
    case 1: { constexpr int kL = 1; CALL; } break;   \
    case 2: { constexpr int kL = 2; CALL; } break;   \
    case 4: { constexpr int kL = 4; CALL; } break;   \
    case 8: { constexpr int kL = 8; CALL; } break;   \
    case 16: { constexpr int kL = 16; CALL; } break; \
    case 32: { constexpr int kL = 32; CALL; } break; \
    default: { constexpr int kL = 64; CALL; } break; \
    }

#define GROOT_DISPATCH_W(W, CALL)                           \
    switch (W) {                                            \
    case kOnes: { constexpr int kW = kOnes; CALL; } break;  \
    case kMean: { constexpr int kW = kMean; CALL; } break;  \
    default: { constexpr int kW = kExplicit; CALL; } break; \
    }

// Signed byte distance between two device addresses that belong to different allocations (the row of zeros
// of a plan, seen from a feature matrix): integer arithmetic on the addresses, not a pointer difference.
inline int64_t byte_distance(const void *from, const void *to)
{
    return (int64_t)((uintptr_t)to - (uintptr_t)from);
}

inline bool grid_ok(int64_t blocks) { return blocks > 0 && blocks <= 0x7fffffffLL; }

// explicit weights need the weight array on the device; the other modes never touch it
inline bool weights_ok(const DevicePlan &dp)
{
    return dp.weight_mode == kOnes || dp.weight_mode == kMean || dp.val != nullptr || dp.nnz == 0;
}

}  // namespace groot
