// Device-side helpers shared by the HIP sources of libgroot (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "groot_internal.h"

namespace groot {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kBlock = 256;                  // threads per workgroup (4 wavefronts)
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kLdTileRows = 64;              // consecutive rows per wavefront tile
constexpr int kLdTileCap = 512;              // non-zeros of a tile that are staged in LDS
constexpr int kXcds = 8;                     // workgroups are dealt round-robin over 8 XCDs

// Orders a wavefront's own accesses to its part of LDS: no other wavefront reads or writes it.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

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
// them (an entry past the row's end reads the row of zeros), the next eight columns beside them: a row of 31 entries is five
// latencies, with its columns fetched when they were needed eight.  Xf: the lane's slice of row 0; zero_off: byte distance to its
// slice of the row of zeros.
template <int W>
__device__ __forceinline__ v4f row_sum_ahead(int64_t s, int64_t e, const int32_t *__restrict__ cols, const char *__restrict__ Xf,
                                             int row_shift, int64_t zero_off)
{
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    if (s >= e) return acc;
    int32_t c[8];
    auto fetch = [&](int64_t p) {
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = cols[p + k < e ? p + k : e - 1];
    };
    fetch(s);
#pragma unroll 1
    for (int64_t p = s; p < e; p += 8) {
        v4f x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = *(const v4f *)(Xf + (p + k < e ? (int64_t)c[k] << row_shift : zero_off));
        if (p + 8 < e) fetch(p + 8);
#pragma unroll
        for (int k = 0; k < 8; ++k) acc += x[k];
    }
    if (W == kMean) acc *= row_weight<kMean>(e - s);
    return acc;
}

// ---------------------------------------------------------------------------
// HD part.  One workgroup per piece of a high-degree row (the plan cuts a row
// into balanced pieces).  Its 256/L lane groups stride over the piece's entries,
// up to 8 gathers in flight each and no branch between them, with a register
// accumulator per float4 slice: the byte offsets of the rows of X (and the
// weights) have been put to LDS by the group's own wavefront, padded with the
// row of zeros.  The group sums meet in LDS and are added by a tree.  The result
// goes to Y (single-piece rows) or to the row's slot of partial sums.
//
// Where the pieces are few, latencies one after the other bound this: the form
// before (every lane group fetched its own four indices, then their rows, again
// and again) had 2 x 16 of them for a piece of 512 entries at F = 128, this one
// has 2 + 8.  Polarized graphs, us before / now: 374 pieces F = 128 23.2 / 18.1,
// 949 F = 64 26.2 / 20.6, F = 128 39.0 / 31.1; 4-LUT shape, 1,024 pieces, F = 64
// 39.5 / 36.5.  Where they are many it is the vector memory units' return path:
// 37,634 pieces F = 128 453 / 420, the offsets no longer computed lane by lane.
// Rows of 33 and 65 entries take what they took.  Entries meet in the order that
// they had (by lane group, four at a time, then the tree), so results have the
// same bits (at F = 4 for pieces of up to 768 entries: no four of a lane group's).
// ---------------------------------------------------------------------------
// gathers of a lane group in flight: no more than a usual piece of 512 entries has for it (F = 4, 18 M entries: with 8 it
// was 119 us, now 69)
constexpr int hd_ahead(int L) { return L >= 4 ? 8 : 2 * L; }
constexpr int hd_slots(int) { return 128; }  // entries of a wavefront that are staged at a time
template <int L>
constexpr int kHdSmemBytes = kWavesPerBlock * hd_slots(L) * 12 + kBlock * 16;

template <int L, int W>
__device__ __forceinline__ void hd_piece(char *smem, const HdChunk ch, const int32_t *__restrict__ col,
                                         const float *__restrict__ val, const char *__restrict__ X, int64_t zero_off,
                                         v4f *__restrict__ Y, v4f *__restrict__ partials, int32_t F4,
                                         const int64_t *__restrict__ out_ids)
{
    constexpr int G = kBlock / L, GW = kWave / L;        // lane groups of the workgroup and of a wavefront
    constexpr int kSlots = hd_slots(L), kRun = kSlots / GW, kHdAhead = hd_ahead(L);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    int64_t *const s_off = (int64_t *)smem + wave * kSlots;
    float *const s_val = (float *)(smem + kWavesPerBlock * kSlots * 8) + wave * kSlots;
    v4f *const s_red = (v4f *)(smem + kWavesPerBlock * kSlots * 12);      // [G][L]
    const int gw = lane / L, f = lane % L;
    const float rw = row_weight<W>(ch.row_nnz);

#pragma unroll 1
    for (int32_t fb = 0; fb < F4; fb += L) {
        const int32_t ff = fb + f;
        const bool live = ff < F4;
        const char *const Xf = X + 16 * ff;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int32_t s = 0; s < ch.len; s += kRun * G) {
            // entry k G + (lane group) of what is left belongs to the group's step k
            const int32_t left = ch.len - s, steps = left < kRun * G ? (left + G - 1) / G : kRun;
            if (s || fb) wave_sync();                    // the run before has been read
            int32_t c[kSlots / kWave];
            float v[kSlots / kWave];
#pragma unroll
            for (int h = 0; h < kSlots / kWave; ++h) {   // past the end: the last entry again, its offset is not used
                const int i = lane + h * kWave, e = i / GW * G + wave * GW + i % GW;
                const int64_t p = ch.begin + s + (e < left ? e : left - 1);
                c[h] = col[p];
                if (W == kExplicit) v[h] = val[p];
            }
#pragma unroll
            for (int h = 0; h < kSlots / kWave; ++h) {
                const int i = lane + h * kWave, e = i / GW * G + wave * GW + i % GW;
                s_off[i] = e < left ? (int64_t)c[h] * (F4 * 16) : zero_off;
                if (W == kExplicit) s_val[i] = e < left ? v[h] : 0.f;
            }
            wave_sync();
            if (!live) continue;                         // idle lanes cost the vector memory units time, too
#pragma unroll 1
            for (int32_t k0 = 0; k0 < steps; k0 += kHdAhead) {
                v4f x[kHdAhead];
                float w[kHdAhead];
#pragma unroll
                for (int k = 0; k < kHdAhead; ++k) {
                    x[k] = *(const v4f *)(Xf + s_off[(k0 + k) * GW + gw]);
                    if (W == kExplicit) w[k] = s_val[(k0 + k) * GW + gw];
                }
                if (W == kExplicit) {
#pragma unroll
                    for (int k = 0; k < kHdAhead; ++k) acc += w[k] * x[k];
                } else if constexpr (kHdAhead < 4) {
#pragma unroll
                    for (int k = 0; k < kHdAhead; ++k) acc += x[k];
                } else if ((k0 + kHdAhead) * G <= left) {
#pragma unroll
                    for (int k = 0; k < kHdAhead; k += 4) acc += (x[k] + x[k + 1]) + (x[k + 2] + x[k + 3]);
                } else {                                 // four entries at a time while there are four, the rest one by one
#pragma unroll
                    for (int k = 0; k < kHdAhead; k += 4) {
                        const v4f four = acc + ((x[k] + x[k + 1]) + (x[k + 2] + x[k + 3]));
                        const v4f fewer = ((acc + x[k]) + x[k + 1]) + x[k + 2];
                        acc = (k0 + k + 3) * G + wave * GW + gw < left ? four : fewer;
                    }
                }
            }
        }
        if (W != kExplicit) acc *= rw;
        s_red[threadIdx.x] = acc;
        __syncthreads();
        if (wave == 0) {
            v4f sum = (s_red[lane] + s_red[lane + 2 * kWave]) + (s_red[lane + kWave] + s_red[lane + 3 * kWave]);
#pragma unroll
            for (int off = kWave / 2; off >= L; off /= 2)
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[c] += __shfl_down(sum[c], off);
            if (gw == 0 && live) {
                if (ch.slot < 0) Y[(out_ids ? out_ids[ch.row] : (int64_t)ch.row) * F4 + ff] = sum;
                else partials[(int64_t)ch.slot * F4 + ff] = sum;
            }
        }
        if (fb + L < F4) __syncthreads();
    }
}

// Y[row] = partials[first] + ... + partials[first+count-1], in that order: lane f of the L lanes of a row.
template <int L>
__device__ __forceinline__ void hd_finish_row(const HdSplitRow sr, const v4f *__restrict__ partials, v4f *__restrict__ Y,
                                              int32_t F4, const int64_t *__restrict__ out_ids, int f)
{
    const int64_t orow = out_ids ? out_ids[sr.row] : (int64_t)sr.row;
    for (int32_t ff = f; ff < F4; ff += L) {
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        const v4f *p = partials + (int64_t)sr.first * F4 + ff;
        int32_t c = 0;
        for (; c + 8 <= sr.count; c += 8, p += 8 * (int64_t)F4) {   // eight loads in flight: a row may have hundreds of pieces
            v4f x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = p[i * (int64_t)F4];
#pragma unroll
            for (int i = 0; i < 8; ++i) acc += x[i];
        }
        for (; c < sr.count; ++c, p += F4) acc += *p;
        Y[orow * F4 + ff] = acc;
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
