// HIP kernels of libgroot for gfx950 (wave64): the low-degree and high-degree
// aggregation kernels, the reduction of split high-degree rows, and the row
// gather / scatter of the partitioned mode.
//
// Feature rows are handled as float4 slices: a row of F floats is covered by
// a "lane group" of L lanes (L = smallest power of two >= F/4, at most 64), so
// one wavefront works on 64/L rows at a time and every load/store of a group
// is one contiguous F*4-byte segment.
#include "groot_device.h"

namespace groot {

// ---------------------------------------------------------------------------
// LD part.  A wavefront owns 64 consecutive rows.  When none of them is
// high-degree and the tile's non-zeros fit, the wavefront first copies the
// tile's column indices (and weights) to LDS with fully coalesced loads; lane
// groups then walk their rows (group g takes rows g, g+G, g+2G, ...), gather
// the feature slices of all neighbours of a row before accumulating them in
// registers, and store the finished slice.  The G groups of a wavefront always
// store G consecutive rows, i.e. one contiguous G*F*4-byte area per store.
// High-degree rows are skipped (HD pieces write them).
// ---------------------------------------------------------------------------
constexpr int kLdsBytes = kWavesPerBlock * (2 * kLdTileCap + kLdTileRows + 1) * 4;

template <int L, int W>
__device__ __forceinline__ void ld_tile(char *smem, int64_t tile, const int64_t *__restrict__ rowptr,
                                        const int32_t *__restrict__ col, const float *__restrict__ val,
                                        const v4f *__restrict__ X, v4f *__restrict__ Y, int64_t n,
                                        int32_t F4, int32_t T, const int64_t *__restrict__ out_ids, int64_t n_out)
{
    constexpr int G = kWave / L;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    int32_t *s_col = (int32_t *)smem + wave * kLdTileCap;
    float *s_val = (float *)smem + (kWavesPerBlock + wave) * kLdTileCap;
    int32_t *s_rel = (int32_t *)smem + 2 * kWavesPerBlock * kLdTileCap + wave * (kLdTileRows + 1);
    const int64_t base = (tile * kWavesPerBlock + wave) * kLdTileRows;   // may lie beyond n: empty tile

    const int64_t r = base + lane;
    int64_t rp0 = 0, rp1 = 0;
    if (r < n) { rp0 = rowptr[r]; rp1 = rowptr[r + 1]; }
    const int64_t tile_begin = rowptr[base < n ? base : n];
    const int64_t tile_end = rowptr[base + kLdTileRows < n ? base + kLdTileRows : n];
    const bool any_hd = __ballot(rp1 - rp0 >= T) != 0;
    const bool staged = !any_hd && (tile_end - tile_begin) <= kLdTileCap;

    if (staged) {
        const int m = (int)(tile_end - tile_begin);
        s_rel[lane] = (r < n) ? (int32_t)(rp0 - tile_begin) : m;
        if (lane == 0) s_rel[kLdTileRows] = m;
        for (int p = lane; p < m; p += kWave) {
            s_col[p] = __builtin_nontemporal_load(&col[tile_begin + p]);
            if (W == kExplicit) s_val[p] = __builtin_nontemporal_load(&val[tile_begin + p]);
        }
    }
    __syncthreads();

    const int g = lane / L, f = lane % L;
    for (int it = 0; it < kLdTileRows / G; ++it) {
        const int lr = it * G + g;
        const int64_t row = base + lr;
        if (row >= n_out) break;                         // n_out <= n: rows past it are not wanted
        const int64_t orow = out_ids ? out_ids[row] : row;
        if (staged) {
            const int64_t s = s_rel[lr], e = s_rel[lr + 1];
            for (int32_t ff = f; ff < F4; ff += L) {
                v4f acc = ld_row_sum<W, true>(s, e, s_col, s_val, X, F4, ff);
                __builtin_nontemporal_store(acc, &Y[orow * F4 + ff]);
            }
        } else {
            const int64_t s = rowptr[row], e = rowptr[row + 1];
            if (e - s >= T) continue;
            for (int32_t ff = f; ff < F4; ff += L) {
                v4f acc = ld_row_sum<W, false>(s, e, col, val, X, F4, ff);
                __builtin_nontemporal_store(acc, &Y[orow * F4 + ff]);
            }
        }
    }
}

// Block t of the LD launch computes the tile of rows [256 t, 256 t + 256).
template <int L, int W>
__global__ __launch_bounds__(kBlock) void ld_kernel(const int64_t *__restrict__ rowptr,
                                                    const int32_t *__restrict__ col,
                                                    const float *__restrict__ val,
                                                    const v4f *__restrict__ X, v4f *__restrict__ Y,
                                                    int64_t n, int32_t F4, int32_t T, int64_t n_tiles,
                                                    int64_t blocks_per_xcd, int remap,
                                                    const int64_t *__restrict__ out_ids, int64_t n_out)
{
    __shared__ __align__(16) char smem[kLdsBytes];
    const int64_t tile = logical_block(blocks_per_xcd, remap);
    if (tile >= n_tiles) return;
    ld_tile<L, W>(smem, tile, rowptr, col, val, X, Y, n, F4, T, out_ids, n_out);
}

// One workgroup per piece.  The pieces stand in the order of their first column, so neighbours in the list gather from the
// same stretch of X; consecutive workgroups land on different XCDs, each with an L2 of its own.  run > 1: the list is dealt
// to the XCDs in runs of that many pieces.
template <int L, int W>
__global__ __launch_bounds__(kBlock) void hd_kernel(const HdChunk *__restrict__ chunks,
                                                    const int32_t *__restrict__ col,
                                                    const float *__restrict__ val,
                                                    const char *__restrict__ X, int64_t zero_off,
                                                    v4f *__restrict__ Y, v4f *__restrict__ partials, int32_t F4,
                                                    const int64_t *__restrict__ out_ids, int64_t n_out, int64_t n_chunks,
                                                    int32_t run)
{
    __shared__ __align__(16) char smem[kHdSmemBytes<L>];
    int64_t piece = blockIdx.x;
    if (run > 1) {
        const int64_t k = blockIdx.x / kXcds;            // the XCD's k-th workgroup
        piece = (k / run * kXcds + blockIdx.x % kXcds) * run + k % run;
        if (piece >= n_chunks) return;                   // the whole workgroup
    }
    const HdChunk ch = chunks[piece];
    if (ch.row >= n_out) return;                         // the whole workgroup: a row that is not wanted
    hd_piece<L, W>(smem, ch, col, val, X, zero_off, Y, partials, F4, out_ids);
}

// Y[row] = partials[first] + ... + partials[first+count-1], in that order.
template <int L>
__global__ __launch_bounds__(kBlock) void hd_finish_kernel(const HdSplitRow *__restrict__ rows,
                                                           int64_t n_rows,
                                                           const v4f *__restrict__ partials,
                                                           v4f *__restrict__ Y, int32_t F4,
                                                           const int64_t *__restrict__ out_ids, int64_t n_out)
{
    constexpr int G = kBlock / L;
    const int64_t k = (int64_t)blockIdx.x * G + threadIdx.x / L;
    if (k >= n_rows) return;
    const HdSplitRow sr = rows[k];
    if (sr.row >= n_out) return;
    hd_finish_row<L>(sr, partials, Y, F4, out_ids, threadIdx.x % L);
}

// out[i] = X[ids[i]]  (kScatter = false)   or   Y[ids[i]] = in[i]  (kScatter = true)
template <int L, bool kScatter>
__global__ __launch_bounds__(kBlock) void rows_move_kernel(const int64_t *__restrict__ ids, int64_t n,
                                                           const v4f *__restrict__ src,
                                                           v4f *__restrict__ dst, int32_t F4)
{
    constexpr int G = kBlock / L;
    const int64_t i = (int64_t)blockIdx.x * G + threadIdx.x / L;
    if (i >= n) return;
    const int64_t id = ids[i];
    for (int32_t ff = threadIdx.x % L; ff < F4; ff += L) {
        if (kScatter) dst[id * F4 + ff] = src[i * F4 + ff];
        else dst[i * F4 + ff] = src[id * F4 + ff];
    }
}

// col[p] = ids[col[p]]: the columns of a part's sub-graph renamed from local ids to rows of the whole graph
__global__ __launch_bounds__(kBlock) void col_map_kernel(int32_t *__restrict__ col, int64_t nnz,
                                                         const int64_t *__restrict__ ids)
{
    for (int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * kBlock)
        col[p] = (int32_t)ids[col[p]];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static int lanes_for(int32_t F4)
{
    int L = 1;
    while (L < F4 && L < kWave) L *= 2;
    return L;
}

#define GROOT_DISPATCH_LW(L, W, CALL)                                  \
    switch (W) {                                                       \
    case kOnes: { constexpr int kW = kOnes; GROOT_DISPATCH_L(L, CALL) } break; \
    case kMean: { constexpr int kW = kMean; GROOT_DISPATCH_L(L, CALL) } break; \
    default: { constexpr int kW = kExplicit; GROOT_DISPATCH_L(L, CALL) } break; \
    }

// The pipelined kernel serves the leading rows of a graph at F = 32, 64 and 128, whole graphs also at the widths between:
// from 20 on with 5 slots per row (512-bit multiplier, plain against pipelined kernel: F = 16 107 and 105 us with more than
// twice the time at 8, F = 20 145 and 122, F = 100 ... 200 a quarter less), from 36 on with 6 to 8 (shape mapped to cells, rows
// of 6: F = 20 50 and 56 us, F = 28 54 and 60; 4-LUT shape: F = 20 55 and 62, F = 36 88 and 88, F = 124 257 and 233), up to 256
// (64 lanes of one float4).  Below F = 32 a graph of middling size without high-degree rows, whose launches it would share, stays
// on the plain kernel (rows of 4 and 5, F = 28: 65,536 rows 13.7 and 12.1 us, 131,072 15.0 and 18.1, 262,144 20.0 and 20.9, 524,288
// 41.6 and 36.4).
static bool ld_pipelined(const DevicePlan &dp, int32_t F4, const RowOut *out)
{
    if (!dp.zero_row || !dp.ld_pipelined) return false;
    if (F4 == 8 || F4 == 16 || F4 == 32) return true;
    if (out || F4 > kWave || F4 <= 4) return false;
    if (F4 > 8) return true;
    return dp.pipe_depth <= 5 && (dp.n_chunks > 0 || dp.n <= 65536 || dp.n >= 524288);
}

// Whether the pieces of the high-degree rows join the low-degree rows' launch.  In the same launch / in one of their own, us:
//   F = 32: 374 pieces (polarized) 13.6 / 17.4, 512 (256-bit multiplier) 32.2 / 33.6, 646 (Booth) 24.8 / 25.9, 757 (polarized)
//     18.8 / 18.5, 949 (polarized) 19.4 / 17.8, 1,024 (multiplier) 34.7 / 33.0, (4-LUT shape) 26.7 / 23.3
//   F = 64: 757 20.8 / 26.5, 949 20.0 / 25.0, 1,024 (multiplier) 48.8 / 52.6, (4-LUT shape, one copy) 33.2 / 31.6, (four) 30.8 / 33.1;
//     2,048 (4-LUT shape) 56.3 / 53.1, (mapped to cells) 70.8 / 66.7, 2,099 (polarized) 36.9 / 41.0
//   F = 100: 512 73.8 / 77.2, 646 48.7 / 56.0, 757 27.3 / 32.5, 1,024 (4-LUT shape) 46.3 / 46.4, (mapped to cells) 57.5 / 59.9: the
//     pieces would gain up to 1,024 here, too; the line is from pieces whose indices were not staged (949 61.1 / 46.9)
//   F = 128, 200: 771 (Booth) 137 / 149, 238 / 250; 1,024 (4-LUT shape) 48.3 / 49.8, 72.8 / 75.0; more than 1,024 (polarized, beside
//     dense rows) 55.3 / 51.6, 92.4 / 81.5
bool ld_takes_hd(const DevicePlan &dp, int32_t F, const RowOut *out)
{
    const int64_t few = F == 64 || F >= 128 ? 1024 : 512;
    return ld_pipelined(dp, F / 4, out) && dp.n_chunks > 0 && dp.n_chunks <= few;
}

int launch_ld(const DevicePlan &dp, const float *X, float *Y, int32_t F, void *stream, const RowOut *out, bool with_hd)
{
    const int32_t F4 = F / 4;
    const int64_t *out_ids = out ? out->ids : nullptr;
    const int64_t n_out = out ? out->n_out : dp.n;
    if (ld_pipelined(dp, F4, out)) return launch_ld_pipelined(dp, X, Y, F, stream, out, with_hd);
    if (with_hd) return (int)hipErrorInvalidValue;
    const int64_t n_tiles = (n_out + kRowsPerLdTile - 1) / kRowsPerLdTile;
    if (n_tiles == 0) return 0;
    const int64_t per_xcd = (n_tiles + kXcds - 1) / kXcds;
    const int remap = dp.xcd_remap && n_tiles >= 4 * kXcds;
    const int64_t grid = remap ? per_xcd * kXcds : n_tiles;
    if (!grid_ok(grid)) return (int)hipErrorInvalidConfiguration;
    if (!weights_ok(dp)) return (int)hipErrorInvalidValue;
    hipStream_t st = (hipStream_t)stream;
    GROOT_DISPATCH_LW(lanes_for(F4), dp.weight_mode,
                      (ld_kernel<kL, kW><<<dim3((unsigned)grid), dim3(kBlock), 0, st>>>(
                          dp.rowptr, dp.col, dp.val, (const v4f *)X, (v4f *)Y, dp.n, F4, dp.threshold, n_tiles,
                          per_xcd, remap, out_ids, n_out)));
    return (int)hipGetLastError();
}

int launch_hd(const DevicePlan &dp, const float *X, float *Y, int32_t F, void *stream, const RowOut *out)
{
    const int32_t F4 = F / 4;
    const int64_t *out_ids = out ? out->ids : nullptr;
    const int64_t n_out = out ? out->n_out : dp.n;
    if (!weights_ok(dp) || !dp.zero_row) return (int)hipErrorInvalidValue;
    hipStream_t st = (hipStream_t)stream;
    // Runs of 64 pieces from F = 64 on, where a stretch of X is large beside an L2.  Whole step, us, with runs / without: polarized
    // graphs, every row of X gathered 40 to 70 times, explicit weights (with others most such pieces are dense rows): 2,905 pieces
    // F = 64 40.9 / 44.8, F = 128 56.3 / 76.3, F = 256 106 / 157; 37,634 pieces F = 128 479 / 485, F = 256 992 / 1,097.  Multipliers,
    // whose rows are gathered once or twice, the same (2,048 pieces, F = 64 235.6 / 235.7); 6,329 pieces of shorter rows F = 128
    // 194 / 189.  Below the line one or the other: 757 pieces F = 128 41.3 / 33.2, 374 20.3 / 23.2.
    const int32_t run = F4 >= 16 && dp.n_chunks >= 2048 ? 64 : 1;
    const int64_t grid = run > 1 ? (dp.n_chunks + kXcds * run - 1) / (kXcds * run) * (kXcds * run) : dp.n_chunks;
    if (!grid_ok(grid)) return (int)hipErrorInvalidConfiguration;
    GROOT_DISPATCH_LW(lanes_for(F4), dp.weight_mode,
                      (hd_kernel<kL, kW><<<dim3((unsigned)grid), dim3(kBlock), 0, st>>>(
                          dp.chunks, dp.col, dp.val, (const char *)X, byte_distance(X, dp.zero_row), (v4f *)Y,
                          (v4f *)dp.partials, F4, out_ids, n_out, dp.n_chunks, run)));
    return (int)hipGetLastError();
}

int launch_hd_finish(const DevicePlan &dp, float *Y, int32_t F, void *stream, const RowOut *out)
{
    const int32_t F4 = F / 4;
    const int64_t *out_ids = out ? out->ids : nullptr;
    const int64_t n_out = out ? out->n_out : dp.n;
    const int L = lanes_for(F4);
    const int64_t grid = (dp.n_split_rows + kBlock / L - 1) / (kBlock / L);
    if (!grid_ok(grid)) return (int)hipErrorInvalidConfiguration;
    hipStream_t st = (hipStream_t)stream;
    GROOT_DISPATCH_L(L, (hd_finish_kernel<kL><<<dim3((unsigned)grid), dim3(kBlock), 0, st>>>(
                            dp.split_rows, dp.n_split_rows, (const v4f *)dp.partials, (v4f *)Y, F4, out_ids, n_out)));
    return (int)hipGetLastError();
}

int launch_col_map(int32_t *col, int64_t nnz, const int64_t *ids, void *stream)
{
    if (nnz <= 0) return 0;
    int64_t grid = (nnz + kBlock - 1) / kBlock;
    if (grid > 65536) grid = 65536;                      // grid-stride loop
    col_map_kernel<<<dim3((unsigned)grid), dim3(kBlock), 0, (hipStream_t)stream>>>(col, nnz, ids);
    return (int)hipGetLastError();
}

int launch_rows_gather(const int64_t *ids, int64_t n, const float *X, float *out, int32_t F, void *stream)
{
    const int32_t F4 = F / 4;
    const int L = lanes_for(F4);
    const int64_t grid = (n + kBlock / L - 1) / (kBlock / L);
    if (!grid_ok(grid)) return (int)hipErrorInvalidConfiguration;
    hipStream_t st = (hipStream_t)stream;
    GROOT_DISPATCH_L(L, (rows_move_kernel<kL, false><<<dim3((unsigned)grid), dim3(kBlock), 0, st>>>(
                            ids, n, (const v4f *)X, (v4f *)out, F4)));
    return (int)hipGetLastError();
}

int launch_rows_scatter(const int64_t *ids, int64_t n, const float *in, float *Y, int32_t F, void *stream)
{
    const int32_t F4 = F / 4;
    const int L = lanes_for(F4);
    const int64_t grid = (n + kBlock / L - 1) / (kBlock / L);
    if (!grid_ok(grid)) return (int)hipErrorInvalidConfiguration;
    hipStream_t st = (hipStream_t)stream;
    GROOT_DISPATCH_L(L, (rows_move_kernel<kL, true><<<dim3((unsigned)grid), dim3(kBlock), 0, st>>>(
                            ids, n, (const v4f *)in, (v4f *)Y, F4)));
    return (int)hipGetLastError();
}

const char *hip_error_text(int err) { return hipGetErrorString((hipError_t)err); }

int dev_upload(void *dst, const void *src, size_t bytes)
{
    return (int)hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice);
}

}  // namespace groot
