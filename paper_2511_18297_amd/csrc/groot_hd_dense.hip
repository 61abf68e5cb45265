// High-degree rows that hold a large part of all columns, as a dense product on the matrix cores (gfx950).
//
// A gather of a feature row for every stored entry reads a row of X as often as high-degree rows name it: on the
// polarized graph of 262,144 rows 70 times, 9.5 GB at F = 128, and the vector memory units return no more than 23 TB/s
// (hd_kernel 380 us).  261 of its rows hold 22 % of all columns each, 83 % of the entries of the high-degree rows.  With
// row-uniform weights the sum of such a row is a product of a row of zeros and ones with X: 16, 32 or 64 rows at a time,
// v_mfma_f32_16x16x4_f32, the zeros and ones expanded from one bit per column, X read once per 64 rows straight into the
// instruction's operand layout.  Products with 1 are exact and the sums are fp32, as they were.
//
// The fp32 matrix instruction does 16 rows x 16 features x 4 columns in 32 cycles, the gathers 41 bytes per cycle and CU:
// a row is cheaper here from about 7 % of the columns on (choose_dense_rows).  One workgroup per CU multiplies, which keeps its
// matrix cores busy; the other high-degree rows' pieces, in the same launch, take the memory system beside it (220 us together at
// F = 128, 156 of them matrix instructions; as two launches 155 + 96; with two workgroups per CU, which leave the pieces no
// room, 252).
//
// 0 x infinity is not 0: where X holds a number that is not finite, rows without that column would get NaN.  A row whose
// sums do not all come out finite is therefore summed again from its entries by the finishing kernel.
#include "groot_device.h"

namespace groot {

constexpr int kDenseUnit = 32;               // columns per step of the loop: eight instructions a row block and feature block
constexpr int kDenseTile = 64;               // features of a workgroup

struct DenseArgs {
    const HdChunk *rows;                     // [n_rows] the whole row as one piece, slot -1
    const uint32_t *mask;                    // [unit / 4][padded row][k < 4]: bit 8 (unit % 4) + j is the unit's column 4 j + k
    float *partials;                         // [k_parts][padded rows][F]
    int32_t n_rows, tile_rows, padded;       // padded: n_rows in whole tiles
    int32_t row_tiles, f_tiles, k_parts;
    int64_t n_units;                         // columns in units of kDenseUnit
    int64_t n_wg;                            // row_tiles x f_tiles x k_parts
};

// First column of a unit: the last one is moved back to end with the last column (there are kDenseUnit columns or more) and
// has bits for those only that the unit before has not.
__device__ __forceinline__ int64_t dense_first_column(int64_t u, int64_t n_units, int64_t n_cols)
{
    return u == n_units - 1 ? n_cols - kDenseUnit : u * kDenseUnit;
}

// One wavefront's part of a tile of 16 MB rows x 16 NV features: columns of the units [u0, u1).
// Lane layout of the instruction: A row and B column are lane % 16, k is lane / 16; D rows are 4 (lane / 16) + r.  Component
// v of the lane's NV features is the operand whose column m is feature NV m + v, so a lane's load of consecutive features
// serves NV instructions as it is.  fp32 matrix and vector instructions of a SIMD do not overlap and changing between them costs
// cycles, so the loop has next to no address arithmetic (a scalar base and constant offsets) and expands the bits of MB
// instructions' rows, then issues their MB NV instructions: with
// addresses per lane and the bits expanded as the compiler placed them the polarized graph took 195 us, now 155.
template <int MB, int NV>
__device__ __forceinline__ void dense_sum(v4f (&acc)[MB][NV], const DenseArgs &d, const char *__restrict__ X, int32_t feature,
                                          int64_t row_bytes, int64_t n_cols, int32_t row0, int64_t u0, int64_t u1)
{
    typedef float vN __attribute__((ext_vector_type(NV)));
    const int lane = threadIdx.x % kWave, m = lane % 16, k4 = lane / 16;
    uint32_t x_at[8], bits_at[MB];
#pragma unroll
    for (int j = 0; j < 8; ++j) x_at[j] = (uint32_t)((4 * j + k4) * (int)row_bytes + 4 * feature);
#pragma unroll
    for (int b = 0; b < MB; ++b) bits_at[b] = (uint32_t)((row0 + 16 * b + m) * 16 + k4 * 4);
    auto load = [&](int64_t u, vN (&x)[8], uint32_t (&w)[MB]) {
        const char *const base = X + dense_first_column(u, d.n_units, n_cols) * row_bytes;
        const uint8_t *const bits = (const uint8_t *)d.mask + (u / 4) * d.padded * 16 + u % 4;
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = *(const vN *)(base + x_at[j]);
#pragma unroll
        for (int b = 0; b < MB; ++b) w[b] = bits[bits_at[b]];
    };
    auto multiply = [&](const vN (&x)[8], const uint32_t (&w)[MB]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float a[MB];
#pragma unroll
            for (int b = 0; b < MB; ++b) a[b] = __builtin_bit_cast(float, __builtin_amdgcn_sbfe(w[b], j, 1) & 0x3f800000);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int v = 0; v < NV; ++v) acc[b][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b], x[j][v], acc[b][v], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    vN xa[8], xb[8];
    uint32_t wa[MB], wb[MB];
    load(u0, xa, wa);
#pragma unroll 1
    for (int64_t u = u0; u < u1; u += 2) {               // one unit is multiplied while the next is on its way
        load(u + 1 < u1 ? u + 1 : u, xb, wb);
        __builtin_amdgcn_sched_barrier(0);               // the compiler would sink the loads to their use
        multiply(xa, wa);
        load(u + 2 < u1 ? u + 2 : u, xa, wa);
        __builtin_amdgcn_sched_barrier(0);
        if (u + 1 < u1) multiply(xb, wb);
    }
}

// The four wavefronts of a workgroup share a tile and split its columns; their sums meet in LDS, (0 + 2) + (1 + 3).
template <int MB, int NV>
__device__ __forceinline__ void dense_tile(v4f *s_sum, const DenseArgs &d, const char *__restrict__ X, int32_t F, int64_t n_cols,
                                           int32_t row_tile, int32_t f0, int32_t k_part)
{
    typedef float vN __attribute__((ext_vector_type(NV)));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave, m = lane % 16;
    const int f = f0 + NV * m;
    v4f acc[MB][NV];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[b][v] = v4f{0.f, 0.f, 0.f, 0.f};
    const int64_t parts = (int64_t)d.k_parts * kWavesPerBlock, part = (int64_t)k_part * kWavesPerBlock + wave;
    const int64_t u0 = d.n_units * part / parts, u1 = d.n_units * (part + 1) / parts;
    if (u0 < u1)
        dense_sum<MB, NV>(acc, d, X, f < F - NV ? f : F - NV, (int64_t)F * 4, n_cols, row_tile * d.tile_rows, u0, u1);
#pragma unroll
    for (int half = 2; half > 0; half /= 2) {
        v4f *const to = s_sum + (wave - half) * MB * NV * kWave, *const from = s_sum + wave * MB * NV * kWave;
        if (half < 2) __syncthreads();
        if (wave >= half && wave < 2 * half) {
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int v = 0; v < NV; ++v) to[(b * NV + v) * kWave + lane] = acc[b][v];
        }
        __syncthreads();
        if (wave < half) {
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int v = 0; v < NV; ++v) acc[b][v] += from[(b * NV + v) * kWave + lane];
        }
    }
    if (wave == 0 && f < F) {
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                vN out;
#pragma unroll
                for (int v = 0; v < NV; ++v) out[v] = acc[b][v][r];
                const int64_t row = (int64_t)k_part * d.padded + row_tile * d.tile_rows + 16 * b + 4 * (lane / 16) + r;
                *(vN *)(d.partials + row * F + f) = out;
            }
    }
}

// Workgroups [0, d.n_wg): the dense rows.  The ones behind: the pieces of the other high-degree rows, which the memory system
// serves meanwhile.
template <int MB, int L, int W>
__global__ __launch_bounds__(kBlock, 3) void hd_dense_kernel(const DenseArgs d, const HdChunk *__restrict__ chunks,
                                                          const int32_t *__restrict__ col, const char *__restrict__ X,
                                                          int64_t zero_off, v4f *__restrict__ Y, v4f *__restrict__ partials,
                                                          int32_t F4, int64_t n_cols)
{
    constexpr int kSums = 2 * MB * 4 * kWave * 16, kPiece = kHdSmemBytes<L>;
    __shared__ __align__(16) char smem[kSums > kPiece ? kSums : kPiece];
    if (blockIdx.x >= d.n_wg) {
        hd_piece<L, W>(smem, chunks[blockIdx.x - d.n_wg], col, nullptr, X, zero_off, Y, partials, F4, nullptr);
        return;
    }
    const int32_t t = (int32_t)blockIdx.x, row_tile = t % d.row_tiles, f_tile = t / d.row_tiles % d.f_tiles;
    const int32_t k_part = t / d.row_tiles / d.f_tiles, F = 4 * F4;
    if (F - f_tile * kDenseTile > kDenseTile / 2)
        dense_tile<MB, 4>((v4f *)smem, d, X, F, n_cols, row_tile, f_tile * kDenseTile, k_part);
    else
        dense_tile<MB, 2>((v4f *)smem, d, X, F, n_cols, row_tile, f_tile * kDenseTile, k_part);
}

// Workgroups [0, d.n_rows): one dense row each, the sums of its column parts and its weight; a row with a sum that is not
// finite is computed from its entries.  The ones behind: the split rows among the others, as in hd_finish_kernel.
template <int L, int W>
__global__ __launch_bounds__(kBlock) void hd_dense_finish_kernel(const DenseArgs d, const HdSplitRow *__restrict__ split,
                                                                 int64_t n_split, const v4f *__restrict__ partials,
                                                                 const int32_t *__restrict__ col, const char *__restrict__ X,
                                                                 int64_t zero_off, v4f *__restrict__ Y, int32_t F4)
{
    constexpr int G = kBlock / L;
    __shared__ __align__(16) char smem[kHdSmemBytes<L>];
    const int g = threadIdx.x / L, f = threadIdx.x % L;
    if (blockIdx.x >= d.n_rows) {
        const int64_t k = (int64_t)(blockIdx.x - d.n_rows) * G + g;
        if (k < n_split) hd_finish_row<L>(split[k], partials, Y, F4, nullptr, f);
        return;
    }
    const HdChunk row = d.rows[blockIdx.x];
    const float rw = row_weight<W>(row.row_nnz);
    v4f *const s_red = (v4f *)smem;                      // [G][L]
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;                     // a barrier lies between this and every use
#pragma unroll 1
    for (int32_t fb = 0; fb < F4; fb += L) {
        const int32_t ff = fb + f;
        const bool live = ff < F4;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        const v4f *p = (const v4f *)d.partials + (int64_t)blockIdx.x * F4 + (live ? ff : 0);
        const int64_t step = (int64_t)d.padded * F4;
        int32_t k = g;
        for (; k + 3 * G < d.k_parts; k += 4 * G) {
            const v4f x0 = p[k * step], x1 = p[(k + G) * step], x2 = p[(k + 2 * G) * step], x3 = p[(k + 3 * G) * step];
            acc += (x0 + x1) + (x2 + x3);
        }
        for (; k < d.k_parts; k += G) acc += p[k * step];
        s_red[threadIdx.x] = acc;
        __syncthreads();
#pragma unroll
        for (int stride = G / 2; stride > 0; stride /= 2) {
            if (g < stride) s_red[threadIdx.x] += s_red[threadIdx.x + stride * L];
            __syncthreads();
        }
        if (g == 0 && live) {
            const v4f sum = s_red[f] * rw;
            if (!(isfinite(sum[0]) && isfinite(sum[1]) && isfinite(sum[2]) && isfinite(sum[3]))) s_bad = 1;
            Y[(int64_t)row.row * F4 + ff] = sum;
        }
        __syncthreads();
    }
    if (s_bad) hd_piece<L, W>(smem, row, col, nullptr, X, zero_off, Y, (v4f *)d.partials, F4, nullptr);   // slot -1: to Y
}

// the four mask words of row r and units 4 b .. 4 b + 3, one thread each; padding rows get zeros
__global__ __launch_bounds__(kBlock) void dense_mask_kernel(const HdChunk *__restrict__ rows, int32_t n_rows, int32_t padded,
                                                            const int32_t *__restrict__ col, int64_t n_cols, int64_t n_units,
                                                            uint4 *__restrict__ mask)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t b = i / padded;
    const int32_t r = (int32_t)(i % padded);
    if (4 * b >= n_units) return;
    uint32_t w[4] = {0, 0, 0, 0};
    if (r < n_rows) {
        const HdChunk row = rows[r];
        const int32_t *const c = col + row.begin;
        const int64_t first = b * 4 * kDenseUnit;
        int32_t lo = 0, hi = row.len;                    // first entry with a column >= first
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo) / 2;
            if (c[mid] < first) lo = mid + 1; else hi = mid;
        }
        for (; lo < row.len && c[lo] < first + 4 * kDenseUnit; ++lo) {
            const int64_t u = c[lo] / kDenseUnit;
            const int at = (int)(c[lo] - dense_first_column(u, n_units, n_cols));
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] |= at % 4 == k ? 1u << (at / 4 + 8 * (int)(u % 4)) : 0u;
        }
    }
    mask[i] = uint4{w[0], w[1], w[2], w[3]};
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static DenseArgs dense_args(const DevicePlan &dp, int32_t F)
{
    DenseArgs d{};
    d.rows = dp.dense_rows;
    d.mask = dp.dense_mask;
    d.partials = dp.dense_partials;
    d.n_rows = dp.n_dense_rows;
    d.tile_rows = dp.dense_tile_rows;
    d.row_tiles = (dp.n_dense_rows + dp.dense_tile_rows - 1) / dp.dense_tile_rows;
    d.padded = d.row_tiles * dp.dense_tile_rows;
    d.f_tiles = (F + kDenseTile - 1) / kDenseTile;
    d.n_units = (dp.n_cols + kDenseUnit - 1) / kDenseUnit;
    // one workgroup per CU while a wavefront has two units or more to sum
    const int32_t tiles = d.row_tiles * d.f_tiles;
    int64_t k = kDenseMaxWorkgroups / tiles;
    const int64_t most = (d.n_units + 2 * kWavesPerBlock - 1) / (2 * kWavesPerBlock);
    if (k > most) k = most;
    d.k_parts = (int32_t)(k < 1 ? 1 : k);
    d.n_wg = (int64_t)tiles * d.k_parts;
    return d;
}

// floats of dense_partials for widths up to max_F: a workgroup's tile each, and one part at least
size_t dense_partials_floats(const DevicePlan &dp, int32_t max_F)
{
    const size_t padded = (size_t)(dp.n_dense_rows + dp.dense_tile_rows - 1) / dp.dense_tile_rows * dp.dense_tile_rows;
    const size_t most = (size_t)kDenseMaxWorkgroups * dp.dense_tile_rows * kDenseTile, one = padded * max_F;
    return most > one ? most : one;
}

// A launch and the finishing kernel more than with the gathers: polarized graphs, whole step, us, gathers / dense product, by
// entries of the dense rows x F: 8 M (16,384 rows, F = 64) 12.5 / 18.7, 15 M (F = 128) 18.1 / 22.0; 24 M (32,768 rows, F = 64)
// 20.4 / 22.0; 37 M (65,536 rows, F = 32) 29.0 / 27.3, 48 M (32,768 rows, F = 128) 31.1 / 27.3, 74 M (65,536 rows, F = 64) 39.5 / 38.6;
// 2.1 G (17 M entries, 262,144 rows): F = 8 108 / 80, F = 32 132 / 88, F = 64 223 / 143, F = 128 414 / 260.
bool hd_dense_serves(const DevicePlan &dp, int32_t F)
{
    return dp.n_dense_rows > 0 && dp.n_cols == dp.n && F >= kDenseMinF && dp.dense_entries * F >= (int64_t)1 << 25;
}

size_t dense_mask_words(const DevicePlan &dp)
{
    const size_t padded = (size_t)(dp.n_dense_rows + dp.dense_tile_rows - 1) / dp.dense_tile_rows * dp.dense_tile_rows;
    const size_t units = (size_t)(dp.n_cols + kDenseUnit - 1) / kDenseUnit;
    return (units + 3) / 4 * padded * 4;
}

int launch_dense_mask(const DevicePlan &dp, void *stream)
{
    const DenseArgs d = dense_args(dp, 4);
    const int64_t grid = ((d.n_units + 3) / 4 * d.padded + kBlock - 1) / kBlock;
    if (!grid_ok(grid) || dp.n_cols < kDenseUnit) return (int)hipErrorInvalidConfiguration;
    dense_mask_kernel<<<dim3((unsigned)grid), dim3(kBlock), 0, (hipStream_t)stream>>>(d.rows, d.n_rows, d.padded, dp.col, dp.n_cols,
                                                                                      d.n_units, (uint4 *)dp.dense_mask);
    return (int)hipGetLastError();
}

#define GROOT_DENSE_L(L, CALL)           \
    switch (L) {                         \
    case 8: { constexpr int kL = 8; CALL; } break;   \
    case 16: { constexpr int kL = 16; CALL; } break; \
    case 32: { constexpr int kL = 32; CALL; } break; \
    default: { constexpr int kL = 64; CALL; } break; \
    }

static int dense_lanes(int32_t F4)
{
    int L = 8;
    while (L < F4 && L < kWave) L *= 2;
    return L;
}

// The dense rows, and the pieces of dp (of the other rows) in the same launch.
int launch_hd_dense(const DevicePlan &dp, const float *X, float *Y, int32_t F, int64_t n_chunks, void *stream)
{
    if (dp.weight_mode == kExplicit || !dp.zero_row) return (int)hipErrorInvalidValue;
    const DenseArgs d = dense_args(dp, F);
    if (!grid_ok(d.n_wg + n_chunks)) return (int)hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)(d.n_wg + n_chunks));
    hipStream_t st = (hipStream_t)stream;
    auto launch = [&](auto mb) {
        constexpr int MB = decltype(mb)::value;
        auto go = [&](auto kernel) {
            kernel<<<grid, dim3(kBlock), 0, st>>>(d, dp.chunks, dp.col, (const char *)X, byte_distance(X, dp.zero_row), (v4f *)Y,
                                                  (v4f *)dp.partials, F / 4, dp.n_cols);
        };
        if (dp.weight_mode == kMean) { GROOT_DENSE_L(dense_lanes(F / 4), (go(hd_dense_kernel<MB, kL, kMean>))) }
        else { GROOT_DENSE_L(dense_lanes(F / 4), (go(hd_dense_kernel<MB, kL, kOnes>))) }
    };
    if (dp.dense_tile_rows == 64) launch(std::integral_constant<int, 4>());
    else if (dp.dense_tile_rows == 32) launch(std::integral_constant<int, 2>());
    else if (dp.dense_tile_rows == 16) launch(std::integral_constant<int, 1>());
    else return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

int launch_hd_dense_finish(const DevicePlan &dp, const float *X, float *Y, int32_t F, void *stream)
{
    const DenseArgs d = dense_args(dp, F);
    hipStream_t st = (hipStream_t)stream;
    const int L = dense_lanes(F / 4);
    const int64_t n_wg = d.n_rows + (dp.n_split_rows + kBlock / L - 1) / (kBlock / L);
    if (!grid_ok(n_wg)) return (int)hipErrorInvalidConfiguration;
    auto go = [&](auto kernel) {
        kernel<<<dim3((unsigned)n_wg), dim3(kBlock), 0, st>>>(d, dp.split_rows, dp.n_split_rows, (const v4f *)dp.partials, dp.col,
                                                             (const char *)X, byte_distance(X, dp.zero_row), (v4f *)Y, F / 4);
    };
    if (dp.weight_mode == kMean) { GROOT_DENSE_L(L, (go(hd_dense_finish_kernel<kL, kMean>))) }
    else { GROOT_DENSE_L(L, (go(hd_dense_finish_kernel<kL, kOnes>))) }
    return (int)hipGetLastError();
}

}  // namespace groot
