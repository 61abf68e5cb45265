// High-degree rows that hold a large part of all columns, as a dense product on the matrix cores (gfx950).
//
// A gather of a feature row for every stored entry reads a row of X as often as high-degree rows name it: on the
// polarized graph of 262,144 rows 70 times, 9.5 GB at F = 128, and the vector memory units return no more than 23 TB/s
// (hd_kernel 380 us).  Its 320 longest rows hold 20 % of all columns each, 92 % of the entries of the high-degree rows.  With
// row-uniform weights the sum of such a row is a product of a row of zeros and ones with X: 16, 32 or 64 rows at a time,
// v_mfma_f32_16x16x4_f32, the zeros and ones expanded from one bit per column, X read once per 64 rows straight into the
// instruction's operand layout.  Products with 1 are exact and the sums are fp32, as they were.
//
// The fp32 matrix instruction does 16 rows x 16 features x 4 columns in 32 cycles, the gathers 41 bytes per cycle and CU:
// a row is cheaper here from about 7 % of the columns on (choose_dense_rows).  One workgroup per CU multiplies, which keeps its
// matrix cores busy; the other high-degree rows' pieces, in the same launch, take the memory system beside it (220 us together at
// F = 128, 156 of them matrix instructions; as two launches 155 + 96; with two workgroups per CU, which leave the pieces no
// room, 252; these times in one chain per wavefront, see dense_args).
//
// 0 x infinity is not 0: where X holds a number that is not finite, rows without that column would get NaN.  So a run of columns
// whose sums do not all come out finite is swept again (DensePass).  Polarized graph, 262,144 rows, F = 128, whole step, gathers / here:
// one NaN in X 453 / 364 us, nothing but NaN 453 / 499 (a row gathered again by one workgroup of the finishing kernel: 893);
// F = 512 2,805 / 1,570 and 2,817 / 2,344; 65,536 rows, F = 64: 46 / 43 and 46 / 44.
#include <algorithm>

#include "groot_device.h"

namespace groot {

constexpr int kDenseUnit = 32;               // columns per step of the loop: eight instructions a row block and feature block
constexpr int kDenseTile = 64;               // features of a workgroup
constexpr int kDenseRun = 16;                // units that a wavefront sums in one chain, at most
// LDS: what the wavefronts exchange (at most eight of a tile's 4 x MB instruction results at a time), the tile's sums, the weights
template <int MB> constexpr int kDensePartBytes = kWavesPerBlock * (MB > 1 ? 8 : 4) * kWave * 16;
template <int MB> constexpr int kDenseOwnBytes = MB * 4 * kWave * 16;
template <int MB> constexpr int kDenseSmemBytes = kDensePartBytes<MB> + kDenseOwnBytes<MB> + 16 * MB * 4;

struct DenseArgs {
    const HdChunk *rows;                     // [n_rows] the whole row as one piece, slot -1
    const uint32_t *mask;                    // [unit / 4][padded row][k < 4]: bit 8 (unit % 4) + j is the unit's column 4 j + k
    float *partials;                         // [k_part and group][padded rows][F]
    int32_t n_rows, tile_rows, padded;       // padded: n_rows in whole tiles
    int32_t row_tiles, f_tiles, k_parts;
    int32_t runs, group;                     // a wavefront's stretch in runs, one chain each; runs that meet in one partial sum
    int32_t n_partials;                      // of a row: k_parts x groups
    int64_t n_units;                         // columns in units of kDenseUnit
    int64_t n_wg;                            // row_tiles x f_tiles x k_parts
};

// First column of a unit: the last one is moved back to end with the last column (there are kDenseUnit columns or more) and
// has bits for those only that the unit before has not.
__device__ __forceinline__ int64_t dense_first_column(int64_t u, int64_t n_units, int64_t n_cols)
{
    return u == n_units - 1 ? n_cols - kDenseUnit : u * kDenseUnit;
}

// What the second and the third sweep over a run of columns multiply, where the first, of X as it is, did not come out finite.
// Codes: in the place of what is not finite in X a number that counts its kind in a field of its own; their sums become the
// infinity or NaN that the accumulators start the last sweep with, over what is finite.
enum DensePass { kDenseCodes, kDenseFinite };
constexpr float kDenseInf = 1.f, kDenseNegInf = 1024.f, kDenseNaN = 1048576.f;
static_assert(kDenseRun * kDenseUnit < 1024, "the count of a run fits its field");

// no branches here: 32 values of a lane each
__device__ __forceinline__ float dense_operand(float x, int pass)
{
    const bool finite = isfinite(x);
    float code = x > 0.f ? kDenseInf : kDenseNegInf;
    code = x != x ? kDenseNaN : code;
    const float where_finite = pass == kDenseFinite ? x : 0.f, elsewhere = pass == kDenseFinite ? 0.f : code;
    return finite ? where_finite : elsewhere;
}

__device__ __forceinline__ float dense_decode(float sum)
{
    const uint32_t n = (uint32_t)sum, pos = n % 1024, neg = n / 1024;
    float inf = pos ? __builtin_inff() : -__builtin_inff();
    inf = (sum >= kDenseNaN) | ((pos != 0) & (neg != 0)) ? __builtin_nanf("") : inf;
    return n ? inf : 0.f;
}

// One workgroup's tile of 16 MB rows x 16 NV features: the columns of a k_part, a quarter for each wavefront.
// Lane layout of the instruction: A row and B column are lane % 16, k is lane / 16; D rows are 4 (lane / 16) + r.  Component
// v of the lane's NV features is the operand whose column m is feature NV m + v, so a lane's load of consecutive features
// serves NV instructions as it is.  fp32 matrix and vector instructions of a SIMD do not overlap and changing between them costs
// cycles, so the loop has next to no address arithmetic (scalar bases and constant offsets) and expands the bits of MB
// instructions' rows, then issues their MB NV instructions: with
// addresses per lane and the bits expanded as the compiler placed them the polarized graph took 195 us, now 155.
//
// A wavefront sums a run of kDenseRun units at most, then the four of them meet in LDS, every one adds up a quarter of the tile,
// (0 + 2) + (1 + 3), and the row's weight times that goes to the quarter's sums, in LDS too (registers for them would cost the third
// workgroup of a CU, where the pieces of the other rows run: 286 us instead of 273).  So chains of additions stay short.
// With mean weights the ones are 1 / 64 and the weights 64 times as large, both exact: a sum of many columns that the weight will
// make small does not overflow before (the gathers apply the weight to the few entries of a lane group, up to 128).
template <int MB, int NV, int W>
__device__ __forceinline__ void dense_tile(char *smem, const DenseArgs &d, const char *__restrict__ X, int32_t F, int64_t n_cols,
                                           int32_t row_tile, int32_t f0, int32_t k_part)
{
    typedef float vN __attribute__((ext_vector_type(NV)));
    constexpr float kOne = W == kMean ? 0x1p-6f : 1.f;
    constexpr int kHalves = MB * NV > 8 ? 2 : 1, kNh = NV / kHalves;              // components exchanged at a time: kNh of a row block
    constexpr int kOwn = MB * kNh > kWavesPerBlock ? MB * kNh / kWavesPerBlock : 1;   // of these a wavefront adds up
    typedef float vOwn __attribute__((ext_vector_type(kHalves * kOwn)));
    v4f *const s_part = (v4f *)smem;                                              // [wavefront][block and component][lane]
    v4f *const s_own = (v4f *)(smem + kDensePartBytes<MB>);                       // [wavefront][half][own][lane]
    float *const s_weight = (float *)(smem + kDensePartBytes<MB> + kDenseOwnBytes<MB>);   // [row]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave, m = lane % 16, k4 = lane / 16;
    const int32_t row0 = row_tile * d.tile_rows;
    const int f = f0 + NV * m;
    if (threadIdx.x < 16 * MB) {
        const int32_t r = row0 + (int32_t)threadIdx.x;
        s_weight[threadIdx.x] = r < d.n_rows ? row_weight<W>(d.rows[r].row_nnz) / kOne : 0.f;
    }
    const int64_t first = d.n_units * k_part / d.k_parts, behind = d.n_units * (k_part + 1) / d.k_parts;
    const int64_t share = (behind - first + kWavesPerBlock - 1) / kWavesPerBlock;
    const int64_t u0 = first + wave * share, u1 = u0 + share < behind ? u0 + share : behind;
    const int64_t run = (share + d.runs - 1) / d.runs;

    const int64_t row_bytes = (int64_t)F * 4;
    const uint32_t x_at = (uint32_t)(k4 * (int)row_bytes + 4 * (f < F - NV ? f : F - NV));
    const uint32_t bits_at = (uint32_t)((row0 + m) * 16 + k4 * 4);
    auto load = [&](int64_t u, vN (&x)[8], uint32_t (&w)[MB]) {
        u = u < d.n_units ? u : d.n_units - 1;
        const char *const base = X + dense_first_column(u, d.n_units, n_cols) * row_bytes;
        const uint8_t *const bits = (const uint8_t *)d.mask + (u / 4) * d.padded * 16 + u % 4;
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = *(const vN *)((base + 4 * j * row_bytes) + x_at);
#pragma unroll
        for (int b = 0; b < MB; ++b) w[b] = (bits + bits_at)[256 * b];
    };
    v4f acc[MB][NV];
    auto multiply = [&](const vN (&x)[8], const uint32_t (&w)[MB]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float a[MB];
#pragma unroll
            for (int b = 0; b < MB; ++b) a[b] = __builtin_bit_cast(float, __builtin_amdgcn_sbfe(w[b], j, 1) & __builtin_bit_cast(int, kOne));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int v = 0; v < NV; ++v) acc[b][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b], x[j][v], acc[b][v], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto clear = [&]() {
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[b][v] = v4f{0.f, 0.f, 0.f, 0.f};
    };
    auto all_finite = [&]() {
        float zero = 0.f;
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int r = 0; r < 4; ++r) zero = __builtin_fmaf(acc[b][v][r], 0.f, zero);
        return __ballot(zero != 0.f) == 0;               // otherwise NaN
    };
    vN xa[8], xb[8];
    uint32_t wa[MB], wb[MB];
    load(u0, xa, wa);
    bool finite = true;                                  // of the run before: if not, this one is not tried as it is
#pragma unroll 1
    for (int32_t i = 0, slot = k_part * (d.n_partials / d.k_parts); i < d.runs; ++i) {
        const int64_t begin = u0 + i * run, to = begin + run < u1 ? begin + run : u1;
        clear();
        if (finite) {
#pragma unroll 1
            for (int64_t u = begin; u < to; u += 2) {    // one unit is multiplied while the next is on its way
                load(u + 1 < to ? u + 1 : u, xb, wb);
                __builtin_amdgcn_sched_barrier(0);       // the compiler would sink the loads to their use
                multiply(xa, wa);
                load(u + 2 < to ? u + 2 : to, xa, wa);   // in the end the next run's first
                __builtin_amdgcn_sched_barrier(0);
                if (u + 1 < to) multiply(xb, wb);
            }
            finite = all_finite();
            if (!finite) clear();
        }
        if (!finite) {
#pragma unroll 1
            for (int pass = kDenseCodes; pass <= kDenseFinite; ++pass) {
#pragma unroll 1
                for (int64_t u = begin; u < to; ++u) {
                    uint32_t any = 0;
                    load(u, xa, wa);
#pragma unroll
                    for (int j = 0; j < 8; ++j)
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            const float x = dense_operand(xa[j][v], pass);
                            any |= __builtin_bit_cast(uint32_t, x);   // (of a vector's component it would be the first one's)
                            xa[j][v] = x;
                        }
                    if (__ballot(any)) multiply(xa, wa);   // usually nothing to code
                }
                if (pass == kDenseCodes) {
#pragma unroll
                    for (int b = 0; b < MB; ++b)
#pragma unroll
                        for (int v = 0; v < NV; ++v)
#pragma unroll
                            for (int r = 0; r < 4; ++r) acc[b][v][r] = dense_decode(acc[b][v][r] / kOne);
                    finite = all_finite();
                }
            }
            load(to, xa, wa);
        }
        const int b_own = wave % MB, v_own = wave / MB * kOwn;
#pragma unroll
        for (int h = 0; h < kHalves; ++h) {
            __syncthreads();                             // what was there has been read
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int v = 0; v < kNh; ++v) s_part[((wave * MB + b) * kNh + v) * kWave + lane] = acc[b][h * kNh + v];
            __syncthreads();
            if (v_own < kNh) {
                const v4f weight = *(const v4f *)(s_weight + 16 * b_own + 4 * k4);
#pragma unroll
                for (int v = 0; v < kOwn; ++v) {
                    const v4f *const p = s_part + (b_own * kNh + v_own + v) * kWave + lane;
                    constexpr int kNext = MB * kNh * kWave;
                    v4f *const own = s_own + ((wave * kHalves + h) * kOwn + v) * kWave + lane;
                    const v4f sum = weight * ((p[0] + p[2 * kNext]) + (p[kNext] + p[3 * kNext]));
                    *own = i % d.group ? *own + sum : sum;
                }
            }
        }
        if ((i + 1) % d.group && i + 1 < d.runs) continue;
        if (v_own < kNh && f < F) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                vOwn out;
#pragma unroll
                for (int v = 0; v < kHalves * kOwn; ++v) out[v] = ((const float *)(s_own + (wave * kHalves * kOwn + v) * kWave + lane))[r];
                const int64_t row = (int64_t)slot * d.padded + row0 + 16 * b_own + 4 * k4 + r;
                *(vOwn *)(d.partials + row * F + f + v_own) = out;
            }
        }
        ++slot;
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
    constexpr int kSums = kDenseSmemBytes<MB>, kPiece = kHdSmemBytes<L>;
    __shared__ __align__(16) char smem[kSums > kPiece ? kSums : kPiece];
    if (blockIdx.x >= d.n_wg) {
        hd_piece<L, W>(smem, chunks[blockIdx.x - d.n_wg], col, nullptr, X, zero_off, Y, partials, F4, nullptr);
        return;
    }
    const int32_t t = (int32_t)blockIdx.x, row_tile = t % d.row_tiles, f_tile = t / d.row_tiles % d.f_tiles;
    const int32_t k_part = t / d.row_tiles / d.f_tiles, F = 4 * F4;
    if (F - f_tile * kDenseTile > kDenseTile / 2)
        dense_tile<MB, 4, W>(smem, d, X, F, n_cols, row_tile, f_tile * kDenseTile, k_part);
    else
        dense_tile<MB, 2, W>(smem, d, X, F, n_cols, row_tile, f_tile * kDenseTile, k_part);
}

// Workgroups [0, d.n_rows): one dense row each, its partial sums meet in fp64.  The ones behind: the split rows among the others, as
// in hd_finish_kernel.
template <int L>
__global__ __launch_bounds__(kBlock) void hd_dense_finish_kernel(const DenseArgs d, const HdSplitRow *__restrict__ split,
                                                                 int64_t n_split, const v4f *__restrict__ partials,
                                                                 v4f *__restrict__ Y, int32_t F4)
{
    constexpr int G = kBlock / L;
    typedef double v4d __attribute__((ext_vector_type(4)));
    auto wide = [](v4f x) { return __builtin_convertvector(x, v4d); };
    __shared__ v4d s_red[kBlock];                        // [G][L]
    const int g = threadIdx.x / L, f = threadIdx.x % L;
    if (blockIdx.x >= d.n_rows) {
        const int64_t k = (int64_t)(blockIdx.x - d.n_rows) * G + g;
        if (k < n_split) hd_finish_row<L>(split[k], partials, Y, F4, nullptr, f);
        return;
    }
    const int64_t row = d.rows[blockIdx.x].row;
#pragma unroll 1
    for (int32_t fb = 0; fb < F4; fb += L) {
        const int32_t ff = fb + f;
        const bool live = ff < F4;
        v4d acc = {0., 0., 0., 0.};
        const v4f *p = (const v4f *)d.partials + (int64_t)blockIdx.x * F4 + (live ? ff : 0);
        const int64_t step = (int64_t)d.padded * F4;
        int32_t k = g;
        for (; k + 3 * G < d.n_partials; k += 4 * G) {
            const v4f x0 = p[k * step], x1 = p[(k + G) * step], x2 = p[(k + 2 * G) * step], x3 = p[(k + 3 * G) * step];
            acc += (wide(x0) + wide(x1)) + (wide(x2) + wide(x3));
        }
        for (; k < d.n_partials; k += G) acc += wide(p[k * step]);
        s_red[threadIdx.x] = acc;
        __syncthreads();
#pragma unroll
        for (int stride = G / 2; stride > 0; stride /= 2) {
            if (g < stride) s_red[threadIdx.x] += s_red[threadIdx.x + stride * L];
            __syncthreads();
        }
        if (g == 0 && live) Y[row * F4 + ff] = __builtin_convertvector(s_red[f], v4f);
        __syncthreads();
    }
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
    const int64_t tiles = (int64_t)d.row_tiles * d.f_tiles;
    int64_t k = kDenseMaxWorkgroups / tiles;
    const int64_t most = (d.n_units + 2 * kWavesPerBlock - 1) / (2 * kWavesPerBlock);
    if (k > most) k = most;
    d.k_parts = (int32_t)(k < 1 ? 1 : k);
    // How long a run is, and how many meet in fp32, so that the error is no larger than that of the gathers, which grows with a
    // row's pieces.  Error of the dense rows in the 2-norm, U(-1, 1), here / gathers, 1e-7, F = 128: polarized graphs of 32,768 rows
    // 0.74 / 1.12, 65,536 1.11 / 1.42, 131,072 1.31 / 1.51, 262,144 1.77 / 2.01 (F = 512 1.96 / 2.11); 64 rows of half of 65,536
    // columns 1.64 / 1.83; 1,024 rows of a twelfth of them 1.10 / 1.20, of a quarter of 20,000 1.06 / 1.22.  In one chain per
    // wavefront the 262,144 rows were at 4.1 (F = 512: 8.2).  A run costs 2 us: 260 us a step in one chain, 272 in six (F = 128).
    const double length = (double)dp.dense_entries / dp.n_dense_rows, pieces = length / 512, per_unit = length / d.n_units;
    const double run = (14 + 1.1 * pieces) / (1 + per_unit);
    const int64_t share = ((d.n_units + d.k_parts - 1) / d.k_parts + kWavesPerBlock - 1) / kWavesPerBlock;
    const int64_t units = run < 2 ? 2 : run > kDenseRun ? kDenseRun : (int64_t)run;
    d.runs = (int32_t)((share + units - 1) / units);
    d.group = 4 + (int32_t)(pieces < 1024 ? pieces / 8 : 128);
    d.n_partials = d.k_parts * ((d.runs + d.group - 1) / d.group);
    d.n_wg = tiles * d.k_parts;
    return d;
}

// floats of dense_partials for widths up to max_F
size_t dense_partials_floats(const DevicePlan &dp, int32_t max_F)
{
    size_t most = 0;
    for (int32_t F = kDenseMinF; F <= max_F; F += 4) {
        const DenseArgs d = dense_args(dp, F);
        most = std::max(most, (size_t)d.n_partials * d.padded * F);
    }
    return most;
}

// A launch and the finishing kernel more than with the gathers: polarized graphs, whole step, us, gathers / dense product, by
// entries of the dense rows x F: 16,384 rows 7.4 M (F = 64) 12.4 / 18.3, 15 M (128) 17.6 / 21.4, 23 M (200) 24.5 / 26.1; 32,768 rows
// 22 M (64) 20.0 / 22.6, 43 M (128) 30.9 / 28.6, 68 M (200) 48.2 / 38.8; 65,536 rows 29 M (32) 28.8 / 27.3, 59 M (64) 38.7 / 38.4, 117 M
// (128) 54.2 / 51.5; 131,072 rows 35 M (8) 38.0 / 38.5, 141 M (32) 54.8 / 47.2, 566 M (128) 134 / 102; 262,144 rows 134 M (8) 90 / 85,
// 534 M (32) 128 / 92, 1.07 G (64) 220 / 145, 2.1 G (128) 423 / 273.
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

int launch_hd_dense_finish(const DevicePlan &dp, float *Y, int32_t F, void *stream)
{
    const DenseArgs d = dense_args(dp, F);
    const int L = dense_lanes(F / 4);
    const int64_t n_wg = d.n_rows + (dp.n_split_rows + kBlock / L - 1) / (kBlock / L);
    if (!grid_ok(n_wg)) return (int)hipErrorInvalidConfiguration;
    GROOT_DENSE_L(L, (hd_dense_finish_kernel<kL><<<dim3((unsigned)n_wg), dim3(kBlock), 0, (hipStream_t)stream>>>(
                         d, dp.split_rows, dp.n_split_rows, (const v4f *)dp.partials, (v4f *)Y, F / 4)));
    return (int)hipGetLastError();
}

}  // namespace groot
