// Weight gradients of the fused GraphSAGE-mean layer for gfx950:
//     dWn = (A_hat X)^T dZ,   dWs = X^T dZ,   X [N, FI], dZ [N, FO], dWn and dWs [FI, FO], FI = 32 or 64, FO = 16, 32 or 64
// for the layer Z = (A_hat X) Wn + X Ws + b with dZ the gradient of the loss at Z (Section "GNN and Edge
// Re-growth After Partition": the model is trained).  Two products with N as the contraction length: as plain
// matrix products over [N, 64] operands they take 58 ms each on 134 M rows with the vendor library, and the
// first needs A_hat X in memory.  Here one pass does both with the aggregation kept on chip.
//
// The aggregation is the fused layer kernel's (groot_sage_pipe.hip: a persistent workgroup per CU, every
// wavefront walks its own 16-row tiles and keeps the next tile's gathers in flight; slot table in LDS, a row of
// zeros for dead slots).  For every tile the wavefront adds [A_hat X | X]^T dZ (2 FI x FO) to accumulators that it
// keeps for its whole sweep.
//
// The contraction runs over rows, and v_mfma_f32_16x16x4_f32 (fp32 in and out) wants exactly what the gathers leave
// in the registers: lane (m = lane % 16, k = lane / 16) holds one value of column m of row k, and at FI = 64 lane l has
// a float4 of row l / 16 of a sweep, columns 4 (l % 16) .. + 3.  So component j of that float4 is the operand whose
// column m is feature 4 m + j, and a sweep's 4 rows are the contraction length of one instruction: no transposition,
// no trip through LDS, and products and sums in fp32 throughout.  dZ is loaded with 16 lanes to a row (FO / 16
// consecutive floats each), so its component i is the operand whose column n is feature (FO / 16) n + i.  At FI = 32 a
// sweep has 8 rows (8 lanes to a row): neighbouring rows 2 k and 2 k + 1 sit in the two halves of 16 lanes, which swap
// half of their float4 (DPP row rotation by 8), giving operands of row 2 k (p = 0) and of row 2 k + 1 (p = 1).
//
// What bounds it: at 64 x 64 the fp32 matrix instructions, 128 of 32 cycles per 16 rows and SIMD (2.09 M cycles of
// the 3.15 M counted at 8.4 M rows, at the 2.05 GHz that the chip grants dense fp32 matrix work), on the other widths the memory
// traffic.  The form before this one passed the operands transposed through LDS, cut into three bf16 pieces, six piece
// products on v_mfma_f32_16x16x16_bf16, whose inner sums truncate: at 8.4 M rows, carry-save multipliers, whole call,
// 64 x 64 2,030 us and 1.3e-5 from the 64-bit result, now 1,431 us and 1.1e-6; on the Booth shape, 4.3 M rows, 64 x 32:
// whole call 966 us and 7e-6, now 559 us and 4e-7.
//
// An accumulator that took a whole sweep's rows one after the other would round N / 2048 times.  Where LDS has room for a
// second set of sums (every width but 64 x 64), the accumulators are added to it every kWgFold tiles and cleared.  At
// the end a workgroup's wavefronts are added in fp64 and written, in fp64, as one slice of a workspace; a second kernel adds the
// slices in a fixed order.  No atomics: the result is the same on every run.
#include <type_traits>

#include "groot_device.h"

namespace groot {

constexpr int kWgRows = 16;                  // rows per tile
constexpr int kWgFold = 32;                  // tiles between two additions to the sums in LDS (512 rows)
constexpr int kWgPending = 32;               // tiles with rows that the slots do not serve, noted per wavefront
// Wavefronts per workgroup (one workgroup per CU), two per SIMD: one's vector work and waits then run beside the other's
// matrix work.  At 64 x 64 the accumulators take 128 of a wavefront's 256 registers (one wavefront per SIMD with a whole
// tile of rows in flight: 1,621 us at 8.4 M rows instead of 1,454).
constexpr int kWgWaves = 8;
constexpr bool wg_folds(int FI, int FO) { return FI * FO < 64 * 64; }    // 64 x 64: the second set of sums would be 256 KB

typedef float wg_f2 __attribute__((ext_vector_type(2)));
typedef double wg_d2 __attribute__((ext_vector_type(2)));

// the value of lane (l + 8) % 16 of the same 16 lanes
__device__ __forceinline__ float wg_other_half(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x128, 0xf, 0xf, false));
}

// feature of column m (0..15) of operand component j of a half (A_hat X or X)
template <int FI>
__device__ __forceinline__ int wg_feature(int m, int j)
{
    return FI == 64 ? 4 * m + j : m < 8 ? 4 * m + j : 4 * (m - 8) + 2 + j;
}

// c[mb][nb] += a[mb] b[nb]^T for 4 x 4 blocks, every sum in place.  (Given the builtin, the compiler lets the sums wander between
// registers, which costs 64 x 64 the last free ones: it spills in the loop, 2,497 us instead of 1,454 at 8.4 M rows.)  The two wait states before the first instruction
// cover operands that a vector instruction has just written, those after the last one a read of the sums by whatever comes next.
__device__ __forceinline__ void wg_mfma_4x4(v4f (&c0)[4], v4f (&c1)[4], v4f (&c2)[4], v4f (&c3)[4], const float (&a)[4], const float (&b)[4])
{
    asm volatile(
        "s_nop 1\n"
        "v_mfma_f32_16x16x4_f32 %0, %16, %20, %0\n"
        "v_mfma_f32_16x16x4_f32 %1, %16, %21, %1\n"
        "v_mfma_f32_16x16x4_f32 %2, %16, %22, %2\n"
        "v_mfma_f32_16x16x4_f32 %3, %16, %23, %3\n"
        "v_mfma_f32_16x16x4_f32 %4, %17, %20, %4\n"
        "v_mfma_f32_16x16x4_f32 %5, %17, %21, %5\n"
        "v_mfma_f32_16x16x4_f32 %6, %17, %22, %6\n"
        "v_mfma_f32_16x16x4_f32 %7, %17, %23, %7\n"
        "v_mfma_f32_16x16x4_f32 %8, %18, %20, %8\n"
        "v_mfma_f32_16x16x4_f32 %9, %18, %21, %9\n"
        "v_mfma_f32_16x16x4_f32 %10, %18, %22, %10\n"
        "v_mfma_f32_16x16x4_f32 %11, %18, %23, %11\n"
        "v_mfma_f32_16x16x4_f32 %12, %19, %20, %12\n"
        "v_mfma_f32_16x16x4_f32 %13, %19, %21, %13\n"
        "v_mfma_f32_16x16x4_f32 %14, %19, %22, %14\n"
        "v_mfma_f32_16x16x4_f32 %15, %19, %23, %15\n"
        "s_nop 15\n"
        : "+v"(c0[0]), "+v"(c0[1]), "+v"(c0[2]), "+v"(c0[3]), "+v"(c1[0]), "+v"(c1[1]), "+v"(c1[2]), "+v"(c1[3]), "+v"(c2[0]), "+v"(c2[1]), "+v"(c2[2]), "+v"(c2[3]), "+v"(c3[0]), "+v"(c3[1]), "+v"(c3[2]), "+v"(c3[3])
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]));
}

// W: kOnes or kMean; FI: width of X; FO: width of dZ; D: gather slots per row on the pipelined path (5, 6 or 8)
template <int W, int FI, int FO, int D>
__global__ __launch_bounds__(kWgWaves * kWave) __attribute__((amdgpu_waves_per_eu(kWgWaves / 4, kWgWaves / 4))) void sage_wgrad_kernel(
    const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col, const char *__restrict__ X, const char *__restrict__ dZ, int64_t zero_off, int64_t n, int64_t nnz, int32_t T, int64_t n_tiles,
    int64_t tiles_per_part, int64_t waves_per_part, int32_t parts, const int32_t *__restrict__ hd_rows, int32_t n_hd,
    const char *__restrict__ hd_agg, wg_d2 *__restrict__ partials)
{
    static_assert(FI == 64 || FI == 32, "width of X");
    static_assert(FO == 64 || FO == 32 || FO == 16, "width of dZ");
    static_assert(W == kOnes || W == kMean, "row-uniform weights");
    constexpr int kL = FI / 4, kRpg = kWave / kL, kG = kWgRows / kRpg, kRowShift = FI == 64 ? 8 : 7;
    constexpr int kZShift = FO == 64 ? 8 : FO == 32 ? 7 : 6;             // log2 of a row of dZ in bytes
    constexpr int kP = kRpg / 4;                                         // contraction groups of 4 rows per sweep
    constexpr int kMc = FI / 16, kMb = 2 * kMc, kNb = FO / 16;           // 16-column blocks of a half, of [A_hat X | X], of dZ
    constexpr int kSlots = kWgRows * D, kH = (kSlots + kWave - 1) / kWave;
    using ZVec = typename std::conditional<kNb == 4, v4f, typename std::conditional<kNb == 2, wg_f2, float>::type>::type;
    __shared__ __align__(16) int64_t s_slot[kWgWaves][kSlots];
    __shared__ float s_inv[kWgWaves][kWgRows];
    constexpr bool kFold = wg_folds(FI, FO);
    // sweeps in flight: half a tile (a whole one: 2 % slower); 64 x 64 one (two: 1,478 us instead of 1,454, the registers are full)
    constexpr int kSets = kFold ? kG / 2 : 1;
    constexpr int kBufs = kFold ? kWgWaves : kWgWaves / 2;
    __shared__ __align__(16) v4f s_sum[kBufs][kMb * kNb][kWave];         // 64 x 64: 32 KB per buffer

    // a scalar: the tile arithmetic below then runs on the scalar unit, and vector instructions are what this kernel is short of
    __shared__ int32_t s_pending[kWgWaves][kWgPending];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int g = l / kL, f = l % kL;
    const int kq = l / 16, jl = l % 16;                  // matrix instruction: contraction index / column of A, of B and of D
    const int64_t part = blockIdx.x % parts, j = (blockIdx.x / parts) * kWgWaves + w;
    const int64_t x_begin = part * tiles_per_part;
    const int64_t x_end = x_begin + tiles_per_part < n_tiles ? x_begin + tiles_per_part : n_tiles;
    const int64_t t_first = x_begin + j, stride = waves_per_part;
    const int64_t n_full = n / kWgRows, x_full = x_end < n_full ? x_end : n_full;   // whole tiles
    const char *Xf = X + 16 * f;

    v4f acc[kMb][kNb];
    auto clear = [&]() {
#pragma unroll
        for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
            for (int nb = 0; nb < kNb; ++nb) acc[mb][nb] = (v4f){0.f, 0.f, 0.f, 0.f};
    };
    auto fold = [&]() {                                  // accumulators -> sums in LDS (every lane its own words)
#pragma unroll
        for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
            for (int nb = 0; nb < kNb; ++nb) {
                s_sum[w][mb * kNb + nb][l] += acc[mb][nb];
                __builtin_amdgcn_sched_barrier(0);       // one block at a time: no registers for more
            }
    };
    clear();
    if constexpr (kFold) {
#pragma unroll
        for (int b = 0; b < kMb * kNb; ++b) s_sum[w][b][l] = (v4f){0.f, 0.f, 0.f, 0.f};
    }

    if (t_first < x_end) {
        // ---- CSR pipeline: rp_a and cc belong to the next tile to be staged, rp_b to the one after
        int64_t rp_a = 0, rp_b = 0;
        int32_t cc[kH];
#pragma unroll
        for (int h = 0; h < kH; ++h) cc[h] = 0;
        bool fix_a = false;                              // the tile has rows that the slots do not serve
        int32_t len_a = 0;                               // lanes 0..15: stored length of the tile's row
        uint32_t live_a = 0;                             // bit h: slot l + 64 h holds an entry
        auto load_rp = [&](int64_t tile) -> int64_t {
            const int64_t ri = tile * kWgRows + (l < kWgRows ? l : kWgRows);
            return rowptr[ri < n ? ri : n];              // lanes 0..16 hold the pointers; rows past the end read rowptr[n]: no entries
        };
        auto load_cols = [&]() {                         // from rp_a: every slot fetches its own entry
            const uint32_t begin_lo = __builtin_amdgcn_readfirstlane((uint32_t)rp_a);
            const int64_t begin = (int64_t)((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)rp_a >> 32)) << 32 | begin_lo);
            const int32_t *const tile_col = col + (begin < nnz ? begin : 0);   // a dead slot reads the tile's first entry, or entry 0
            const int32_t rel = (int32_t)((uint32_t)rp_a - begin_lo);
            len_a = __shfl_down(rel, 1) - rel;
            fix_a = __ballot(l < kWgRows && (len_a > D || len_a >= T)) != 0;
            live_a = 0;
#pragma unroll
            for (int h = 0; h < kH; ++h) {               // unconditional loads: the number of loads in flight stays known
                const int s = l + kWave * h;             // slot s: row r, entry k
                const int r = s / D, k = s - r * D;
                const int32_t lo = __shfl(rel, r), len = __shfl(rel, r + 1) - lo;
                const bool live = s < kSlots && k < len && len <= D && len < T;
                live_a |= (uint32_t)live << h;
                cc[h] = __builtin_nontemporal_load(&tile_col[live ? (uint32_t)(lo + k) : 0u]);
            }
        };
        auto stage = [&]() -> bool {                     // cc, live_a, len_a -> slot table and row weights; -> fix_a
#pragma unroll
            for (int h = 0; h < kH; ++h) {
                const int s = l + kWave * h;
                if (s < kSlots) s_slot[w][s] = ((live_a >> h) & 1) ? ((int64_t)cc[h] << kRowShift) : zero_off;
            }
            if (W == kMean && l < kWgRows) s_inv[w][l] = row_weight<kMean>(len_a);
            wave_sync();
            return fix_a;
        };
        // ---- one sweep: kRpg rows, one per lane group: the row's D slots, its own features; and the rows of dZ
        struct Regs {
            v4f xs[D], self;
            ZVec dz[kP];
            float inv;
        };
        Regs rr[kSets];
        const uint32_t x_lane = (uint32_t)g << kRowShift | 16 * f, z_lane = (uint32_t)(kq * kP) << kZShift | 4 * kNb * jl;
        auto load_self = [&](int64_t tile, int grp) -> v4f {
            return *(const v4f *)(X + (tile << kRowShift) * kWgRows + x_lane + ((grp * kRpg) << kRowShift));
        };
        auto load_z = [&](int64_t tile, int grp, int p) -> ZVec {
            return __builtin_nontemporal_load((const ZVec *)(dZ + (tile << kZShift) * kWgRows + z_lane + ((grp * kRpg + p) << kZShift)));
        };
        auto issue = [&](Regs &q, int64_t tile, int grp) {   // the tile whose slots are staged
            const int lr = grp * kRpg + g;               // row (inside the tile) that this lane holds a float4 of X of
            if (W == kMean) q.inv = s_inv[w][lr];
#pragma unroll
            for (int k = 0; k < D; ++k) q.xs[k] = *(const v4f *)(Xf + s_slot[w][lr * D + k]);
            q.self = load_self(tile, grp);
#pragma unroll
            for (int p = 0; p < kP; ++p) q.dz[p] = load_z(tile, grp, p);
        };
        auto sum = [&](const Regs &q) -> v4f {
            v4f a = q.xs[0];
#pragma unroll
            for (int k = 1; k < D; ++k) a += q.xs[k];
            if (W == kMean) a *= q.inv;
            return a;
        };
        // acc[mb0 ..] += (this half's columns)^T dz, over the rows of one sweep
        auto multiply = [&](int mb0, const v4f &x, const ZVec (&dz)[kP]) {
#pragma unroll
            for (int p = 0; p < kP; ++p) {
                float a[kMc], b[kNb];
                if constexpr (FI == 64) {
#pragma unroll
                    for (int c = 0; c < kMc; ++c) a[c] = x[c];
                } else {                                 // the two halves of 16 lanes hold rows 2 k and 2 k + 1
                    const bool odd = (jl & 8) != 0;
#pragma unroll
                    for (int c = 0; c < kMc; ++c) {
                        const float lo = p == 0 ? x[c] : wg_other_half(x[c]);
                        const float hi = p == 0 ? wg_other_half(x[2 + c]) : x[2 + c];
                        a[c] = odd ? hi : lo;
                    }
                }
                if constexpr (kNb == 1) b[0] = dz[p];
                else {
#pragma unroll
                    for (int c = 0; c < kNb; ++c) b[c] = dz[p][c];
                }
                if constexpr (kMc == 4 && kNb == 4) wg_mfma_4x4(acc[mb0], acc[mb0 + 1], acc[mb0 + 2], acc[mb0 + 3], a, b);
                else {
#pragma unroll
                    for (int mb = 0; mb < kMc; ++mb)
#pragma unroll
                        for (int nb = 0; nb < kNb; ++nb)
                            acc[mb0 + mb][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mb], b[nb], acc[mb0 + mb][nb], 0, 0, 0);
                }
            }
        };
        int until_fold = kWgFold;                        // tiles that may still be added before the next fold
        auto fold_now = [&]() {
            fold();
            clear();
            until_fold = kWgFold;
        };
        int64_t tile = t_first;
        while (tile < x_end) {
            int pending = 0;
            if (tile < x_full) {
                // ---- prologue: the first kSets sweeps are in flight; the CSR of the next two tiles is on its way
                rp_a = load_rp(tile);
                load_cols();
                bool fix_cur = stage(), fix_next = false;
                rp_a = load_rp(tile + stride);
                load_cols();
                rp_b = load_rp(tile + 2 * stride);
#pragma unroll
                for (int grp = 0; grp < kSets; ++grp) issue(rr[grp], tile, grp);
                __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0): the loop's own order of loads is the only one from here on

                for (; tile < x_full && pending < kWgPending; tile += stride) {
                    const int64_t next = tile + stride < n_full ? tile + stride : n_full - 1;
#pragma unroll
                    for (int grp = 0; grp < kG; ++grp) {
                        if (grp == kG - kSets) {         // this tile's sweeps are all issued: CSR of the next tile -> slot table
                            fix_next = stage();
                            rp_a = rp_b;
                            load_cols();
                            rp_b = load_rp(tile + 3 * stride);
                        }
                        // this sweep's values out of the register set, which takes the sweep kSets later
                        Regs &q = rr[grp % kSets];
                        const v4f a = sum(q), s = q.self;   // a row that the slots do not serve: the sum is zero
                        ZVec z[kP];
#pragma unroll
                        for (int p = 0; p < kP; ++p) z[p] = q.dz[p];
                        issue(q, grp + kSets < kG ? tile : next, (grp + kSets) % kG);
                        // Matrix instructions in one run: fp32 ones and vector instructions do not overlap within a
                        // wavefront and alternating costs (left to the scheduler, 64 x 64 took 1,872 us); at a raised
                        // priority, so that the SIMD's two wavefronts take turns (1,475 against 1,484 us).
                        __builtin_amdgcn_sched_barrier(0);
                        __builtin_amdgcn_s_setprio(1);
                        multiply(0, a, z);
                        multiply(kMc, s, z);
                        __builtin_amdgcn_s_setprio(0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (fix_cur) {
                        if (l == 0) s_pending[w][pending] = (int32_t)tile;
                        ++pending;
                    }
                    fix_cur = fix_next;
                    if constexpr (kFold) {
                        if (--until_fold == 0) fold_now();
                    }
                }
            }
            if (tile >= x_full && tile < x_end && pending < kWgPending) {   // the ragged last tile
                if (l == 0) s_pending[w][pending] = (int32_t)tile;
                ++pending;
                tile += stride;
            }
            // ---- the noted tiles, straight from global memory: A_hat X of the rows that had no live slots (more entries
            //      than slots, or high-degree: their sums come from the side buffer), for which the loop above has
            //      added zeros, and all of the ragged tile.  Outside the loop because the registers that hold its rows
            //      in flight are needed here (inside it they were spilled), and so that its loads are all unconditional.
            wave_sync();
            static_assert(kWgPending <= kWgFold, "the noted tiles fit between two folds");
            if constexpr (kFold) {
                if (pending > until_fold) fold_now();
            }
#pragma unroll 1
            for (int i = 0; i < pending; ++i) {
                const int64_t t = __builtin_amdgcn_readfirstlane(s_pending[w][i]);
                const bool ragged = t >= n_full;
                const int64_t rp = load_rp(t);           // rows past the end: no entries
                const int64_t next_rp = __shfl_down(rp, 1);
                const bool here = t * kWgRows + l < n;
                // rows past the end of the matrix are in no sum
                uint32_t redo = (uint32_t)__ballot(l < kWgRows && here && (ragged || next_rp - rp > D || next_rp - rp >= T));
                const uint32_t hd = (uint32_t)__ballot(l < kWgRows && next_rp - rp >= T);
                const int32_t place = hd ? hd_place(hd_rows, n_hd, t * kWgRows) : 0;   // of the tile's first high-degree row
                // kRpg rows at a time, whichever they are: lane group g holds the g-th of what is left.  (By sweeps, whose rows
                // stand side by side, a tile with one such row in every sweep took kG turns: 79 thousand rows of a multiplier, 32 x 64,
                // whole call 28.8 us, now 27.7; Booth shape, 10 thousand rows, 64 x 64 32.8, now 31.1.)
#pragma unroll 1
                while (redo) {
                    int lr[kRpg];                        // scalars: the turn's rows, -1 past the last
#pragma unroll
                    for (int i = 0; i < kRpg; ++i) {
                        lr[i] = redo ? __builtin_ctz(redo) : -1;
                        redo &= redo - 1;
                    }
                    int mine = lr[0], of_z[kP];          // of the lane's float4 of X, of its values of dZ
#pragma unroll
                    for (int p = 0; p < kP; ++p) of_z[p] = lr[p];
#pragma unroll
                    for (int i = 1; i < kRpg; ++i) {
                        if (g == i) mine = lr[i];
#pragma unroll
                        for (int p = 0; p < kP; ++p)
                            if (kq * kP + p == i) of_z[p] = lr[i];
                    }
                    const v4f zero = {0.f, 0.f, 0.f, 0.f};
                    ZVec z[kP];
#pragma unroll
                    for (int p = 0; p < kP; ++p)
                        z[p] = of_z[p] >= 0 ? __builtin_nontemporal_load((const ZVec *)(dZ + ((t * kWgRows + of_z[p]) << kZShift) + 4 * kNb * jl))
                                            : (ZVec)(0.f);
                    const int row = mine >= 0 ? mine : 0;
                    const int64_t s = __shfl(rp, row), e = __shfl(rp, row + 1);
                    v4f a = zero, own = zero;
                    if (mine >= 0) {
                        if (ragged) own = *(const v4f *)(Xf + ((t * kWgRows + mine) << kRowShift));
                        if ((hd >> mine) & 1)
                            a = *(const v4f *)(hd_agg + ((int64_t)(place + __popc(hd & ((1u << mine) - 1))) << kRowShift) + 16 * f);
                        else if (ragged || e - s > D)
                            a = row_sum_ahead<W>(s, e, col, Xf, kRowShift, zero_off);
                    }
                    multiply(0, a, z);
                    if (ragged) multiply(kMc, own, z);
                }
            }
            if constexpr (kFold) {
                until_fold -= pending;
                if (until_fold == 0) fold_now();
            }
        }
    }
    // ---- the workgroup's slice of the workspace: its wavefronts' sums, in wavefront order, in fp64; stored as the
    //      accumulators lie (block, lane, register), which the reducing kernel undoes
    constexpr int kVecs = kMb * kNb * kWave, kMine = (kVecs + kWgWaves * kWave - 1) / (kWgWaves * kWave);
    double t[kMine][4];
#pragma unroll
    for (int i = 0; i < kMine; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) t[i][r] = 0.0;
    if constexpr (kFold) fold();
#pragma unroll 1
    for (int first = 0; first < kWgWaves; first += kBufs) {
        if constexpr (!kFold) {                          // kBufs wavefronts at a time
            if (w >= first && w < first + kBufs) {
#pragma unroll
                for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
                    for (int nb = 0; nb < kNb; ++nb) s_sum[w - first][mb * kNb + nb][l] = acc[mb][nb];
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const int e = i * kWgWaves * kWave + threadIdx.x;
            if (e < kVecs)
                for (int q = 0; q < kBufs; ++q) {
                    const v4f v = (&s_sum[q][0][0])[e];
#pragma unroll
                    for (int r = 0; r < 4; ++r) t[i][r] += (double)v[r];
                }
        }
        __syncthreads();
    }
    wg_d2 *mine = partials + (int64_t)blockIdx.x * kVecs * 2;
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int e = i * kWgWaves * kWave + threadIdx.x;
        if (e < kVecs) {
            mine[e] = (wg_d2){t[i][0], t[i][1]};         // registers 0 and 1 of all lanes, then 2 and 3: whole lines per store
            mine[kVecs + e] = (wg_d2){t[i][2], t[i][3]};
        }
    }
}

// dWn[m][n] (m < FI) and dWs[m - FI][n] = sum over the workgroups' slices in fp64, in a fixed order.  A workgroup takes
// 16 pairs of a slice's numbers; its 16 groups of 16 threads take every 16th slice each, so that a slice count of 256 is 16
// loads in flight per thread and one latency (one thread per element walking 2,048 slices took 42 us at 64 x 64 and 94 us at
// 32 x 32, where 8 workgroups had it all), then the groups are added in order.
constexpr int kWgRedVec = 16, kWgRedGroups = kBlock / kWgRedVec;
template <int FI, int FO>
__global__ __launch_bounds__(kBlock) void sage_wgrad_reduce_kernel(const wg_d2 *__restrict__ partials, int64_t slices,
                                                                   float *__restrict__ dWn, float *__restrict__ dWs)
{
    constexpr int kMc = FI / 16, kNb = FO / 16, kPairs = 2 * FI * FO / 2;
    static_assert(kPairs % kWgRedVec == 0, "whole workgroups");
    __shared__ double s_part[kWgRedGroups][kWgRedVec][2];
    const int v = threadIdx.x % kWgRedVec, grp = threadIdx.x / kWgRedVec;
    wg_d2 t = {0.0, 0.0};
#pragma unroll 16
    for (int64_t k = grp; k < slices; k += kWgRedGroups) t += partials[k * kPairs + blockIdx.x * kWgRedVec + v];
    s_part[grp][v][0] = t[0];
    s_part[grp][v][1] = t[1];
    __syncthreads();
    if (threadIdx.x >= kWgRedVec * 2) return;
    double sum = 0.0;
    for (int q = 0; q < kWgRedGroups; ++q) sum += (&s_part[q][0][0])[threadIdx.x];
    // pair of the slice: registers 0 and 1 of every block and lane, then registers 2 and 3
    const int at = blockIdx.x * kWgRedVec + threadIdx.x / 2, half = at / (kPairs / 2), e = at % (kPairs / 2);
    const int blk = e / kWave, lane = e % kWave, r = 2 * half + threadIdx.x % 2;
    const int mb = blk / kNb, nb = blk % kNb;            // accumulator acc[mb][nb]: rows 4 (lane / 16) + r, column lane % 16
    float *out = mb < kMc ? dWn : dWs;
    out[wg_feature<FI>(4 * (lane / 16) + r, mb % kMc) * FO + kNb * (lane % 16) + nb] = (float)sum;
}

static int64_t wgrad_workgroups()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return -1;
    int64_t n_wg = cus / kXcds * kXcds;                  // one workgroup per CU; consecutive workgroup ids land on different XCDs
    return n_wg < kXcds ? kXcds : n_wg;
}

// bytes of workspace that launch_sage_wgrad asks for at these widths on the current device (0 on failure): 2 F_in F_out
// floats per SIMD (F_in = 64) or twice that (32).  The kernel fills 2 F_in F_out doubles per workgroup, a half or a quarter of
// it; the size is part of the interface.
size_t sage_wgrad_workspace_bytes(int32_t FI, int32_t FO)
{
    const int64_t n_wg = wgrad_workgroups();
    return n_wg < 0 ? 0 : (size_t)n_wg * (FI == 64 ? 4 : 8) * 2 * (size_t)FI * (size_t)FO * sizeof(float);
}

template <int FI, int FO>
static int wgrad_launch(const DevicePlan &dp, const float *X, const float *dZ, float *dWn, float *dWs, void *workspace,
                        hipStream_t st)
{
    const int64_t cu_wg = wgrad_workgroups();
    if (cu_wg < 0) return (int)hipErrorInvalidDevice;
    const int64_t n_tiles = (dp.n + kWgRows - 1) / kWgRows;
    const int32_t parts = dp.xcd_remap ? kXcds : 1;
    const int64_t tiles_per_part = (n_tiles + parts - 1) / parts;
    // no more workgroups than tiles: a slice without rows would be written and read for nothing
    const int64_t wanted = (tiles_per_part + kWgWaves - 1) / kWgWaves * parts;
    const int64_t n_wg = wanted < cu_wg ? wanted : cu_wg / parts * parts;
    const int64_t waves_per_part = n_wg / parts * kWgWaves;
    if (!grid_ok(n_wg) || n_tiles <= 0) return (int)hipErrorInvalidConfiguration;
    // the kernel reads entry 0 of the index array from idle lanes: give it something to read when the matrix has no entries
    const int32_t *col_arg = dp.col ? dp.col : (const int32_t *)dp.rowptr;
#define GROOT_WGRAD_LAUNCH(WM, DD)                                                                                      \
    sage_wgrad_kernel<WM, FI, FO, DD><<<dim3((unsigned)n_wg), dim3(kWgWaves * kWave), 0, st>>>(                            \
        dp.rowptr, col_arg, (const char *)X, (const char *)dZ, byte_distance(X, dp.zero_row), dp.n, dp.nnz, dp.threshold, \
        n_tiles, tiles_per_part, waves_per_part, parts, dp.hd_rows, (int32_t)dp.n_hd_rows, (const char *)dp.hd_agg,    \
        (wg_d2 *)workspace)
    if (dp.weight_mode == kMean) {
        if (dp.sage_depth == 5) GROOT_WGRAD_LAUNCH(kMean, 5);
        else if (dp.sage_depth == 6) GROOT_WGRAD_LAUNCH(kMean, 6);
        else GROOT_WGRAD_LAUNCH(kMean, 8);
    } else {
        if (dp.sage_depth == 5) GROOT_WGRAD_LAUNCH(kOnes, 5);
        else if (dp.sage_depth == 6) GROOT_WGRAD_LAUNCH(kOnes, 6);
        else GROOT_WGRAD_LAUNCH(kOnes, 8);
    }
#undef GROOT_WGRAD_LAUNCH
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return (int)err;
    sage_wgrad_reduce_kernel<FI, FO><<<dim3(2 * FI * FO / 2 / kWgRedVec), dim3(kBlock), 0, st>>>((const wg_d2 *)workspace, n_wg, dWn, dWs);
    return (int)hipGetLastError();
}

int launch_sage_wgrad(const DevicePlan &dp, const float *X, const float *dZ, float *dWn, float *dWs, int32_t FI, int32_t FO,
                      void *workspace, void *stream)
{
    if (!weights_ok(dp) || !dp.zero_row || (FI != 64 && FI != 32) || (FO != 64 && FO != 32 && FO != 16) || !workspace)
        return (int)hipErrorInvalidValue;
    if (dp.weight_mode == kExplicit) return (int)hipErrorInvalidValue;
    if (dp.n_hd_rows && (!dp.hd_rows || !dp.hd_agg)) return (int)hipErrorInvalidValue;
    hipStream_t st = (hipStream_t)stream;
    if (FI == 64) {
        if (FO == 64) return wgrad_launch<64, 64>(dp, X, dZ, dWn, dWs, workspace, st);
        if (FO == 32) return wgrad_launch<64, 32>(dp, X, dZ, dWn, dWs, workspace, st);
        return wgrad_launch<64, 16>(dp, X, dZ, dWn, dWs, workspace, st);
    }
    if (FO == 64) return wgrad_launch<32, 64>(dp, X, dZ, dWn, dWs, workspace, st);
    if (FO == 32) return wgrad_launch<32, 32>(dp, X, dZ, dWn, dWs, workspace, st);
    return wgrad_launch<32, 16>(dp, X, dZ, dWn, dWs, workspace, st);
}

}  // namespace groot
