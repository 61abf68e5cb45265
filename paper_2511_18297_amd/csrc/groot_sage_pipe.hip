// Fused GraphSAGE-mean layer for gfx950, self-contained wavefronts (two per SIMD):
//     H = act((A_hat X) Wn + X Ws + b),   X [N, FI], Wn and Ws [FI, FO], H [N, FO], FI = 32 or 64, FO = 16, 32 or 64
//     (described below for FI = FO = 64).
//
// The aggregation is the software-pipelined LD kernel's (a persistent workgroup per CU, every wavefront walks
// its own tiles and keeps a whole tile of gathers in flight; slot table in LDS, zero row for dead slots, no
// workgroup barrier after the start).  A tile here is 16 rows, the height of a matrix instruction.  Instead
// of storing the 16 sums, the wavefront parks [A_hat X | X] of its tile in its own LDS region, multiplies it
// with the stacked weights [Wn; Ws] (128 x 64) on the matrix cores and stores the result from the accumulators, whole
// 128-byte lines per instruction.  Nothing is shared between wavefronts, so nothing
// waits for another wavefront; while a wavefront multiplies, the gathers of its next tile are in flight, and
// the second wavefront of its SIMD issues whenever the first one waits (with one wavefront per SIMD, which
// could keep the weights in registers, every wait of that wavefront idles the SIMD: 25.9 against 24.5 ms of
// the 12-wavefront kernel).
//
// The dense product keeps fp32 accuracy on the bf16 matrix instruction (v_mfma_f32_16x16x32_bf16, a sixteenth
// of the fp32 instruction's time per multiply-add): every fp32 operand is cut into three bf16 pieces,
// x = hi + mid + lo up to 2^-24 |x|, and a product keeps the six piece products down to 2^-16 relative size
// (hi hi, hi mid, mid hi, hi lo, lo hi, mid mid; the dropped ones are below 2^-24), summed in fp32 in the
// instruction's accumulator.  The weights are cut once per workgroup into LDS, in the operand layout of the
// instruction (48 KB, one 16-byte read per lane and operand); the tile is cut when it is parked.
// With two pieces instead of three (template argument P; a knob of the library, off by default) a product keeps
// hi hi, hi mid and mid hi: what is dropped and what the two pieces do not represent stays below 3 x 2^-18 of
// |x| |w| per product, a bar twice as wide as fp32's for half the matrix instructions.
//
// The layer's gradient with respect to its input runs through the same kernel (template argument SD).  With
// dZ the gradient at the layer's pre-activation output, dX = A_hat^T (dZ Wn^T) + dZ Ws^T = (A_hat^T dZ) Wn^T + dZ Ws^T,
// and for a symmetric adjacency with mean weights A_hat^T = A D^-1: the aggregation is the plain (unit-weight)
// sum of the rows of dZ / deg, which the caller hands over, and the row's own part is that row times its length
// again.  So SD is the layer with unit weights whose own-row operand is scaled by the row's stored length.
//
// High-degree rows are aggregated beforehand by the HD kernel into a side buffer of the plan, one row per
// high-degree row in ascending order of their ids.  Such a row, and one with more than D entries, has no live slot: the
// loop's own sum of it is zero, and before the tile is multiplied a branch parks the right one over it, straight from
// global memory or from the side buffer (the row's place in it by a search over the list of high-degree rows).  The same
// path computes the ragged last tile behind the loop.  All other loads and stores of the loop are unconditional.
// A tile that was dropped, noted and computed as a whole behind the loop, high-degree rows by binary search, instead:
// 1 M rows, 1 in 100 of 9 to 12 entries, 64 -> 64 309 us, now 209; 1 in 25 474, now 230; polarized degrees, 1 M rows 635,
// now 483; multipliers, where one tile in 600 has such a row, the same to 2 % better.
//
// What bounds it: at 64 x 64 the power the chip grants dense bf16 matrix work beside the memory traffic (it runs at
// 1.4 to 1.7 GHz).  Scalar tile arithmetic, the result stored from the accumulators, whole tiles only in the loop
// (390 instead of 500 vector instructions per tile): 8.4 M rows of carry-save multipliers, 64 -> 64: 1,285 -> 1,215 us,
// 32 -> 32: 617 -> 580 us (lines stored by halves instead: 1,364 and 675 us, 9 % more bytes written).
#include <type_traits>

#include "groot_device.h"

namespace groot {

constexpr int kSpRows = 16;                  // rows per tile: the height of a matrix instruction

// Shapes for FI input and FO output features and NW wavefronts per workgroup (one workgroup per CU).
template <int FI, int FO, int NW>
struct SpCfg {
    static constexpr int kWaves = NW;
    static constexpr int kL = FI / 4;                // lanes per input row, one float4 each
    static constexpr int kRpg = kWave / kL;          // input rows per lane-group sweep
    static constexpr int kG = kSpRows / kRpg;        // sweeps per tile
    static constexpr int kRowShift = FI == 64 ? 8 : 7;   // log2 of an input row's bytes
    static constexpr int kK = 2 * FI;                // contraction length: [agg | self]
    static constexpr int kKs = kK / 32;              // k blocks of a matrix instruction
    static constexpr int kNb = FO / 16;              // blocks of 16 output columns
    static constexpr int kBRow = kK * 2 + 16;        // bytes per LDS row of one bf16 plane (16 B of padding: conflict-free)
    static constexpr int kPlane = kSpRows * kBRow;
    static constexpr int kORowShift = FO == 64 ? 8 : FO == 32 ? 7 : 6;   // log2 of an output row's bytes
    static_assert(FI == 64 || FI == 32, "input width");
    static_assert(FO == 64 || FO == 32 || FO == 16, "output width");
};

typedef __bf16 sp_bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 sp_bf8 __attribute__((ext_vector_type(8)));
typedef unsigned int sp_u4 __attribute__((ext_vector_type(4)));
typedef unsigned int sp_u2 __attribute__((ext_vector_type(2)));
typedef float sp_f2 __attribute__((ext_vector_type(2)));

// two fp32 values -> their bf16 roundings (nearest even), packed: a in the low half
__device__ __forceinline__ unsigned sp_pack2(float a, float b)
{
    const sp_f2 x = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(x, sp_bf2));
}

// (a, b) = hi + mid + lo, three packed bf16 pairs; the remainders are exact in fp32
__device__ __forceinline__ void sp_split3(float a, float b, unsigned &hi, unsigned &mid, unsigned &lo)
{
    hi = sp_pack2(a, b);
    float ra = a - __builtin_bit_cast(float, hi << 16), rb = b - __builtin_bit_cast(float, hi & 0xffff0000u);
    mid = sp_pack2(ra, rb);
    ra -= __builtin_bit_cast(float, mid << 16);
    rb -= __builtin_bit_cast(float, mid & 0xffff0000u);
    lo = sp_pack2(ra, rb);
}

// four consecutive elements k..k+3 of tile row `row` into the P planes (row stride kBRow, plane size kPlane)
template <int kBRow, int kPlane, int P>
__device__ __forceinline__ void sp_park(char *tile, int row, int k, v4f x)
{
    unsigned h0, m0, l0, h1, m1, l1;
    sp_split3(x[0], x[1], h0, m0, l0);                   // P = 2: the third piece is never used and is not computed
    sp_split3(x[2], x[3], h1, m1, l1);
    char *p = tile + row * kBRow + k * 2;
    *(sp_u2 *)p = (sp_u2){h0, h1};
    *(sp_u2 *)(p + kPlane) = (sp_u2){m0, m1};
    if constexpr (P == 3) *(sp_u2 *)(p + 2 * kPlane) = (sp_u2){l0, l1};
}

// W: kOnes or kMean; D: gather slots per row on the pipelined path; P: bf16 pieces per fp32 operand, 3 or 2
template <int W, int FI, int FO, int NW, int D, int P, bool SD = false>
__global__ __launch_bounds__(NW * kWave) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void sage_pipe_kernel(
    const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col, const char *__restrict__ X, char *H, int64_t zero_off,
    const float *__restrict__ Wn, const float *__restrict__ Ws, const float *__restrict__ bias, int relu, int64_t n, int64_t nnz,
    int32_t T, int64_t n_tiles, int64_t tiles_per_part, int64_t waves_per_part, int32_t parts,
    const int32_t *__restrict__ hd_rows, int32_t n_hd, const char *__restrict__ hd_agg)
{
    static_assert(P == 3 || P == 2, "pieces per operand");
    static_assert(!SD || W == kOnes, "the own-row operand is scaled by the row length in the unit-weight form only");
    static_assert(W == kOnes || W == kMean, "row-uniform weights");
    using C = SpCfg<FI, FO, NW>;
    constexpr int F = FI;
    constexpr int kSpD = D, kSpSlots = kSpRows * kSpD, kSpH = (kSpSlots + kWave - 1) / kWave;
    constexpr int kSpWaves = C::kWaves, kSpL = C::kL, kSpRpg = C::kRpg, kSpG = C::kG, kRowShift = C::kRowShift;
    constexpr int kKs = C::kKs, kNb = C::kNb, kSpBRow = C::kBRow, kSpPlane = C::kPlane;
    __shared__ __align__(16) int64_t s_slot[kSpWaves][kSpSlots];
    __shared__ float s_inv[kSpWaves][kSpRows];
    __shared__ __align__(16) char s_A[kSpWaves][P * kSpPlane];           // F = 64, P = 3: 13,056 B per wavefront
    __shared__ __align__(16) sp_u4 s_W[kNb][kKs][P][kWave];              // F = 64, P = 3: 49,152 B: [nb][ks][piece][lane] weight operands
    __shared__ __align__(16) float s_bias[FO];

    // the wavefront's number as a scalar: the tile arithmetic below then runs on the scalar unit, and vector instructions
    // are what this kernel is short of
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int g = l / kSpL, f = l % kSpL;
    const int kq = l / 16, jl = l % 16;                  // matrix instruction: k block / weight column (A), tile row (B, D)
    const int64_t part = blockIdx.x % parts, j = (blockIdx.x / parts) * kSpWaves + w;
    const int64_t x_begin = part * tiles_per_part;
    const int64_t x_end = x_begin + tiles_per_part < n_tiles ? x_begin + tiles_per_part : n_tiles;
    const int64_t t_first = x_begin + j, stride = waves_per_part;
    const int64_t n_full = n / kSpRows, x_full = x_end < n_full ? x_end : n_full;   // whole tiles
    const char *Xf = X + 16 * f;

    // ---- CSR pipeline: rp_a and cc belong to the next tile to be staged, rp_b to the one after
    int64_t rp_a = 0, rp_b = 0;
    int32_t cc[kSpH];
    bool fix_a = false;                                  // the tile has rows that the slots do not serve
    int32_t len_a = 0;                                   // lanes 0..kSpRows-1: stored length of the tile's row
    uint32_t live_a = 0;                                 // bit h: slot l + 64 h holds an entry
    auto load_rp = [&](int64_t tile) -> int64_t {
        const int64_t ri = tile * kSpRows + (l < kSpRows ? l : kSpRows);
        return rowptr[ri < n ? ri : n];                  // lanes 0..kSpRows hold the pointers; rows past the end read rowptr[n]: no entries
    };
    auto load_cols = [&]() {                             // from rp_a: every slot fetches its own entry
        const uint32_t begin_lo = __builtin_amdgcn_readfirstlane((uint32_t)rp_a);
        const int64_t begin = (int64_t)((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)rp_a >> 32)) << 32 | begin_lo);
        const int32_t *const tile_col = col + (begin < nnz ? begin : 0);   // a dead slot reads the tile's first entry, or entry 0
        const int32_t rel = (int32_t)((uint32_t)rp_a - begin_lo);
        len_a = __shfl_down(rel, 1) - rel;
        // a row with more entries than slots, or a high-degree row, has no live slot: patch() serves it
        fix_a = __ballot(l < kSpRows && (len_a > kSpD || len_a >= T)) != 0;
        live_a = 0;
        // unconditional loads: the number of loads in flight stays known
#pragma unroll
        for (int h = 0; h < kSpH; ++h) {
            const int s = l + kWave * h;                 // slot s: row r, entry k
            const int r = s / kSpD, k = s - r * kSpD;
            const int32_t lo = __shfl(rel, r), len = __shfl(rel, r + 1) - lo;
            const bool live = s < kSpSlots && k < len && len <= kSpD && len < T;
            live_a |= (uint32_t)live << h;
            cc[h] = __builtin_nontemporal_load(&tile_col[live ? (uint32_t)(lo + k) : 0u]);
        }
    };
    auto stage = [&]() -> bool {                         // cc, live_a, len_a -> slot table and row weights; -> fix_a
#pragma unroll
        for (int h = 0; h < kSpH; ++h) {
            const int s = l + kWave * h;
            if (s < kSpSlots) s_slot[w][s] = ((live_a >> h) & 1) ? ((int64_t)cc[h] << kRowShift) : zero_off;
        }
        if (W == kMean && l < kSpRows) s_inv[w][l] = row_weight<kMean>(len_a);
        if (SD && l < kSpRows) s_inv[w][l] = (float)len_a;   // exact: a row that the slots serve has few entries
        wave_sync();
        return fix_a;
    };

    // ---- the row pointers of the first tiles, then the weights, then the first tile's columns are on their way, and the weights
    //      are cut while those arrive: three latencies before the first gather is issued instead of six.  On small graphs, one
    //      tile per wavefront, that is most of the launch (kernel on 32 thousand rows, 32 -> 32: 7.8 us, now 7.1; call on 157 thousand, 64 -> 64:
    //      33.5, now 32.0; a training step on 32 thousand rows is bound by the host and takes what it took).
    rp_a = load_rp(t_first);
    const int64_t rp_second = load_rp(t_first + stride);
    rp_b = load_rp(t_first + 2 * stride);
    // The weights, cut once per workgroup: s_W[nb][ks][piece][lane] is the operand of output columns
    // 16 nb .. 16 nb + 15 for k = 32 ks + 8 kq + e, e = 0..7.  The wavefronts share the (nb, ks) pairs.
    // Every wavefront reaches this barrier (none has left yet).
    {
        constexpr int kPairs = kNb * kKs, kMine = (kPairs + kSpWaves - 1) / kSpWaves;
        float raw[kMine][8];
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const int c = w + i * kSpWaves < kPairs ? w + i * kSpWaves : 0, nb = c / kKs, ks = c % kKs, jcol = 16 * nb + jl;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = 32 * ks + 8 * kq + e;
                raw[i][e] = k < F ? Wn[k * FO + jcol] : Ws[(k - F) * FO + jcol];
            }
        }
        if (threadIdx.x < FO) s_bias[threadIdx.x] = bias ? bias[threadIdx.x] : 0.0f;
        __builtin_amdgcn_sched_barrier(0);
        load_cols();                                     // also without a tile: rows past the end have no entries
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const int c = w + i * kSpWaves, nb = c / kKs, ks = c % kKs;
            if (c < kPairs) {
                sp_u4 pc[3];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    unsigned h, m, lo_;
                    sp_split3(raw[i][e], raw[i][e + 1], h, m, lo_);
                    pc[0][e / 2] = h;
                    pc[1][e / 2] = m;
                    pc[2][e / 2] = lo_;
                }
#pragma unroll
                for (int q = 0; q < P; ++q) s_W[nb][ks][q][l] = pc[q];
            }
        }
    }
    __syncthreads();
    if (t_first >= x_end) return;

    // ---- one group: kSpRpg rows, one per lane group: the row's own features and its kSpD slots
    struct Regs {
        v4f xs[kSpD], self;
        float inv;
    };
    constexpr int kSets = D <= 6 ? kSpG : kSpG / 2;      // sweeps in flight: a whole tile (half of it: 2 % slower), or what registers allow
    Regs rr[kSets];
    // Whether the next tile's gathers arrive before this tile is multiplied.  Where the matrix instructions bound the kernel
    // they are left in flight; on the other widths the memory system does better with fewer requests (8.4 M rows of
    // carry-save multipliers, left in flight and drained: 64 -> 64 1,215 and 1,212 us, on 4.3 M rows of the Booth shape 682 and
    // 691; 64 -> 16 868 and 828, 32 -> 64 804 and 782, 32 -> 16 506 and 484; two pieces per operand, 64 -> 64 1,125 and 1,109,
    // 32 -> 32 576 and 552).  With 8 slots only half a tile is in flight: 4-LUT shape, 64 -> 64 254 and 260 us.
    constexpr bool kDrain = D <= 6 && !(FI == 64 && FO == 64 && P == 3);
    const uint32_t x_lane = (uint32_t)g << kRowShift | 16 * f;
    auto issue = [&](Regs &q, int64_t tile, int grp) {   // the tile whose slots are staged; a whole one
        const int lr = grp * kSpRpg + g;
        if (W == kMean || SD) q.inv = s_inv[w][lr];
#pragma unroll
        for (int k = 0; k < kSpD; ++k) q.xs[k] = *(const v4f *)(Xf + s_slot[w][lr * kSpD + k]);
        q.self = *(const v4f *)(X + (tile << kRowShift) * kSpRows + x_lane + ((grp * kSpRpg) << kRowShift));
    };
    auto sum = [&](const Regs &q) -> v4f {
        v4f a = q.xs[0];
#pragma unroll
        for (int k = 1; k < kSpD; ++k) a += q.xs[k];
        if (W == kMean) a *= q.inv;
        return a;
    };
    char *const a_tile = s_A[w];
    v4f bias4[kNb];                                      // this lane's output features 16 nb + 4 kq .. + 3
#pragma unroll
    for (int nb = 0; nb < kNb; ++nb) bias4[nb] = *(const v4f *)&s_bias[16 * nb + 4 * kq];
    // ---- [Wn; Ws]^T (FO x 2F) times the parked tile [agg | self]^T (2F x 16), + bias: the weights are the instruction's
    //      first operand, so that lane (jl, kq) ends with features 16 nb + 4 kq .. + 3 of tile row jl and stores them as
    //      they are.  (With the tile as first operand a lane holds one feature of four rows, and the result went through
    //      LDS once more.)
    auto multiply = [&](v4f (&acc)[kNb]) {
        const char *a_lane = a_tile + jl * kSpBRow + 16 * kq;
        // P kKs steps (ks, weight piece pb = hi, mid, lo), each against the tile pieces whose product is kept
        // (P = 3: hi with lo, mid, hi; mid with mid, hi; lo with hi.  P = 2: hi with mid, hi; mid with hi), on kNb
        // independent accumulators.  The weight operands of step s + 1 are read from LDS while step s runs; a tile
        // piece of the next ks is read as soon as its register is dead (the last piece after the first step, the one
        // before it after the second, hi after the last step, where the first matrix instructions of the next ks do
        // not need it yet).
        sp_u4 aop[P], bop[2][kNb];
        auto read_a = [&](int ks, int pc) { aop[pc] = *(const sp_u4 *)(a_lane + pc * kSpPlane + 64 * ks); };
        auto read_b = [&](int s_) {
            const int ks = s_ / P, pb = s_ % P;
#pragma unroll
            for (int nb = 0; nb < kNb; ++nb) bop[s_ & 1][nb] = s_W[nb][ks][pb][l];
        };
#pragma unroll
        for (int pc = P - 1; pc >= 0; --pc) read_a(0, pc);
        read_b(0);
#pragma unroll
        for (int s_ = 0; s_ < P * kKs; ++s_) {
            const int ks = s_ / P, pb = s_ % P;
            if (s_ + 1 < P * kKs) read_b(s_ + 1);
            if (ks + 1 < kKs && pb >= 1) read_a(ks + 1, P - pb);     // piece P - pb was last used in the step before this one
            __builtin_amdgcn_sched_barrier(0);                       // the reads stay ahead of this step's matrix instructions
#pragma unroll
            for (int pa = P - 1 - pb; pa >= 0; --pa)
#pragma unroll
                for (int nb = 0; nb < kNb; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(sp_bf8, bop[s_ & 1][nb]),
                                                                      __builtin_bit_cast(sp_bf8, aop[pa]),
                                                                      s_ == 0 && pa == P - 1 ? bias4[nb] : acc[nb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (ks + 1 < kKs && pb == P - 1) read_a(ks + 1, 0);      // hi after the last step
        }
        if (relu) {
#pragma unroll
            for (int nb = 0; nb < kNb; ++nb)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[nb][r] = acc[nb][r] > 0.0f ? acc[nb][r] : 0.0f;
        }
    };
    // whole 128-byte lines per store instruction: neighbouring lanes (tile rows 2 i and 2 i + 1) swap half of their blocks
    const bool odd = (jl & 1) != 0;
    const uint32_t h_lane = (uint32_t)(kNb > 1 ? jl & ~1 : jl) << C::kORowShift | (kNb > 1 && odd ? 64 : 0) | 16 * kq;
    auto swap1 = [](float x) -> float {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, false));
    };
    auto store = [&](char *rows, const v4f (&acc)[kNb], int live) {   // live: rows of the tile that exist
        if constexpr (kNb == 1) {
            if (jl < live) __builtin_nontemporal_store(acc[0], (v4f *)(rows + h_lane));
        } else {
#pragma unroll
            for (int nb = 0; nb < kNb; nb += 2) {
                v4f x, y;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float got = swap1(odd ? acc[nb][r] : acc[nb + 1][r]);
                    x[r] = odd ? got : acc[nb][r];
                    y[r] = odd ? acc[nb + 1][r] : got;
                }
                if ((jl & ~1) < live) __builtin_nontemporal_store(x, (v4f *)(rows + h_lane + 64 * nb));
                if ((jl | 1) < live) __builtin_nontemporal_store(y, (v4f *)(rows + h_lane + 64 * nb + (1 << C::kORowShift)));
            }
        }
    };

    // ---- rows of a tile straight from global memory into the parked tile (A_hat X only), one per lane group: rows with more
    //      entries than slots are summed here, high-degree rows come from the side buffer
    auto patch = [&](int64_t t, bool all) {
        const int64_t rp = load_rp(t), next_rp = __shfl_down(rp, 1);
        const int64_t mine = l < kSpRows ? next_rp - rp : 0;
        const uint32_t hd = (uint32_t)__ballot(l < kSpRows && mine >= T);
        const int32_t place = hd ? hd_place(hd_rows, n_hd, t * kSpRows) : 0;   // of the tile's first high-degree row
        uint32_t rows = (uint32_t)__ballot(l < kSpRows && (all || mine > kSpD || mine >= T));
#pragma unroll 1
        while (rows) {
            uint32_t left = rows;                        // lane group g takes the g-th row that is left
#pragma unroll
            for (int i = 0; i < kSpRpg; ++i) {
                if (i < g) left &= left - 1;
                rows &= rows - 1;
            }
            const int lr = left ? __builtin_ctz(left) : 0;
            const int64_t s = __shfl(rp, lr), e = __shfl(rp, lr + 1);
            if (left) {
                const v4f a = (hd >> lr) & 1
                    ? *(const v4f *)(hd_agg + ((int64_t)(place + __popc(hd & ((1u << lr) - 1))) << kRowShift) + 16 * f)
                    : row_sum_ahead<W>(s, e, col, Xf, kRowShift, zero_off);
                sp_park<kSpBRow, kSpPlane, P>(a_tile, lr, 4 * f, a);
            }
        }
    };

    int64_t tile = t_first;
    if (tile < x_full) {
        // ---- prologue: the first tile is staged and put in flight, the CSR of the next two is on its way
        bool fix_cur = stage();
        rp_a = rp_second;
        load_cols();
#pragma unroll
        for (int grp = 0; grp < kSets; ++grp) issue(rr[grp], tile, grp);
        __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): the loop's own order of loads is the only one from here on

        for (; tile < x_full; tile += stride) {
            const int64_t next = tile + stride < n_full ? tile + stride : n_full - 1;
            bool fix_next = false;
            // sums of this tile -> LDS, cut into bf16 pieces; a register set then takes the sweep kSets later
#pragma unroll
            for (int grp = 0; grp < kSpG; ++grp) {
                if (grp == kSpG - kSets) {               // this tile's sweeps are all issued: CSR of the next tile -> slot table
                    fix_next = stage();
                    rp_a = rp_b;
                    load_cols();
                    rp_b = load_rp(tile + 3 * stride);
                }
                Regs &q = rr[grp % kSets];
                const v4f a = sum(q);
                sp_park<kSpBRow, kSpPlane, P>(a_tile, grp * kSpRpg + g, 4 * f, a);
                sp_park<kSpBRow, kSpPlane, P>(a_tile, grp * kSpRpg + g, F + 4 * f, SD ? q.self * q.inv : q.self);
                issue(q, grp + kSets < kSpG ? tile : next, (grp + kSets) % kSpG);
            }
            if (fix_cur) patch(tile, false);             // the rows that had no live slots, parked again
            if constexpr (kDrain) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
            wave_sync();
            v4f acc[kNb];
            multiply(acc);
            store(H + (tile << C::kORowShift) * kSpRows, acc, kSpRows);
            wave_sync();                              // the tile in LDS is free for the next round
            fix_cur = fix_next;
        }
    }
    if (tile < x_end) {                                  // the ragged last tile
        const int64_t rp = load_rp(tile), next_rp = __shfl_down(rp, 1);
#pragma unroll 1
        for (int grp = 0; grp < kSpG; ++grp) {
            const int lr = grp * kSpRpg + g;
            const int64_t row = tile * kSpRows + lr;
            v4f own = *(const v4f *)(Xf + ((row < n ? row : n - 1) << kRowShift));   // past the end: not stored
            if (SD) own *= (float)__shfl(next_rp - rp, lr);
            sp_park<kSpBRow, kSpPlane, P>(a_tile, lr, F + 4 * f, own);
        }
        patch(tile, true);                               // rows past the end: no entries
        wave_sync();
        v4f acc[kNb];
        multiply(acc);
        store(H + (tile << C::kORowShift) * kSpRows, acc, (int)(n - tile * kSpRows));
    }
}

// out[i, :] = Z[i, :] / (stored length of row i), one lane per float4; out may be Z
__global__ __launch_bounds__(kBlock) void rows_over_degree_kernel(const int64_t *__restrict__ rowptr, const v4f *Z, v4f *out,
                                                                  int64_t n, int32_t F4)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n * F4) return;
    const int64_t row = i / F4;
    const float d = (float)(rowptr[row + 1] - rowptr[row]);
    const v4f z = Z[i];
    out[i] = d > 0.f ? (v4f){z[0] / d, z[1] / d, z[2] / d, z[3] / d} : (v4f){0.f, 0.f, 0.f, 0.f};
}

int launch_rows_over_degree(const DevicePlan &dp, const float *Z, float *out, int32_t F, void *stream)
{
    const int64_t total = dp.n * (int64_t)(F / 4), grid = (total + kBlock - 1) / kBlock;
    if (total == 0) return 0;
    if (!grid_ok(grid)) return (int)hipErrorInvalidConfiguration;
    rows_over_degree_kernel<<<dim3((unsigned)grid), dim3(kBlock), 0, (hipStream_t)stream>>>(dp.rowptr, (const v4f *)Z, (v4f *)out,
                                                                                          dp.n, F / 4);
    return (int)hipGetLastError();
}

int launch_sage_pipe(const DevicePlan &dp, const float *X, float *H, const float *Wn, const float *Ws, const float *bias,
                     int relu, int32_t FI, int32_t FO, int pieces, int self_times_degree, void *stream)
{
    if (!weights_ok(dp) || !dp.zero_row || (FI != 64 && FI != 32) || (FO != 64 && FO != 32 && FO != 16) ||
        (pieces != 2 && pieces != 3))
        return (int)hipErrorInvalidValue;
    // row-uniform weights only: with explicit weights the slot table is twice as large and LDS does not hold it
    if (dp.weight_mode == kExplicit) return (int)hipErrorInvalidValue;
    const int wm = self_times_degree ? (int)kOnes : dp.weight_mode;
    if (dp.n_hd_rows && (!dp.hd_rows || !dp.hd_agg)) return (int)hipErrorInvalidValue;
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return (int)e;
    // wavefronts per workgroup: two per SIMD (at F = 32 three fit and are slower: 11.4 against 10.2 ms)
    constexpr int kNwRun = 8;
    const int64_t n_tiles = (dp.n + kSpRows - 1) / kSpRows;
    // one workgroup per CU; consecutive workgroup ids land on different XCDs
    int64_t n_wg = cus / kXcds * kXcds;
    if (n_wg < kXcds) n_wg = kXcds;
    const int32_t parts = dp.xcd_remap ? kXcds : 1;
    const int64_t tiles_per_part = (n_tiles + parts - 1) / parts;
    const int64_t waves_per_part = n_wg / parts * kNwRun;
    if (!grid_ok(n_wg) || n_tiles <= 0) return (int)hipErrorInvalidConfiguration;
    // the kernel reads entry 0 of the index array from idle lanes: give it something to read when the matrix has no entries
    const int32_t *col_arg = dp.col ? dp.col : (const int32_t *)dp.rowptr;
    hipStream_t st = (hipStream_t)stream;
#define GROOT_SAGE_PIPE_LAUNCH(WM, FFI, FFO, DD, PP)                                                                   \
    sage_pipe_kernel<WM, FFI, FFO, kNwRun, DD, PP, SDV><<<dim3((unsigned)n_wg), dim3(kNwRun * kWave), 0, st>>>(        \
        dp.rowptr, col_arg, (const char *)X, (char *)H, byte_distance(X, dp.zero_row), Wn, Ws, bias, relu, \
        dp.n, dp.nnz, dp.threshold, n_tiles, tiles_per_part, waves_per_part, parts, dp.hd_rows, (int32_t)dp.n_hd_rows,         \
        (const char *)dp.hd_agg)
#define GROOT_SAGE_PIPE_P(WM, FFI, FFO, DD)                               \
    if (pieces == 2) GROOT_SAGE_PIPE_LAUNCH(WM, FFI, FFO, DD, 2);         \
    else GROOT_SAGE_PIPE_LAUNCH(WM, FFI, FFO, DD, 3)
#define GROOT_SAGE_PIPE_D(WM, FFI, FFO)                                   \
    if (dp.sage_depth == 5) { GROOT_SAGE_PIPE_P(WM, FFI, FFO, 5); }       \
    else if (dp.sage_depth == 6) { GROOT_SAGE_PIPE_P(WM, FFI, FFO, 6); }  \
    else { GROOT_SAGE_PIPE_P(WM, FFI, FFO, 8); }
#define GROOT_SAGE_PIPE_FO(WM, FFI)                            \
    if (FO == 64) { GROOT_SAGE_PIPE_D(WM, FFI, 64); }          \
    else if (FO == 32) { GROOT_SAGE_PIPE_D(WM, FFI, 32); }     \
    else { GROOT_SAGE_PIPE_D(WM, FFI, 16); }
    if (self_times_degree) {
        constexpr bool SDV = true;
        if (FI == 64) { GROOT_SAGE_PIPE_FO(kOnes, 64); }
        else { GROOT_SAGE_PIPE_FO(kOnes, 32); }
    } else {
        constexpr bool SDV = false;
        if (FI == 64) {
            if (wm == kMean) { GROOT_SAGE_PIPE_FO(kMean, 64); }
            else { GROOT_SAGE_PIPE_FO(kOnes, 64); }
        } else {
            if (wm == kMean) { GROOT_SAGE_PIPE_FO(kMean, 32); }
            else { GROOT_SAGE_PIPE_FO(kOnes, 32); }
        }
    }
#undef GROOT_SAGE_PIPE_D
#undef GROOT_SAGE_PIPE_P
#undef GROOT_SAGE_PIPE_FO
#undef GROOT_SAGE_PIPE_LAUNCH
    return (int)hipGetLastError();
}

}  // namespace groot
