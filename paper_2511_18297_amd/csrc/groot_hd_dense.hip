// High-degree rows that hold a large part of all columns, as a dense product on the matrix cores (gfx950).
//
// A gather of a feature row for every stored entry reads a row of X as often as high-degree rows name it: on the
// polarized graph of 262,144 rows 70 times, 9.5 GB at F = 128, and the vector memory units return no more than 23 TB/s
// (hd_kernel 380 us).  Its 448 longest rows hold 15 % of all columns each, 97 % of the entries of the high-degree rows.  With
// row-uniform weights the sum of such a row is a product of a row of zeros and ones with X.
//
// The product runs on v_mfma_f32_16x16x32_bf16.  A number of X is cut into three bf16 pieces by truncation, x = hi + mid + lo, exactly:
// three times 8 significant bits (bf16 has the exponents of fp32).  Products with a power of two are exact.  What the instruction adds up
// is truncated to the 24 bits of the accumulator, so the hi pieces, of 8 bits, have one of their own, and next to nothing is cut off
// where the numbers of 128 columns are of similar size.  Where they are not, the small ones lose bits at every instruction: four of
// them, 128 columns, are one chain, which a vector addition, rounded to nearest, puts to the sum.  mid and lo, 2^-8 of it, stay in one
// chain.  Error of the dense rows in the 2-norm, 1e-8, gathers / fp32 instructions / here (131,072 rows, 448 dense, F = 128; 65,536, 64, 512):
// U(-1, 1) 15.7 / 14.7 / 3.6, 19.3 / 16.4 / 4.1; exp(4 N) 13.7 / 10.9 / 9.0, 11.7 / 10.0 / 10.4; 2^U(-40, 0) 9.7 / 3.9 / 3.5, 12.3 / 4.6 / 4.1.  (In
// chains of 2,048 columns exp(4 N) 21.8 and 32.7.)  In 20,011 rows, one step or two per workgroup, exp(4 N) 9.5 / 7.9 / 11.1.
// Chains of two (five other seeds: 7.1 to 9.3 there instead of 7.1 to 10.8, where the gathers have 9.4 to 13.3; the same elsewhere) take 224 us a
// call on the polarized graph instead of 177.
// v_mfma_f32_16x16x4_f32 on X as it is, one bit expanded per operand, does 16 rows x 16 features x 32 columns in 256 cycles, the
// three pieces take 48.
//
// One workgroup of eight wavefronts per CU takes a stretch of the columns, 64 features and up to 448 rows, so that X is read
// once and cut once: 128 columns at a time, every wavefront loads and cuts an eighth (32 columns x 32 features; eight columns of a
// lane are the eight k of an operand, so nothing is transposed) and puts the operands to LDS, from where the wavefronts of a
// feature half multiply them with the bits of their rows.  One barrier per 128 columns, loads stay in flight across it.
//
// Polarized graph, F = 128, 448 rows: 86 to 89 us (24 with 16 rows or fewer, which is X at 5.5 TB/s), 1.02 to 1.05 PFLOP/s of the pieces'
// products.  Counters: matrix units busy in 42 % of the cycles (of 2.3 GHz), vector instructions issued in 31 %, three beside each matrix
// instruction (bits to operands, cut, sums), no bank conflicts.  Neither is at its end: two wavefronts per SIMD, all that the accumulators leave room for, wait for each other at every barrier and for operands.
// Operands of the next unit read ahead, where registers allow it, make no difference.
//
// 0 x infinity is not 0, and numbers from 2^104 on are too large for the scale of the cut, which checks itself.  Where 128 columns hold
// such a number, it is left out there and these columns' exceptions are multiplied once more (`special`).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "groot_device.h"

namespace groot {

constexpr int kDenseUnit = 32;               // columns of a matrix instruction
constexpr int kDenseStep = 128;              // columns between two barriers: the columns of a mask word and its three neighbours
constexpr int kDenseTile = 64;               // features of a workgroup
constexpr int kDenseWaves = 8;               // wavefronts per workgroup, one workgroup per CU
constexpr int kDenseGroup = 256;             // steps that meet in one partial sum, at most
constexpr int kDenseMaxBlocks = 7;           // row blocks of 16 per wavefront, at most: three sets of 8 registers each
typedef unsigned int dense_u4 __attribute__((ext_vector_type(4)));
typedef __bf16 dense_b8 __attribute__((ext_vector_type(8)));
typedef __bf16 dense_b2 __attribute__((ext_vector_type(2)));

constexpr int kDenseOperandBytes = 2 * (kDenseStep / kDenseUnit) * 2 * 2 * 3 * kWave * 16;   // LDS, 96 KB: two steps' operands
constexpr int kDenseBlockSumBytes = kDenseWaves * 2 * kWave * 16;                            // 16 KB: a row block of every wavefront

// Row blocks of a wavefront whose sums are in LDS: with those of all seven in registers, of which there are 256, others spill in the loop, and
// a reload waits for the loads of X, too (polarized graph, F = 128, whole call 198 us; with three blocks' in LDS 175)
constexpr int dense_lds_blocks(int MB) { return MB == kDenseMaxBlocks ? 3 : 0; }

struct DenseArgs {
    const HdChunk *rows;                     // [n_rows] the whole row as one piece, slot -1
    const uint32_t *mask;                    // [step][padded row][kq < 4]: bit 4 u + i is column 8 kq + 2 i of unit u, bit 16 + 4 u + i the one behind it
    float *partials;                         // [k_part, unit share and group][padded rows][F]
    int32_t n_rows, tile_rows, padded;       // padded: n_rows in whole tiles
    int32_t blocks;                          // row blocks of 16 of a wavefront
    int32_t row_tiles, f_tiles, k_parts;
    int32_t groups, group;                   // partial sums of a workgroup's stretch of columns, and the steps that meet in one
    int32_t n_partials;                      // of a row
    int64_t n_steps;                         // columns in units of kDenseStep
    int64_t n_wg;                            // row_tiles x f_tiles x k_parts
    uint32_t one_bits;                       // the product's ones, one part in the columns of a partial sum or less, as bf16
    float down, up;                          // from sums of numbers that were cut 2^24 times and 2^-24 times as large to partial sums
    double weight_scale;                     // the finishing kernel's, times the row's weight
};

// Numbers are cut 2^24 times as large: all bits of a subnormal number, too, are then in three pieces that are normal numbers.  What
// becomes infinite by that, from 2^104 on, is an exception and is cut 2^-24 times as large, in a pass of its own.  The product's ones are
// one part in the columns that meet in a partial sum, exact, so no sum of numbers below 2^104 overflows.
constexpr float kDenseUp = 0x1p24f, kDenseDown = 0x1p-24f;
constexpr int kDenseScaleExp = 24;
// With mean weights partial sums are stored as one part in 64 or less: the sum of unweighted numbers, which the weight will make small,
// overflows where they are 1 / 32 of the largest float in every column, or later, however many columns meet in it (the gathers apply the
// weight to the few entries of a lane group, up to 128 of them).  With smaller parts subnormal results would be rounded more coarsely.
constexpr int kDenseStoreExp = 6, kDenseHeadExp = 5;

// (a, b) -> packed bf16 pieces, a in the low halves, of finite numbers exactly; NaN and infinity make z NaN.  a - hi by
// v_dot2_f32_bf16 with (-1, 0), one instruction instead of an unpacking and a subtraction; a neighbour that is not finite makes NaN of
// it, too, and that is seen.
__device__ __forceinline__ void dense_cut(float a, float b, unsigned &hi, unsigned &mid, unsigned &lo, float &z)
{
    unsigned pick_a = 0x0000bf80u, pick_b = 0xbf800000u;
    asm("" : "+s"(pick_a), "+s"(pick_b));                // in registers: as a literal operand 0x0000bf80 came out as (-1, -1)
    const dense_b2 first = __builtin_bit_cast(dense_b2, pick_a), second = __builtin_bit_cast(dense_b2, pick_b);
    auto upper = [](float x, float y) {
        return __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, y), __builtin_bit_cast(unsigned, x), 0x07060302u);
    };
    hi = upper(a, b);
    float ra = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dense_b2, hi), first, a, false);
    float rb = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dense_b2, hi), second, b, false);
    mid = upper(ra, rb);
    ra = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dense_b2, mid), first, ra, false);
    rb = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dense_b2, mid), second, rb, false);
    lo = upper(ra, rb);
    z += ra;
    z += rb;
}

// What is multiplied in place of x: all that is finite 2^24 times as large; then, where a step holds anything else, the infinities and
// NaN (a one in the first piece for +infinity and NaN, in the second for -infinity and NaN), and the very large numbers.
enum DensePass { kDenseMain, kDenseCodes, kDenseLarge };

// First column that the unit at `column` loads: a unit that would end behind the last column is moved back to end with it, and has bits only
// for columns from `column` on (there are kDenseUnit columns or more).
__device__ __forceinline__ int64_t dense_first_column(int64_t column, int64_t n_cols)
{
    return column < n_cols - kDenseUnit ? column : n_cols - kDenseUnit;
}

// Orders LDS accesses of the workgroup; loads from global memory stay in flight.
__device__ __forceinline__ void dense_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One workgroup's tile of 16 MB RG rows x 32 NV features over a stretch of the columns.  Matrix instruction: A row and B column are
// lane % 16, k = 8 (lane / 16) + e; D rows are 4 (lane / 16) + r.  B column m of half h and component v is feature
// 32 h NV / 2 + NV m + v.  RG: wavefronts that share the rows; the 4 / RG groups of wavefronts share a step's units of 32 columns.
template <int MB, int RG, int NV>
__device__ __forceinline__ void dense_tile(char *smem, const DenseArgs &d, const char *__restrict__ X, int32_t F, int64_t n_cols,
                                           int32_t row_tile, int32_t f0, int32_t k_part)
{
    typedef float vN __attribute__((ext_vector_type(NV)));
    constexpr int kUnits = kDenseStep / kDenseUnit, kShares = 4 / RG;
    dense_u4 (*const s_b)[kUnits][2][NV][3][kWave] = (dense_u4(*)[kUnits][2][NV][3][kWave])smem;    // [2]: two steps
    __shared__ int32_t s_special[2];                                              // which passes the step needs beside the main one
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave, m = lane % 16, kq = lane / 16;
    const int half = wave % 2, cut_unit = wave / 2, rg = wave / 2 % RG, share = wave / 2 / RG;
    const int f = f0 + (half * 16 + m) * NV;                                      // first feature of the lane, cutting and storing
    const int64_t row_bytes = (int64_t)F * 4;
    const uint32_t x_at = (uint32_t)(8 * kq * (int)row_bytes + 4 * (f < F - NV ? f : F - NV));
    const uint32_t w_at = (uint32_t)(16 * m + 4 * kq), p_at = (uint32_t)(4 * (4 * kq * F + f));
    const int64_t s0 = d.n_steps * k_part / d.k_parts, s1 = d.n_steps * (k_part + 1) / d.k_parts;
    const int32_t n_blocks = d.padded / 16, block0 = (row_tile * RG + rg) * MB;   // the last tile may have blocks past the end

    auto load = [&](int64_t s, vN (&x)[8]) {             // without a branch, see the loop
        const char *const base = X + dense_first_column(s * kDenseStep + cut_unit * kDenseUnit, n_cols) * row_bytes;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = *(const vN *)((base + e * row_bytes) + x_at);
    };
    auto mask_of = [&](int64_t s, int b) -> uint32_t {
        const int32_t block = block0 + b < n_blocks ? block0 + b : n_blocks - 1;
        return *(const uint32_t *)((const char *)d.mask + (s * d.padded + 16 * block) * 16 + w_at);
    };
    auto put = [&](int buf, int v, const dense_u4 (&op)[3]) {
#pragma unroll
        for (int q = 0; q < 3; ++q) s_b[buf][cut_unit][half][v][q][lane] = op[q];
    };
    auto cut = [&](int buf, const vN (&x)[8]) {
        float z = 0.f;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            dense_u4 op[3];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                unsigned q0, q1, q2;
                dense_cut(x[2 * p][v] * kDenseUp, x[2 * p + 1][v] * kDenseUp, q0, q1, q2, z);
                op[0][p] = q0;
                op[1][p] = q1;
                op[2][p] = q2;
            }
            put(buf, v, op);
        }
        if (__ballot(z != z)) {                          // put again, without the exceptions
            int32_t kinds = 0;
#pragma unroll 1
            for (int v = 0; v < NV; ++v) {
                dense_u4 op[3];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const float a = v ? x[2 * p][NV - 1] : x[2 * p][0], b = v ? x[2 * p + 1][NV - 1] : x[2 * p + 1][0];
                    const bool a_ok = isfinite(a * kDenseUp), b_ok = isfinite(b * kDenseUp);
                    if (__ballot(!isfinite(a) || !isfinite(b))) kinds |= 1 << kDenseCodes;
                    if (__ballot((!a_ok && isfinite(a)) || (!b_ok && isfinite(b)))) kinds |= 1 << kDenseLarge;
                    unsigned q0, q1, q2;
                    dense_cut(a_ok ? a * kDenseUp : 0.f, b_ok ? b * kDenseUp : 0.f, q0, q1, q2, z);
                    op[0][p] = q0;
                    op[1][p] = q1;
                    op[2][p] = q2;
                }
                put(buf, v, op);
            }
            if (lane == 0) atomicOr(&s_special[buf], kinds);
        }
    };
    // unit u's bits of a row -> the eight ones and zeros of an operand
    auto ones = [&](uint32_t w, int u) -> dense_b8 {
        const uint32_t t = w >> (4 * u);
        dense_u4 a;
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = __umul24(t & (0x00010001u << i), d.one_bits >> i);
        return __builtin_bit_cast(dense_b8, a);
    };
    // sums of one step's leading pieces, of the others, of all steps' leading pieces; the last in LDS where registers end
    constexpr int kLdsBlocks = dense_lds_blocks(MB), kRegBlocks = MB - kLdsBlocks;
    v4f hi[MB][NV], rest[MB][NV], sum[kRegBlocks][NV];
    v4f *const s_sum = (v4f *)(smem + kDenseOperandBytes);
    const v4f zero = {0.f, 0.f, 0.f, 0.f};
    auto at_sum = [&](int b, int v) -> v4f * { return s_sum + ((wave * kLdsBlocks + b - kRegBlocks) * NV + v) * kWave + lane; };
    auto add = [&](int b, int v) {
        if (b < kRegBlocks) sum[b][v] += hi[b][v];
        else *at_sum(b, v) += hi[b][v];
    };
    uint32_t w[MB];                                      // bits of the step that is multiplied next
    auto multiply = [&](int buf) {
        constexpr int kMine = kUnits / kShares;
        // while there are registers, a unit's operands are read and a block's ones expanded ahead
        constexpr int kAhead = MB < 6 && kMine > 1 ? 2 : 1;
        constexpr bool kRoom = MB < kDenseMaxBlocks;
        dense_b8 x[kAhead][NV][3];
        auto read = [&](int k) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int q = 0; q < 3; ++q) x[k % kAhead][v][q] = __builtin_bit_cast(dense_b8, s_b[buf][k * kShares + share][half][v][q][lane]);
        };
        read(0);
        dense_b8 a = {};
        if (kRoom) a = ones(w[0], share);
#pragma unroll
        for (int k = 0; k < kMine; ++k) {
            if (kAhead == 2 && k + 1 < kMine) read(k + 1);
            __builtin_amdgcn_sched_barrier(0);           // the reads stay ahead of this unit's matrix instructions
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                dense_b8 next = a;
                const int to = b + 1 < MB ? k : k + 1 < kMine ? k + 1 : k;
                if (kRoom) next = ones(w[b + 1 < MB ? b + 1 : 0], to * kShares + share);
                else a = ones(w[b], k * kShares + share);
#pragma unroll
                for (int v = 0; v < NV; ++v)
                    hi[b][v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, x[k % kAhead][v][0], k ? hi[b][v] : zero, 0, 0, 0);
#pragma unroll
                for (int q = 1; q < 3; ++q)
#pragma unroll
                    for (int v = 0; v < NV; ++v)
                        rest[b][v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, x[k % kAhead][v][q], rest[b][v], 0, 0, 0);
                if (b > 0 && k == kMine - 1)             // of the block before: its instructions have ended
#pragma unroll
                    for (int v = 0; v < NV; ++v) add(b - 1, v);
                a = next;
                __builtin_amdgcn_sched_barrier(0);       // no more of them at a time: registers
            }
            if (kAhead == 1 && k + 1 < kMine) read(k + 1);
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) add(MB - 1, v);
    };
    int64_t slot = 0;                                    // partial sum that the present run goes to
    bool started = false;                                // something has been written there
    auto partial = [&](int64_t at, int b) -> char * { return (char *)d.partials + (at * d.padded + 16 * (block0 + b)) * row_bytes + p_at; };
    // The step's exceptions, over the operands in LDS, which have been multiplied.  Every wavefront of the workgroup gets here.
    auto special = [&](int64_t s, int buf, int32_t kinds) {
#pragma unroll 1
        for (int pass = kDenseCodes; pass <= kDenseLarge; ++pass) {
            if (!(kinds >> pass & 1)) continue;
            dense_barrier();                             // what is there has been read
            vN x[8];
            load(s, x);
            if (threadIdx.x == 0) s_special[buf] = 0;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                dense_u4 op[3] = {};
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const float ab[2] = {x[2 * p][v], x[2 * p + 1][v]};
                    float t[2];
                    unsigned plus[2], minus[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const bool nan = ab[i] != ab[i], in_main = isfinite(ab[i] * kDenseUp);
                        plus[i] = nan || ab[i] == __builtin_inff() ? 0x3f80u : 0u;
                        minus[i] = nan || ab[i] == -__builtin_inff() ? 0x3f80u : 0u;
                        t[i] = in_main || plus[i] || minus[i] ? 0.f : ab[i] * kDenseDown;
                    }
                    unsigned q0, q1, q2;
                    float z = 0.f;
                    dense_cut(t[0], t[1], q0, q1, q2, z);
                    op[0][p] = pass == kDenseCodes ? plus[0] | plus[1] << 16 : q0;
                    op[1][p] = pass == kDenseCodes ? minus[0] | minus[1] << 16 : q1;
                    op[2][p] = pass == kDenseCodes ? 0u : q2;
                }
                put(buf, v, op);
            }
            dense_barrier();
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    v4f t0 = zero, t1 = zero;
                    const uint32_t bits = mask_of(s, b);
#pragma unroll 1
                    for (int k = 0; k < kUnits / kShares; ++k) {
                        const int u = k * kShares + share;
                        const dense_b8 a = ones(bits, u);
                        const dense_u4 (*const op)[kWave] = s_b[buf][u][half][v];
                        t0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(dense_b8, op[0][lane]), t0, 0, 0, 0);
                        t1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(dense_b8, op[1][lane]), t1, 0, 0, 0);
                        t1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(dense_b8, op[2][lane]), t1, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float inf = t0[r] > 0.f ? __builtin_inff() : -__builtin_inff();
                        const float code = t0[r] > 0.f && t1[r] > 0.f ? __builtin_nanf("") : t0[r] > 0.f || t1[r] > 0.f ? inf : 0.f;
                        t0[r] = pass == kDenseCodes ? code : (t0[r] + t1[r]) * d.up;
                    }
                    int64_t at = slot;
                    asm("" : "+s"(at));                  // no addresses kept from one pass to the next: registers
                    if (block0 + b < n_blocks && f < F) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            float *const p = (float *)(partial(at, b) + r * row_bytes) + v;
                            *p = started ? *p + t0[r] : t0[r];
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            started = true;
        }
    };

    vN x[8];
    if (threadIdx.x < 2) s_special[threadIdx.x] = 0;
    load(s0, x);
#pragma unroll
    for (int b = 0; b < MB; ++b) w[b] = mask_of(s0, b);
    dense_barrier();
    cut(0, x);
    load(s0 + 1 < s1 ? s0 + 1 : s0, x);
    dense_barrier();
    int64_t s = s0;
#pragma unroll 1
    for (int32_t i = 0; i < d.groups; ++i) {
        const int64_t to = s0 + (i + 1) * (int64_t)d.group < s1 ? s0 + (i + 1) * (int64_t)d.group : s1;
        slot = ((int64_t)k_part * kShares + share) * d.groups + i;
        started = false;
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                rest[b][v] = zero;
                if (b < kRegBlocks) sum[b][v] = zero;
                else *at_sum(b, v) = zero;
            }
#pragma unroll 1
        for (; s < to; ++s) {
            const int buf = (int)(s - s0) & 1;
            // The last step, too, cuts and loads for one that does not come: where there are paths with and without loads, the compiler
            // counts on the fewest and has the bits and the next step wait for the loads of X that were issued last (12 rows of half of
            // 262,144 columns, this kernel, F = 128 and 512: 30.4 and 132 us, now 24.2 and 96).
            uint32_t next_w[MB];
#pragma unroll
            for (int b = 0; b < MB; ++b) next_w[b] = mask_of(s + 1 < s1 ? s + 1 : s, b);
            cut(buf ^ 1, x);
            load(s + 2 < s1 ? s + 2 : s, x);
            multiply(buf);
            const int32_t kinds = __builtin_amdgcn_readfirstlane(s_special[buf]);
            if (kinds) special(s, buf, kinds);
#pragma unroll
            for (int b = 0; b < MB; ++b) w[b] = next_w[b];
            dense_barrier();
        }
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            if (block0 + b >= n_blocks || f >= F) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                vN *const p = (vN *)(partial(slot, b) + r * row_bytes);
                vN out;
#pragma unroll
                for (int v = 0; v < NV; ++v) out[v] = ((b < kRegBlocks ? sum[b < kRegBlocks ? b : 0][v] : *at_sum(b, v))[r] + rest[b][v][r]) * d.down;
                *p = started ? *p + out : out;
            }
        }
    }
}

template <int MB, int RG>
__global__ __launch_bounds__(kDenseWaves * kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void hd_dense_kernel(
    const DenseArgs d, const char *__restrict__ X, int32_t F4, int64_t n_cols, int64_t wgs_per_xcd, int remap)
{
    __shared__ __align__(16) char smem[kDenseOperandBytes + dense_lds_blocks(MB) * kDenseBlockSumBytes];
    // the tiles of a stretch of columns on one XCD, whose L2 they share
    const int32_t t = (int32_t)logical_block(wgs_per_xcd, remap), row_tile = t % d.row_tiles, f_tile = t / d.row_tiles % d.f_tiles;
    const int32_t k_part = t / d.row_tiles / d.f_tiles, F = 4 * F4;
    if (F - f_tile * kDenseTile > kDenseTile / 2)
        dense_tile<MB, RG, 2>(smem, d, X, F, n_cols, row_tile, f_tile * kDenseTile, k_part);
    else
        dense_tile<MB, RG, 1>(smem, d, X, F, n_cols, row_tile, f_tile * kDenseTile, k_part);
}

// Workgroups [0, n_dense): kDenseFinishLanes x 4 features of a dense row each, whose partial sums meet in fp64 and get the row's weight.
// The ones behind: the split rows among the others, as in hd_finish_kernel.  A few dense rows are a few workgroups, and what one takes is
// latencies: 32 lane groups share a row's partial sums (up to 1,024 as a rule), 4 or 16 of each in flight.  12 rows of 512 partial sums, F = 128,
// and of 128, F = 512, 4.8 and 5.0 us; with a workgroup per row 8.8 and 8.7.
constexpr int kDenseFinishLanes = 8;
template <int L, int W>
__global__ __launch_bounds__(kBlock) void hd_dense_finish_kernel(const DenseArgs d, int32_t n_dense, const HdSplitRow *__restrict__ split,
                                                                 int64_t n_split, const v4f *__restrict__ partials,
                                                                 v4f *__restrict__ Y, int32_t F4)
{
    constexpr int G = kBlock / kDenseFinishLanes;
    typedef double v4d __attribute__((ext_vector_type(4)));
    auto wide = [](v4f x) { return __builtin_convertvector(x, v4d); };
    __shared__ v4d s_red[kBlock];                        // [G][kDenseFinishLanes]
    if ((int32_t)blockIdx.x >= n_dense) {
        const int64_t k = (int64_t)((int32_t)blockIdx.x - n_dense) * (kBlock / L) + threadIdx.x / L;
        if (k < n_split) hd_finish_row<L>(split[k], partials, Y, F4, nullptr, threadIdx.x % L);
        return;
    }
    const int g = threadIdx.x / kDenseFinishLanes, f_blocks = (F4 + kDenseFinishLanes - 1) / kDenseFinishLanes;
    const int32_t r = (int32_t)blockIdx.x / f_blocks, f = (int32_t)blockIdx.x % f_blocks * kDenseFinishLanes + threadIdx.x % kDenseFinishLanes;
    const HdChunk row = d.rows[r];
    v4d acc = {0., 0., 0., 0.};
    const v4f *p = (const v4f *)d.partials + (int64_t)r * F4 + (f < F4 ? f : 0);
    const int64_t step = (int64_t)d.padded * F4;
    int32_t k = g;
    auto take = [&](auto ahead) {
        constexpr int kAhead = decltype(ahead)::value;
        v4f x[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) x[i] = p[(k + i * G < d.n_partials ? k + i * G : k) * step];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (k + i * G < d.n_partials) acc += wide(x[i]);
        k += kAhead * G;
    };
    while (k + 4 * G < d.n_partials) take(std::integral_constant<int, 16>());
    if (k < d.n_partials) take(std::integral_constant<int, 4>());
    s_red[threadIdx.x] = acc;
    __syncthreads();
#pragma unroll
    for (int stride = G / 2; stride > 0; stride /= 2) {
        if (g < stride) s_red[threadIdx.x] += s_red[threadIdx.x + stride * kDenseFinishLanes];
        __syncthreads();
    }
    const double weight = (double)row_weight<W>(row.row_nnz) * d.weight_scale;
    if (g == 0 && f < F4) Y[(int64_t)row.row * F4 + f] = __builtin_convertvector(s_red[threadIdx.x] * weight, v4f);
}

// the four mask words of row r and step b, one thread each; padding rows get zeros
__global__ __launch_bounds__(kBlock) void dense_mask_kernel(const HdChunk *__restrict__ rows, int32_t n_rows, int32_t padded,
                                                            const int32_t *__restrict__ col, int64_t n_cols, int64_t n_steps,
                                                            uint4 *__restrict__ mask)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t b = i / padded;
    const int32_t r = (int32_t)(i % padded);
    if (b >= n_steps) return;
    uint32_t w[4] = {0, 0, 0, 0};
    if (r < n_rows) {
        const HdChunk row = rows[r];
        const int32_t *const c = col + row.begin;
        const int64_t first = b * kDenseStep;
        int32_t lo = 0, hi = row.len;                    // first entry with a column >= first
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo) / 2;
            if (c[mid] < first) lo = mid + 1; else hi = mid;
        }
        for (; lo < row.len && c[lo] < first + kDenseStep; ++lo) {
            const int unit = (int)(c[lo] - first) / kDenseUnit;
            const int at = (int)(c[lo] - dense_first_column(first + unit * kDenseUnit, n_cols)), e = at % 8;
            const uint32_t bit = 1u << (4 * unit + e / 2 + 16 * (e % 2));
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] |= at / 8 == k ? bit : 0u;
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
    const int32_t tiles = (dp.n_dense_rows + dp.dense_tile_rows - 1) / dp.dense_tile_rows;   // a wavefront has a row block of each
    d.padded = tiles * dp.dense_tile_rows;
    // Row blocks of a wavefront and workgroups beside each other, as few blocks in all as may be, those past the last row among them; what
    // every workgroup does for itself, the cut above all, is half a block's work.
    const int32_t most = dp.dense_tile_rows == 64 ? kDenseMaxBlocks : 1, least = (tiles + most - 1) / most;
    for (int32_t t = least; t < 2 * least + 1; ++t) {
        const int32_t blocks = (tiles + t - 1) / t;
        if (t > least && t * (2 * blocks + 1) >= d.row_tiles * (2 * d.blocks + 1)) continue;
        d.row_tiles = t;
        d.blocks = blocks;
    }
    d.f_tiles = (F + kDenseTile - 1) / kDenseTile;
    d.n_steps = (dp.n_cols + kDenseStep - 1) / kDenseStep;
    const int64_t wgs = (int64_t)d.row_tiles * d.f_tiles;
    int64_t k = kDenseMaxWorkgroups / wgs;               // one workgroup per CU while it has a step or more
    if (k > d.n_steps) k = d.n_steps;
    d.k_parts = (int32_t)(k < 1 ? 1 : k);
    const int64_t share = (d.n_steps + d.k_parts - 1) / d.k_parts;
    d.groups = (int32_t)((share + kDenseGroup - 1) / kDenseGroup);
    d.group = (int32_t)((share + d.groups - 1) / d.groups);
    d.n_partials = d.k_parts * (64 / dp.dense_tile_rows) * d.groups;
    d.n_wg = wgs * d.k_parts;
    const int64_t columns = (int64_t)d.group * kDenseStep / (64 / dp.dense_tile_rows);
    int one = 0, store = kDenseStoreExp;                 // exponents: parts in 2^one and 2^store
    while ((int64_t)1 << one < columns) ++one;
    while ((int64_t)1 << (store + kDenseHeadExp) < columns) ++store;
    if (dp.weight_mode != kMean) store = 0;
    d.one_bits = (uint32_t)(127 - one) << 7;
    d.down = (float)std::ldexp(1., one - store - kDenseScaleExp);
    d.up = (float)std::ldexp(1., one - store + kDenseScaleExp);
    d.weight_scale = std::ldexp(1., store);
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

// Where the product takes less than the gathers of the same rows, in femtoseconds: a gather 300 per entry and feature; the product 4 us of launches, 150 per
// column and feature to read and cut X, 4.7 per padded row, column and feature.  Whole calls, us, gathers / product, polarized graphs: 16,384
// rows (64 dense), F = 64 12.2 / 15.8, 128 17.6 / 19.0, 200 24.2 / 22.9; 32,768 rows (64) F = 32 17.2 / 16.2, 64 20.0 / 20.2, 128 30.4 / 24.4; 65,536
// rows (128) F = 8 19.3 / 21.4, 12 25.9 / 25.2, 16 28.6 / 23.7, 128 54.1 / 35.4; 131,072 rows (256) F = 8 37.8 / 31.2; 262,144 rows F = 8 89.8 / 56.0.  Rows of one
// length: 64 of 5 % of 262,144 columns F = 8 23.4 / 25.2, 16 33.0 / 30.9, 128 118 / 93; 16 of 10 % F = 32 34.0 / 34.0, 48 51.5 / 50.0, 128 93.8 / 90.5; of 65,536
// columns 64 of 5 % F = 64 21.9 / 27.3, 128 32.6 / 31.9, 200 49.4 / 46.3; 300 of 3 % F = 32 22.5 / 26.7, 64 33.7 / 36.6, 128 51.1 / 44.5; 16 of 10 % F = 200 40.4 / 44.9.
bool hd_dense_serves(const DevicePlan &dp, int32_t F)
{
    if (dp.n_dense_rows < 1 || dp.n_cols != dp.n || F < kDenseMinF) return false;
    const int64_t padded = (dp.n_dense_rows + dp.dense_tile_rows - 1) / dp.dense_tile_rows * dp.dense_tile_rows;
    return 300. * dp.dense_entries * F >= 4e9 + (150 + 4.7 * padded) * dp.n_cols * F;
}

size_t dense_mask_words(const DevicePlan &dp)
{
    const size_t padded = (size_t)(dp.n_dense_rows + dp.dense_tile_rows - 1) / dp.dense_tile_rows * dp.dense_tile_rows;
    const size_t steps = (size_t)(dp.n_cols + kDenseStep - 1) / kDenseStep;
    return steps * padded * 4;
}

int launch_dense_mask(const DevicePlan &dp, void *stream)
{
    const DenseArgs d = dense_args(dp, 4);
    const int64_t grid = (d.n_steps * d.padded + kBlock - 1) / kBlock;
    if (!grid_ok(grid) || dp.n_cols < kDenseUnit) return (int)hipErrorInvalidConfiguration;
    dense_mask_kernel<<<dim3((unsigned)grid), dim3(kBlock), 0, (hipStream_t)stream>>>(d.rows, d.n_rows, d.padded, dp.col, dp.n_cols, d.n_steps,
                                                                                      (uint4 *)dp.dense_mask);
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

int launch_hd_dense(const DevicePlan &dp, const float *X, int32_t F, void *stream)
{
    if (dp.weight_mode == kExplicit) return (int)hipErrorInvalidValue;
    const DenseArgs d = dense_args(dp, F);
    if (!grid_ok(d.n_wg)) return (int)hipErrorInvalidConfiguration;
    const int remap = dp.xcd_remap && d.n_wg % kXcds == 0;
    auto launch = [&](auto kernel) {
        kernel<<<dim3((unsigned)d.n_wg), dim3(kDenseWaves * kWave), 0, (hipStream_t)stream>>>(d, (const char *)X, F / 4, dp.n_cols,
                                                                                              d.n_wg / kXcds, remap);
    };
    if (dp.dense_tile_rows == 16) launch(hd_dense_kernel<1, 1>);
    else if (dp.dense_tile_rows == 32) launch(hd_dense_kernel<1, 2>);
    else if (dp.dense_tile_rows != 64) return (int)hipErrorInvalidValue;
    else switch (d.blocks) {
    case 1: launch(hd_dense_kernel<1, 4>); break;
    case 2: launch(hd_dense_kernel<2, 4>); break;
    case 3: launch(hd_dense_kernel<3, 4>); break;
    case 4: launch(hd_dense_kernel<4, 4>); break;
    case 5: launch(hd_dense_kernel<5, 4>); break;
    case 6: launch(hd_dense_kernel<6, 4>); break;
    default: launch(hd_dense_kernel<7, 4>); break;
    }
    return (int)hipGetLastError();
}

int launch_hd_dense_finish(const DevicePlan &dp, float *Y, int32_t F, void *stream)
{
    const DenseArgs d = dense_args(dp, F);
    const int L = dense_lanes(F / 4);
    const int64_t n_dense = (int64_t)d.n_rows * ((F / 4 + kDenseFinishLanes - 1) / kDenseFinishLanes);
    const int64_t n_wg = n_dense + (dp.n_split_rows + kBlock / L - 1) / (kBlock / L);
    if (!grid_ok(n_wg)) return (int)hipErrorInvalidConfiguration;
    auto launch = [&](auto kernel) {
        kernel<<<dim3((unsigned)n_wg), dim3(kBlock), 0, (hipStream_t)stream>>>(d, (int32_t)n_dense, dp.split_rows, dp.n_split_rows,
                                                                               (const v4f *)dp.partials, (v4f *)Y, F / 4);
    };
    if (dp.weight_mode == kMean) { GROOT_DENSE_L(L, (launch(hd_dense_finish_kernel<kL, kMean>))) }
    else { GROOT_DENSE_L(L, (launch(hd_dense_finish_kernel<kL, kOnes>))) }
    return (int)hipGetLastError();
}

}  // namespace groot
