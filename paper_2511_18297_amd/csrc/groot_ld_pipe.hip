// Software-pipelined LD kernel for gfx950: the low-degree rows of graphs whose rows are short (an AIG
// with self-loops has 2 to 6 entries per low-degree row), F = 20 to 256 (32, 64 and 128 without
// idle lanes).
//
// One persistent workgroup of four wavefronts per CU, i.e. one wavefront per SIMD.  Every wavefront walks
// its own tiles of G lane groups x (64 / L) rows (L = F / 4 lanes per row) and keeps a whole tile in
// flight: G register sets of D gathered float4 each (D = 5 to 8 slots per row, chosen per plan).  Right
// after the rows of a group of tile t have been summed and stored, the same register set is loaded with
// the group's rows of tile t+1, so the wavefront never waits with nothing in flight.  Compared with the
// plain LD kernel (32 wavefronts per CU, four rows in flight each, all of them drained at every tile) this
// keeps fewer requests in flight per CU (measured to be what the memory system of this chip prefers for
// this access pattern) and never lets the stream of requests stop.
//
// What makes the pipeline work (each item was a measured dead end without it):
//  * All address arithmetic is done once per tile, lane-parallel: lane s owns slot s = D r + k of a
//    wavefront-private table in LDS (byte offset of the k-th neighbour of row r); it fetches that entry's
//    column index itself, two tiles ahead, from the row pointers that arrived three tiles ahead (register
//    shuffles hand every slot its row's extent).  A slot past a row's end points at a row of zeros outside
//    X: the sum of a row is the plain sum of its D slots, in CSR order.
//  * The steady state has no branch and no conditional load or store, so the compiler's vmcnt waits are
//    exact: the wait before a group's sum leaves the G-1 younger groups in flight.  A row that does not
//    fit (more than D entries, or a high-degree row) is masked: all its slots point at the zero row and
//    its sum is stored to a trash area instead of Y, or past the end of a buffer descriptor, where the
//    hardware drops it (an address select, not a branch); the high-degree kernel, or a workgroup behind the sweep for low-degree rows longer than D, computes it.  Only the ragged
//    last tile is masked as a whole and redone by a plain, unoverlapped path.
//  * No workgroup barrier after the start (the list of hot rows is copied to LDS once): wavefronts share
//    nothing else.
#include <type_traits>

#include "groot_device.h"

namespace groot {

constexpr int kPipeWaves = 4;                // wavefronts per workgroup, one workgroup per CU
// lane-group sweeps (register sets) in flight per wavefront, by lanes per row.  Measured on the headline graph:
// 16 lanes (F = 64), LD kernels with X and Y where they run fastest: 13.08 / 12.75 / 12.94 / 12.63 / 12.75 ms for
// 4 / 5 / 6 / 7 / 8 (with both matrices in one class of address ranges 5 was the best: 16.9 / 14.4 / 14.2 / 13.7 /
// 14.0 / 13.8 / 13.9 ms for 2..8); 8 lanes (F = 32): 6.46 / 6.36 ms for 5 / 7; 32 lanes (F = 128): 31.0 / 30.5 /
// 31.3 ms per step for 5 / 7 / 8
constexpr int pipe_groups(int) { return 7; }
// S = 2: rows of a tile.  As many as the sweeps' 64 lanes hold; pipe_max_rows: at the narrowest width (9, 17, 33 float4) that is
// served with L lanes' template.
constexpr int pipe_max_rows(int L) { return pipe_groups(L) * kWave / (L / 2 + 1); }

// Whether rows take F4 lanes (S = 2): the rows of a tile, or 0.  They do where that fills a quarter more of the lanes: with L lanes
// per row and 9 of 16, 17 of 32 or 34 of 64 in use a sweep did half of what it costs.  2.1 M rows of a carry-save multiplier,
// us, L / F4 lanes: F = 36 192 / 154, 72 357 / 284, 136 689 / 550, 164 759 / 700; 4-LUT shape, 1.1 M rows: 36 142 / 120, 72
// 298 / 257, 136 567 / 490.  With less to gain the lines that two sweeps share cost more: F = 60 (15 of 16) 245 / 260, 28 (7 of 8)
// 120 / 123; F = 100 (25 of 32; 16 of 17.9 rows) 424 / 406, but 79.5 / 81.8 at 0.5 M rows and 369 / 375 on the 4-LUT shape;
// F = 180 (45 of 64) 815 / 790, 4-LUT 685 / 703.  With 5 slots the kernel has a little more than half of the registers, so what
// rides along waits for the sweep, and small graphs lose: below 64 MB of X 12.0 / 12.7 (64-bit multiplier x 2, F = 36), 43 / 46.5
// (polarized, 65,536 rows, F = 72), at 75 MB 47 / 39 (128-bit x 4, F = 36); with 6 to 8 slots it is so either way.
static int pipe_tile_rows(int L, int32_t F4, int depth, int64_t n_rows)
{
    const int lanes = pipe_groups(L) * kWave, by_lanes = pipe_groups(L) * (kWave / L);
    if (L < 16 || F4 == L || (depth == 5 && n_rows * F4 * 16 < (int64_t)64 << 20)) return 0;
    int rows = lanes / F4;
    // whole 128-byte lines per tile where that leaves three quarters of the lanes in use: the sweeps' stores, 1 KB each,
    // then begin and end with a line
    int unit = 8;
    for (int32_t f = F4; unit > 1 && f % 2 == 0; f /= 2) unit /= 2;
    const int whole = rows / unit * unit;
    if (whole * F4 * 4 >= lanes * 3) rows = whole;
    return rows * 4 >= by_lanes * 5 ? rows : 0;
}

typedef int pipe_i4 __attribute__((ext_vector_type(4)));
constexpr int kHotAhead = 8;                  // 16-byte loads of the hot list that a lane has in flight

typedef unsigned int pipe_u4 __attribute__((ext_vector_type(4)));
constexpr int kPipeRawBuffer = 0x00027000;   // last word of a buffer descriptor: raw 32-bit data, offsets checked against the size
constexpr int kPipeNontemporal = 2;
constexpr uint32_t kPipeDropped = 0x40000000;

// What a launch does beside the sweep, in workgroups of their own behind it: the low-degree rows that the pipeline masks,
// one lane group per row, where they are few (rows_beside_sweep), and, where those are few (ld_takes_hd), the pieces of the
// high-degree rows.  On small
// graphs the launches were most of the time: 32-bit multiplier, F = 32, three kernels of 10 + 3.5 + 3.4 us, now one of 8.0;
// 256-bit, F = 64, 48 + 7.6 + 5 and the gaps (75 us), now one of 48 (65 us).  A graph of many pieces keeps the kernel of
// their own: it wants all wavefronts of a CU, this one has registers for one or two per SIMD.
struct SideWork {
    int64_t n_ld;                            // workgroups of the sweep
    const int32_t *rows;                     // the row list
    int64_t n_rows, n_row_wg;
    const HdChunk *chunks;                   // one workgroup per piece
    float *partials;
};

// The compact form of the CSR (C = true: 4-byte row pointers, 2-byte column codes, the list of high-degree
// rows that a code can name; see groot_compress.hip) replaces the loads of the pipeline; the plain path and the
// side work keep reading the full arrays.
struct CompactCsr {
    const uint32_t *rp32;
    const uint16_t *col16;
    const int32_t *hot;
    int32_t n_hot;
};

// M: the sum of row r goes to row out_ids[r] of Y (the owned rows of a part written into place in the matrix of
// the whole graph); n is then the number of leading rows that are wanted.  Only without the compact matrix.
// S: rows of F4 float4, any number up to L (0: F4 = L).  1: a row has L lanes, the ones past its end do what the lane of its last
// float4 does, and store the same value to the same place.  2: a row has F4 lanes, the sweeps deal the tile's float4 out to all
// of them, 64 after 64, whatever row they belong to (pipe_tile_rows says where).  No trash area here: parts of a line written to one place by all
// wavefronts wait for one another (lanes past the end, 4-LUT shape, 0.5 M rows, F = 124: 574 us, now 233; masked rows, 4 M
// rows, one in 27 masked, F = 100: 2,140 us, now 1,095).  With whole lines it costs next to nothing and the plain store is
// the faster one (8.4 M rows of carry-save multipliers, F = 32: 491 us, through the descriptor 502; F = 64 942 and 951).
// The workgroups behind the first n_ld of the grid compute the rows of the row list, then (n_hd of them) the pieces of the
// high-degree rows: see SideWork.
template <int L, int W, int G, int D, bool C, bool M = false, int S = 0>
__global__ __launch_bounds__(kPipeWaves * kWave) __attribute__((amdgpu_waves_per_eu(1, 2))) void ld_pipe_kernel(
    const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col, const float *__restrict__ val,
    const CompactCsr cz, const char *__restrict__ X, char *__restrict__ Y, int64_t zero_off, char *trash, int64_t n,
    int32_t T, int64_t n_tiles, int64_t tiles_per_part, int64_t waves_per_part, int32_t parts,
    const int64_t *__restrict__ out_ids, int32_t F4, int32_t tile_rows, const SideWork side)
{
    static_assert(!(C && M) && !(S && M), "the row-mapped form reads the plain arrays and has rows of L float4");
    constexpr int kRpg = kWave / L;                      // rows per lane group sweep (S < 2)
    constexpr int kMaxRows = S == 2 ? pipe_max_rows(L) : G * kRpg;
    const int kTileRows = S == 2 ? tile_rows : G * kRpg; // rows of a tile, a constant with S < 2
    constexpr int kPipeD = D;                            // slots per row
    constexpr int kSlots = kMaxRows * kPipeD, kH = (kSlots + kWave - 1) / kWave;
    constexpr int kRowShift = L == 8 ? 7 : L == 16 ? 8 : L == 32 ? 9 : 10;   // log2 of a feature row's bytes
    static_assert(L == 8 || L == 16 || L == 32 || L == 64, "one float4 per lane");
    auto row_bytes = [&](int64_t row) -> int64_t { return S ? row * (F4 * 16) : row << kRowShift; };
    static_assert(kMaxRows + 1 <= kWave, "row pointers of a tile fit one wavefront");
    // a slot: byte offset of the gathered row from X; with explicit weights the entry's weight rides in the
    // same 16-byte slot, so that one LDS read per slot serves both
    struct SlotW { int64_t off; float w; float pad; };
    using Slot = typename std::conditional<W == kExplicit, SlotW, int64_t>::type;
    constexpr int kSlotBytes = kPipeWaves * kSlots * (int)sizeof(Slot), kHdBytes = kHdSmemBytes<L>;
    __shared__ __align__(16) char s_buf[kSlotBytes > kHdBytes ? kSlotBytes : kHdBytes];
    Slot (*const s_slot)[kSlots] = (Slot(*)[kSlots])s_buf;
    __shared__ float s_inv[kPipeWaves][kMaxRows];       // row weight (1 unless W == kMean), or -1: the row is masked
    __shared__ int64_t s_oid[M ? kPipeWaves : 1][M ? kMaxRows : 1];   // M: byte offset of the row's place in Y

    if (blockIdx.x >= side.n_ld) {
        const int64_t b = blockIdx.x - side.n_ld;
        if (b < side.n_row_wg) {
            const int64_t k = b * (kBlock / L) + threadIdx.x / L;
            const int ff = threadIdx.x % L;
            if (k >= side.n_rows || ff >= F4) return;
            const int64_t row = side.rows[k];
            if (row >= n) return;                        // a row that is not wanted (row-mapped calls: boundary rows)
            __builtin_nontemporal_store(ld_row_sum<W, false>(rowptr[row], rowptr[row + 1], col, val, (const v4f *)X, F4, ff),
                                        (v4f *)Y + (M ? out_ids[row] : row) * F4 + ff);
        } else {
            const HdChunk ch = side.chunks[b - side.n_row_wg];
            if (ch.row >= n) return;                     // the whole workgroup
            hd_piece<L, W>(s_buf, ch, col, val, X, zero_off, (v4f *)Y, (v4f *)side.partials, F4, M ? out_ids : nullptr);
        }
        return;
    }
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), l = threadIdx.x % kWave;
    const int g = l / L, f = S == 2 ? 0 : S == 1 ? (l % L < F4 ? l % L : F4 - 1) : l % L;
    // S = 2.  slot_at: byte offset of the first slot of the lane's row in the slot table; f_at: byte offset of its float4 in the
    // row.  Both move on with every sweep that is issued (a pair of registers per sweep would cost the second wavefront of a
    // SIMD, where the pieces of the high-degree rows run).
    constexpr int kRowSlots = kPipeD * (int)sizeof(Slot);
    const int slot_0 = S == 2 ? l / F4 * kRowSlots : 0, f_0 = S == 2 ? l % F4 * 16 : 0;
    const int slot_step = S == 2 ? kWave / F4 * kRowSlots : 0, f_step = S == 2 ? kWave % F4 * 16 : 0;
    int slot_at = slot_0, f_at = f_0;
    // Part x (an XCD) owns tiles [x TP, (x+1) TP); its wavefronts take them round-robin, so that the
    // part sweeps a narrow window of rows at any time.
    const int64_t part = blockIdx.x % parts, j = (blockIdx.x / parts) * kPipeWaves + w;
    const int64_t x_begin = part * tiles_per_part;
    const int64_t x_end = x_begin + tiles_per_part < n_tiles ? x_begin + tiles_per_part : n_tiles;
    const int64_t t_first = x_begin + j, stride = waves_per_part;
    extern __shared__ __align__(16) int32_t s_hot[];     // C: the hot list (hot_ints of it)
    const int n_hot4 = C ? hot_ints(cz.n_hot) / 4 : 0;
    const char *Xf = X + 16 * f;

    // ---- CSR pipeline: rp_a and cc/vv belong to the next tile to be staged, rp_b to the one after
    int64_t rp_a = 0, rp_b = 0;
    int32_t cc[kH];
    float vv[kH];
#pragma unroll
    for (int h = 0; h < kH; ++h) { cc[h] = 0; vv[h] = 0.f; }
    bool ok_a = false;
    int32_t len_a = 0;                                   // lanes 0..kTileRows-1: stored length of the tile's row
    uint32_t live_a = 0;                                 // bit h: slot l + 64 h holds an entry
    int32_t base_a = 0;                                  // C: first row of the tile that cc belongs to
    int64_t oid_a = 0, oid_b = 0;                        // M: out_ids of the rows that rp_a / rp_b belong to
    auto load_oid = [&](int64_t tile) -> int64_t {
        if constexpr (!M) return 0;
        const int64_t ri = tile * kTileRows + (l < kTileRows ? l : 0);
        return out_ids[ri < n ? ri : 0];                 // rows past the end: any valid entry, never used
    };
    auto load_rp = [&](int64_t tile) -> int64_t {
        const int64_t ri = tile * kTileRows + (l < kTileRows ? l : kTileRows);
        // lanes 0..kTileRows hold the pointers; rows past the end read rowptr[n]
        if constexpr (C) return (int64_t)cz.rp32[ri < n ? ri : n];       // all of them below 2^32
        else return rowptr[ri < n ? ri : n];
    };
    auto load_cols = [&](int64_t tile) {                 // from rp_a: every slot fetches its own entry
        // a tile takes part in the pipeline when all its rows exist; a row that does not fit its slots (too long,
        // or high-degree) has no live slot, whatever its length: it does not disturb the rows around it
        ok_a = (tile + 1) * kTileRows <= n && tile < x_end;
        base_a = ok_a ? (int32_t)(tile * kTileRows) : 0;
        const int64_t begin = __shfl(rp_a, 0);
        const int32_t rel = ok_a ? (int32_t)(rp_a - begin) : 0;
        len_a = __shfl_down(rel, 1) - rel;
        live_a = 0;
        // unconditional loads (a dead slot reads entry 0): the number of loads in flight stays known
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            const int s = l + kWave * h;                 // slot s: row r, entry k
            const int r = s / kPipeD, k = s - r * kPipeD;
            const int32_t lo = __shfl(rel, r), len = __shfl(rel, r + 1) - lo;
            const bool live = s < kSlots && k < len && len <= kPipeD && len < T;
            live_a |= (uint32_t)live << h;
            const int64_t i = live ? begin + lo + k : 0;
            // (plain loads, no streaming hint: the cache line a tile's entries end in is the one the next tile's
            // begin in, and that tile belongs to another wavefront of the same XCD, a moment later; 1.7 % of a step)
            if constexpr (C) cc[h] = cz.col16[i];
            else cc[h] = col[i];
            if (W == kExplicit) vv[h] = val[i];
        }
    };
    auto stage = [&]() -> bool {                         // cc, vv, live_a, len_a -> slot table and row weights
        uint64_t badm[kH];                               // C: slots whose entry no code expresses
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            const int s = l + kWave * h;
            bool live = (live_a >> h) & 1;
            int32_t c = cc[h];
            if constexpr (C) {                           // code -> column: near the row, or one of the hot rows
                const bool bad = live && c == kCodeBad;
                badm[h] = __ballot(bad);
                live = live && !bad;
                const int32_t hot_c = s_hot[live && c >= kCodeHot ? c - kCodeHot : 0];
                c = c >= kCodeHot ? hot_c : base_a + s / kPipeD + c - kCodeNear;
            }
            if (s < kSlots) {
                const int64_t off = live ? row_bytes(c) : zero_off;
                if constexpr (W == kExplicit) s_slot[w][s] = SlotW{off, live ? vv[h] : 0.f, 0.f};
                else s_slot[w][s] = off;
            }
        }
        bool row_ok = ok_a && len_a <= kPipeD && len_a < T;
        if constexpr (C) {                               // a row with a bad slot is masked as a whole: slots l D .. l D + D - 1
            const int sb = l * kPipeD, sh = sb & 63;
            uint64_t w0 = 0, w1 = 0;
#pragma unroll
            for (int q = 0; q < kH; ++q) {
                w0 = (sb >> 6) == q ? badm[q] : w0;
                w1 = (sb >> 6) + 1 == q ? badm[q] : w1;
            }
            const uint64_t bits = (w0 >> sh) | (sh ? w1 << (64 - sh) : 0);
            row_ok = row_ok && (bits & ((1u << kPipeD) - 1)) == 0;
        }
        if (l < kTileRows) s_inv[w][l] = row_ok ? row_weight<W == kMean ? kMean : kOnes>(len_a) : -1.0f;
        if constexpr (M) {
            if (l < kTileRows) s_oid[w][l] = oid_a << kRowShift;
        }
        wave_sync();
        return ok_a;
    };

    // ---- one group: kRpg rows, one per lane group
    struct Regs {
        v4f xs[kPipeD];
        float ws[W == kExplicit ? kPipeD : 1];
        float inv;
        int64_t oid;                                     // M: where the row's sum goes
    };
    Regs rr[G];
    auto issue = [&](Regs &q, int grp) {
        const int lr = grp * kRpg + g;
        const int last = (kTileRows - 1) * kRowSlots;    // past the tile's last float4: its last row again, not stored
        const uint32_t at = (uint32_t)(slot_at < last ? slot_at : last);
        const Slot *const slots = S == 2 ? (const Slot *)((const char *)s_slot[w] + at) : s_slot[w] + lr * kPipeD;
        const char *const Xg = S == 2 ? X + f_at : Xf;
        q.inv = S == 2 ? s_inv[w][at / kRowSlots] : s_inv[w][lr];
        if constexpr (M) q.oid = s_oid[w][lr];
#pragma unroll
        for (int k = 0; k < kPipeD; ++k) {
            if constexpr (W == kExplicit) {
                const SlotW sl = slots[k];
                q.xs[k] = *(const v4f *)(Xg + sl.off);
                q.ws[k] = sl.w;
            } else {
                q.xs[k] = *(const v4f *)(Xg + slots[k]);
            }
        }
        if constexpr (S == 2) {                          // on to the next sweep; after the last one from the start
            const int f_next = f_at + f_step;
            const bool over = f_next >= F4 * 16;
            f_at = grp == G - 1 ? f_0 : over ? f_next - F4 * 16 : f_next;
            slot_at = grp == G - 1 ? slot_0 : slot_at + slot_step + (over ? kRowSlots : 0);
        }
    };
    auto sum = [&](const Regs &q) -> v4f {
        v4f a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kPipeD; ++k) {
            if (W == kExplicit) a += q.ws[k] * q.xs[k];
            else a += q.xs[k];
        }
        if (W == kMean) a *= q.inv;
        return a;
    };

    char *const tbase = trash + 16 * f;
    // ---- prologue: the first tile is staged and put in flight, the CSR of the next two is on its way.  The hot list is copied
    // meanwhile, 32 KB in flight at a time: a load and a store at a time, before the first row pointer was used, the copy
    // was a latency per 256 rows of the list in front of everything (4-LUT shape, 1 M rows, 4,096 of them hot, F = 64: 220 us, now 213).
    // Every wavefront takes part, also one without a tile: its loads read what exists.
    rp_a = load_rp(t_first);
    oid_a = load_oid(t_first);
    pipe_i4 hot_a[kHotAhead];
    auto load_hot = [&](int base) {
#pragma unroll
        for (int k = 0; k < kHotAhead; ++k) {
            const int i = base + k * (kPipeWaves * kWave) + threadIdx.x;
            hot_a[k] = ((const pipe_i4 *)cz.hot)[i < n_hot4 ? i : 0];
        }
    };
    auto store_hot = [&](int base) {
#pragma unroll
        for (int k = 0; k < kHotAhead; ++k) {
            const int i = base + k * (kPipeWaves * kWave) + threadIdx.x;
            if (i < n_hot4) ((pipe_i4 *)s_hot)[i] = hot_a[k];
        }
    };
    if constexpr (C) load_hot(0);
    load_cols(t_first);
    rp_b = load_rp(t_first + stride);                    // arrives with the columns
    oid_b = load_oid(t_first + stride);
    if constexpr (C) {
        store_hot(0);
#pragma unroll 1
        for (int base = kHotAhead * kPipeWaves * kWave; base < n_hot4; base += kHotAhead * kPipeWaves * kWave) {
            load_hot(base);
            store_hot(base);
        }
        __syncthreads();                                 // every wavefront of the sweep gets here: none has left
    }
    if (t_first >= x_end) return;
    bool ok_cur = stage();
#pragma unroll
    for (int grp = 0; grp < G; ++grp) issue(rr[grp], grp);
    rp_a = rp_b;
    oid_a = oid_b;
    load_cols(t_first + stride);
    rp_b = load_rp(t_first + 2 * stride);
    oid_b = load_oid(t_first + 2 * stride);
    // Everything above has arrived before the loop starts: the loop's own order of loads is then the
    // only one the compiler has to account for at the loop head, and its waits stay exact.
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)

    for (int64_t tile = t_first; tile < x_end; tile += stride) {
        const bool ok_next = stage();                    // CSR of the next tile -> slot table (this tile's groups are all issued)
        rp_a = rp_b;
        oid_a = oid_b;
        load_cols(tile + 2 * stride);
        rp_b = load_rp(tile + 3 * stride);
        oid_b = load_oid(tile + 3 * stride);
        const int64_t base = tile * kTileRows;
        char *const ybase = Y + row_bytes(base) + 16 * f;
        const __amdgpu_buffer_rsrc_t ytile =             // S: the tile's rows of Y; a store past their end is dropped
            __builtin_amdgcn_make_buffer_rsrc(Y + row_bytes(base), 0, (int)row_bytes(kTileRows), kPipeRawBuffer);
#pragma unroll
        for (int grp = 0; grp < G; ++grp) {
            const v4f a = sum(rr[grp]);
            const int lr = grp * kRpg + g;
            // a masked row (every row of a tile that is not ok) is not stored: a select of the address, no branch
            if constexpr (S) {
                const uint32_t at = S == 2 ? 16 * (grp * kWave + l) : (uint32_t)row_bytes(lr) + 16 * f;   // past the tile's end: dropped
                const uint32_t off = rr[grp].inv >= 0.f ? at : kPipeDropped;
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(pipe_u4, a), ytile, (int)off, 0, kPipeNontemporal);
            } else {
                char *const yrow = M ? Y + rr[grp].oid + 16 * f : ybase + (int)row_bytes(lr);
                char *const dst = rr[grp].inv >= 0.f ? yrow : tbase + (lr << kRowShift);
                __builtin_nontemporal_store(a, (v4f *)dst);
            }
            issue(rr[grp], grp);                         // the same rows of the next tile
        }
        if (!ok_cur) {
            // plain path: the rows of this tile that the pipeline serves elsewhere, straight from global memory
#pragma unroll 1
            for (int grp = 0; grp < G; ++grp) {
                const int i = grp * kWave + l, lr = S == 2 ? i / F4 : grp * kRpg + g, fr = S == 2 ? i % F4 : f;
                const int64_t row = base + lr;
                if (lr < kTileRows && row < n) {
                    const int64_t s = rowptr[row], e = rowptr[row + 1];
                    if (e - s < T && e - s <= kPipeD)
                        __builtin_nontemporal_store(ld_row_sum<W, false>(s, e, col, val, (const v4f *)X, S ? F4 : L, fr),
                                                    (v4f *)(Y + row_bytes(M ? out_ids[row] : row) + 16 * fr));
                }
            }
        }
        ok_cur = ok_next;
    }
}

// A long row list in a launch of its own, at full occupancy: one lane group per row.
template <int L, int W>
__global__ __launch_bounds__(kBlock) void ld_rows_kernel(const int32_t *__restrict__ rows, int64_t n_rows,
                                                         const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                                         const float *__restrict__ val, const v4f *__restrict__ X,
                                                         v4f *__restrict__ Y, int32_t F4, const int64_t *__restrict__ out_ids,
                                                         int64_t n)
{
    const int64_t k = (int64_t)blockIdx.x * (kBlock / L) + threadIdx.x / L;
    const int ff = threadIdx.x % L;
    if (k >= n_rows || ff >= F4) return;
    const int64_t row = rows[k];
    if (row >= n) return;                                // a row that is not wanted (row-mapped calls: boundary rows)
    __builtin_nontemporal_store(ld_row_sum<W, false>(rowptr[row], rowptr[row + 1], col, val, X, F4, ff),
                                Y + (out_ids ? out_ids[row] : row) * F4 + ff);
}

struct PipeArgs {
    const int64_t *rowptr;
    const int32_t *col;
    const float *val;
    CompactCsr cz;
    bool compact;
    const char *X;
    char *Y;
    int64_t zero_off;                        // byte distance from X to the plan's row of zeros
    char *trash;
    int64_t n;
    int32_t T;
    int64_t n_tiles, tiles_per_part, waves_per_part;
    int32_t parts;
    int64_t n_wg;
    hipStream_t st;
    const int64_t *out_ids;                  // row-mapped form, else NULL
    int32_t F4;                              // float4 per row
    int32_t tile_rows;                       // S = 2: rows of a tile; else 0
    SideWork side;
    int64_t n_hd;                            // pieces of high-degree rows in this launch
};

template <int L, int W, int G, int D>
static void pipe_launch(const PipeArgs &a)
{
    const dim3 grid((unsigned)(a.n_wg + a.side.n_row_wg + a.n_hd));
    if (a.out_ids) {
        ld_pipe_kernel<L, W, G, D, false, true><<<grid, dim3(kPipeWaves * kWave), 0, a.st>>>(
            a.rowptr, a.col, a.val, a.cz, a.X, a.Y, a.zero_off, a.trash, a.n, a.T, a.n_tiles, a.tiles_per_part,
            a.waves_per_part, a.parts, a.out_ids, a.F4, a.tile_rows, a.side);
    } else if (a.compact) {
        const size_t lds = (size_t)hot_ints(a.cz.n_hot) * sizeof(int32_t);
        ld_pipe_kernel<L, W, G, D, true><<<grid, dim3(kPipeWaves * kWave), lds, a.st>>>(
            a.rowptr, a.col, a.val, a.cz, a.X, a.Y, a.zero_off, a.trash, a.n, a.T, a.n_tiles, a.tiles_per_part,
            a.waves_per_part, a.parts, nullptr, a.F4, a.tile_rows, a.side);
    } else {
        ld_pipe_kernel<L, W, G, D, false><<<grid, dim3(kPipeWaves * kWave), 0, a.st>>>(
            a.rowptr, a.col, a.val, a.cz, a.X, a.Y, a.zero_off, a.trash, a.n, a.T, a.n_tiles, a.tiles_per_part,
            a.waves_per_part, a.parts, nullptr, a.F4, a.tile_rows, a.side);
    }
}

template <int L, int W, int G, int D, int S>
static void pipe_launch_any(const PipeArgs &a)
{
    const dim3 grid((unsigned)(a.n_wg + a.side.n_row_wg + a.n_hd));
    if (a.compact) {
        const size_t lds = (size_t)hot_ints(a.cz.n_hot) * sizeof(int32_t);
        ld_pipe_kernel<L, W, G, D, true, false, S><<<grid, dim3(kPipeWaves * kWave), lds, a.st>>>(
            a.rowptr, a.col, a.val, a.cz, a.X, a.Y, a.zero_off, a.trash, a.n, a.T, a.n_tiles, a.tiles_per_part,
            a.waves_per_part, a.parts, nullptr, a.F4, a.tile_rows, a.side);
    } else {
        ld_pipe_kernel<L, W, G, D, false, false, S><<<grid, dim3(kPipeWaves * kWave), 0, a.st>>>(
            a.rowptr, a.col, a.val, a.cz, a.X, a.Y, a.zero_off, a.trash, a.n, a.T, a.n_tiles, a.tiles_per_part,
            a.waves_per_part, a.parts, nullptr, a.F4, a.tile_rows, a.side);
    }
}

template <int W>
static void rows_dispatch_l(int L, int64_t n_wg, int64_t n_rows, const PipeArgs &a)
{
    auto launch = [&](auto kernel) {
        kernel<<<dim3((unsigned)n_wg), dim3(kBlock), 0, a.st>>>(a.side.rows, n_rows, a.rowptr, a.col, a.val, (const v4f *)a.X,
                                                                (v4f *)a.Y, a.F4, a.out_ids, a.n);
    };
    if (L == 8) launch(ld_rows_kernel<8, W>);
    else if (L == 16) launch(ld_rows_kernel<16, W>);
    else if (L == 32) launch(ld_rows_kernel<32, W>);
    else launch(ld_rows_kernel<64, W>);
}

template <int W, int D>
static void pipe_dispatch_l(int32_t F4, const PipeArgs &a)
{
    if (F4 == 8) pipe_launch<8, W, pipe_groups(8), D>(a);
    else if (F4 == 16) pipe_launch<16, W, pipe_groups(16), D>(a);
    else if (F4 == 32) pipe_launch<32, W, pipe_groups(32), D>(a);
    else if (F4 < 8) pipe_launch_any<8, W, pipe_groups(8), D, 1>(a);
    else if (F4 < 16) a.tile_rows ? pipe_launch_any<16, W, pipe_groups(16), D, 2>(a) : pipe_launch_any<16, W, pipe_groups(16), D, 1>(a);
    else if (F4 < 32) a.tile_rows ? pipe_launch_any<32, W, pipe_groups(32), D, 2>(a) : pipe_launch_any<32, W, pipe_groups(32), D, 1>(a);
    else a.tile_rows ? pipe_launch_any<64, W, pipe_groups(64), D, 2>(a) : pipe_launch_any<64, W, pipe_groups(64), D, 1>(a);
}

template <int W>
static void pipe_dispatch_d(int depth, int32_t F4, const PipeArgs &a)
{
    switch (depth) {
    case 5: pipe_dispatch_l<W, 5>(F4, a); break;
    case 6: pipe_dispatch_l<W, 6>(F4, a); break;
    case 7: pipe_dispatch_l<W, 7>(F4, a); break;
    default: pipe_dispatch_l<W, 8>(F4, a); break;
    }
}

// The compact form keeps the hot list in dynamic LDS, up to 128 KB: the runtime wants to be told once per
// kernel that more than its default limit may be asked for.  Called when a plan gets its compact CSR (not at
// launch, which may be under stream capture).
template <int L, int W, int D, int S>
static int pipe_allow_lds()
{
    return (int)hipFuncSetAttribute((const void *)&ld_pipe_kernel<L, W, pipe_groups(L), D, true, false, S>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, hot_ints(kCodeMaxHot) * (int)sizeof(int32_t));
}
template <int W, int D>
static int pipe_allow_lds_l()
{
    int err = pipe_allow_lds<8, W, D, 0>();
    if (!err) err = pipe_allow_lds<16, W, D, 0>();
    if (!err) err = pipe_allow_lds<32, W, D, 0>();
    if (!err) err = pipe_allow_lds<8, W, D, 1>();
    if (!err) err = pipe_allow_lds<16, W, D, 1>();
    if (!err) err = pipe_allow_lds<32, W, D, 1>();
    if (!err) err = pipe_allow_lds<64, W, D, 1>();
    if (!err) err = pipe_allow_lds<16, W, D, 2>();
    if (!err) err = pipe_allow_lds<32, W, D, 2>();
    if (!err) err = pipe_allow_lds<64, W, D, 2>();
    return err;
}
template <int W>
static int pipe_allow_lds_d()
{
    int err = pipe_allow_lds_l<W, 5>();
    if (!err) err = pipe_allow_lds_l<W, 6>();
    if (!err) err = pipe_allow_lds_l<W, 7>();
    if (!err) err = pipe_allow_lds_l<W, 8>();
    return err;
}
int pipe_compact_prepare()
{
    static std::atomic<int> state{-1};                   // -1 not tried, else the result
    int s = state.load();
    if (s >= 0) return s;
    int err = pipe_allow_lds_d<kOnes>();
    if (!err) err = pipe_allow_lds_d<kMean>();
    if (!err) err = pipe_allow_lds_d<kExplicit>();
    state.store(err);
    return err;
}

// Rows of the list that the sweep's launch takes along.  They run there at the sweep's occupancy, so a long list wants a launch
// of its own.  Rows of 9 to 14 entries, beside the sweep / in a launch of their own, us:
//   5 slots, F = 24    155,625 of 4 M rows     315 / 333
//   5 slots, F = 32     11,001 of 0.5 M       43.6 / 44.5    21,332 of 1 M     71.7 / 69.7    155,625 of 4 M  392 / 325
//   5 slots, F = 64      2,861 of 0.5 M       55.9 / 60.3    11,001 of 0.5 M   68.6 / 61.9    155,625 of 4 M  618 / 645
//   5 slots, F = 100     3,238 of 0.1 M       33.3 / 36.9    11,001 of 0.5 M   99.1 / 86.5    155,625 of 4 M  1,095 / 1,117
//   5 slots, F = 128     5,043 of 1 M          276 / 285     155,625 of 4 M   1,206 / 1,244
//   8 slots, F = 32      5,043 of 1 M         72.7 / 83.1    21,332 of 1 M     86.1 / 87.0
//   8 slots, F = 100     5,043 of 1 M          343 / 339     21,332 of 1 M      392 / 349
// From F = 36 on with 5 slots it depends on whether X stays in the last-level cache (F = 64, 0.5 M rows): a sweep that
// waits for the memory has room for any list.
static int64_t rows_beside_sweep(int depth, int32_t F4, int64_t n_rows)
{
    constexpr int64_t kCacheBytes = (int64_t)256 << 20;
    if (depth == 5 && F4 < 8) return n_rows;
    if (F4 <= 8) return 16384;
    if (depth > 5) return 8192;
    return n_rows * F4 * 16 < kCacheBytes ? 4096 : n_rows;
}

// Whether a whole-graph call reads the compact matrix.  It halves the bytes of the matrix and costs the decoding of every
// slot, so it pays where the feature matrices come from HBM.  Whole step, us, compact / plain arrays, by the bytes of X:
//   5 slots: 67 MB (multiplier, F = 32) 36.0 / 32.4; 134 MB (F = 32) 59.9 / 55.9, (F = 64) 49.3 / 48.7, (Booth, F = 32) 66.6 / 63.3;
//     208 MB (F = 100) 77.7 / 78.5, (Booth, F = 128) 82.8 / 81.0; 267 MB (F = 32) 123.7 / 124.0, (F = 64) 118.9 / 118.4, (F = 128)
//     117.5 / 124.2; 535 MB (F = 64) 233.9 / 238.3; 2.1 GB (F = 64) 941 / 962
//   6 and 7 slots: 134 MB (4-LUT, F = 32) 104.8 / 94.4; 271 MB (cells, F = 32) 172.7 / 166.0, (4-LUT, F = 64) 212.2 / 215.4; 424 MB
//     (4-LUT, F = 100) 369.8 / 364.2; 540 MB (F = 64) 423.9 / 423.6, (cells) 317.5 / 316.4; 844 MB 710.1 / 710.8; 1.1 GB (4-LUT, F = 32)
//     803 / 811, (cells) 628 / 640
// (All from the second pass on.  On inputs that no cache holds 5 slots are even at 67 MB and 1.5 to 3 % faster with the compact matrix
// at 134 MB, 84.9 / 86.1 (F = 64) and 94.6 / 97.0 (F = 32), 4 to 6 % slower at 140 and 167 MB, 105.5 / 99.6 and 109.9 / 105.9; 6 to 8 slots
// 1 to 2 % slower up to 424 MB.)
bool compact_pays(const DevicePlan &dp, int32_t F)
{
    const int64_t line = dp.pipe_depth <= 5 ? (int64_t)192 << 20 : (int64_t)1 << 30;
    return dp.compact_always || dp.n_cols * F * 4 >= line;
}

bool ld_reads_compact(const DevicePlan &dp, int32_t F)
{
    return dp.compressed && dp.rp32 && dp.col16 && dp.hot_cols && compact_pays(dp, F);
}

// Whether a plan for widths up to max_F gets it: where some width reads it.  For no reader it would be 4 n + 2 nnz bytes, two
// kernels over the matrix and, in groot_plan_upload, a wait.
bool ld_builds_compact(const DevicePlan &dp, int32_t max_F, int knob)
{
    return dp.ld_pipelined && knob && compact_pays(dp, max_F < kPipeMaxF ? max_F : kPipeMaxF);
}

// out: the leading out->n_out rows only, row r written to row out->ids[r] of Y (ids NULL: to row r)
int launch_ld_pipelined(const DevicePlan &dp, const float *X, float *Y, int32_t F, void *stream, const RowOut *out, bool with_hd)
{
    const int64_t n_rows = out ? out->n_out : dp.n;
    const int64_t *out_ids = out ? out->ids : nullptr;
    if (n_rows < 0 || n_rows > dp.n) return (int)hipErrorInvalidValue;
    if (n_rows == 0) return 0;
    const int32_t F4 = F / 4;
    if (F4 <= 4 || F4 > kWave || (out && F4 != 8 && F4 != 16 && F4 != 32)) return (int)hipErrorInvalidValue;
    if (!weights_ok(dp) || !dp.zero_row) return (int)hipErrorInvalidValue;
    if (dp.pipe_depth < kPipeMinDepth || dp.pipe_depth > kPipeMaxDepth) return (int)hipErrorInvalidValue;
    if (dp.n_mid_rows && !dp.mid_rows) return (int)hipErrorInvalidValue;
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return (int)e;
    int L = 8;                                           // lanes per row
    while (L < F4) L *= 2;
    const int packed_rows = pipe_tile_rows(L, F4, dp.pipe_depth, n_rows), tile_rows = packed_rows ? packed_rows : pipe_groups(L) * (kWave / L);
    const int64_t n_tiles = (n_rows + tile_rows - 1) / tile_rows;
    // one workgroup per CU; consecutive workgroup ids land on different XCDs
    int64_t n_wg = cus / kXcds * kXcds;
    if (n_wg < kXcds) n_wg = kXcds;
    const int32_t parts = dp.xcd_remap ? kXcds : 1;
    const int64_t tiles_per_part = (n_tiles + parts - 1) / parts;
    const int64_t wanted = (tiles_per_part + kPipeWaves - 1) / kPipeWaves * parts;   // a small graph: a wavefront per tile
    n_wg = wanted < n_wg ? wanted : n_wg / parts * parts;
    const int64_t waves_per_part = n_wg / parts * kPipeWaves;
    if (!grid_ok(n_wg) || n_tiles <= 0) return (int)hipErrorInvalidConfiguration;
    // the kernel reads entry 0 of the index (and weight) array from idle lanes: give it something to read
    // when the matrix has no entries, or no weight array
    const int32_t *col_arg = dp.col ? dp.col : (const int32_t *)dp.rowptr;
    const float *val_arg = dp.val ? dp.val : (const float *)dp.rowptr;
    char *trash = (char *)(dp.zero_row + kZeroRowFloats);
    static_assert(pipe_groups(8) <= 8 && pipe_groups(16) <= 8 && pipe_groups(32) <= 8 && 8 * kWave * 16 <= kTrashFloats * 4,
                  "a tile's masked sums fit the trash area");
    hipStream_t st = (hipStream_t)stream;
    // the compact matrix codes rows that the row list serves as uncoded, which only holds for whole-graph calls
    const bool compact = !out && ld_reads_compact(dp, F);
    // the low-degree rows with more entries than the pipeline has slots; the rows that the compact matrix cannot
    // code stand at the end of the list and are the pipeline's own whenever it reads the plain arrays
    const int64_t n_mid = compact ? dp.n_mid_rows : dp.n_mid_rows - dp.n_bad_rows;
    const int64_t list_wg = n_mid > 0 ? (n_mid + kBlock / L - 1) / (kBlock / L) : 0;
    const bool own_list = n_mid > rows_beside_sweep(dp.pipe_depth, F4, n_rows);
    const int64_t n_row_wg = own_list ? 0 : list_wg;
    const int64_t n_hd = with_hd ? dp.n_chunks : 0;
    if (!grid_ok(n_wg + n_row_wg + n_hd)) return (int)hipErrorInvalidConfiguration;
    const PipeArgs a{dp.rowptr, col_arg, val_arg, CompactCsr{dp.rp32, dp.col16, dp.hot_cols, dp.n_hot}, compact,
                     (const char *)X, (char *)Y, byte_distance(X, dp.zero_row), trash, n_rows,
                     dp.threshold, n_tiles, tiles_per_part, waves_per_part, parts, n_wg, st, out_ids, F4, packed_rows,
                     SideWork{n_wg, dp.mid_rows, n_mid, n_row_wg, dp.chunks, dp.partials}, n_hd};
    GROOT_DISPATCH_W(dp.weight_mode, (pipe_dispatch_d<kW>(dp.pipe_depth, F4, a)));
    e = hipGetLastError();
    if (e != hipSuccess || !own_list) return (int)e;
    GROOT_DISPATCH_W(dp.weight_mode, (rows_dispatch_l<kW>(L, list_wg, n_mid, a)));
    return (int)hipGetLastError();
}

}  // namespace groot
