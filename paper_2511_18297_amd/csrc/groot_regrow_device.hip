// Device-side partition with boundary edge re-growth for gfx950 (paper: Section "GNN and Edge Re-growth
// After Partition", Eq. (1), Eq. (2), Algorithm 1), one part per call, from the CSR that an uploaded plan
// keeps on the device.  All integer work; the result is bit-identical to the host's groot_partition_regrow.
//
// A node set is one bit per node of the whole graph plus the number of set bits before every 32-bit word, so a node's place in
// it is two loads from arrays of N / 8 bytes (which an L2 holds; one int32 per node does not fit one, had to be cleared, and was
// read twice to be compacted).  For part p with node set S_p:
//   rg_mark      (or rg_mark_slices) every owned row flags its columns in other parts: B_p (Eq. (1)), and counts them
//   rg_count / rg_place
//                flags to bits and bits per workgroup, then places before every word and the ids themselves, ascending: S_p
//                first, B_p after (global_id).  S_p under the built-in rule is one slice of every copy and needs neither bits nor loads.
//   rg_row_len (+ rg_row_len_long where a long row has to be walked, one wavefront per row)
//                stored length of every local row: an owned row keeps its whole neighbourhood, a boundary
//                row keeps its self-loop and its edges into S_p (the crossing edges C_p of Eq. (2))
//   rg_len_write exclusive prefix of the lengths: the sub-graph's row pointer
//   rg_fill      the sub-graph's columns (and weights): local ids are monotone in the global id inside
//                S_p and inside B_p, so a row sorted by global column becomes sorted by local column by
//                writing its owned columns first and its boundary columns after
// Seven launches where long rows need no walk.  The parts are small, so launches and the latencies inside them are most of the
// time: with 14 launches and the int32 numbering a part of 10 thousand rows (109-bit multiplier, 9 parts) took 66 us of kernels,
// now 30, one of a million rows (512-bit x 4, 8 parts) 191, now 95.
#include "groot_device.h"

namespace groot {

constexpr int kRgWords = 4;                                        // words of a node set per thread
constexpr int kRgBlockWords = kBlock * kRgWords;                   // ... per workgroup: 32,768 nodes
constexpr int kRgLenBlock = 1024;                                  // rows per workgroup of the length kernels
constexpr int kRgFusedSums = 4096;                                 // up to so many of them every workgroup adds up those before it
// ... so many workgroups of words, 134 M nodes.  Every one adding up those before it is quadratic; rg_place without / with the scan and its time, us:
// 42 M nodes 14.2 / 16.5, 134 M 19.4 / 20.1 (and the launch); at 2^31 nodes 2 x 10^9 loads, or a scan.
constexpr int kRgFusedCounts = 4096;
constexpr int kRgMark = 8;                                         // entries in flight per thread of rg_mark_slices
constexpr int kRgShort = 16;                                       // longest row that one lane walks alone
constexpr int kRgUnroll = 4;                                       // 64-entry chunks of a long row in flight
constexpr int kRgLongBlocks = 2048;                                // workgroups that share the long rows, at most
constexpr int kRgSlots = 64;                                       // counters that share the additions to one total

// totals on the device, kRgSlots 64-bit counters each, then two 32-bit numbers
enum : int { kRgHalo = 0, kRgOwned = kRgSlots, kRgCross = 2 * kRgSlots, kRgNnz = 3 * kRgSlots, kRgEnd = 4 * kRgSlots };

// sum of x over the workgroup, for thread 0 (every thread calls); Waves: wavefronts of the workgroup
template <int Waves>
__device__ __forceinline__ int64_t rg_block_sum(int64_t x)
{
    __shared__ int64_t s_sum[Waves];
    for (int off = kWave / 2; off > 0; off >>= 1) x += __shfl_down(x, off);
    __syncthreads();                                     // an earlier sum has been read
    if (threadIdx.x % kWave == 0) s_sum[threadIdx.x / kWave] = x;
    __syncthreads();
    int64_t t = 0;
    for (int w = 0; w < Waves; ++w) t += s_sum[w];
    return t;
}

// One addition per workgroup, to one of kRgSlots counters: one address took 10 ns per addition
__device__ __forceinline__ void rg_add(unsigned long long *__restrict__ slots, int64_t x)
{
    if (x) atomicAdd(&slots[blockIdx.x % kRgSlots], (unsigned long long)x);
}

struct RgGraph {
    const int64_t *rowptr;
    const int32_t *col;
    const float *val;          // NULL unless the weights are explicit
    int64_t n, n1;
    const int32_t *part_of;    // NULL: the built-in rule
    int32_t p;
    uint32_t lo, hi;           // built-in rule: part p owns the nodes with lo <= (v mod n1) < hi
    bool sliced;               // the built-in rule on whole copies (whose edges stay inside them): S_p needs no bits
    bool regrow;
    bool symmetric;            // every edge is known to be stored in both directions
    uint8_t *halo_flag;        // one byte per node: it is in B_p
    uint32_t *halo, *own;      // bits of B_p, of S_p (NULL if sliced)
    uint32_t *halo_before, *own_before;   // set bits before every word
    int64_t n_owned;           // known from the launch of rg_place on
};

// Is node v in part p?  The caller's array, or the p-th contiguous slice of every copy:
// floor(r P / n1) = p  <=>  ceil(p n1 / P) <= r < ceil((p + 1) n1 / P)  for r = v mod n1 (n < 2^31).
__device__ __forceinline__ bool rg_in_part(const RgGraph &g, int64_t v)
{
    if (g.part_of) return g.part_of[v] == g.p;
    const uint32_t r = (uint32_t)v % (uint32_t)g.n1;
    return r >= g.lo && r < g.hi;
}

__device__ __forceinline__ int64_t rg_rank(const uint32_t *__restrict__ bits, const uint32_t *__restrict__ before, uint32_t u)
{
    return (int64_t)before[u / 32] + __popc(bits[u / 32] & ((1u << (u % 32)) - 1));
}

// The part's nodes as seen from row v: its columns lie in v's copy.
struct RgOwn {
    uint32_t first, end;       // sliced: the part's nodes of the copy
    int64_t base;              // ... and the place of the first of them
};

__device__ __forceinline__ RgOwn rg_own(const RgGraph &g, int64_t copy)
{
    return RgOwn{(uint32_t)(copy * g.n1) + g.lo, (uint32_t)(copy * g.n1) + g.hi, copy * (int64_t)(g.hi - g.lo)};
}

__device__ __forceinline__ bool rg_owned(const RgGraph &g, const RgOwn &o, uint32_t u)
{
    return g.sliced ? u >= o.first && u < o.end : (g.own[u / 32] >> (u % 32) & 1) != 0;
}

// place of an owned node
__device__ __forceinline__ int64_t rg_own_place(const RgGraph &g, const RgOwn &o, uint32_t u)
{
    return g.sliced ? o.base + (u - o.first) : rg_rank(g.own, g.own_before, u);
}

// local row k -> global row and the part's nodes of its copy
__device__ __forceinline__ int64_t rg_global(const RgGraph &g, const int64_t *__restrict__ global_id, int64_t k, RgOwn &o)
{
    if (!g.sliced) {
        o = RgOwn{0, 0, 0};
        return global_id[k];
    }
    if (k < g.n_owned) {
        const uint32_t slice = g.hi - g.lo, copy = (uint32_t)k / slice;
        o = rg_own(g, copy);
        return (int64_t)o.first + ((uint32_t)k - copy * slice);
    }
    const int64_t v = global_id[k];
    o = rg_own(g, (uint32_t)v / (uint32_t)g.n1);
    return v;
}

__global__ __launch_bounds__(kBlock) void rg_fill_i32(int32_t *__restrict__ a, int64_t n, int32_t value)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) a[i] = value;
}

__global__ __launch_bounds__(kBlock) void rg_clear(uint4 *__restrict__ a, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) a[i] = make_uint4(0, 0, 0, 0);
}

// bits of S_p, whole workgroups of words; flag[0] = 1 when a caller-supplied part id lies outside [0, P)
__global__ __launch_bounds__(kBlock) void rg_own_bits(RgGraph g, int32_t P, int32_t *__restrict__ flag)
{
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    bool in = false;
    if (v < g.n) {
        in = rg_in_part(g, v);
        if (g.part_of && (g.part_of[v] < 0 || g.part_of[v] >= P)) atomicOr(flag, 1);
    }
    const uint64_t m = __ballot(in);
    if (threadIdx.x % kWave == 0) *(uint64_t *)&g.own[v / 32] = m;
}

// Every owned row marks its columns of other parts, each of which is a crossing pair.  One byte per node, so that rows which mark
// the same node (the primary inputs: thousands) store the same value and need no atomics: with an atomic OR on the bits, skipped
// where the bit is seen to be set, 709 us for a part of the 512-bit multiplier x 4, with bytes 13.
__global__ __launch_bounds__(kBlock) void rg_mark(RgGraph g, unsigned long long *__restrict__ totals)
{
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const RgOwn none{0, 0, 0};
    int64_t cross = 0;
    if (v < g.n && rg_owned(g, none, (uint32_t)v)) {
        const int64_t b = g.rowptr[v], e = g.rowptr[v + 1];
        for (int64_t q = b; q < e; ++q) {
            const uint32_t u = (uint32_t)g.col[q];
            if (!rg_owned(g, none, u)) {
                g.halo_flag[u] = 1;
                ++cross;
            }
        }
    }
    cross = rg_block_sum<kWavesPerBlock>(cross);
    if (threadIdx.x == 0) rg_add(totals + kRgCross, cross);
}

// The same for slices: the part's rows of a copy (blockIdx.y) are consecutive, and so are their entries; which row
// an entry belongs to does not matter.  By rows the part that owns the primary inputs of a multiplier took 367 us (a lane walked
// 513 entries one after the other), and 346 with a wavefront per such row, 64 of which stand side by side; the others 13.
__global__ __launch_bounds__(kBlock) void rg_mark_slices(RgGraph g, unsigned long long *__restrict__ totals)
{
    const RgOwn o = rg_own(g, blockIdx.y);
    const int64_t b = g.rowptr[o.first], e = g.rowptr[o.end], step = (int64_t)gridDim.x * kBlock;
    const int32_t *__restrict__ const col = g.col;
    uint8_t *__restrict__ const flag = g.halo_flag;
    int32_t cross = 0;
    for (int64_t q = b + (int64_t)blockIdx.x * kBlock + threadIdx.x; q < e; q += kRgMark * step) {
        uint32_t u[kRgMark];
#pragma unroll
        for (int k = 0; k < kRgMark; ++k) u[k] = (uint32_t)col[q + k * step < e ? q + k * step : q];
#pragma unroll
        for (int k = 0; k < kRgMark; ++k)
            if (u[k] < o.first || u[k] >= o.end) {
                flag[u[k]] = 1;
                cross += q + k * step < e;
            }
    }
    const int64_t sum = rg_block_sum<kWavesPerBlock>(cross);
    if (threadIdx.x == 0) rg_add(totals + kRgCross, sum);
}

// Set bits of a workgroup's words: B_p (blockIdx.y = 0), whose flags become bits here, S_p (1); cnt[set][workgroup]
__global__ __launch_bounds__(kBlock) void rg_count(RgGraph g, int32_t *__restrict__ cnt, unsigned long long *__restrict__ totals)
{
    int32_t mine = 0;
    if (blockIdx.y) {
        const uint4 w = ((const uint4 *)g.own)[(int64_t)blockIdx.x * kBlock + threadIdx.x];
        mine = __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
    } else {
        constexpr int kRuns = kRgBlockWords * 32 / 16 / kBlock;          // 16 flags per thread and run
        const int64_t first = (int64_t)blockIdx.x * kRgBlockWords * 2;
        uint4 f[kRuns];
#pragma unroll
        for (int i = 0; i < kRuns; ++i) f[i] = ((const uint4 *)g.halo_flag)[first + i * kBlock + threadIdx.x];
#pragma unroll
        for (int i = 0; i < kRuns; ++i) {
            // four flags -> bits 28..31 of the product, no two terms of which meet
            const uint32_t half = f[i].x * 0x10204080u >> 28 | f[i].y * 0x10204080u >> 28 << 4 | f[i].z * 0x10204080u >> 28 << 8 |
                                  f[i].w * 0x10204080u >> 28 << 12;
            mine += __popc(half);
            const uint32_t other = __shfl_down(half, 1);
            if (threadIdx.x % 2 == 0) g.halo[(first + i * kBlock + threadIdx.x) / 2] = half | other << 16;
        }
    }
    const int64_t sum = rg_block_sum<kWavesPerBlock>(mine);
    if (threadIdx.x == 0) {
        cnt[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = (int32_t)sum;
        rg_add(totals + (blockIdx.y ? kRgOwned : kRgHalo), sum);
    }
}

// exclusive prefix of x over the workgroup's threads (every thread calls)
template <int Waves>
__device__ __forceinline__ int64_t rg_block_prefix(int64_t x)
{
    __shared__ int64_t s_w[Waves];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    int64_t incl = x;
    for (int off = 1; off < kWave; off <<= 1) {
        const int64_t up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    if (lane == kWave - 1) s_w[wave] = incl;
    __syncthreads();
    int64_t run = incl - x;
    for (int w = 0; w < wave; ++w) run += s_w[w];
    return run;
}

// One workgroup per array of n_sums numbers: they become the sums of those before them, which T holds.
template <class T>
__global__ __launch_bounds__(kRgLenBlock) void rg_scan_sums(T *__restrict__ sums, int64_t n_sums)
{
    sums += blockIdx.x * n_sums;
    const int64_t seg = (n_sums + kRgLenBlock - 1) / kRgLenBlock;
    const int64_t b0 = (int64_t)threadIdx.x * seg < n_sums ? (int64_t)threadIdx.x * seg : n_sums;
    const int64_t b1 = b0 + seg < n_sums ? b0 + seg : n_sums;
    int64_t sum = 0;
    for (int64_t b = b0; b < b1; ++b) sum += (int64_t)sums[b];
    int64_t run = rg_block_prefix<kRgLenBlock / kWave>(sum);
    for (int64_t b = b0; b < b1; ++b) {
        const int64_t v = (int64_t)sums[b];
        sums[b] = (T)run;
        run += v;
    }
}

// Set bits before every word and the ids of the set, ascending; grid as rg_count.  scanned: cnt holds prefixes already; else a workgroup adds
// up the counts of those before it by itself, up to kRgFusedCounts of them, one per 32,768 nodes.
__global__ __launch_bounds__(kBlock) void rg_place(RgGraph g, const int32_t *__restrict__ cnt, bool scanned, int64_t *__restrict__ global_id,
                                                   unsigned long long *__restrict__ sums, int64_t n_sums)
{
    if (blockIdx.y == 0)                                 // rg_row_len adds to them
        for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n_sums; i += (int64_t)gridDim.x * kBlock) sums[i] = 0;
    const bool own = blockIdx.y != 0;
    const uint32_t *const bits = own ? g.own : g.halo;
    cnt += (int64_t)blockIdx.y * gridDim.x;
    int64_t before = 0;
    if (scanned) {
        before = cnt[blockIdx.x];
    } else {
        for (int64_t b = threadIdx.x; b < blockIdx.x; b += kBlock) before += cnt[b];
        before = rg_block_sum<kWavesPerBlock>(before);
    }
    const int64_t at = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const uint4 w4 = ((const uint4 *)bits)[at];
    const uint32_t w[kRgWords] = {w4.x, w4.y, w4.z, w4.w};
    int64_t run = before + rg_block_prefix<kWavesPerBlock>(__popc(w[0]) + __popc(w[1]) + __popc(w[2]) + __popc(w[3]));
    uint32_t r[kRgWords];
    int64_t *const ids = global_id + (own ? 0 : g.n_owned);
#pragma unroll
    for (int k = 0; k < kRgWords; ++k) {
        r[k] = (uint32_t)run;
        for (uint32_t m = w[k]; m; m &= m - 1) ids[run++] = (at * kRgWords + k) * 32 + __ffs(m) - 1;
    }
    ((uint4 *)(own ? g.own_before : g.halo_before))[at] = make_uint4(r[0], r[1], r[2], r[3]);
}

// first entry in [lo, hi) whose column is at least u (columns ascending)
__device__ __forceinline__ int64_t rg_lower_bound(const RgGraph &g, int64_t lo, int64_t hi, uint32_t u)
{
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if ((uint32_t)g.col[mid] < u) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// is u a stored column of row v?
__device__ __forceinline__ bool rg_row_has(const RgGraph &g, int64_t v, uint32_t u)
{
    const int64_t e = g.rowptr[v + 1], at = rg_lower_bound(g, g.rowptr[v], e, u);
    return at < e && (uint32_t)g.col[at] == u;
}

// Is the entry (row v, column u) part of the sub-graph?  An owned row keeps its owned and (all of B_p being marked by it) its
// boundary columns, a boundary row its owned ones and its self-loop; a boundary-boundary edge is not in E_p+.
__device__ __forceinline__ bool rg_keep(const RgGraph &g, bool row_owned, int64_t v, uint32_t u, bool u_owned)
{
    return u_owned || (row_owned ? g.regrow : u == (uint32_t)v);
}

// A long row of slices need not be walked: its owned columns are consecutive.
__host__ __device__ __forceinline__ bool rg_long_by_search(const RgGraph &g) { return g.sliced && g.symmetric; }

// len[k] = stored length of local row k, sums[] += the lengths of kRgLenBlock rows each, and the rest of the crossing pairs: an edge stored only in
// the boundary row is one that its owned end did not count.  The slice's global ids, which no earlier kernel wrote, too.
// A lane walks a short row alone; a row above kRgShort entries (the primary inputs of a multiplier have
// thousands) is put on long_list (n_long[0] entries, any order) for rg_fill, and is walked by rg_row_len_long if it has to be.
// A workgroup's wavefronts take runs of 64 rows that lie far apart: side by side, the 4,096 rows of primary inputs fell to four
// CUs, whose vector memory units then bound the launch (a part of the 512-bit multiplier x 4: 36 us, now 25; eight ways instead of two, so four latencies with 21 loads each: 47 side by side).
__global__ __launch_bounds__(kBlock) void rg_row_len(RgGraph g, int64_t *__restrict__ global_id, int64_t n_loc,
                                                     int32_t *__restrict__ len, unsigned long long *__restrict__ sums,
                                                     unsigned long long *__restrict__ totals,
                                                     int32_t *__restrict__ long_list, int32_t *__restrict__ n_long)
{
    const int64_t run = (int64_t)(threadIdx.x / kWave) * gridDim.x + blockIdx.x, k = run * kWave + threadIdx.x % kWave;
    int64_t cross = 0;
    int32_t count = 0;
    if (k < n_loc) {
        RgOwn o;
        const int64_t v = rg_global(g, global_id, k, o);
        const bool row_owned = k < g.n_owned, whole = row_owned && g.regrow;
        if (g.sliced && row_owned) global_id[k] = v;
        const int64_t b = g.rowptr[v], e = g.rowptr[v + 1];
        const bool is_long = e - b > kRgShort;
        if (is_long) long_list[atomicAdd(n_long, 1)] = (int32_t)k;
        if (whole) {
            count = (int32_t)(e - b);
        } else if (!is_long) {
            for (int64_t q = b; q < e; q += 8) {         // eight columns in flight at a time
                uint32_t c[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) c[i] = (uint32_t)g.col[q + i < e ? q + i : e - 1];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const bool own = rg_owned(g, o, c[i]);
                    if (q + i < e && rg_keep(g, row_owned, v, c[i], own)) ++count;
                    if (q + i < e && own && !row_owned && !g.symmetric && !rg_row_has(g, c[i], (uint32_t)v)) ++cross;
                }
            }
        } else if (rg_long_by_search(g)) {
            // places of the slice's two ends and of v, the three searches in step: one latency per halving
            int64_t at[3] = {b, b, b};
            const uint32_t want[3] = {o.first, o.end, (uint32_t)v};
            uint32_t c[3];
            for (int64_t left = e - b; left > 1;) {
                const int64_t half = left / 2;
#pragma unroll
                for (int i = 0; i < 3; ++i) c[i] = (uint32_t)g.col[at[i] + half - 1];
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (c[i] < want[i]) at[i] += half;
                left -= half;
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) c[i] = (uint32_t)g.col[at[i]];
            const int64_t first = at[0] + (c[0] < want[0]), end = at[1] + (c[1] < want[1]);
            bool self = c[2] == want[2];
            if (c[2] < want[2]) self = at[2] + 1 < e && (uint32_t)g.col[at[2] + 1] == want[2];
            count = (int32_t)(end - first) + (!row_owned && self);
        }
        len[k] = count;
    }
    int64_t of_run = count;
    for (int off = kWave / 2; off > 0; off >>= 1) of_run += __shfl_down(of_run, off);
    if (threadIdx.x % kWave == 0 && of_run) atomicAdd(&sums[run * kWave / kRgLenBlock], (unsigned long long)of_run);
    const int64_t sum = rg_block_sum<kWavesPerBlock>(count);
    if (threadIdx.x == 0) rg_add(totals + kRgNnz, sum);
    if (!g.symmetric) {
        cross = rg_block_sum<kWavesPerBlock>(cross);
        if (threadIdx.x == 0) rg_add(totals + kRgCross, cross);
    }
}

// The rows of long_list that rg_row_len left open, one wavefront per row at a time (kRgUnroll x 64 entries in flight).
__global__ __launch_bounds__(kBlock) void rg_row_len_long(RgGraph g, const int64_t *__restrict__ global_id,
                                                          int32_t *__restrict__ len, unsigned long long *__restrict__ sums,
                                                          unsigned long long *__restrict__ totals,
                                                          const int32_t *__restrict__ long_list,
                                                          const int32_t *__restrict__ n_long)
{
    const int lane = threadIdx.x % kWave;
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerBlock;
    const int32_t n_rows = n_long[0];
    int64_t cross = 0, nnz = 0;
    for (int64_t i = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave; i < n_rows; i += n_waves) {
        const int64_t k = long_list[i];
        RgOwn o;
        const int64_t v = rg_global(g, global_id, k, o);
        const bool row_owned = k < g.n_owned;
        if (row_owned && g.regrow) continue;
        const int64_t b = g.rowptr[v], e = g.rowptr[v + 1];
        int32_t count = 0;
        for (int64_t q0 = b; q0 < e; q0 += kRgUnroll * kWave) {
            uint32_t c[kRgUnroll];
#pragma unroll
            for (int u = 0; u < kRgUnroll; ++u) {
                const int64_t q = q0 + u * kWave + lane;
                c[u] = (uint32_t)g.col[q < e ? q : e - 1];
            }
#pragma unroll
            for (int u = 0; u < kRgUnroll; ++u) {
                const bool in = q0 + u * kWave + lane < e, own = rg_owned(g, o, c[u]);
                count += __popcll(__ballot(in && rg_keep(g, row_owned, v, c[u], own)));
                if (in && own && !row_owned && !g.symmetric && !rg_row_has(g, c[u], (uint32_t)v)) ++cross;
            }
        }
        if (lane == 0) {
            len[k] = count;
            atomicAdd(&sums[k / kRgLenBlock], (unsigned long long)count);
            nnz += count;
        }
    }
    nnz = rg_block_sum<kWavesPerBlock>(nnz);
    cross = rg_block_sum<kWavesPerBlock>(cross);
    if (threadIdx.x == 0) {
        rg_add(totals + kRgNnz, nnz);
        rg_add(totals + kRgCross, cross);
    }
}

// rowptr[k] = lengths before row k, four rows per thread.  scanned: sums holds prefixes already; else every workgroup adds up
// those before it (a scan in between would be a launch of 4 us; above kRgFusedSums the reads would be more than that).  A part of
// a million rows: one row per thread 12.5 us, now 8.0.
__global__ __launch_bounds__(kBlock) void rg_len_write(const int32_t *__restrict__ len, int64_t n,
                                                       const unsigned long long *__restrict__ sums, bool scanned,
                                                       int64_t *__restrict__ rowptr)
{
    constexpr int kPer = kRgLenBlock / kBlock;
    const int64_t k = (int64_t)blockIdx.x * kRgLenBlock + threadIdx.x * kPer;
    int32_t mine[kPer];
    int64_t all = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) mine[i] = k + i < n ? len[k + i] : 0;
    int64_t before = 0;
    if (scanned) {
        before = (int64_t)sums[blockIdx.x];
    } else {
        for (int64_t b = threadIdx.x; b < blockIdx.x; b += kBlock) before += (int64_t)sums[b];
        before = rg_block_sum<kWavesPerBlock>(before);
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) all += mine[i];
    int64_t run = before + rg_block_prefix<kWavesPerBlock>(all);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (k + i < n) rowptr[k + i] = run;
        run += mine[i];
        if (k + i == n - 1) rowptr[n] = run;
    }
}

// local id of a column that the row keeps
__device__ __forceinline__ int64_t rg_local(const RgGraph &g, const RgOwn &o, bool row_owned, int64_t k, uint32_t u, bool u_owned)
{
    if (u_owned) return rg_own_place(g, o, u);
    return row_owned ? g.n_owned + rg_rank(g.halo, g.halo_before, u) : k;   // a boundary row keeps no boundary column but its own
}

// One wavefront per row of long_list at a time; positions inside a row by ballot ranks in lane order.
__device__ __forceinline__ void rg_fill_long(const RgGraph &g, const int64_t *__restrict__ global_id,
                                             const int64_t *__restrict__ sub_rowptr, int32_t *__restrict__ sub_col,
                                             float *__restrict__ sub_val, const int32_t *__restrict__ long_list, int32_t n_rows,
                                             int64_t first, int64_t n_waves)
{
    const int lane = threadIdx.x % kWave;
    const uint64_t lt_mask = lane ? (~0ULL >> (64 - lane)) : 0ULL;
    for (int64_t i = first; i < n_rows; i += n_waves) {
        const int64_t k = long_list[i];
        RgOwn o;
        const int64_t v = rg_global(g, global_id, k, o);
        const int64_t b = g.rowptr[v], e = g.rowptr[v + 1];
        const bool row_owned = k < g.n_owned;
        int64_t w = sub_rowptr[k];
        const int64_t w_end = sub_rowptr[k + 1];
        for (int pass = 0; pass < 2; ++pass)
            for (int64_t q0 = b; q0 < e && w < w_end; q0 += kRgUnroll * kWave) {
                uint32_t c[kRgUnroll];
#pragma unroll
                for (int u = 0; u < kRgUnroll; ++u) {
                    const int64_t q = q0 + u * kWave + lane;
                    c[u] = (uint32_t)g.col[q < e ? q : e - 1];
                }
#pragma unroll
                for (int u = 0; u < kRgUnroll; ++u) {
                    const int64_t q = q0 + u * kWave + lane;
                    const bool own = rg_owned(g, o, c[u]);
                    const bool keep = q < e && rg_keep(g, row_owned, v, c[u], own) && own == (pass == 0);
                    const uint64_t m = __ballot(keep);
                    const int64_t at = w + __popcll(m & lt_mask);
                    if (keep && at < w_end) {
                        sub_col[at] = (int32_t)rg_local(g, o, row_owned, k, c[u], own);
                        if (sub_val) sub_val[at] = g.val[q];
                    }
                    w += __popcll(m);
                }
            }
    }
}

// Columns (and weights) of the sub-graph: per row the kept entries with an owned column, in order, then those
// with a boundary column.  The first long_blocks workgroups take the rows of long_list, a wavefront each, the others short rows,
// a lane each.
__global__ __launch_bounds__(kBlock) void rg_fill(RgGraph g, const int64_t *__restrict__ global_id, int64_t n_loc,
                                                  const int64_t *__restrict__ sub_rowptr, int32_t *__restrict__ sub_col,
                                                  float *__restrict__ sub_val, const int32_t *__restrict__ long_list,
                                                  const int32_t *__restrict__ n_long, int32_t long_blocks)
{
    if ((int32_t)blockIdx.x < long_blocks) {
        rg_fill_long(g, global_id, sub_rowptr, sub_col, sub_val, long_list, n_long[0],
                     (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave, (int64_t)long_blocks * kWavesPerBlock);
        return;
    }
    const int64_t k = (int64_t)(blockIdx.x - long_blocks) * kBlock + threadIdx.x;
    if (k >= n_loc) return;
    RgOwn o;
    const int64_t v = rg_global(g, global_id, k, o);
    const int64_t b = g.rowptr[v], e = g.rowptr[v + 1];
    if (e - b > kRgShort) return;
    const bool row_owned = k < g.n_owned;
    int64_t w = sub_rowptr[k];
    const int64_t w_end = sub_rowptr[k + 1];
    if (e - b <= 8 && e > b) {                                   // nearly all rows: everything loaded before anything is placed
        uint32_t c[8];
        int32_t lc[8];
        float val[8];
        uint32_t kept = 0, owned = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t q = b + i < e ? b + i : e - 1;
            c[i] = (uint32_t)g.col[q];
            if (sub_val) val[i] = g.val[q];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bool own = rg_owned(g, o, c[i]), keep = b + i < e && rg_keep(g, row_owned, v, c[i], own);
            kept |= (uint32_t)keep << i;
            owned |= (uint32_t)(keep && own) << i;
            lc[i] = keep ? (int32_t)rg_local(g, o, row_owned, k, c[i], own) : 0;
        }
        const int n_own = __popc(owned);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t before = (1u << i) - 1, bit = 1u << i;
            const int64_t at = w + ((owned & bit) ? __popc(owned & before) : n_own + __popc(kept & ~owned & before));
            if ((kept & bit) && at < w_end) {                    // always true when the lengths match this walk
                sub_col[at] = lc[i];
                if (sub_val) sub_val[at] = val[i];
            }
        }
        return;
    }
    for (int pass = 0; pass < 2; ++pass)
        for (int64_t q = b; q < e; ++q) {
            const uint32_t c = (uint32_t)g.col[q];
            const bool own = rg_owned(g, o, c);
            if (own != (pass == 0) || !rg_keep(g, row_owned, v, c, own)) continue;
            if (w < w_end) {                                     // always true when the lengths match this walk
                sub_col[w] = (int32_t)rg_local(g, o, row_owned, k, c, own);
                if (sub_val) sub_val[w] = g.val[q];
            }
            ++w;
        }
}

namespace {

inline unsigned rg_grid(int64_t items, int per_block) { return (unsigned)((items + per_block - 1) / per_block); }

struct Scratch {
    void *p[8] = {};
    int used = 0;
    ~Scratch() { for (int i = 0; i < used; ++i) dev_free(p[i]); }
    template <class T>
    bool get(T **out, size_t count)
    {
        void *q = nullptr;
        if (used >= 8 || dev_alloc(&q, (count ? count : 1) * sizeof(T)) != 0) return false;
        p[used++] = q;
        *out = (T *)q;
        return true;
    }
};

int64_t rg_sum_slots(const int64_t *slots)
{
    int64_t t = 0;
    for (int i = 0; i < kRgSlots; ++i) t += slots[i];
    return t;
}

}  // namespace

void free_device_part(DevicePart &part)
{
    dev_free(part.global_id);
    dev_free(part.rowptr);
    dev_free(part.col);
    dev_free(part.val);
    part = DevicePart{};
}

// Returns 0, a hipError_t, kErrOutOfDeviceMemory, or kErrBadPartId (a part id outside [0, P)).
int launch_regrow_device(const DevicePlan &dp, int64_t n1, int32_t P, const int32_t *part_of_dev, int32_t p,
                         int regrow, bool symmetric, void *stream, DevicePart *out)
{
    hipStream_t st = (hipStream_t)stream;
    const int64_t n = dp.n;
    *out = DevicePart{};
    if (n < 1 || n > 0x7fffffffLL || n1 < 1 || n1 > n || P < 1 || p < 0 || p >= P) return (int)hipErrorInvalidValue;
    const int64_t copies = n / n1;
    const bool sliced = !part_of_dev && n % n1 == 0 && copies <= 65535;     // copies are a grid dimension of rg_mark_slices
    // slice of the built-in rule: ceil(p n1 / P) .. ceil((p + 1) n1 / P), exact in 64 bits (n1, P < 2^31)
    const uint32_t lo = (uint32_t)(((int64_t)p * n1 + P - 1) / P), hi = (uint32_t)(((int64_t)(p + 1) * n1 + P - 1) / P);
    const int64_t words = ((n + 31) / 32 + kRgBlockWords - 1) / kRgBlockWords * kRgBlockWords, blocks = words / kRgBlockWords;
    const unsigned sets = sliced ? 1 : 2;

    Scratch scratch;
    int32_t *cnt = nullptr, *len = nullptr, *long_list = nullptr;
    uint32_t *sets_dev = nullptr;                                           // totals and the flags of B_p (cleared together), the bits
    unsigned long long *sums = nullptr;
    constexpr int64_t kTotalWords = (2 * (kRgEnd + 1) + 3) / 4 * 4;
    if (!scratch.get(&sets_dev, (size_t)(kTotalWords + (8 + 2 * sets) * words)) || !scratch.get(&cnt, (size_t)(sets * blocks)))
        return kErrOutOfDeviceMemory;
    unsigned long long *const totals = (unsigned long long *)sets_dev;
    int32_t *const flag = (int32_t *)(totals + kRgEnd), *const n_long = flag + 1;
    RgGraph g{dp.rowptr, dp.col, dp.graph_weight_mode == kExplicit ? dp.val : nullptr, n, n1, part_of_dev, p, lo, hi, sliced,
              regrow != 0, symmetric, (uint8_t *)(sets_dev + kTotalWords), sets_dev + kTotalWords + 8 * words, nullptr, nullptr, nullptr, 0};
    g.halo_before = g.halo + words;
    if (!sliced) {
        g.own = g.halo_before + words;
        g.own_before = g.own + words;
    }

    DevicePart part;
    hipError_t e = hipSuccess;
    auto done = [&](int code) {
        (void)hipStreamSynchronize(st);                          // scratch and partial results are freed next
        free_device_part(part);
        return code;
    };

    const int64_t clear = kTotalWords + 8 * words;
    rg_clear<<<dim3(rg_grid(clear / 4, kBlock)), dim3(kBlock), 0, st>>>((uint4 *)sets_dev, clear / 4);
    if (!sliced) rg_own_bits<<<dim3(rg_grid(words * 32, kBlock)), dim3(kBlock), 0, st>>>(g, P, flag);
    if (regrow && sliced) {
        int64_t per_copy = dp.nnz / copies / P / (kRgMark * kBlock) + 1;        // workgroups that walk a copy's entries once, about
        if (per_copy > 2048) per_copy = 2048;
        rg_mark_slices<<<dim3((unsigned)per_copy, (unsigned)copies), dim3(kBlock), 0, st>>>(g, totals);
    } else if (regrow) {
        rg_mark<<<dim3(rg_grid(n, kBlock)), dim3(kBlock), 0, st>>>(g, totals);
    }
    rg_count<<<dim3((unsigned)blocks, sets), dim3(kBlock), 0, st>>>(g, cnt, totals);
    if ((e = hipGetLastError()) != hipSuccess) return done((int)e);
    int64_t h_total[kRgEnd + 1] = {};
    if ((e = hipMemcpyAsync(h_total, totals, sizeof h_total, hipMemcpyDeviceToHost, st)) != hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
        return done((int)e);
    if ((int32_t)h_total[kRgEnd]) return done(kErrBadPartId);
    part.n_owned = sliced ? copies * (int64_t)(hi - lo) : rg_sum_slots(h_total + kRgOwned);
    part.n_halo = rg_sum_slots(h_total + kRgHalo);
    const int64_t n_loc = part.n_owned + part.n_halo;
    if (part.n_owned < 0 || part.n_halo < 0 || n_loc > n) return done((int)hipErrorUnknown);
    g.n_owned = part.n_owned;

    if (dev_alloc((void **)&part.global_id, (size_t)(n_loc ? n_loc : 1) * sizeof(int64_t)) != 0 ||
        dev_alloc((void **)&part.rowptr, (size_t)(n_loc + 1) * sizeof(int64_t)) != 0)
        return done(kErrOutOfDeviceMemory);
    const int64_t n_sums = (n_loc + kRgLenBlock - 1) / kRgLenBlock;
    if (!scratch.get(&len, (size_t)n_loc) || !scratch.get(&sums, (size_t)n_sums) || !scratch.get(&long_list, (size_t)n_loc))
        return done(kErrOutOfDeviceMemory);

    if (n_loc) {
        const bool scanned = blocks > kRgFusedCounts;
        if (scanned) rg_scan_sums<<<dim3(sets), dim3(kRgLenBlock), 0, st>>>(cnt, blocks);
        rg_place<<<dim3((unsigned)blocks, sets), dim3(kBlock), 0, st>>>(g, cnt, scanned, part.global_id, sums, n_sums);
        rg_row_len<<<dim3(rg_grid(n_loc, kBlock)), dim3(kBlock), 0, st>>>(g, part.global_id, n_loc, len, sums, totals, long_list,
                                                                          n_long);
        if (!rg_long_by_search(g))
            rg_row_len_long<<<dim3(kRgLongBlocks), dim3(kBlock), 0, st>>>(g, part.global_id, len, sums, totals,
                                                                          long_list, n_long);
    } else {
        rg_fill_i32<<<dim3(1), dim3(kBlock), 0, st>>>((int32_t *)part.rowptr, 2, 0);
    }
    if ((e = hipGetLastError()) != hipSuccess) return done((int)e);
    if ((e = hipMemcpyAsync(h_total + kRgCross, totals + kRgCross, 2 * kRgSlots * sizeof(int64_t), hipMemcpyDeviceToHost, st)) != hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
        return done((int)e);
    part.n_crossing = rg_sum_slots(h_total + kRgCross);
    part.nnz = rg_sum_slots(h_total + kRgNnz);
    if (part.nnz < 0 || part.nnz > dp.nnz) return done((int)hipErrorUnknown);

    if (dev_alloc((void **)&part.col, (size_t)(part.nnz ? part.nnz : 1) * sizeof(int32_t)) != 0)
        return done(kErrOutOfDeviceMemory);
    if (g.val && dev_alloc((void **)&part.val, (size_t)(part.nnz ? part.nnz : 1) * sizeof(float)) != 0)
        return done(kErrOutOfDeviceMemory);
    if (n_loc) {
        const bool scanned = n_sums > kRgFusedSums;
        if (scanned) rg_scan_sums<<<dim3(1), dim3(kRgLenBlock), 0, st>>>(sums, n_sums);
        rg_len_write<<<dim3((unsigned)n_sums), dim3(kBlock), 0, st>>>(len, n_loc, sums, scanned, part.rowptr);
        // no more workgroups for long rows than the graph has entries for
        const int64_t most = dp.nnz / (kRgShort + 1) / kWavesPerBlock + 1;
        const int32_t long_blocks = (int32_t)(most < kRgLongBlocks ? most : kRgLongBlocks);
        rg_fill<<<dim3(long_blocks + rg_grid(n_loc, kBlock)), dim3(kBlock), 0, st>>>(g, part.global_id, n_loc, part.rowptr, part.col,
                                                                                   part.val, long_list, n_long, long_blocks);
    }
    if ((e = hipGetLastError()) != hipSuccess) return done((int)e);
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return done((int)e);   // the scratch is freed on return
    *out = part;
    return 0;
}

// Milliseconds per call of fn(ctx), which enqueues work on the stream: one untimed call, then `reps` calls between two
// events.  Synchronises the stream.  0, or the first HIP error (fn returns 0 or an error of its own).
int device_time_ms(void *stream, int reps, int (*fn)(void *ctx), void *ctx, float *ms)
{
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t a = nullptr, b = nullptr;
    hipError_t e = hipEventCreate(&a);
    if (e == hipSuccess) e = hipEventCreate(&b);
    int err = (int)e;
    if (!err) err = fn(ctx);
    if (!err) err = (int)hipEventRecord(a, st);
    for (int r = 0; r < reps && !err; ++r) err = fn(ctx);
    if (!err) err = (int)hipEventRecord(b, st);
    if (!err) err = (int)hipEventSynchronize(b);
    float t = 0.f;
    if (!err) err = (int)hipEventElapsedTime(&t, a, b);
    if (a) (void)hipEventDestroy(a);
    if (b) (void)hipEventDestroy(b);
    if (err) (void)hipStreamSynchronize(st);
    *ms = reps > 0 ? t / (float)reps : 0.f;
    return err;
}

int device_download(void *dst_host, const void *src_dev, size_t bytes, void *stream)
{
    if (!bytes) return 0;
    hipStream_t st = (hipStream_t)stream;
    hipError_t err = hipMemcpyAsync(dst_host, src_dev, bytes, hipMemcpyDeviceToHost, st);
    hipError_t err2 = hipStreamSynchronize(st);
    return (int)(err != hipSuccess ? err : err2);
}

int device_wait(void *stream) { return (int)hipStreamSynchronize((hipStream_t)stream); }

}  // namespace groot
