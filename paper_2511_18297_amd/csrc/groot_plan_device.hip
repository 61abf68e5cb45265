// Device-side degree plan for gfx950: the LD kernel's "step B" of the paper on the GPU -- every row's
// degree from the row pointer, its class, and a stable counting sort of the low-degree rows by degree
// (linear time, as the paper notes for count sort).  All integer work; the lists are bit-identical to
// the host plan's.
//
// Launches over blocks of 4096 consecutive rows (16 wavefronts of 256 consecutive rows, four per lane, which are all loaded
// before any is looked at: with 16 one after the other for each of 4 wavefronts, plan_scatter took 18 us on 10 thousand rows and
// 25 on a million, now 6 and 11):
//   plan_count    per block: number of low-degree rows of every degree < T, of LD rows, of HD rows
//   plan_scan     per column of that table: exclusive prefix over the blocks (+ totals); only for tables of more than
//                 kPlanFusedTable numbers, smaller ones are added up by every block of plan_scatter, which costs less than the
//                 launch (4 us)
//   plan_scatter  the degree offsets are the exclusive prefix of the per-degree totals; per block again: every row gets its
//                 position = column start + rows of the same column in earlier blocks + in earlier wavefronts of the block +
//                 earlier in its own wavefront (ballot ranks in lane order), which is exactly the stable order
#include <mutex>

#include "groot_device.h"

namespace groot {

constexpr int kPlanRowsPerLane = 4;
constexpr int kPlanRowsPerWave = kPlanRowsPerLane * kWave;
constexpr int kPlanBlock = 1024, kPlanWaves = kPlanBlock / kWave;
constexpr int kPlanRowsPerBlock = kPlanRowsPerWave * kPlanWaves;       // 4096
constexpr int64_t kPlanFusedTable = 16384;
constexpr int kPlanMaxCols = kPlanDeviceMaxThreshold + 2;              // degrees 0..T-1, LD count, HD count
static_assert(kErrOutOfDeviceMemory == (int)hipErrorOutOfMemory, "error code shared with the host side");

// stored lengths of a lane's rows first, first + 64, ... (-1: past the end); a row pointer that runs backwards counts as an
// empty row
__device__ __forceinline__ void plan_degrees(const int64_t *__restrict__ rowptr, int64_t n, int64_t first,
                                             int64_t (&d)[kPlanRowsPerLane])
{
    int64_t b[kPlanRowsPerLane], e[kPlanRowsPerLane];
#pragma unroll
    for (int k = 0; k < kPlanRowsPerLane; ++k) {
        const int64_t i = first + (int64_t)k * kWave;
        b[k] = rowptr[i < n ? i : n];
        e[k] = rowptr[i < n ? i + 1 : n];
    }
#pragma unroll
    for (int k = 0; k < kPlanRowsPerLane; ++k) {
        const int64_t len = e[k] - b[k];
        d[k] = first + (int64_t)k * kWave < n ? (len < 0 ? 0 : len) : -1;
    }
}

// f(degree, lanes) for every degree that low-degree rows of the wavefront have, once
template <class F>
__device__ __forceinline__ void plan_each_degree(int64_t d, bool ld, F f)
{
    uint64_t remaining = __ballot(ld);
    while (remaining) {
        const int dl = (int)__shfl((int)d, __ffsll((unsigned long long)remaining) - 1);
        const uint64_t peers = __ballot(ld && (int)d == dl);
        f(dl, peers);
        remaining &= ~peers;
    }
}

// hist[block * cols + c]
__global__ __launch_bounds__(kPlanBlock) void plan_count(const int64_t *__restrict__ rowptr, int64_t n, int32_t T,
                                                         int32_t cols, int32_t *__restrict__ hist,
                                                         uint8_t *__restrict__ row_class)
{
    __shared__ int32_t s_cnt[kPlanMaxCols];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    for (int c = threadIdx.x; c < cols; c += kPlanBlock) s_cnt[c] = 0;
    const int64_t first = (int64_t)blockIdx.x * kPlanRowsPerBlock + wave * kPlanRowsPerWave + lane;
    int64_t d[kPlanRowsPerLane];
    plan_degrees(rowptr, n, first, d);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPlanRowsPerLane; ++k) {
        const bool hd = d[k] >= T, ld = d[k] >= 0 && !hd;
        if (row_class && d[k] >= 0) row_class[first + (int64_t)k * kWave] = hd ? 1 : 0;
        const uint64_t m_hd = __ballot(hd), m_ld = __ballot(ld);
        if (lane == 0) {
            if (m_ld) atomicAdd(&s_cnt[T], __popcll(m_ld));
            if (m_hd) atomicAdd(&s_cnt[T + 1], __popcll(m_hd));
        }
        plan_each_degree(d[k], ld, [&](int dl, uint64_t peers) {
            if (lane == 0) atomicAdd(&s_cnt[dl], __popcll(peers));
        });
    }
    __syncthreads();
    for (int c = threadIdx.x; c < cols; c += kPlanBlock) hist[(int64_t)blockIdx.x * cols + c] = s_cnt[c];
}

// exclusive prefix of x over the workgroup's Waves wavefronts; every thread calls
template <int Waves>
__device__ __forceinline__ int64_t plan_block_prefix(int64_t x, int64_t *total)
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
    int64_t run = incl - x, all = 0;
    for (int w = 0; w < Waves; ++w) {
        if (w < wave) run += s_w[w];
        all += s_w[w];
    }
    *total = all;
    return run;
}

// One workgroup per column: hist[., c] -> exclusive prefix over the blocks, total[c] = column sum.
__global__ __launch_bounds__(kBlock) void plan_scan(int32_t *__restrict__ hist, int64_t n_blocks, int32_t cols,
                                                    int64_t *__restrict__ total)
{
    const int c = blockIdx.x;
    const int64_t seg = (n_blocks + kBlock - 1) / kBlock;
    const int64_t b0 = (int64_t)threadIdx.x * seg < n_blocks ? (int64_t)threadIdx.x * seg : n_blocks;
    const int64_t b1 = b0 + seg < n_blocks ? b0 + seg : n_blocks;
    int64_t sum = 0, all;
    for (int64_t b = b0; b < b1; ++b) sum += hist[b * cols + c];
    int64_t run = plan_block_prefix<kWavesPerBlock>(sum, &all);
    if (threadIdx.x == 0) total[c] = all;
    for (int64_t b = b0; b < b1; ++b) {
        const int32_t v = hist[b * cols + c];
        hist[b * cols + c] = (int32_t)run;
        run += v;
    }
}

// table: plan_count's (n_blocks rows; total NULL), or plan_scan's prefixes with the columns' totals.
// deg_offsets[d] = number of LD rows of degree < d (d = 0..T); counts = {n_hd, n_ld}.  The lists: ld_rows may be NULL; by_degree
// receives the rows of at least `from` entries only, so its first is the first of those.
__global__ __launch_bounds__(kPlanBlock) void plan_scatter(const int64_t *__restrict__ rowptr, int64_t n, int32_t T,
                                                           int32_t cols, const int32_t *__restrict__ table, int64_t n_blocks,
                                                           const int64_t *__restrict__ total,
                                                           int32_t *__restrict__ hd_rows, int32_t *__restrict__ ld_rows,
                                                           int32_t *__restrict__ by_degree, int32_t from,
                                                           int64_t *__restrict__ deg_offsets, int64_t *__restrict__ counts)
{
    __shared__ int32_t s_pos[kPlanWaves][kPlanMaxCols];
    __shared__ int32_t s_before[kPlanMaxCols], s_total[kPlanMaxCols];
    __shared__ int32_t s_from;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const uint64_t lt_mask = lane ? (~0ULL >> (64 - lane)) : 0ULL;
    const int64_t first = (int64_t)blockIdx.x * kPlanRowsPerBlock + wave * kPlanRowsPerWave + lane;

    int64_t d[kPlanRowsPerLane];
    plan_degrees(rowptr, n, first, d);
    for (int c = lane; c < cols; c += kWave) s_pos[wave][c] = 0;
    for (int c = threadIdx.x; c < cols; c += kPlanBlock) {
        s_before[c] = total && n_blocks ? table[(int64_t)blockIdx.x * cols + c] : 0;
        s_total[c] = total ? (int32_t)total[c] : 0;
    }
    __syncthreads();
    if (!total)
        for (uint32_t i = threadIdx.x; i < (uint32_t)(n_blocks * cols); i += kPlanBlock) {
            const int32_t v = table[i];
            const uint32_t b = i / (uint32_t)cols, c = i - b * (uint32_t)cols;
            if (v) atomicAdd(&s_total[c], v);
            if (v && b < blockIdx.x) atomicAdd(&s_before[c], v);
        }
    // per-wavefront counts of every column
#pragma unroll
    for (int k = 0; k < kPlanRowsPerLane; ++k) {
        const bool hd = d[k] >= T, ld = d[k] >= 0 && !hd;
        const uint64_t m_hd = __ballot(hd), m_ld = __ballot(ld);
        if (lane == 0) { s_pos[wave][T] += __popcll(m_ld); s_pos[wave][T + 1] += __popcll(m_hd); }
        plan_each_degree(d[k], ld && d[k] >= from, [&](int dl, uint64_t peers) {
            if (lane == 0) s_pos[wave][dl] += __popcll(peers);
        });
    }
    __syncthreads();
    // start of every degree
    static_assert(kPlanBlock >= kPlanDeviceMaxThreshold, "a thread per degree");
    int64_t n_ld;
    const int64_t start = plan_block_prefix<kPlanWaves>((int)threadIdx.x < T ? s_total[threadIdx.x] : 0, &n_ld);
    if ((int)threadIdx.x == from) s_from = (int32_t)start;
    if (blockIdx.x == 0) {
        if ((int)threadIdx.x < T) deg_offsets[threadIdx.x] = start;
        if (threadIdx.x == 0) {
            deg_offsets[T] = n_ld;
            counts[0] = s_total[T + 1];
            counts[1] = n_ld;
        }
    }
    // start position of every (wavefront, column): earlier blocks + earlier wavefronts (+ the degree's offset)
    __syncthreads();
    for (int c = threadIdx.x; c < cols; c += kPlanBlock) {
        int32_t run = s_before[c] + (c < T ? (int32_t)start - s_from : 0);       // c < T: c is the thread
        for (int w = 0; w < kPlanWaves; ++w) {
            const int32_t v = s_pos[w][c];
            s_pos[w][c] = run;
            run += v;
        }
    }
    __syncthreads();
    // rows in order: 64 at a time, rank among equal columns by ballot in lane order
#pragma unroll
    for (int k = 0; k < kPlanRowsPerLane; ++k) {
        const int32_t i = (int32_t)(first + (int64_t)k * kWave);
        const bool hd = d[k] >= T, ld = d[k] >= 0 && !hd;
        const uint64_t m_hd = __ballot(hd), m_ld = __ballot(ld);
        if (hd) hd_rows[s_pos[wave][T + 1] + __popcll(m_hd & lt_mask)] = i;
        if (ld && ld_rows) ld_rows[s_pos[wave][T] + __popcll(m_ld & lt_mask)] = i;
        wave_sync();
        if (lane == 0) { s_pos[wave][T + 1] += __popcll(m_hd); s_pos[wave][T] += __popcll(m_ld); }
        plan_each_degree(d[k], ld && d[k] >= from, [&](int dl, uint64_t peers) {
            if ((peers >> lane) & 1) by_degree[s_pos[wave][dl] + __popcll(peers & lt_mask)] = i;
            wave_sync();
            if (lane == 0) s_pos[wave][dl] += __popcll(peers);
            wave_sync();
        });
        wave_sync();
    }
}

namespace {

// the launches on the caller's stream, with the block table and the column totals where the caller says
int plan_launches(const int64_t *rowptr_dev, int64_t n, int32_t T, int32_t cols, int64_t n_blocks, int32_t *hist,
                  int64_t *total, uint8_t *row_class, int32_t *hd_rows, int32_t *ld_rows, int32_t *by_degree, int32_t from,
                  int64_t *deg_offsets, int64_t *counts, hipStream_t st)
{
    const bool fused = n_blocks * cols <= kPlanFusedTable;
    if (n_blocks)
        plan_count<<<dim3((unsigned)n_blocks), dim3(kPlanBlock), 0, st>>>(rowptr_dev, n, T, cols, hist, row_class);
    if (!fused) plan_scan<<<dim3((unsigned)cols), dim3(kBlock), 0, st>>>(hist, n_blocks, cols, total);
    plan_scatter<<<dim3((unsigned)(n_blocks ? n_blocks : 1)), dim3(kPlanBlock), 0, st>>>(     // an empty graph: all totals 0
        rowptr_dev, n, T, cols, hist, n_blocks, fused ? nullptr : total, hd_rows, ld_rows, by_degree, from, deg_offsets, counts);
    return (int)hipGetLastError();
}

// Scratch of the entry point that may not allocate: the column totals (int64 [cols]) at offset 0 and the
// block table (int32 [n_blocks][cols]) behind them.  One copy per GPU, held until the process ends; every
// call on a GPU uses the same bytes.  In host code `scratch` is only a handle for hipGetSymbolAddress: the
// device address it yields is what kernels, copies and clears are given.
static __device__ __align__(256) unsigned char scratch[kPlanStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char *g_scratch_ptr[kMaxDevices] = {};

// device address of the current device's copy of `scratch` (looked up once per device)
int static_scratch(unsigned char **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        if (!p) return (int)hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = (unsigned char *)p;
    }
    *out = g_scratch_ptr[dev];
    return 0;
}

constexpr size_t plan_totals_bytes(int32_t cols) { return ((size_t)cols * sizeof(int64_t) + 255) / 256 * 256; }

}  // namespace

int launch_plan_device(const int64_t *rowptr_dev, int64_t n, int32_t T, uint8_t *row_class, int32_t *hd_rows,
                       int32_t *ld_rows, int32_t *by_degree, int64_t *deg_offsets, int64_t *counts, void *stream, bool wait,
                       int32_t from)
{
    hipStream_t st = (hipStream_t)stream;
    const int32_t cols = T + 2;
    const int64_t n_blocks = (n + kPlanRowsPerBlock - 1) / kPlanRowsPerBlock;
    if (T < 1 || cols > kPlanMaxCols || n < 0 || n > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    int32_t *hist = nullptr;
    int64_t *total = nullptr;
    if (dev_alloc((void **)&hist, (size_t)(n_blocks ? n_blocks : 1) * cols * sizeof(int32_t))) return (int)hipErrorOutOfMemory;
    if (dev_alloc((void **)&total, (size_t)cols * sizeof(int64_t))) { dev_free(hist); return (int)hipErrorOutOfMemory; }
    const int err = plan_launches(rowptr_dev, n, T, cols, n_blocks, hist, total, row_class, hd_rows, ld_rows, by_degree, from,
                                  deg_offsets, counts, st);
    const hipError_t e2 = wait ? hipStreamSynchronize(st) : hipSuccess;
    dev_free(hist);                                          // may still be in use (see dev_free)
    dev_free(total);
    return err ? err : (int)e2;
}

size_t plan_static_scratch_needed(int64_t n, int32_t T)
{
    const int64_t n_blocks = (n + kPlanRowsPerBlock - 1) / kPlanRowsPerBlock;
    return plan_totals_bytes(T + 2) + (size_t)n_blocks * (size_t)(T + 2) * sizeof(int32_t);
}

int launch_plan_device_static(const int64_t *rowptr_dev, int64_t n, int32_t T, uint8_t *row_class, int32_t *hd_rows,
                              int32_t *ld_rows, int32_t *by_degree, int64_t *deg_offsets, int64_t *counts,
                              void *stream)
{
    const int32_t cols = T + 2;
    const int64_t n_blocks = (n + kPlanRowsPerBlock - 1) / kPlanRowsPerBlock;
    if (T < 1 || cols > kPlanMaxCols || n < 0 || n > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    if (plan_static_scratch_needed(n, T) > kPlanStaticScratchBytes) return (int)hipErrorInvalidValue;
    unsigned char *base = nullptr;
    const int err = static_scratch(&base);
    if (err) return err;
    // Nothing in the scratch has to start at zero: plan_count writes every column of every block's table
    // entry, plan_scan (where it runs) every total, before anything reads them.
    int64_t *total = (int64_t *)base;
    int32_t *hist = (int32_t *)(base + plan_totals_bytes(cols));
    return plan_launches(rowptr_dev, n, T, cols, n_blocks, hist, total, row_class, hd_rows, ld_rows, by_degree, 0,
                         deg_offsets, counts, (hipStream_t)stream);
}

}  // namespace groot
