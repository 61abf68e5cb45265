// Schedule of the high-degree rows built on the device (gfx950), for plans whose matrix lives there.
// Section "Kernel Design - GROOT-GPU": the non-zeros of a high-degree row are partitioned statically; here a
// row of d entries is cut into ceil(d / hd_chunk) balanced pieces, a row with more than one piece gets a run of
// partial-sum slots, and the pieces run in the order of their first column (pieces of different rows that read
// the same stretch of feature rows then run close together).  Integer work; the arrays are bit-identical to what
// the host builds from the same rows (groot_spmm_plan): pieces in row order, then a stable sort by first column.
#include <algorithm>
#include <cstring>

#include <hip/hip_runtime.h>
#include <rocprim/device/device_radix_sort.hpp>

#include "groot_device.h"

namespace groot {

namespace {


__device__ __forceinline__ int64_t hs_pieces(int64_t d, int64_t chunk)
{
    const int64_t p = (d + chunk - 1) / chunk;
    return p < 1 ? 1 : p;
}

// Before every high-degree row: pieces, partial-sum slots (none for a row of a single piece) and split rows (one workgroup walks
// the rows in runs of four per thread; one per thread, about 4,200 rows took 14.7 us, now 7.4); the totals and the number of
// entries of all high-degree rows.
constexpr int kScanRows = 4;
__global__ __launch_bounds__(1024) void hs_scan(const int64_t *__restrict__ rowptr, const int32_t *__restrict__ hd_rows,
                                                const int64_t *__restrict__ n_hd_dev, int64_t chunk, int64_t *__restrict__ pieces,
                                                int64_t *__restrict__ slots, int64_t *__restrict__ split,
                                                HdTotals *__restrict__ totals)
{
    const int64_t n_hd = *n_hd_dev;
    __shared__ int64_t s_part[3][16];                    // per wavefront
    __shared__ int64_t s_carry[4];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    if (threadIdx.x < 4) s_carry[threadIdx.x] = 0;
    __syncthreads();
    int64_t nnz = 0;
    for (int64_t base = 0; base < n_hd; base += 1024 * kScanRows) {
        const int64_t k = base + threadIdx.x * kScanRows;
        int64_t row[kScanRows], d[kScanRows], p[kScanRows];
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) row[i] = hd_rows[k + i < n_hd ? k + i : n_hd - 1];
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) d[i] = rowptr[row[i] + 1] - rowptr[row[i]];
        int64_t v[3] = {0, 0, 0};
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) {
            const bool here = k + i < n_hd;
            p[i] = here ? hs_pieces(d[i] < 0 ? 0 : d[i], chunk) : 0;
            nnz += here ? d[i] : 0;
            v[0] += p[i];
            v[1] += p[i] > 1 ? p[i] : 0;
            v[2] += p[i] > 1 ? 1 : 0;
        }
        int64_t incl[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {                    // inclusive scan inside the wavefront
            int64_t x = v[a];
#pragma unroll
            for (int off = 1; off < kWave; off *= 2) {
                const int64_t y = __shfl_up(x, off);
                if (lane >= off) x += y;
            }
            incl[a] = x;
            if (lane == kWave - 1) s_part[a][wave] = x;
        }
        __syncthreads();
        int64_t before[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            int64_t b = s_carry[a];
            for (int w2 = 0; w2 < wave; ++w2) b += s_part[a][w2];
            before[a] = b;
        }
        int64_t run[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) run[a] = before[a] + incl[a] - v[a];
#pragma unroll
        for (int i = 0; i < kScanRows; ++i) {
            if (k + i < n_hd) {
                pieces[k + i] = run[0];
                slots[k + i] = run[1];
                split[k + i] = run[2];
            }
            run[0] += p[i];
            run[1] += p[i] > 1 ? p[i] : 0;
            run[2] += p[i] > 1 ? 1 : 0;
        }
        __syncthreads();
        if (threadIdx.x == 1023) {
#pragma unroll
            for (int a = 0; a < 3; ++a) s_carry[a] = before[a] + incl[a];
        }
        __syncthreads();
    }
    // entries of the high-degree rows: per-thread sums -> one number (integer, order-free)
#pragma unroll
    for (int off = kWave / 2; off > 0; off /= 2) nnz += __shfl_down(nnz, off);
    if (lane == 0) s_part[0][wave] = nnz;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w2 = 0; w2 < 16; ++w2) t += s_part[0][w2];
        totals->n_chunks = (unsigned long long)s_carry[0];
        totals->n_slots = (unsigned long long)s_carry[1];
        totals->n_split = (unsigned long long)s_carry[2];
        totals->nnz_hd = (unsigned long long)t;
    }
}

// One thread per high-degree row writes its pieces (in row order), its split-row record, the sort keys and the
// identity permutation (order may be NULL); the *_rank arrays name the row by its place k in hd_rows instead of its id.
__global__ __launch_bounds__(kBlock) void hs_fill(const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                                  const int32_t *__restrict__ hd_rows, int64_t n_hd, int64_t chunk,
                                                  const int64_t *__restrict__ piece_off, const int64_t *__restrict__ slot_off,
                                                  const int64_t *__restrict__ split_off, HdChunk *__restrict__ chunks,
                                                  HdChunk *__restrict__ chunks_rank, int32_t *__restrict__ keys,
                                                  int32_t *__restrict__ order, HdSplitRow *__restrict__ split_rows,
                                                  HdSplitRow *__restrict__ split_rows_rank)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n_hd) return;
    const int32_t row = hd_rows[k];
    const int64_t b = rowptr[row];
    int64_t d = rowptr[row + 1] - b;
    if (d < 0) d = 0;
    const int64_t pieces = hs_pieces(d, chunk), per = (d + pieces - 1) / pieces;
    const int64_t o = piece_off[k], sl = slot_off[k];
    if (pieces > 1) {
        split_rows[split_off[k]] = HdSplitRow{row, (int32_t)sl, (int32_t)pieces, 0};
        split_rows_rank[split_off[k]] = HdSplitRow{(int32_t)k, (int32_t)sl, (int32_t)pieces, 0};
    }
    for (int64_t c = 0; c < pieces; ++c) {
        const int64_t lo = c * per, hi = d < lo + per ? d : lo + per;
        HdChunk ch;
        ch.begin = b + lo;
        ch.len = (int32_t)(hi > lo ? hi - lo : 0);
        ch.row = row;
        ch.slot = pieces > 1 ? (int32_t)(sl + c) : -1;
        ch.row_nnz = (int32_t)(d < 0x7fffffffLL ? d : 0x7fffffffLL);
        chunks[o + c] = ch;
        ch.row = (int32_t)k;
        chunks_rank[o + c] = ch;
        keys[o + c] = ch.len > 0 ? col[ch.begin] : 0x7fffffff;
        if (order) order[o + c] = (int32_t)(o + c);
    }
}

__global__ __launch_bounds__(kBlock) void hs_permute(const HdChunk *__restrict__ in, const HdChunk *__restrict__ in_rank,
                                                     const int32_t *__restrict__ order, int64_t n,
                                                     HdChunk *__restrict__ out, HdChunk *__restrict__ out_rank)
{
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c >= n) return;
    out[c] = in[order[c]];
    out_rank[c] = in_rank[order[c]];
}

// hs_permute for few pieces, which finds their order as well: a piece's place is the number of pieces with a smaller key, or
// the same key and before it.  A wavefront counts for kRankPieces pieces at a time, 64 keys per comparison, kRankAhead loads in
// flight.
constexpr int kRankPieces = 4, kRankAhead = 8;
__global__ __launch_bounds__(kBlock) void hs_rank(const HdChunk *__restrict__ in, const HdChunk *__restrict__ in_rank,
                                                  const int32_t *__restrict__ keys, int32_t n,
                                                  HdChunk *__restrict__ out, HdChunk *__restrict__ out_rank)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int32_t first = (blockIdx.x * kWavesPerBlock + wave) * kRankPieces;
    if (first >= n) return;
    int32_t mine[kRankPieces], place[kRankPieces];
#pragma unroll
    for (int i = 0; i < kRankPieces; ++i) {
        mine[i] = keys[first + i < n ? first + i : n - 1];
        place[i] = 0;
    }
    for (int32_t j0 = 0; j0 < n; j0 += kRankAhead * kWave) {
        int32_t key[kRankAhead];
#pragma unroll
        for (int a = 0; a < kRankAhead; ++a) key[a] = keys[j0 + a * kWave + lane < n ? j0 + a * kWave + lane : n - 1];
#pragma unroll
        for (int a = 0; a < kRankAhead; ++a) {
            const int32_t j = j0 + a * kWave + lane;
#pragma unroll
            for (int i = 0; i < kRankPieces; ++i)
                place[i] += __popcll(__ballot(j < n && (key[a] < mine[i] || (key[a] == mine[i] && j < first + i))));
        }
    }
#pragma unroll
    for (int i = 0; i < kRankPieces; ++i)
        if (lane == i && first + i < n) {
            out[place[i]] = in[first + i];
            out_rank[place[i]] = in_rank[first + i];
        }
}

struct Tmp {                                             // device memory freed on scope exit
    void *p[12] = {};
    int used = 0;
    ~Tmp() { for (int i = 0; i < used; ++i) dev_free(p[i]); }
    template <class T>
    bool get(T **out, size_t count)
    {
        void *q = nullptr;
        if (used >= 12 || dev_alloc(&q, (count ? count : 1) * sizeof(T)) != 0) return false;
        p[used++] = q;
        *out = (T *)q;
        return true;
    }
};

__global__ __launch_bounds__(kBlock) void plan_finish(float *__restrict__ zero_row, int32_t *__restrict__ mid, const int32_t *__restrict__ mid_src,
                                                      int64_t n_mid, int32_t *__restrict__ hd, const int32_t *__restrict__ hd_src, int64_t n_hd)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n_mid || i < n_hd || i < kZeroRowFloats + kTrashFloats;
         i += (int64_t)gridDim.x * kBlock) {
        if (i < kZeroRowFloats + kTrashFloats) zero_row[i] = 0.f;
        if (i < n_mid) mid[i] = mid_src[i];
        if (i < n_hd) hd[i] = hd_src[i];
    }
}

}  // namespace

int launch_plan_finish(float *zero_row, int32_t *mid, const int32_t *mid_src, int64_t n_mid, int32_t *hd, const int32_t *hd_src,
                       int64_t n_hd, void *stream)
{
    const int64_t most = std::max<int64_t>({n_mid, n_hd, kZeroRowFloats + kTrashFloats}), grid = (most + kBlock - 1) / kBlock;
    plan_finish<<<dim3((unsigned)std::min<int64_t>(grid, 4096)), dim3(kBlock), 0, (hipStream_t)stream>>>(zero_row, mid, mid_src, n_mid, hd,
                                                                                                          hd_src, n_hd);
    return (int)hipGetLastError();
}

void free_device_hd_schedule(DeviceHdSchedule &s)
{
    dev_free(s.chunks); dev_free(s.chunks_rank); dev_free(s.split_rows); dev_free(s.split_rows_rank);
    s = DeviceHdSchedule{};
}

void free_hd_counts(HdCounts &c)
{
    dev_free(c.pieces); dev_free(c.slots); dev_free(c.split);
    c = HdCounts{};
}

// Enqueues the counting of pieces, slots and split rows.  n_hd_dev: number of high-degree rows, on the device, at most `most`;
// totals_dev receives the sizes.  The counts belong to the caller.
int launch_hd_schedule_count(const int64_t *rowptr_dev, const int32_t *hd_rows_dev, const int64_t *n_hd_dev, int64_t most,
                             int32_t hd_chunk, void *stream, HdTotals *totals_dev, HdCounts *out)
{
    hipStream_t st = (hipStream_t)stream;
    HdCounts c;
    const size_t bytes = (size_t)(most > 0 ? most : 1) * sizeof(int64_t);
    if (dev_alloc((void **)&c.pieces, bytes) || dev_alloc((void **)&c.slots, bytes) || dev_alloc((void **)&c.split, bytes)) {
        free_hd_counts(c);
        return kErrOutOfDeviceMemory;
    }
    hs_scan<<<dim3(1), dim3(1024), 0, st>>>(rowptr_dev, hd_rows_dev, n_hd_dev, hd_chunk < 64 ? 64 : hd_chunk, c.pieces, c.slots, c.split,
                                            totals_dev);
    *out = c;
    return (int)hipGetLastError();
}

// hd_rows_dev: the n_hd high-degree rows, ascending; counts and h from launch_hd_schedule_count, h read back since.  The schedule is
// complete when the stream has reached the end of what is enqueued here.  kErrOutOfDeviceMemory when an allocation
// fails, kErrTooManyPieces when the slots do not fit 31 bits.
int launch_hd_schedule_device(const int64_t *rowptr_dev, const int32_t *col_dev, const int32_t *hd_rows_dev, int64_t n_hd,
                              int32_t hd_chunk, const HdCounts &counts, const HdTotals &h, void *stream, DeviceHdSchedule *out)
{
    *out = DeviceHdSchedule{};
    if (n_hd <= 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    const int64_t chunk = hd_chunk < 64 ? 64 : hd_chunk;
    Tmp tmp;
    int64_t *const pieces = counts.pieces, *const slots = counts.slots, *const split = counts.split;
    const unsigned grid_rows = (unsigned)((n_hd + kBlock - 1) / kBlock);
    hipError_t e = hipSuccess;
    if (h.n_slots > 0x3fffffffULL || h.n_chunks > 0x7fffffffULL) return kErrTooManyPieces;
    const int64_t n_chunks = (int64_t)h.n_chunks, n_split = (int64_t)h.n_split;

    HdChunk *raw = nullptr, *raw_rank = nullptr;
    int32_t *keys = nullptr, *keys_sorted = nullptr, *order = nullptr, *order_sorted = nullptr;
    DeviceHdSchedule s;
    // Up to 5,120 pieces their order is counted out, n^2 / 64 comparisons in one launch (100 pieces 3.4 us, about 4,200 13.5,
    // 8,200 38), above it is sorted, three or four launches and hs_permute (100 pieces 11.5 us, 4,200 23)
    const bool count_out = n_chunks <= 5120;
    if (!tmp.get(&raw, (size_t)n_chunks) || !tmp.get(&raw_rank, (size_t)n_chunks) || !tmp.get(&keys, (size_t)n_chunks) ||
        (!count_out && (!tmp.get(&keys_sorted, (size_t)n_chunks) || !tmp.get(&order, (size_t)n_chunks) ||
                        !tmp.get(&order_sorted, (size_t)n_chunks))))
        return kErrOutOfDeviceMemory;
    auto own = [&](auto **p, size_t count) {
        return dev_alloc((void **)p, (count ? count : 1) * sizeof(**p)) == 0;
    };
    if (!own(&s.chunks, (size_t)n_chunks) || !own(&s.chunks_rank, (size_t)n_chunks) || !own(&s.split_rows, (size_t)n_split) ||
        !own(&s.split_rows_rank, (size_t)n_split)) {
        (void)hipGetLastError();
        free_device_hd_schedule(s);
        return kErrOutOfDeviceMemory;
    }
    hs_fill<<<dim3(grid_rows), dim3(kBlock), 0, st>>>(rowptr_dev, col_dev, hd_rows_dev, n_hd, chunk, pieces, slots, split, raw,
                                                      raw_rank, keys, order, s.split_rows, s.split_rows_rank);
    e = hipGetLastError();
    if (e == hipSuccess && count_out) {
        constexpr int kPer = kWavesPerBlock * kRankPieces;
        hs_rank<<<dim3((unsigned)((n_chunks + kPer - 1) / kPer)), dim3(kBlock), 0, st>>>(raw, raw_rank, keys, (int32_t)n_chunks, s.chunks,
                                                                                      s.chunks_rank);
        e = hipGetLastError();
    }
    // stable sort of the pieces by their first column: radix sort of (key, position) pairs
    size_t sort_bytes = 0;
    void *sort_tmp = nullptr;
    if (e == hipSuccess && !count_out)
        e = rocprim::radix_sort_pairs(nullptr, sort_bytes, keys, keys_sorted, order, order_sorted, (size_t)n_chunks, 0, 32, st);
    if (e == hipSuccess && !count_out && !tmp.get((char **)&sort_tmp, sort_bytes)) {
        free_device_hd_schedule(s);
        return kErrOutOfDeviceMemory;
    }
    if (e == hipSuccess && !count_out)
        e = rocprim::radix_sort_pairs(sort_tmp, sort_bytes, keys, keys_sorted, order, order_sorted, (size_t)n_chunks, 0, 32, st);
    if (e == hipSuccess && !count_out) {
        hs_permute<<<dim3((unsigned)((n_chunks + kBlock - 1) / kBlock)), dim3(kBlock), 0, st>>>(raw, raw_rank, order_sorted,
                                                                                            n_chunks, s.chunks, s.chunks_rank);
        e = hipGetLastError();
    }
    if (e != hipSuccess) {
        free_device_hd_schedule(s);
        return (int)e;
    }
    s.n_chunks = n_chunks;
    s.n_split_rows = n_split;
    s.n_partials = (int64_t)h.n_slots;
    s.nnz_hd = (int64_t)h.nnz_hd;
    *out = s;
    return 0;
}

}  // namespace groot
