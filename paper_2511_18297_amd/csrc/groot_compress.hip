// Compact form of the device CSR for the pipelined LD kernel (gfx950): 4-byte row pointers and 2-byte column
// codes, built on the device from the resident CSR.  The aggregation is bound by the bytes it moves, and for
// the short rows of an EDA graph (Section "Kernel Design - GROOT-GPU": the low-degree class) the matrix
// itself is 5 % of them: 8 bytes of row pointer per row and 4 bytes per entry.  Nearly every entry of a
// low-degree row points either at a row close by (the gates of the same and of the neighbouring cells) or
// at one of the few high-degree rows (the primary inputs), which is what the two code ranges cover:
//     code <  0x8000:  column = row + code - 0x4000          (within -16384 .. +16383 rows)
//     code >= 0x8000:  column = hot[code - 0x8000]           (one of up to 32767 high-degree rows)
//     code == 0xFFFF:  neither (a primary output and its driver, say): the whole row joins the
//                      list of rows that are computed one by one, from the plain arrays
// Only rows that the pipelined kernel can serve are encoded (no more entries than it has slots, not
// high-degree); if more than one row in 50 cannot be encoded the plan keeps using the plain arrays.
#include "groot_device.h"

namespace groot {

// One thread per row, which copies the low half of its row pointer, too.  An entry that fits neither range gets kCodeBad and
// its row is appended to bad_rows (in no particular order): the pipelined kernel masks such a row, which is then computed by list.
__global__ __launch_bounds__(kBlock) void col16_kernel(const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                                       int64_t n, int32_t T, int32_t depth, const int32_t *__restrict__ hot,
                                                       int32_t n_hot, uint32_t *__restrict__ rp32, uint16_t *__restrict__ out,
                                                       int32_t *__restrict__ bad_rows, int32_t bad_cap,
                                                       int32_t *__restrict__ n_bad)
{
    for (int64_t row = (int64_t)blockIdx.x * kBlock + threadIdx.x; row < n; row += (int64_t)gridDim.x * kBlock) {
        const int64_t s = rowptr[row], e = rowptr[row + 1];
        rp32[row] = (uint32_t)s;
        if (row == n - 1) rp32[n] = (uint32_t)e;
        if (e - s > depth || e - s >= T) continue;                  // never read in compact form
        bool bad = false;
        for (int64_t p = s; p < e; ++p) {
            const int64_t c = col[p], delta = c - row;
            uint32_t code = kCodeBad;
            if (delta >= -kCodeNear && delta < kCodeNear) {
                code = (uint32_t)(delta + kCodeNear);
            } else {
                int32_t lo = 0, hi = n_hot;                         // first hot row >= c
                while (lo < hi) {
                    const int32_t mid = (lo + hi) / 2;
                    if (hot[mid] < c) lo = mid + 1; else hi = mid;
                }
                if (lo < n_hot && hot[lo] == c) code = kCodeHot + (uint32_t)lo;
                else bad = true;
            }
            out[p] = (uint16_t)code;
        }
        if (bad) {
            const int32_t k = atomicAdd(n_bad, 1);
            if (k < bad_cap) bad_rows[k] = (int32_t)row;
        }
    }
}

// hot_cols (padding included) from the list of high-degree rows, and the count of rows without a code
__global__ __launch_bounds__(kBlock) void hot_kernel(const int32_t *__restrict__ hd_rows, int32_t n_hot, int32_t *__restrict__ hot,
                                                     int32_t *__restrict__ n_bad)
{
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < hot_ints(n_hot)) hot[i] = i < n_hot ? hd_rows[i] : 0;
    if (i == 0) *n_bad = 0;
}

int32_t csr_bad_capacity(int64_t n) { return (int32_t)(n / 50 + 1024); }

// Enqueues the building of dp.rp32 / dp.col16 / dp.hot_cols from the resident CSR and the (device) list of high-degree rows,
// ascending.  The rows without a code go to bad_rows (room for csr_bad_capacity), their number to n_bad_dev; once that has been
// read, csr_compress_end decides.  *begun: whether there is anything to decide (not for matrices without entries or with too many
// for 32-bit row pointers, and not without memory: no error, the plain arrays serve).
int csr_compress_begin(DevicePlan &dp, const int32_t *hd_rows_dev, int64_t n_hd, int32_t *bad_rows, int32_t *n_bad_dev, void *stream,
                       bool *begun)
{
    hipStream_t st = (hipStream_t)stream;
    dp.compressed = 0;
    *begun = false;
    if (dp.n <= 0 || dp.nnz <= 0 || dp.nnz >= ((int64_t)1 << 32)) return 0;
    dp.n_hot = (int32_t)(n_hd < kCodeMaxHot ? n_hd : kCodeMaxHot);
    if (dev_alloc((void **)&dp.rp32, (size_t)(dp.n + 1) * 4) != 0 ||
        dev_alloc((void **)&dp.col16, (size_t)dp.nnz * 2) != 0 ||
        dev_alloc((void **)&dp.hot_cols, (size_t)hot_ints(dp.n_hot) * 4) != 0) {
        (void)hipGetLastError();
        csr_compress_drop(dp);
        return 0;
    }
    hot_kernel<<<dim3((unsigned)((hot_ints(dp.n_hot) + kBlock - 1) / kBlock)), dim3(kBlock), 0, st>>>(hd_rows_dev, dp.n_hot, dp.hot_cols,
                                                                                                   n_bad_dev);
    const int64_t grid = (dp.n + kBlock - 1) / kBlock;
    col16_kernel<<<dim3((unsigned)(grid < 16384 ? grid : 16384)), dim3(kBlock), 0, st>>>(
        dp.rowptr, dp.col, dp.n, dp.threshold, dp.pipe_depth, dp.hot_cols, dp.n_hot, dp.rp32, dp.col16, bad_rows,
        csr_bad_capacity(dp.n), n_bad_dev);
    const int err = (int)hipGetLastError();
    if (err) csr_compress_drop(dp);
    *begun = !err;
    return err;
}

// h_bad: rows without a code.  False, and the compact form is gone, when they are more than one row in 50; else they are part
// of dp.mid_rows already or become it now (the caller's business) and count here.
bool csr_compress_end(DevicePlan &dp, int32_t h_bad)
{
    if (h_bad < 0 || h_bad > csr_bad_capacity(dp.n) || (int64_t)h_bad * 50 > dp.n) {
        csr_compress_drop(dp);
        return false;
    }
    dp.n_mid_rows += h_bad;
    dp.n_bad_rows = h_bad;
    dp.compressed = 1;
    return true;
}

void csr_compress_drop(DevicePlan &dp)
{
    dev_free(dp.rp32); dev_free(dp.col16); dev_free(dp.hot_cols);
    dp.rp32 = nullptr; dp.col16 = nullptr; dp.hot_cols = nullptr; dp.n_hot = 0;
}

// Builds the compact form and appends the rows it cannot encode to dp.mid_rows.  Synchronises the stream.  On return
// dp.compressed says whether it is usable; when it is not its arrays are released and 0 is returned all the same.
int launch_csr_compress(DevicePlan &dp, const int32_t *hd_rows_dev, int64_t n_hd, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    int32_t *n_bad = nullptr, *rows = nullptr;
    bool begun = false;
    dp.compressed = 0;
    if (dp.n <= 0) return 0;
    if (dev_alloc((void **)&rows, ((size_t)dp.n_mid_rows + csr_bad_capacity(dp.n)) * 4) != 0 || dev_alloc((void **)&n_bad, 4) != 0) {
        (void)hipGetLastError();
        dev_free(rows);
        return 0;                                                    // no memory: the plain arrays serve
    }
    hipError_t e = dp.n_mid_rows ? hipMemcpyAsync(rows, dp.mid_rows, (size_t)dp.n_mid_rows * 4, hipMemcpyDeviceToDevice, st) : hipSuccess;
    int err = e != hipSuccess ? (int)e : csr_compress_begin(dp, hd_rows_dev, n_hd, rows + dp.n_mid_rows, n_bad, stream, &begun);
    int32_t h_bad = -1;
    if (!err && begun) {
        err = device_download(&h_bad, n_bad, 4, stream);             // waits for the stream
        if (err) csr_compress_drop(dp);
    } else {
        (void)hipStreamSynchronize(st);
    }
    if (!err && begun && csr_compress_end(dp, h_bad) && h_bad > 0) {
        dev_free(dp.mid_rows);
        dp.mid_rows = rows;
        rows = nullptr;
    }
    dev_free(rows);
    dev_free(n_bad);
    return err;
}

}  // namespace groot
