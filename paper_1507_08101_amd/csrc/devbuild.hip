// devbuild.hip -- construction of SELL-C-sigma on the device from a CSR matrix that is already
// in device memory (GHOST paper, Sec. 5.1: the format, the sigma-window sort, padding to the
// chunk's longest row, column-major storage inside a chunk).
//
// The steps are the host builder's, as device kernels and library primitives, and the result
// is identical to it entry for entry:
//   row lengths; inside each window of sigma rows a stable sort by descending length (a stable
//   radix sort of the 64-bit keys (window, 2^31 - 1 - length), which keeps equal keys in row
//   order); chunk lengths as the maximum over the chunk's slots; chunk starts as an exclusive
//   prefix sum of C * length; a thread per slot (several where chunks are long) writes its row's
//   entries and its padding (column -1, value 0), converted to the storage type.
// The small per-chunk arrays, the permutation and the row pointers are copied back to the host
// (the matrix keeps them there, as a host-built one does), where the work partition is made.
//
// The CSR row pointers that value updates need and the SELL copy of A^T (a stable sort of the entries by
// column, then the steps above), with the place in it of each entry, are made here too, from the matrix's own
// device arrays. On the host, from an export of the matrix, the first backward pass over the 100^3
// Laplacian (FP32, b = 8) took 99 to 118 ms; with the device steps, which are bound by their
// allocations and copies of metadata, 5.1 ms.
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <new>
#include <vector>

#include "convert.h"
#include "internal.h"

namespace sellcs {

namespace {

constexpr int kT = 256;

unsigned grid_for(int64_t n) {
    int64_t g = (n + kT - 1) / kT;
    if (g < 1) g = 1;
    if (g > 65535) g = 65535;
    return unsigned(g);
}

// A grid of one thread per slot whose chunks' entries are shared by gridDim.y workgroups, 64 entries each at
// least and 2^16 workgroups in all at most: a thread alone with a row of a third of the matrix keeps every
// other one waiting (300,000 rows, one of them full, first transposed product 86 ms, now 3.4; from the host,
// where the row is walked in the cache, 66; 20,000 rows 5.7, 0.5 and 1.6).
dim3 grid_over_entries(int64_t nslots, const std::vector<int32_t> &cl) {
    const int64_t longest = cl.empty() ? 0 : *std::max_element(cl.begin(), cl.end());
    const unsigned gx = grid_for(nslots);
    return dim3(gx, unsigned(std::max<int64_t>(1, std::min<int64_t>(longest / 64, 65536 / gx))));
}

// flags[0] = 1 when the row pointers decrease or a row is 2^31 entries or longer;
// flags[1] = 1 when a column index is out of range. Plain stores of the same value.
__global__ void __launch_bounds__(kT) check_kernel(const int64_t *rowptr, const int32_t *col, int64_t nrows,
                                                   int64_t ncols, int64_t nnz, int32_t *flags) {
    const int64_t stride = int64_t(gridDim.x) * kT;
    for (int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x; i < nrows; i += stride) {
        const int64_t d = rowptr[i + 1] - rowptr[i];
        if (d < 0 || d >= (int64_t(1) << 31)) flags[0] = 1;
    }
    for (int64_t p = int64_t(blockIdx.x) * kT + threadIdx.x; p < nnz; p += stride) {
        const int32_t c = col[p];
        if (c < 0 || int64_t(c) >= ncols) flags[1] = 1;
    }
}

// len[i] = row length; with sorting, the key (window, 2^31 - 1 - length) and the row index.
__global__ void __launch_bounds__(kT) lengths_kernel(const int64_t *rowptr, int64_t nrows, int64_t sigma,
                                                     int32_t *len, uint64_t *keys, int32_t *rows) {
    for (int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x; i < nrows; i += int64_t(gridDim.x) * kT) {
        const int32_t l = int32_t(rowptr[i + 1] - rowptr[i]);
        len[i] = l;
        if (keys) {
            keys[i] = (uint64_t(i / sigma) << 32) | uint64_t(uint32_t(0x7fffffff - l));
            rows[i] = int32_t(i);
        }
    }
}

// slot -> row for the slots past the sorted rows (-1), and flags[2] = 1 when a slot holds
// another row than its own index.
__global__ void __launch_bounds__(kT) perm_tail_kernel(int32_t *slot_row, int64_t nrows, int64_t nslots,
                                                       int32_t *flags) {
    for (int64_t s = int64_t(blockIdx.x) * kT + threadIdx.x; s < nslots; s += int64_t(gridDim.x) * kT) {
        if (s >= nrows)
            slot_row[s] = -1;
        else if (slot_row[s] != int32_t(s))
            flags[2] = 1;
    }
}

// cl[c] = the longest row of chunk c; csz[c] = C * cl[c] (csz[nch] = 0 for the prefix sum).
__global__ void __launch_bounds__(kT) chunk_len_kernel(const int32_t *len, const int32_t *slot_row, int64_t nrows,
                                                       int64_t nch, int32_t C, int32_t *cl, int64_t *csz) {
    for (int64_t c = int64_t(blockIdx.x) * kT + threadIdx.x; c <= nch; c += int64_t(gridDim.x) * kT) {
        if (c == nch) {
            csz[c] = 0;
            continue;
        }
        int32_t m = 0;
        for (int32_t r = 0; r < C; ++r) {
            const int64_t s = c * C + r;
            const int64_t row = slot_row ? int64_t(slot_row[s]) : (s < nrows ? s : -1);
            if (row >= 0) m = max(m, len[row]);
        }
        cl[c] = m;
        csz[c] = int64_t(C) * m;
    }
}

// One thread per slot: the row's entries and the padding of its chunk column.
template <class V>
__global__ void __launch_bounds__(kT) fill_kernel(const int64_t *rowptr, const int32_t *col_in,
                                                  const double *val_in, const int32_t *len, const int32_t *slot_row,
                                                  const int32_t *cl, const int64_t *cs, int64_t nrows, int64_t nslots,
                                                  int32_t C, int32_t *col, V *val) {
    for (int64_t s = int64_t(blockIdx.x) * kT + threadIdx.x; s < nslots; s += int64_t(gridDim.x) * kT) {
        const int64_t c = s / C, r = s - c * C;
        const int64_t row = slot_row ? int64_t(slot_row[s]) : (s < nrows ? s : -1);
        const int32_t n = row >= 0 ? len[row] : 0;
        const int64_t p0 = row >= 0 ? rowptr[row] : 0;
        const int32_t m = cl[c];
        const int64_t base = cs[c] + r;
        for (int32_t k = int32_t(blockIdx.y); k < m; k += int32_t(gridDim.y)) {
            const bool real = k < n;
            col[base + int64_t(k) * C] = real ? col_in[p0 + k] : -1;
            val[base + int64_t(k) * C] = Conv<V, double>::go(real ? val_in[p0 + k] : 0.0);
        }
    }
}

// One thread per slot: len[row] = the row's entries, by bisection (padding, column -1, only follows
// them); len[nrows] = 0 for the prefix sum.
__global__ void __launch_bounds__(kT) row_lengths_kernel(const int32_t *col, const int32_t *cl, const int64_t *cs,
                                                         const int32_t *perm, int64_t nrows, int32_t C, int64_t *len) {
    for (int64_t s = int64_t(blockIdx.x) * kT + threadIdx.x; s <= nrows; s += int64_t(gridDim.x) * kT) {
        if (s == nrows) {
            len[nrows] = 0;
            continue;
        }
        const int64_t c = s / C, row = perm ? int64_t(perm[s]) : s, base = cs[c] + (s - c * C);
        int32_t n = 0, past = cl[c];
        while (n < past) {
            const int32_t mid = n + (past - n) / 2;
            if (col[base + int64_t(mid) * C] >= 0)
                n = mid + 1;
            else
                past = mid;
        }
        len[row] = n;
    }
}

// One thread per slot: the entries of its row in CSR order, as (column, own position) for the sort,
// with their row and their value as the double it represents.
template <class V>
__global__ void __launch_bounds__(kT) expand_kernel(const int32_t *col, const V *val, const int64_t *cs,
                                                    const int32_t *perm, const int64_t *rowptr, int64_t nrows,
                                                    int32_t C, uint32_t *key, int32_t *pos, int32_t *row_of,
                                                    double *value) {
    for (int64_t s = int64_t(blockIdx.x) * kT + threadIdx.x; s < nrows; s += int64_t(gridDim.x) * kT) {
        const int64_t c = s / C, row = perm ? int64_t(perm[s]) : s, base = cs[c] + (s - c * C);
        const int64_t p0 = rowptr[row], n = rowptr[row + 1] - p0;
        for (int64_t k = blockIdx.y; k < n; k += gridDim.y) {
            const int64_t e = base + k * C;
            key[p0 + k] = uint32_t(col[e]);
            pos[p0 + k] = int32_t(p0 + k);
            row_of[p0 + k] = int32_t(row);
            value[p0 + k] = Conv<double, V>::go(val[e]);
        }
    }
}

// CSR of A^T from the entries sorted by column: row pointer t is the first entry whose column is at
// least t (binary search), entry q's column and value those of the entry of A it came from.
__global__ void __launch_bounds__(kT) transposed_csr_kernel(const uint32_t *key, const int32_t *pos,
                                                            const int32_t *row_of, const double *value, int64_t nnz,
                                                            int64_t ncols, int64_t *trp, int32_t *tcol, double *tval) {
    const int64_t stride = int64_t(gridDim.x) * kT, first = int64_t(blockIdx.x) * kT + threadIdx.x;
    for (int64_t t = first; t <= ncols; t += stride) {
        int64_t lo = 0, hi = nnz;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (int64_t(key[mid]) < t)
                lo = mid + 1;
            else
                hi = mid;
        }
        trp[t] = lo;
    }
    for (int64_t q = first; q < nnz; q += stride) {
        const int32_t p = pos[q];
        tcol[q] = row_of[p];
        tval[q] = value[p];
    }
}

// slot_of[row] = slot of a permuted matrix
__global__ void __launch_bounds__(kT) inverse_kernel(const int32_t *perm, int64_t nrows, int32_t *slot_of) {
    for (int64_t s = int64_t(blockIdx.x) * kT + threadIdx.x; s < nrows; s += int64_t(gridDim.x) * kT)
        slot_of[perm[s]] = int32_t(s);
}

// tpos[p] = position in the SELL arrays of A^T of CSR entry p of A
template <class P>
__global__ void __launch_bounds__(kT) tpos_kernel(const uint32_t *key, const int32_t *pos, int64_t nnz,
                                                  const int64_t *trp, const int32_t *slot_of, const int64_t *cs,
                                                  int32_t C, P *tpos) {
    for (int64_t q = int64_t(blockIdx.x) * kT + threadIdx.x; q < nnz; q += int64_t(gridDim.x) * kT) {
        const int64_t t = key[q], slot = slot_of ? int64_t(slot_of[t]) : t, c = slot / C;
        tpos[pos[q]] = P(cs[c] + (q - trp[t]) * C + (slot - c * C));
    }
}

struct DevTemp {
    std::vector<void *> p;
    ~DevTemp() {
        for (void *q : p) (void)lib_free(q);
    }
    hipError_t alloc(void **q, size_t bytes) {
        *q = nullptr;
        hipError_t e = lib_malloc(q, bytes ? bytes : 16);
        if (e == hipSuccess) p.push_back(*q);
        return e;
    }
};

int herr(hipError_t e) { return e == hipErrorOutOfMemory ? SELL_ERR_OOM : SELL_ERR_HIP; }

}  // namespace

// Builds into M (fresh, not yet on the device). Returns SELL_OK or an error; on error the
// caller frees whatever device arrays M holds.
int build_device_sell(sell_mat *M, int64_t nrows, int64_t ncols, const int64_t *rowptr, const int32_t *col,
                      const double *val, int32_t C, int64_t sigma, int vdt, hipStream_t s) {
#define DCHK(x)                                  \
    do {                                         \
        hipError_t e_ = (x);                     \
        if (e_ != hipSuccess) return herr(e_);   \
    } while (0)
    HostSell &h = M->h;
    if (nrows < 0 || ncols < 0 || nrows >= (int64_t(1) << 31) || ncols >= (int64_t(1) << 31)) return SELL_ERR_ARG;
    if (C < 1 || C > (1 << 20) || sigma < 1) return SELL_ERR_ARG;
    if (vdt != SELL_F64 && vdt != SELL_F32 && vdt != SELL_BF16) return SELL_ERR_DTYPE;
    if (!rowptr) return SELL_ERR_ARG;
    DCHK(hipGetDevice(&M->device));
    // row pointers to the host (the matrix keeps them), first and last entries checked there
    h = HostSell();
    h.rowptr.resize(size_t(nrows) + 1);
    DCHK(hipMemcpyAsync(h.rowptr.data(), rowptr, sizeof(int64_t) * (size_t(nrows) + 1), hipMemcpyDeviceToHost, s));
    DCHK(hipStreamSynchronize(s));
    if (h.rowptr[0] != 0) return SELL_ERR_ARG;
    const int64_t nnz = h.rowptr[size_t(nrows)];
    if (nnz < 0) return SELL_ERR_ARG;
    if (nnz > 0 && (!col || !val)) return SELL_ERR_ARG;
    const int64_t nch = (nrows + C - 1) / C, nslots = nch * C;
    const int64_t win = std::min<int64_t>(sigma, std::max<int64_t>(nrows, 1));
    const bool sort = win > 1;

    DevTemp T;
    int32_t *flags, *len, *slot_row = nullptr;
    int64_t *csz;
    DCHK(T.alloc(reinterpret_cast<void **>(&flags), 4 * sizeof(int32_t)));
    DCHK(hipMemsetAsync(flags, 0, 4 * sizeof(int32_t), s));
    hipLaunchKernelGGL(check_kernel, dim3(grid_for(std::max(nrows, nnz))), dim3(kT), 0, s, rowptr, col, nrows, ncols,
                       nnz, flags);
    DCHK(hipGetLastError());
    DCHK(T.alloc(reinterpret_cast<void **>(&len), sizeof(int32_t) * size_t(std::max<int64_t>(nrows, 1))));
    uint64_t *keys = nullptr, *keys_out = nullptr;
    int32_t *rows = nullptr;
    if (sort) {
        DCHK(T.alloc(reinterpret_cast<void **>(&keys), sizeof(uint64_t) * size_t(nrows)));
        DCHK(T.alloc(reinterpret_cast<void **>(&keys_out), sizeof(uint64_t) * size_t(nrows)));
        DCHK(T.alloc(reinterpret_cast<void **>(&rows), sizeof(int32_t) * size_t(nrows)));
        DCHK(lib_malloc(reinterpret_cast<void **>(&slot_row), sizeof(int32_t) * size_t(nslots)));
        M->d_perm = slot_row;  // owned by the matrix from here on (freed with it, or dropped below)
    }
    if (nrows > 0) {
        hipLaunchKernelGGL(lengths_kernel, dim3(grid_for(nrows)), dim3(kT), 0, s, rowptr, nrows, win, len, keys, rows);
        DCHK(hipGetLastError());
    }
    int32_t hflags[4] = {0, 0, 0, 0};
    if (sort && nrows > 0) {
        int nwin_bits = 0;
        while ((int64_t(1) << nwin_bits) < (nrows + win - 1) / win) ++nwin_bits;
        const int end_bit = 32 + nwin_bits;
        size_t tmp_bytes = 0;
        DCHK(hipcub::DeviceRadixSort::SortPairs(nullptr, tmp_bytes, keys, keys_out, rows, slot_row, int(nrows), 0,
                                                end_bit, s));
        void *tmp = nullptr;
        DCHK(T.alloc(&tmp, tmp_bytes));
        DCHK(hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, keys, keys_out, rows, slot_row, int(nrows), 0,
                                                end_bit, s));
    }
    if (sort) {
        hipLaunchKernelGGL(perm_tail_kernel, dim3(grid_for(nslots)), dim3(kT), 0, s, slot_row, nrows, nslots, flags);
        DCHK(hipGetLastError());
    }
    DCHK(hipMemcpyAsync(hflags, flags, 4 * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    DCHK(hipStreamSynchronize(s));
    if (hflags[0] || hflags[1]) return SELL_ERR_ARG;
    const bool has_perm = sort && hflags[2];
    if (sort && !has_perm) {  // the sort kept every row in place: no permutation
        DCHK(lib_free(slot_row));
        M->d_perm = nullptr;
        slot_row = nullptr;
    }

    // chunk lengths and starts
    DCHK(lib_malloc(reinterpret_cast<void **>(&M->d_cl), sizeof(int32_t) * size_t(std::max<int64_t>(nch, 1))));
    DCHK(lib_malloc(reinterpret_cast<void **>(&M->d_cs), sizeof(int64_t) * (size_t(nch) + 1)));
    DCHK(T.alloc(reinterpret_cast<void **>(&csz), sizeof(int64_t) * (size_t(nch) + 1)));
    hipLaunchKernelGGL(chunk_len_kernel, dim3(grid_for(nch + 1)), dim3(kT), 0, s, len, slot_row, nrows, nch, C,
                       M->d_cl, csz);
    DCHK(hipGetLastError());
    {
        size_t tmp_bytes = 0;
        DCHK(hipcub::DeviceScan::ExclusiveSum(nullptr, tmp_bytes, csz, M->d_cs, int(nch + 1), s));
        void *tmp = nullptr;
        DCHK(T.alloc(&tmp, tmp_bytes));
        DCHK(hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, csz, M->d_cs, int(nch + 1), s));
    }
    h.cl.resize(size_t(nch));
    h.cs.resize(size_t(nch) + 1);
    if (nch > 0) DCHK(hipMemcpyAsync(h.cl.data(), M->d_cl, sizeof(int32_t) * size_t(nch), hipMemcpyDeviceToHost, s));
    DCHK(hipMemcpyAsync(h.cs.data(), M->d_cs, sizeof(int64_t) * (size_t(nch) + 1), hipMemcpyDeviceToHost, s));
    DCHK(hipStreamSynchronize(s));
    const int64_t stored = h.cs[size_t(nch)];

    // the fill
    const int vb = dtype_bytes(vdt);
    DCHK(lib_malloc(reinterpret_cast<void **>(&M->d_col), sizeof(int32_t) * size_t(std::max<int64_t>(stored, 1))));
    DCHK(lib_malloc(&M->d_val, size_t(vb) * size_t(std::max<int64_t>(stored, 1))));
    if (nslots > 0) {
        const dim3 gf = grid_over_entries(nslots, h.cl);
        if (vdt == SELL_F64)
            hipLaunchKernelGGL(fill_kernel<double>, gf, dim3(kT), 0, s, rowptr, col, val, len,
                               slot_row, M->d_cl, M->d_cs, nrows, nslots, C, M->d_col,
                               static_cast<double *>(M->d_val));
        else if (vdt == SELL_F32)
            hipLaunchKernelGGL(fill_kernel<float>, gf, dim3(kT), 0, s, rowptr, col, val, len,
                               slot_row, M->d_cl, M->d_cs, nrows, nslots, C, M->d_col, static_cast<float *>(M->d_val));
        else
            hipLaunchKernelGGL(fill_kernel<uint16_t>, gf, dim3(kT), 0, s, rowptr, col, val, len,
                               slot_row, M->d_cl, M->d_cs, nrows, nslots, C, M->d_col,
                               static_cast<uint16_t *>(M->d_val));
        DCHK(hipGetLastError());
    }
    if (has_perm) {
        h.perm.resize(size_t(nslots));
        DCHK(hipMemcpyAsync(h.perm.data(), slot_row, sizeof(int32_t) * size_t(nslots), hipMemcpyDeviceToHost, s));
    }

    // the work partition, made on the host from the chunk lengths
    h.nrows = nrows;
    h.ncols = ncols;
    h.nnz = nnz;
    h.stored = stored;
    h.nch = nch;
    h.sigma = sigma;
    h.C = C;
    h.vdt = vdt;
    h.has_perm = has_perm;
    make_tiles(h.cl, C, default_tile_count(nch), h.tiles);
    h.batch = choose_batch_len(h.cl);
    h.batch_wide = choose_batch_len(h.cl, true);
    h.waves = choose_waves(h.cl);
    h.ulen = uniform_chunk_len(h.cl);
    DCHK(lib_malloc(reinterpret_cast<void **>(&M->d_tiles), sizeof(int32_t) * h.tiles.size()));
    DCHK(hipMemcpyAsync(M->d_tiles, h.tiles.data(), sizeof(int32_t) * h.tiles.size(), hipMemcpyHostToDevice, s));
    DCHK(hipStreamSynchronize(s));
    M->ntiles = int32_t(h.tiles.size()) - 1;
    M->matrix_bytes = int64_t(stored) * (4 + vb) + nch * 12 + 8 + (has_perm ? nslots * 4 : 0) +
                      int64_t(h.tiles.size()) * 4;
    M->on_device = true;
    return SELL_OK;
#undef DCHK
}

#define DCHK(x)                                \
    do {                                       \
        hipError_t e_ = (x);                   \
        if (e_ != hipSuccess) return herr(e_); \
    } while (0)

int device_row_pointers(const sell_mat *A, int64_t **rowptr, hipStream_t s) {
    const HostSell &h = A->h;
    if (h.nrows + 1 > INT32_MAX) return SELL_ERR_UNSUPPORTED;  // the scan counts its items in 32 bits
    DevTemp T, keep;
    int64_t *len, *rp;
    DCHK(keep.alloc(reinterpret_cast<void **>(&rp), sizeof(int64_t) * (size_t(h.nrows) + 1)));
    DCHK(T.alloc(reinterpret_cast<void **>(&len), sizeof(int64_t) * (size_t(h.nrows) + 1)));
    hipLaunchKernelGGL(row_lengths_kernel, dim3(grid_for(h.nrows + 1)), dim3(kT), 0, s, A->d_col, A->d_cl, A->d_cs, A->d_perm,
                       h.nrows, h.C, len);
    DCHK(hipGetLastError());
    size_t bytes = 0;
    void *tmp = nullptr;
    DCHK(hipcub::DeviceScan::ExclusiveSum(nullptr, bytes, len, rp, int(h.nrows + 1), s));
    DCHK(T.alloc(&tmp, bytes));
    DCHK(hipcub::DeviceScan::ExclusiveSum(tmp, bytes, len, rp, int(h.nrows + 1), s));
    DCHK(hipStreamSynchronize(s));
    keep.p.clear();
    *rowptr = rp;
    return SELL_OK;
}

int device_transpose(const sell_mat *A, sell_mat **out, void **out_tpos, bool *wide, hipStream_t s) {
    const HostSell &h = A->h;
    if (h.nnz > INT32_MAX || h.nnz == 0) return SELL_ERR_UNSUPPORTED;  // positions are sorted as 32-bit payloads
    DevTemp T, keep;
    uint32_t *key, *key_s;
    int32_t *pos, *pos_s, *row_of, *tcol, *slot_of = nullptr;
    double *value, *tval;
    int64_t *trp;
    void *tpos = nullptr;
    const size_t nnz = size_t(h.nnz);
    DCHK(T.alloc(reinterpret_cast<void **>(&key), 4 * nnz));
    DCHK(T.alloc(reinterpret_cast<void **>(&key_s), 4 * nnz));
    DCHK(T.alloc(reinterpret_cast<void **>(&pos), 4 * nnz));
    DCHK(T.alloc(reinterpret_cast<void **>(&pos_s), 4 * nnz));
    DCHK(T.alloc(reinterpret_cast<void **>(&row_of), 4 * nnz));
    DCHK(T.alloc(reinterpret_cast<void **>(&tcol), 4 * nnz));
    DCHK(T.alloc(reinterpret_cast<void **>(&value), 8 * nnz));
    DCHK(T.alloc(reinterpret_cast<void **>(&tval), 8 * nnz));
    DCHK(T.alloc(reinterpret_cast<void **>(&trp), 8 * (size_t(h.ncols) + 1)));
    const dim3 gr = grid_over_entries(h.nrows, h.cl), gz(grid_for(h.nnz)), bl(kT);
    if (h.vdt == SELL_F64)
        hipLaunchKernelGGL(expand_kernel<double>, gr, bl, 0, s, A->d_col, static_cast<const double *>(A->d_val), A->d_cs,
                           A->d_perm, A->d_rowptr, h.nrows, h.C, key, pos, row_of, value);
    else if (h.vdt == SELL_F32)
        hipLaunchKernelGGL(expand_kernel<float>, gr, bl, 0, s, A->d_col, static_cast<const float *>(A->d_val), A->d_cs,
                           A->d_perm, A->d_rowptr, h.nrows, h.C, key, pos, row_of, value);
    else
        hipLaunchKernelGGL(expand_kernel<uint16_t>, gr, bl, 0, s, A->d_col, static_cast<const uint16_t *>(A->d_val),
                           A->d_cs, A->d_perm, A->d_rowptr, h.nrows, h.C, key, pos, row_of, value);
    DCHK(hipGetLastError());
    // stable: entries of a column keep A's order, rows ascending
    int bits = 1;
    while ((int64_t(1) << bits) < h.ncols) ++bits;
    size_t bytes = 0;
    void *tmp = nullptr;
    DCHK(hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, key, key_s, pos, pos_s, int(h.nnz), 0, bits, s));
    DCHK(T.alloc(&tmp, bytes));
    DCHK(hipcub::DeviceRadixSort::SortPairs(tmp, bytes, key, key_s, pos, pos_s, int(h.nnz), 0, bits, s));
    hipLaunchKernelGGL(transposed_csr_kernel, dim3(grid_for(std::max(h.nnz, h.ncols + 1))), bl, 0, s, key_s, pos_s, row_of,
                       value, h.nnz, h.ncols, trp, tcol, tval);
    DCHK(hipGetLastError());
    sell_mat *M = new (std::nothrow) sell_mat();
    if (!M) return SELL_ERR_OOM;
    int rc = SELL_ERR_OOM;
    try {
        rc = build_device_sell(M, h.ncols, h.nrows, trp, tcol, tval, h.C, h.sigma, h.vdt, s);
        *wide = M->h.stored > INT32_MAX;
        hipError_t e = hipSuccess;
        if (rc == SELL_OK) e = keep.alloc(&tpos, (*wide ? 8 : 4) * nnz);
        if (rc == SELL_OK && e == hipSuccess && M->d_perm)
            e = T.alloc(reinterpret_cast<void **>(&slot_of), 4 * size_t(h.ncols));
        if (e != hipSuccess) rc = herr(e);
    } catch (const std::bad_alloc &) {
        rc = SELL_ERR_OOM;
    }
    if (rc == SELL_OK) {
        if (slot_of) hipLaunchKernelGGL(inverse_kernel, dim3(grid_for(h.ncols)), bl, 0, s, M->d_perm, h.ncols, slot_of);
        if (*wide)
            hipLaunchKernelGGL(tpos_kernel<int64_t>, gz, bl, 0, s, key_s, pos_s, h.nnz, trp, slot_of, M->d_cs, h.C,
                               static_cast<int64_t *>(tpos));
        else
            hipLaunchKernelGGL(tpos_kernel<int32_t>, gz, bl, 0, s, key_s, pos_s, h.nnz, trp, slot_of, M->d_cs, h.C,
                               static_cast<int32_t *>(tpos));
        if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) rc = SELL_ERR_HIP;
    }
    if (rc) {
        M->on_device = true;  // release whatever device arrays the build made
        sell_destroy(M);
        return rc;
    }
    keep.p.clear();
    *out = M;
    *out_tpos = tpos;
    return SELL_OK;
}
#undef DCHK

}  // namespace sellcs
