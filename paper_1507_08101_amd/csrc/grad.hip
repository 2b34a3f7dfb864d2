// grad.hip -- kernels for derivatives with respect to the stored matrix values.
//
// For a product Y = A X the gradient of a scalar loss with respect to the value of stored
// entry p = (i, k) is sum_j G[i, j] X[k, j] with G = dL/dY: an outer product restricted to
// the sparsity pattern.
#include "convert.h"
#include "devutil.h"
#include "internal.h"

namespace sellcs {

// dval[rowptr[row] + k] (+)= scale sum_p c_p sum_j G_p[row, j] X_p[col(row, k), j] for every stored entry k
// of every row, over the pairs (G_p, X_p) of the launch, written straight to the CSR order.
//
// L = 2^LL lanes serve one row slot, lane vg owning VPT consecutive columns of the row of G (in
// registers) and of the gathered rows of X; consecutive slots go to consecutive lane groups, so
// the indices stream coalesced and a row of X is gathered by L lanes with contiguous addresses.
// The entries are taken U at a time: U indices, U gathers per pair, and the lanes' partial sums of
// the U entries are reduced over the group by exchanging halves (each step halves the entries a
// lane holds), which leaves every lane with U / L finished entries to store. A row's entries are
// consecutive in dval, so a wave's stores fill whole lines of it.
//
// What bounds it: the gathers of X (a row of b elements per stored entry) through the CU's vector
// memory path. 100^3 Laplacian, FP32 vectors, b = 8: 34.9 us (147 MB that it cannot do without,
// 4.2 TB/s) against 285 us for one lane per row with element loads, added into a zeroed array in the
// SELL order that two more kernels cleared and mapped to CSR. 64^3 Anderson matrix, FP64, b = 1, ten
// pairs in a launch: 21.9 us against 10 x 12.1.
// RAG: b is not VPT * L; the last lanes' pieces are shifted back to end at column b - 1 and the
// columns that a lane shares with its neighbour are left to the neighbour.
constexpr int kGradU = 8;

template <class TX, int VPT, int LL, bool RAG>
__global__ void __launch_bounds__(256) grad_kernel(const int32_t *__restrict__ col, const int64_t *__restrict__ cs,
                                                   const int32_t *__restrict__ perm,
                                                   const int64_t *__restrict__ rowptr, int64_t row0, int64_t nrows,
                                                   int32_t C, int32_t cshift, int32_t b, GradPairs pairs, int64_t ldg,
                                                   int64_t ldx, int accumulate, double *__restrict__ dval) {
    constexpr int L = 1 << LL, U = kGradU;
    const int64_t s = row0 + int64_t(xcd_block(blockIdx.x, gridDim.x)) * (256 / L) + (threadIdx.x >> LL);
    if (s >= nrows) return;  // the whole lane group
    const int vg = threadIdx.x & (L - 1);
    const int64_t c = cshift >= 0 ? (s >> cshift) : s / C;
    const int64_t row = perm ? int64_t(perm[s]) : s;
    const int64_t base = cs[c] + (s - c * C);
    const int64_t p0 = rowptr[row];
    const int len = int(rowptr[row + 1] - p0);
    const int jb = RAG ? min(vg * VPT, b - VPT) : vg * VPT;
    const int skip = RAG ? vg * VPT - jb : 0;  // leading columns that belong to the neighbour
    for (int k0 = 0; k0 < len; k0 += U) {
        int64_t xo[U];
        double acc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = min(k0 + u, len - 1);
            xo[u] = int64_t(col[base + int64_t(k) * C]) * ldx + jb;
            acc[u] = 0.0;
        }
        for (int q = 0; q < pairs.n; ++q) {
            const TX *gp = static_cast<const TX *>(pairs.g[q]) + row * ldg + jb;
            const TX *xp = static_cast<const TX *>(pairs.x[q]);
            const double cq = pairs.c[q];
            double g[VPT];
            TX x[U][VPT];
#pragma unroll
            for (int t = 0; t < VPT; ++t) g[t] = cq * double(gp[t]);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int t = 0; t < VPT; ++t) x[u][t] = xp[xo[u] + t];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int t = 0; t < VPT; ++t) {
                    const double f = fma(g[t], double(x[u][t]), acc[u]);
                    acc[u] = !RAG || t >= skip ? f : acc[u];
                }
        }
        // reduce over the lane group, scattering the entries over its lanes
        int e0 = 0;       // first entry of the batch that this lane ends up with
        bool own = true;  // false: another lane holds the same sum
#pragma unroll
        for (int st = 0; st < LL; ++st) {
            const int m = L >> (st + 1), cnt = U >> st;
            const bool up = (vg & m) != 0;
            if (cnt > 1) {
                const int half = cnt / 2;
#pragma unroll
                for (int i = 0; i < half; ++i) {
                    const double send = up ? acc[i] : acc[i + half];
                    const double keep = up ? acc[i + half] : acc[i];
                    acc[i] = keep + __shfl_xor(send, m, 64);
                }
                e0 += up ? half : 0;
            } else {
                acc[0] += __shfl_xor(acc[0], m, 64);
                own = own && !up;
            }
        }
        constexpr int left = (U >> LL) > 0 ? (U >> LL) : 1;
        double *d = dval + p0 + k0 + e0;
        // (applied to the sums: with the rows of G scaled first, a factor and a row that are small or
        // large together left the range of a double where their products with X do not)
#pragma unroll
        for (int i = 0; i < left; ++i) acc[i] *= pairs.scale;
        if (accumulate) {
            double old[left];
#pragma unroll
            for (int i = 0; i < left; ++i) old[i] = own && k0 + e0 + i < len ? d[i] : 0.0;
#pragma unroll
            for (int i = 0; i < left; ++i) acc[i] += old[i];
        }
#pragma unroll
        for (int i = 0; i < left; ++i)
            if (own && k0 + e0 + i < len) d[i] = acc[i];
    }
}

// y = alpha x + beta y over n rows of b columns (row-major, leading dimension ld); y is not
// read when beta == 0.
template <class T>
__global__ void __launch_bounds__(256) axpby_kernel(int64_t n, int32_t b, int64_t ld, double alpha, const T *x,
                                                    double beta, T *y) {
    const int64_t N = n * b;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < N; e += int64_t(gridDim.x) * blockDim.x) {
        const int64_t i = e / b, k = i * ld + (e - i * b);
        const double v = alpha * double(x[k]);
        y[k] = T(beta != 0.0 ? v + beta * double(y[k]) : v);
    }
}

static unsigned ggrid(int64_t n) {
    int64_t g = (n + 255) / 256;
    if (g < 1) g = 1;
    if (g > 8192) g = 8192;
    return unsigned(g);
}

namespace {

template <class TX, int VPT, int LL, bool RAG>
void go_grad(const sell_mat *A, const GradPairs &p, int64_t ldg, int64_t ldx, int32_t b, int accumulate, double *dval,
             hipStream_t s) {
    const HostSell &h = A->h;
    const int32_t cshift = (h.C & (h.C - 1)) == 0 ? __builtin_ctz(unsigned(h.C)) : -1;
    for (int64_t row0 = 0; row0 < h.nrows; row0 += kGradGrid * (256 >> LL))
        hipLaunchKernelGGL((grad_kernel<TX, VPT, LL, RAG>), dim3(grad_grid(h.nrows - row0, LL)), dim3(256), 0, s, A->d_col,
                           A->d_cs, A->d_perm, A->d_rowptr, row0, h.nrows, h.C, cshift, b, p, ldg, ldx, accumulate, dval);
}

// Lanes per row for b columns: one up to b = 4 (VPT = b), else the power of two that holds
// ceil(b / 4) lanes of 4 columns.
template <class TX>
void dispatch_grad(const sell_mat *A, const GradPairs &p, int64_t ldg, int64_t ldx, int32_t b, int accumulate,
                   double *dval, hipStream_t s) {
#define SELL_GRAD(VPT, LL)                                                                            \
    (b == VPT << LL ? go_grad<TX, VPT, LL, false>(A, p, ldg, ldx, b, accumulate, dval, s)             \
                    : go_grad<TX, VPT, LL, (LL > 0)>(A, p, ldg, ldx, b, accumulate, dval, s))
    switch (b) {
        case 1: SELL_GRAD(1, 0); return;
        case 2: SELL_GRAD(2, 0); return;
        case 3: SELL_GRAD(3, 0); return;
        case 4: SELL_GRAD(4, 0); return;
        default: break;
    }
    if (b <= 8) SELL_GRAD(4, 1);
    else if (b <= 16) SELL_GRAD(4, 2);
    else if (b <= 32) SELL_GRAD(4, 3);
    else SELL_GRAD(4, 4);
#undef SELL_GRAD
}

}  // namespace

int launch_grad(const sell_mat *A, const GradPairs &pairs, int64_t ldg, int64_t ldx, int vec_dt, int32_t b,
                int accumulate, double *dval, hipStream_t s) {
    if (A->h.nrows == 0 || A->h.nnz == 0) return SELL_OK;
    const int esize = dtype_bytes(vec_dt);
    // blocks wider than a slice: one launch per slice, the later ones adding
    for (int32_t j = 0; j < b; j += kMaxSliceCols) {
        GradPairs p = pairs;
        for (int q = 0; q < p.n; ++q) {
            p.g[q] = static_cast<const char *>(pairs.g[q]) + int64_t(j) * esize;
            p.x[q] = static_cast<const char *>(pairs.x[q]) + int64_t(j) * esize;
        }
        const int32_t w = b - j < kMaxSliceCols ? b - j : kMaxSliceCols;
        if (vec_dt == SELL_F64)
            dispatch_grad<double>(A, p, ldg, ldx, w, accumulate || j > 0, dval, s);
        else
            dispatch_grad<float>(A, p, ldg, ldx, w, accumulate || j > 0, dval, s);
        if (hipGetLastError() != hipSuccess) return SELL_ERR_HIP;
    }
    return SELL_OK;
}

int launch_axpby(int vec_dt, int64_t n, int32_t b, int64_t ld, double alpha, const void *x, double beta, void *y,
                 hipStream_t s) {
    if (n * b == 0) return SELL_OK;
    if (vec_dt == SELL_F64)
        hipLaunchKernelGGL(axpby_kernel<double>, dim3(ggrid(n * b)), dim3(256), 0, s, n, b, ld, alpha,
                           static_cast<const double *>(x), beta, static_cast<double *>(y));
    else
        hipLaunchKernelGGL(axpby_kernel<float>, dim3(ggrid(n * b)), dim3(256), 0, s, n, b, ld, alpha,
                           static_cast<const float *>(x), beta, static_cast<float *>(y));
    return hipGetLastError() == hipSuccess ? SELL_OK : SELL_ERR_HIP;
}

}  // namespace sellcs
