// tsm.hip -- tall-skinny block-vector kernels (GHOST paper Sec. 5.2), FP64, row-major.
//   tsmttsm:      X = alpha V^T W + beta X   (V: n x m, W: n x k, X: m x k small)
//   tsmm:         W = alpha V X + beta W     (X: m x k small)
//   tsmm_inplace: V = alpha V X + beta V     (X: m x m small)
// m, k <= 64. They are streaming kernels (bandwidth-bound for small m, k). tsmttsm keeps 4 x 4
// blocks of the result in registers per thread and reduces deterministically (per-workgroup
// partials, then a fixed-order sum), with an optional Neumaier-compensated summation (the
// paper adds a Kahan-summed variant of this reduction for accuracy on long vectors); tsmm and
// tsmm_inplace keep the small matrix X in LDS. Wider blocks are dense contractions and run on the
// matrix cores (FP64 MFMA), which take each element once from memory and keep the small matrix in
// registers; the rules that choose stand with the launchers.
#include <algorithm>
#include <type_traits>

#include "devutil.h"
#include "internal.h"

namespace sellcs {

constexpr int kTT = 256;     // threads per workgroup

__device__ __forceinline__ void neumaier_add(double &s, double &comp, double term) {
    const double t = s + term;
    if (fabs(s) >= fabs(term))
        comp += (s - t) + term;
    else
        comp += (term - t) + s;
    s = t;
}

// Partial sums of V^T W over this workgroup's row range [g n / G, (g + 1) n / G). The m x k
// result is cut into 4 x 4 blocks; thread t accumulates block t % nblk in registers over the
// rows t / nblk, + groups, ... of the range (groups = 256 / nblk row groups), so every loaded
// row piece feeds 16 multiply-adds. The row groups' blocks are then added in group order
// through LDS; output q = l * k + j lands in partials[q * G + g]. KAHAN: Neumaier-compensated
// sums in both stages.
// VEC (m and k multiples of 4, V and W rows 16-byte aligned): each thread loads its 4 + 4
// values as 16-byte pieces with no bounds checks and keeps TV rows in flight; the rows are
// visited in the same order, so the sums are the same bit for bit. V^T W with n = 4 M,
// m = k = 8: 98.8 us against 118.9 for the per-element loads (1, 2, 4 or 8 rows in flight
// within 3 %). The compensated sums keep the per-element loads: with 16-byte loads they ran
// 156-163 us with 1 or 2 rows in flight against 157 us (within the noise between runs) and
// 197 us with 8 rows (the Neumaier updates of more rows hold more registers).
constexpr int kTV = 4;
typedef double tsm_d2 __attribute__((ext_vector_type(2)));

template <bool KAHAN, bool VEC, int TV = kTV>
__global__ void __launch_bounds__(kTT) tsmttsm_partial_kernel(const double *__restrict__ V, int64_t ldv,
                                                              const double *__restrict__ W, int64_t ldw, int64_t n,
                                                              int m, int k, double *partials) {
    __shared__ double red[kTT][17];
    const int G = gridDim.x, g = blockIdx.x, tid = threadIdx.x;
    const int64_t r0 = int64_t(g) * n / G, r1 = int64_t(g + 1) * n / G;
    const int nbk = (k + 3) / 4, nblk = ((m + 3) / 4) * nbk;  // at most 256 blocks
    const int groups = kTT / nblk;
    const int blk = tid % nblk, grp = tid / nblk;
    const int l0 = (blk / nbk) * 4, j0 = (blk % nbk) * 4;
    double acc[16], comp[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = comp[e] = 0.0;
    if (VEC && grp < groups) {
        const int64_t st = groups;
        for (int64_t i = r0 + grp; i < r1; i += TV * st) {
            tsm_d2 v[TV][2], w[TV][2];
#pragma unroll
            for (int u = 0; u < TV; ++u)
                if (i + u * st < r1) {
                    const tsm_d2 *vp = reinterpret_cast<const tsm_d2 *>(V + (i + u * st) * ldv + l0);
                    const tsm_d2 *wp = reinterpret_cast<const tsm_d2 *>(W + (i + u * st) * ldw + j0);
                    v[u][0] = vp[0];
                    v[u][1] = vp[1];
                    w[u][0] = wp[0];
                    w[u][1] = wp[1];
                }
#pragma unroll
            for (int u = 0; u < TV; ++u)
                if (i + u * st < r1) {
#pragma unroll
                    for (int a = 0; a < 4; ++a)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const double va = v[u][a >> 1][a & 1], wc = w[u][c >> 1][c & 1];
                            if (KAHAN)
                                neumaier_add(acc[a * 4 + c], comp[a * 4 + c], va * wc);
                            else
                                acc[a * 4 + c] = fma(va, wc, acc[a * 4 + c]);
                        }
                }
        }
    } else if (grp < groups) {
#pragma unroll 2
        for (int64_t i = r0 + grp; i < r1; i += groups) {
            double v[4], w[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                v[t] = l0 + t < m ? V[i * ldv + l0 + t] : 0.0;
                w[t] = j0 + t < k ? W[i * ldw + j0 + t] : 0.0;
            }
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (KAHAN)
                        neumaier_add(acc[a * 4 + c], comp[a * 4 + c], v[a] * w[c]);
                    else
                        acc[a * 4 + c] = fma(v[a], w[c], acc[a * 4 + c]);
                }
        }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) red[tid][e] = acc[e] + comp[e];
    __syncthreads();
    for (int o = tid; o < nblk * 16; o += kTT) {
        const int b = o >> 4, e = o & 15;
        const int l = (b / nbk) * 4 + (e >> 2), j = (b % nbk) * 4 + (e & 3);
        if (l >= m || j >= k) continue;
        double sum = 0.0, c2 = 0.0;
        for (int gg = 0; gg < groups; ++gg) {
            if (KAHAN)
                neumaier_add(sum, c2, red[gg * nblk + b][e]);
            else
                sum += red[gg * nblk + b][e];
        }
        partials[size_t(l * k + j) * G + g] = sum + c2;
    }
}

// X[q] = alpha * sum_g partials[q * G + g] + beta * X[q], one workgroup per entry.
__global__ void __launch_bounds__(kTT) tsmttsm_finish_kernel(const double *partials, int G, int k, int kahan,
                                                             double alpha, double beta, double *X, int64_t ldx) {
    const int q = blockIdx.x;
    const double *p = partials + size_t(q) * G;
    double s = 0.0, comp = 0.0;
    for (int t = threadIdx.x; t < G; t += kTT) {
        if (kahan)
            neumaier_add(s, comp, p[t]);
        else
            s += p[t];
    }
    const double tot = block_sum_256(s) + block_sum_256(comp);
    if (threadIdx.x == 0) {
        const int l = q / k, j = q - l * k;
        double *x = X + int64_t(l) * ldx + j;
        const double v = alpha * tot;
        *x = beta != 0.0 ? v + beta * *x : v;
    }
}

// W = alpha V X + beta W: a tile of R rows of V is staged in LDS with coalesced loads (consecutive
// lanes read consecutive entries), then thread (r, j) of the tile forms output (r, j) from the
// staged row and X, also staged in LDS. The LDS holds exactly m k + R m doubles (dynamic), so
// small blocks do not limit the workgroups per compute unit.
__host__ __device__ inline int tsmm_rows(int m, int k) {
    const int r = kTT / k;
    return r * m > 2048 ? 2048 / m : r;
}

__global__ void __launch_bounds__(kTT) tsmm_kernel(const double *__restrict__ V, int64_t ldv, const double *Xs,
                                                   int64_t ldx, int m, int k, int64_t n, double alpha, double beta,
                                                   double *W, int64_t ldw) {
    extern __shared__ double lds[];
    double *sx = lds, *sv = lds + m * k;
    for (int e = threadIdx.x; e < m * k; e += kTT) sx[e] = Xs[int64_t(e / k) * ldx + e % k];
    const int R = tsmm_rows(m, k);
    const int r = threadIdx.x / k, j = threadIdx.x - r * k;
    for (int64_t t0 = int64_t(blockIdx.x) * R; t0 < n; t0 += int64_t(gridDim.x) * R) {
        const int rows = n - t0 < R ? int(n - t0) : R;
        __syncthreads();
        for (int e = threadIdx.x; e < rows * m; e += kTT) {
            const int rr = e / m;
            sv[e] = V[(t0 + rr) * ldv + (e - rr * m)];
        }
        __syncthreads();
        if (r < rows) {
            double s = 0.0;
            for (int l = 0; l < m; ++l) s = fma(sv[r * m + l], sx[l * k + j], s);
            double *w = W + (t0 + r) * ldw + j;
            const double v = alpha * s;
            *w = beta != 0.0 ? v + beta * *w : v;
        }
    }
}

// V = alpha V X + beta V: rows staged in LDS before any of them is overwritten.
__global__ void __launch_bounds__(kTT) tsmm_inplace_kernel(double *V, int64_t ldv, const double *Xs, int64_t ldx,
                                                           int m, int64_t n, double alpha, double beta) {
    extern __shared__ double lds[];
    double *sv = lds, *sx = lds + kTT;  // LDS: kTT + m m doubles (dynamic)
    for (int e = threadIdx.x; e < m * m; e += kTT) sx[e] = Xs[int64_t(e / m) * ldx + e % m];
    const int rows = kTT / m;  // rows per tile
    for (int64_t t0 = int64_t(blockIdx.x) * rows; t0 < n; t0 += int64_t(gridDim.x) * rows) {
        const int r = threadIdx.x / m, j = threadIdx.x - (threadIdx.x / m) * m;
        const bool act = r < rows && t0 + r < n;
        __syncthreads();
        if (act) sv[r * m + j] = V[(t0 + r) * ldv + j];
        __syncthreads();
        if (act) {
            double s = 0.0;
            for (int l = 0; l < m; ++l) s += sv[r * m + l] * sx[l * m + j];
            const double v = alpha * s;
            V[(t0 + r) * ldv + j] = beta != 0.0 ? v + beta * sv[r * m + j] : v;
        }
    }
}

// ---------------------------------------------------------------- matrix-core kernels
// v_mfma_f64_16x16x4: D (16 x 16) += A (16 x 4) B (4 x 16). Lane l holds A[l % 16][l / 16],
// B[l / 16][l % 16] and D[4 r + l / 16][l % 16], r = 0..3.
typedef double tsm_d4 __attribute__((ext_vector_type(4)));
typedef double tsm_d2u __attribute__((ext_vector_type(2), aligned(8)));  // a 16-byte load of any two doubles

constexpr int kMB = 512;        // threads per workgroup of the V^T W kernel
constexpr int kMW = kMB / 64;   // its waves

// A row piece of a block of M columns (M <= 16 NB) for the 16 lanes of a row: column block q's
// column i is col(q, i). Two blocks at a time are loaded as pairs of neighbouring columns (16
// bytes per lane, block 2p the even ones and 2p + 1 the odd ones); which columns make up a
// block does not matter, since the result is put back by column. Columns past M give 0.
template <int NB>
struct TsmCols {
    int off[(NB + 1) / 2];
    bool ok0[(NB + 1) / 2], ok1[(NB + 1) / 2];
    __device__ static int col(int q, int i) { return q + 1 == NB && NB % 2 ? 16 * q + i : 32 * (q / 2) + 2 * i + (q & 1); }
    __device__ void init(int M, int i) {
#pragma unroll
        for (int p = 0; p < (NB + 1) / 2; ++p) {
            const int c = col(2 * p, i);
            ok0[p] = c < M;
            ok1[p] = c + 1 < M;
            const bool pair = 2 * p + 1 < NB;
            off[p] = pair ? (c < M - 2 ? c : M - 2) : (c < M - 1 ? c : M - 1);  // M > 16 where pairs are
        }
    }
    // v[q] = row[col(q, i)], 0 outside the block or with live false
    __device__ void load(const double *row, bool live, double (&v)[NB]) const {
#pragma unroll
        for (int p = 0; p < (NB + 1) / 2; ++p) {
            if (2 * p + 1 < NB) {
                const tsm_d2u t = *reinterpret_cast<const tsm_d2u *>(row + off[p]);
                v[2 * p] = live && ok0[p] ? (ok1[p] ? t[0] : t[1]) : 0.0;
                v[2 * p + 1] = live && ok1[p] ? t[1] : 0.0;
            } else {
                const double t = row[off[p]];
                v[2 * p] = live && ok0[p] ? t : 0.0;
            }
        }
    }
};

// Partial V^T W of this workgroup's rows [g n / G, (g + 1) n / G) on the matrix cores: a wave takes
// 16 rows at a time (four per instruction) and keeps the whole m x k result (MB x KB blocks of
// 16 x 16) in registers, so every element of V and W is loaded once. The waves' results are added
// in wave order through LDS; entry (l, j) lands in partials[g m k + l k + j]. The next rows' loads are
// in flight during the products (up to 8 KB per wave). Bound by HBM up to 32 x 32 (n = 937,500 again
// and again: 94.7 us, 5.07 TB/s; n = 1,000,000 after a kernel that wrote V: 128 us, 4.0 TB/s), by the partial results that fit the workspace (192 workgroups) at 64 x 64 (n =
// 468,750: 175 us, 2.74 TB/s, 22 TFLOP/s).
__host__ __device__ constexpr int tsm_vtw_u(int blocks) { return blocks <= 2 ? 8 : blocks <= 4 ? 4 : 2; }

template <int MB, int KB>
__global__ void __launch_bounds__(kMB) tsmttsm_mfma_kernel(const double *__restrict__ V, int64_t ldv,
                                                           const double *__restrict__ W, int64_t ldw, int64_t n,
                                                           int m, int k, double *__restrict__ partials) {
    __shared__ double red[MB * KB * 256];
    const int G = gridDim.x, g = blockIdx.x, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, i16 = lane & 15, q4 = lane >> 4;
    const int64_t r0 = int64_t(g) * n / G, r1 = int64_t(g + 1) * n / G;
    TsmCols<MB> cv;
    TsmCols<KB> cw;
    cv.init(m, i16);
    cw.init(k, i16);
    tsm_d4 acc[MB][KB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int c = 0; c < KB; ++c) acc[a][c] = tsm_d4{0.0, 0.0, 0.0, 0.0};
    constexpr int U = tsm_vtw_u(MB + KB);
    constexpr int64_t step = 4 * U * kMW;
    double v[U][MB], w[U][KB];
    auto load = [&](int64_t i) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t r = i + 4 * u + q4, rc = r < r1 ? r : r1 - 1;
            cv.load(V + rc * ldv, r < r1, v[u]);
            cw.load(W + rc * ldw, r < r1, w[u]);
        }
    };
    int64_t i = r0 + 4 * U * wave;
    if (i < r1) load(i);
    while (i < r1) {
        double vc[U][MB], wc[U][KB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int a = 0; a < MB; ++a) vc[u][a] = v[u][a];
#pragma unroll
            for (int c = 0; c < KB; ++c) wc[u][c] = w[u][c];
        }
        i += step;
        if (i < r1) load(i);  // in flight during this step's products
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int c = 0; c < KB; ++c)
                    acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(vc[u][a], wc[u][c], acc[a][c], 0, 0, 0);
    }
    for (int ww = 0; ww < kMW; ++ww) {
        if (wave == ww)
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int c = 0; c < KB; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        double *d = red + ((a * KB + c) * 4 + r) * 64 + lane;
                        *d = ww ? *d + acc[a][c][r] : acc[a][c][r];
                    }
        __syncthreads();
    }
    for (int o = tid; o < MB * KB * 256; o += kMB) {
        const int ln = o & 63, r = (o >> 6) & 3, blk = o >> 8;
        const int l = TsmCols<MB>::col(blk / KB, 4 * r + (ln >> 4)), j = TsmCols<KB>::col(blk % KB, ln & 15);
        if (l < m && j < k) partials[size_t(g) * (m * k) + l * k + j] = red[o];
    }
}

// X[q] = alpha * sum_g partials[g mk + q] + beta * X[q]: a workgroup sums 32 neighbouring entries,
// 8 threads each over every 8th partial, added in thread order.
__global__ void __launch_bounds__(kTT) tsmttsm_mfma_finish_kernel(const double *partials, int G, int mk, int k,
                                                                  double alpha, double beta, double *X, int64_t ldx) {
    __shared__ double red[8][32];
    const int e = threadIdx.x & 31, sl = threadIdx.x >> 5, q = blockIdx.x * 32 + e;
    double s = 0.0;
    if (q < mk)
#pragma unroll 8
        for (int g = sl; g < G; g += 8) s += partials[size_t(g) * mk + q];
    red[sl][e] = s;
    __syncthreads();
    if (sl || q >= mk) return;
#pragma unroll
    for (int t = 1; t < 8; ++t) s += red[t][e];
    const int l = q / k, j = q - l * k;
    double *x = X + int64_t(l) * ldx + j;
    const double v = alpha * s;
    *x = beta != 0.0 ? v + beta * *x : v;
}

// W = alpha V X + beta W on the matrix cores: a wave takes tiles of 16 rows. Lane l loads the column
// pairs (8 c + 2 (l / 16), + 1) of row l % 16, 16 bytes per lane and 64 contiguous bytes per row, and
// the instruction of (c, e) takes columns 8 c + 2 (l / 16) + e as its four terms; X, cut the same
// way, stays in registers. One or two tiles are loaded before the first is used. V and W may be the same
// block (k = m): a wave reads its tiles completely before it stores them, and no other wave reads
// those rows. Bound by HBM: 32 x 32, n = 937,500: 92 us (5.2 TB/s), in place 77 us (6.2 TB/s).
__host__ __device__ constexpr int tsm_vx_tiles(int MC, int KB) { return MC * KB > 12 ? 1 : 2; }

template <int MC, int KB>
__global__ void __launch_bounds__(kTT) tsmm_mfma_kernel(const double *V, int64_t ldv, const double *Xs, int64_t ldx,
                                                        int m, int k, int64_t n, double alpha, double beta, double *W,
                                                        int64_t ldw) {
    constexpr int kRT = tsm_vx_tiles(MC, KB);
    const int lane = threadIdx.x & 63, i16 = lane & 15, q4 = lane >> 4;
    const int64_t wave = int64_t(blockIdx.x) * (kTT / 64) + (threadIdx.x >> 6);
    const int64_t stride = int64_t(gridDim.x) * (kTT / 64) * (16 * kRT);
    double x[MC][2][KB];
    int off[MC];
    bool ok0[MC], ok1[MC];
#pragma unroll
    for (int c = 0; c < MC; ++c) {
        const int l = 8 * c + 2 * q4;
        ok0[c] = l < m;
        ok1[c] = l + 1 < m;
        off[c] = l < m - 2 ? l : m - 2;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                const int j = 16 * b + i16;
                x[c][e][b] = l + e < m && j < k ? Xs[int64_t(l + e) * ldx + j] : 0.0;
            }
    }
    for (int64_t t0 = wave * (16 * kRT); t0 < n; t0 += stride) {
        double v[kRT][MC][2];
#pragma unroll
        for (int t = 0; t < kRT; ++t) {
            const int64_t r = t0 + 16 * t + i16;
            const double *row = V + (r < n ? r : n - 1) * ldv;
#pragma unroll
            for (int c = 0; c < MC; ++c) {
                const tsm_d2u p = *reinterpret_cast<const tsm_d2u *>(row + off[c]);
                v[t][c][0] = ok0[c] ? (ok1[c] ? p[0] : p[1]) : 0.0;
                v[t][c][1] = ok1[c] ? p[1] : 0.0;
            }
        }
        double old[kRT][KB][4];
        if (beta != 0.0)
#pragma unroll
            for (int t = 0; t < kRT; ++t)
#pragma unroll
                for (int b = 0; b < KB; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int64_t row = t0 + 16 * t + 4 * r + q4;
                        const int j = 16 * b + i16;
                        old[t][b][r] = row < n && j < k ? W[row * ldw + j] : 0.0;
                    }
        tsm_d4 acc[kRT][KB];
#pragma unroll
        for (int t = 0; t < kRT; ++t)
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                acc[t][b] = tsm_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int c = 0; c < MC; ++c)
#pragma unroll
                    for (int e = 0; e < 2; ++e)
                        acc[t][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t][c][e], x[c][e][b], acc[t][b], 0, 0, 0);
            }
#pragma unroll
        for (int t = 0; t < kRT; ++t)
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t row = t0 + 16 * t + 4 * r + q4;
                    const int j = 16 * b + i16;
                    const double a = alpha * acc[t][b][r];
                    if (row < n && j < k) W[row * ldw + j] = beta != 0.0 ? a + beta * old[t][b][r] : a;
                }
    }
}

static unsigned tgrid(int64_t work, unsigned cap) {
    int64_t g = (work + kTT - 1) / kTT;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return unsigned(g);
}

// Calls f(std::integral_constant<int, c>) for c = 1..4.
template <class F>
static void with_blocks(int c, F &&f) {
    switch (c) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 3: f(std::integral_constant<int, 3>()); break;
        default: f(std::integral_constant<int, 4>()); break;
    }
}

// Matrix cores for V^T W? The register kernel loads an element of V for each of the k / 4 blocks
// beside it and one of W m / 4 times, m k / (2 (m + k)) times the bytes of the blocks through the L1,
// which bounds it from about 4 times on, and from 2.75 where it loads single elements. Below that
// line the matrix-core kernel's own loads (8 bytes per lane up to 16 columns, lanes idle past m and
// k) are the slower ones. Aligned, n (m + k) = 60 M: 16 x 16 110 us against 130 on the matrix cores,
// 64 x 8 106 against 102, 20 x 20 136 against 99, 32 x 32 184 against 95, 64 x 64 512 against 175;
// element loads: 11 x 11 149 against 168, 17 x 9 188 against 136, 21 x 11 188 against 118.
static bool mfma_vtw(int m, int k, bool vec) { return 2 * m * k > (vec ? 16 : 11) * (m + k); }

// Matrix cores for V X? Not where a row is a few elements: half of the lanes' 16-byte pieces lie past
// m or half of the stored columns past k (m = k = 4: 42 us against 49; 6 x 2: 48 against 53, with
// beta 55 against 74), while the LDS kernel streams well there. From 10 columns in all (12 where k
// <= 2) on they are at least level (4 x 6: 78 against 67; 12 x 2 97 against 91) and then ahead:
// 8 x 8 104 against 94, 16 x 16 121 against 87, 32 x 32 191 against 92, 64 x 64 392 against 134. In
// place: m = 6 61 against 64, m = 8 78 against 73, m = 32 178 against 77, m = 64 365 against 115.
// With beta a row of W costs a second load and two columns of it leave the LDS kernel, whose rows of V then
// conflict in no bank unless 16 divides m, little else: n = 600 K, k = 1, m = 12 16.3 against 17.1, 17 19.8 and
// 21.6, 16 26.7 and 19.7, 20 23.2 and 22.4.
static bool mfma_vx(int m, int k, double beta) {
    return m >= 2 && m + k >= 10 && (k > 2 || (beta != 0.0 ? m >= 20 || m == 16 : m >= 12));
}
static bool mfma_vx_inplace(int m) { return m >= 7; }

// W = alpha V X + beta W (W may be V) on the matrix cores, m >= 2
static int go_tsmm_mfma(const double *V, int64_t ldv, const double *X, int64_t ldx, int m, int k, int64_t n,
                        double alpha, double beta, double *W, int64_t ldw, hipStream_t s) {
    with_blocks((m + 7) / 8 > 4 ? (m + 7) / 8 - 4 : (m + 7) / 8, [&](auto c) {
        with_blocks((k + 15) / 16, [&](auto b) {
            constexpr int MC = decltype(c)::value, KB = decltype(b)::value;
            const int64_t rows = 16 * (m > 32 ? tsm_vx_tiles(MC + 4, KB) : tsm_vx_tiles(MC, KB)) * (kTT / 64);
            const unsigned g = unsigned(std::min<int64_t>((n + rows - 1) / rows, 2048));
            hipLaunchKernelGGL((m > 32 ? tsmm_mfma_kernel<MC + 4, KB> : tsmm_mfma_kernel<MC, KB>), dim3(g), dim3(kTT),
                               0, s, V, ldv, X, ldx, m, k, n, alpha, beta, W, ldw);
        });
    });
    return hipGetLastError() == hipSuccess ? SELL_OK : SELL_ERR_HIP;
}

int launch_tsmttsm(const double *V, int64_t ldv, const double *W, int64_t ldw, int64_t n, int m, int k, double alpha,
                   double beta, double *X, int64_t ldx, int kahan, double *partials, int64_t max_partials,
                   hipStream_t s) {
    const int mk = m * k;
    const bool vec = m % 4 == 0 && k % 4 == 0 && ldv % 2 == 0 && ldw % 2 == 0 &&
                     (reinterpret_cast<uintptr_t>(V) & 15u) == 0 && (reinterpret_cast<uintptr_t>(W) & 15u) == 0;
    if (!kahan && n > 0 && mfma_vtw(m, k, vec)) {
        int64_t G = (n + 16 * kMW - 1) / (16 * kMW);
        G = std::max<int64_t>(1, std::min<int64_t>(G, std::min<int64_t>(512, max_partials / mk)));
        with_blocks((m + 15) / 16, [&](auto a) {
            with_blocks((k + 15) / 16, [&](auto c) {
                hipLaunchKernelGGL((tsmttsm_mfma_kernel<decltype(a)::value, decltype(c)::value>), dim3(unsigned(G)),
                                   dim3(kMB), 0, s, V, ldv, W, ldw, n, m, k, partials);
            });
        });
        if (hipGetLastError() != hipSuccess) return SELL_ERR_HIP;
        hipLaunchKernelGGL(tsmttsm_mfma_finish_kernel, dim3((mk + 31) / 32), dim3(kTT), 0, s, partials, int(G), mk, k,
                           alpha, beta, X, ldx);
        return hipGetLastError() == hipSuccess ? SELL_OK : SELL_ERR_HIP;
    }
    int64_t G = (n + 63) / 64;
    if (G > 1024) G = 1024;
    if (G > max_partials / mk) G = max_partials / mk;
    if (G < 1) G = 1;
    auto kern = kahan ? tsmttsm_partial_kernel<true, false>
                      : (vec ? tsmttsm_partial_kernel<false, true> : tsmttsm_partial_kernel<false, false>);
    hipLaunchKernelGGL(kern, dim3(unsigned(G)), dim3(kTT), 0, s, V, ldv, W, ldw, n, m, k, partials);
    if (hipGetLastError() != hipSuccess) return SELL_ERR_HIP;
    hipLaunchKernelGGL(tsmttsm_finish_kernel, dim3(mk), dim3(kTT), 0, s, partials, int(G), k, kahan, alpha, beta, X,
                       ldx);
    return hipGetLastError() == hipSuccess ? SELL_OK : SELL_ERR_HIP;
}

int launch_tsmm(const double *V, int64_t ldv, const double *X, int64_t ldx, int m, int k, int64_t n, double alpha,
                double beta, double *W, int64_t ldw, hipStream_t s) {
    if (n == 0) return SELL_OK;
    if (mfma_vx(m, k, beta)) return go_tsmm_mfma(V, ldv, X, ldx, m, k, n, alpha, beta, W, ldw, s);
    const int R = tsmm_rows(m, k);
    const size_t lds = size_t(m * k + R * m) * sizeof(double);
    hipLaunchKernelGGL(tsmm_kernel, dim3(tgrid((n + R - 1) / R * kTT, 8192)), dim3(kTT), lds, s, V, ldv, X, ldx, m,
                       k, n, alpha, beta, W, ldw);
    return hipGetLastError() == hipSuccess ? SELL_OK : SELL_ERR_HIP;
}

int launch_tsmm_inplace(double *V, int64_t ldv, const double *X, int64_t ldx, int m, int64_t n, double alpha,
                        double beta, hipStream_t s) {
    if (n == 0) return SELL_OK;
    if (mfma_vx_inplace(m)) return go_tsmm_mfma(V, ldv, X, ldx, m, m, n, alpha, beta, V, ldv, s);
    const int rows = kTT / m;
    hipLaunchKernelGGL(tsmm_inplace_kernel, dim3(tgrid((n + rows - 1) / rows * kTT, 8192)), dim3(kTT),
                       size_t(kTT + m * m) * sizeof(double), s, V, ldv, X, ldx, m, n, alpha, beta);
    return hipGetLastError() == hipSuccess ? SELL_OK : SELL_ERR_HIP;
}

}  // namespace sellcs
