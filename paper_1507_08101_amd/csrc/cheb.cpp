// cheb.cpp -- derivatives with respect to the stored matrix values.
//
//  * sell_grad_values: dL/dval for Y = A X given G = dL/dY (pattern-restricted outer product).
//  * sell_cheb_filter: Z = sum_m coef_m T_m(A~) X, the chained axpby of the augmented product
//    accumulating z = z + coef_m+1 v_m+1 in the step that forms v_m+1.
//  * sell_cheb_forward / sell_cheb_backward: Y = T_N(A~) X with A~ = (A - c I) / s by the
//    three-term Chebyshev recurrence (each step one augmented product), and its adjoint.
//    The forward pass keeps the pair (v_kK, v_kK+1) every K steps; the backward pass walks
//    the segments from the last to the first, recomputes each segment's vectors from its
//    checkpoint and runs the adjoint recurrence
//        w_m = 2 A~^T w_m+1 - w_m+2,   dval += (2/s) outer(w_m+1, v_m)
//    (A~^T w via the forward kernel on the SELL copy of A^T), ending with the first step
//    w_0 = A~^T w_1 - w_2,  dval += (1/s) outer(w_1, v_0).
//    Every step of a recurrence is one launch: the augmented product reads the vector of two
//    steps before from one block and writes the new one to another, so nothing is copied between
//    them, and the vectors that a checkpoint or the result needs are written in place. The outer
//    products of several steps share a launch (16 columns' worth), which then reads and writes
//    the gradient once for all of them.
#include <algorithm>
#include <cmath>
#include <utility>
#include <vector>

#include "internal.h"

using namespace sellcs;

namespace {

#define HIPCHK(x)                                                                             \
    do {                                                                                      \
        hipError_t e_ = (x);                                                                  \
        if (e_ != hipSuccess) return e_ == hipErrorOutOfMemory ? SELL_ERR_OOM : SELL_ERR_HIP; \
    } while (0)

int vec_dt_of(const sell_mat *A) { return A->h.vdt == SELL_F64 ? SELL_F64 : SELL_F32; }

int check_block(const sell_mat *A, const sell_bv *v, int64_t nrows, int b) {
    if (!v) return SELL_ERR_ARG;
    if (v->dt != vec_dt_of(A)) return SELL_ERR_DTYPE;
    if (v->nrows != nrows || v->ncols != b) return SELL_ERR_SHAPE;
    if (v->lay != SELL_ROW_MAJOR || v->ld != v->ncols) return SELL_ERR_UNSUPPORTED;
    if (!v->ptr && nrows * b > 0) return SELL_ERR_ARG;
    return SELL_OK;
}

int check_matrix(const sell_mat *A) {
    if (!A) return SELL_ERR_ARG;
    if (!A->on_device) return SELL_ERR_STATE;
    int cur = -1;
    HIPCHK(hipGetDevice(&cur));
    return cur == A->device ? SELL_OK : SELL_ERR_STATE;
}

// Stream-ordered temporaries, released in stream order.
struct Temps {
    hipStream_t s;
    std::vector<void *> ptrs;
    explicit Temps(hipStream_t st) : s(st) {}
    ~Temps() {
        for (void *p : ptrs) (void)lib_free_async(p, s);
    }
    int alloc(void **p, size_t bytes) {
        *p = nullptr;
        HIPCHK(lib_malloc_async(p, bytes ? bytes : 16, s));
        ptrs.push_back(*p);
        return SELL_OK;
    }
};

sell_bv block(void *p, int64_t n, int b, int dt) {
    sell_bv v;
    v.nrows = n;
    v.ncols = b;
    v.dt = dt;
    v.lay = SELL_ROW_MAJOR;
    v.ptr = p;
    v.ld = b;
    v.owned = false;
    return v;
}

// y <- alpha (M x - c x) - w  (w == nullptr: no w; w may be y itself)
int shifted_product(const sell_mat *M, const sell_bv &x, sell_bv &y, double alpha, double c, const sell_bv *w,
                    hipStream_t s) {
    sell_spmv_opts o = SELL_SPMV_OPTS_INIT;
    o.flags = SELL_SPMV_SCALE | SELL_SPMV_SHIFT | (w ? SELL_SPMV_AXPBY : 0u);
    o.alpha = alpha;
    o.gamma = c;
    o.beta = w ? -1.0 : 0.0;
    return aug_impl(M, &x, &y, nullptr, o, true, s, nullptr, nullptr, nullptr, w);
}

bool overlap(const void *p, size_t pbytes, const void *q, size_t qbytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a < b + qbytes && b < a + pbytes;
}

// The array that a value gradient is computed in: dval itself, or where it overlaps what is still read (or
// written) meanwhile a temporary, which finish() copies to it.
struct GradTarget {
    double *dval, *work;
    size_t bytes;
    hipStream_t s;
    int init(Temps &T, double *d, size_t nnz, bool apart, bool accumulate) {
        dval = work = d;
        bytes = nnz * sizeof(double);
        s = T.s;
        if (apart) return SELL_OK;
        void *p;
        const int rc = T.alloc(&p, bytes);
        if (rc) return rc;
        work = static_cast<double *>(p);
        if (accumulate) HIPCHK(hipMemcpyAsync(work, dval, bytes, hipMemcpyDeviceToDevice, s));
        return SELL_OK;
    }
    int finish() {
        if (work != dval) HIPCHK(hipMemcpyAsync(dval, work, bytes, hipMemcpyDeviceToDevice, s));
        return SELL_OK;
    }
};

}  // namespace

extern "C" {

int sell_grad_values(const sell_mat *A, const sell_bv *G, const sell_bv *X, double alpha, int accumulate,
                     double *dval, void *stream) {
    int rc = check_matrix(A);
    if (rc) return rc;
    if (!G || !X) return SELL_ERR_ARG;
    const int b = G->ncols;
    if ((rc = check_block(A, G, A->h.nrows, b)) || (rc = check_block(A, X, A->h.ncols, b))) return rc;
    if (!dval && A->h.nnz > 0) return SELL_ERR_ARG;
    if (A->h.nnz == 0) return SELL_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if ((rc = ensure_row_pointers(const_cast<sell_mat *>(A), s))) return rc;
    GradPairs p;
    p.n = 1;
    p.g[0] = G->ptr;
    p.x[0] = X->ptr;
    p.c[0] = 1.0;
    p.scale = alpha;
    const size_t row = size_t(b) * dtype_bytes(G->dt), bytes = size_t(A->h.nnz) * sizeof(double);
    Temps T(s);
    GradTarget d;
    if ((rc = d.init(T, dval, size_t(A->h.nnz),
                     !overlap(dval, bytes, G->ptr, size_t(A->h.nrows) * row) &&
                         !overlap(dval, bytes, X->ptr, size_t(A->h.ncols) * row),
                     accumulate != 0)) ||
        (rc = launch_grad(A, p, G->ld, X->ld, G->dt, b, accumulate ? 1 : 0, d.work, s)))
        return rc;
    return d.finish();
}

int sell_cheb_forward(const sell_mat *A, const sell_bv *X, sell_bv *Y, int64_t N, double scale, double c,
                      int64_t K, void *ckpt, void *stream) {
    int rc = check_matrix(A);
    if (rc) return rc;
    if (A->h.nrows != A->h.ncols) return SELL_ERR_SHAPE;
    if (!X || !Y) return SELL_ERR_ARG;
    const int64_t n = A->h.nrows;
    const int b = X->ncols;
    if ((rc = check_block(A, X, n, b)) || (rc = check_block(A, Y, n, b))) return rc;
    if (b > kMaxSliceCols) return SELL_ERR_UNSUPPORTED;
    if (N < 1 || K < 1 || !(scale != 0.0) || !std::isfinite(scale) || !std::isfinite(c)) return SELL_ERR_ARG;
    if (n == 0) return SELL_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int dt = vec_dt_of(A);
    const size_t vb = size_t(n) * b * (dt == SELL_F64 ? 8 : 4);
    Temps T(s);
    void *p0, *p1, *px;
    if ((rc = T.alloc(&p0, vb)) || (rc = T.alloc(&p1, vb))) return rc;
    char *ck = static_cast<char *>(ckpt);
    const int64_t nseg = (N + K - 1) / K;
    // operands inside the checkpoints: X from a copy, v_N to Y last
    auto in_ckpt = [&](const void *p) { return ck && overlap(p, vb, ck, 2 * size_t(nseg) * vb); };
    const bool y_last = in_ckpt(Y->ptr);
    sell_bv V0 = *X;
    if (in_ckpt(X->ptr)) {
        if ((rc = T.alloc(&px, vb))) return rc;
        V0 = block(px, n, b, dt);
        if ((rc = launch_copy(&V0, X, s))) return rc;
    }
    // the block of v_i in the checkpoints (-1: none); with K = 1 also v_i as the second of the pair before
    auto first = [&](int64_t i) { return ck && i % K == 0 && i / K < nseg ? 2 * (i / K) : int64_t(-1); };
    auto second = [&](int64_t i) {
        return ck && i > 0 && (i - 1) % K == 0 && (i - 1) / K < nseg ? 2 * ((i - 1) / K) + 1 : int64_t(-1);
    };
    auto at = [&](int64_t slot) { return block(ck + size_t(slot) * vb, n, b, dt); };
    if (first(0) >= 0) {
        sell_bv c0 = at(first(0));
        if ((rc = launch_copy(&c0, &V0, s))) return rc;
    }
    // v_i goes to its checkpoint block, v_N to Y (where a checkpoint does not want it, and X is not
    // in its way), every other v_i to the work block that does not hold v_i-1; v_i-2, which the
    // step reads element by element as it writes v_i, may be in that one
    sell_bv prev = V0, cur = V0;
    for (int64_t i = 1; i <= N; ++i) {
        const int64_t sl = first(i) >= 0 ? first(i) : second(i);
        const bool last = i == N && y_last;
        sell_bv out = sl >= 0 && !last                                    ? at(sl)
                      : i == N && !last && !overlap(X->ptr, vb, Y->ptr, vb) ? *Y
                                                                            : block(cur.ptr == p0 ? p1 : p0, n, b, dt);
        if ((rc = shifted_product(A, cur, out, (i == 1 ? 1.0 : 2.0) / scale, c, i == 1 ? nullptr : &prev, s))) return rc;
        if (sl >= 0 && (last || (first(i) >= 0 && second(i) >= 0))) {  // (v_N is never the first of a pair)
            sell_bv again = at(last ? sl : second(i));
            if ((rc = launch_copy(&again, &out, s))) return rc;
        }
        prev = cur;
        cur = out;
    }
    return cur.ptr == Y->ptr ? SELL_OK : launch_copy(Y, &cur, s);
}

int sell_cheb_filter(const sell_mat *A, const sell_bv *X, sell_bv *Z, int64_t N, const double *coef, double scale,
                     double c, void *stream) {
    int rc = check_matrix(A);
    if (rc) return rc;
    if (A->h.nrows != A->h.ncols) return SELL_ERR_SHAPE;
    if (!X || !Z || !coef) return SELL_ERR_ARG;
    const int64_t n = A->h.nrows;
    const int b = X->ncols;
    if ((rc = check_block(A, X, n, b)) || (rc = check_block(A, Z, n, b))) return rc;
    if (b > kMaxSliceCols) return SELL_ERR_UNSUPPORTED;
    if (N < 0 || !(scale != 0.0) || !std::isfinite(scale) || !std::isfinite(c)) return SELL_ERR_ARG;
    if (X->ptr == Z->ptr && n > 0) return SELL_ERR_ARG;
    if (n == 0) return SELL_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int dt = vec_dt_of(A);
    // z = coef_0 x
    if ((rc = launch_axpby(dt, n, b, b, coef[0], X->ptr, 0.0, Z->ptr, s))) return rc;
    if (N == 0) return SELL_OK;
    const size_t vb = size_t(n) * b * (dt == SELL_F64 ? 8 : 4);
    Temps T(s);
    void *p0, *p1;
    if ((rc = T.alloc(&p0, vb)) || (rc = T.alloc(&p1, vb))) return rc;
    sell_bv V0 = block(p0, n, b, dt), V1 = block(p1, n, b, dt);
    // every step: one augmented product forming v_m+1 with the chained z = z + coef_m+1 v_m+1
    sell_spmv_opts o = SELL_SPMV_OPTS_INIT;
    o.flags = SELL_SPMV_SCALE | SELL_SPMV_SHIFT | SELL_SPMV_CHAIN;
    o.alpha = 1.0 / scale;
    o.gamma = c;
    o.delta = 1.0;
    o.eta = coef[1];
    if ((rc = aug_impl(A, X, &V1, Z, o, true, s))) return rc;  // v_1 = A~ v_0
    o.flags |= SELL_SPMV_AXPBY;
    o.alpha = 2.0 / scale;
    o.beta = -1.0;
    for (int64_t m = 1; m < N; ++m) {
        // v_m+1 = 2 A~ v_m - v_m-1, written over v_m-1 (v_0 is X, which stays)
        o.eta = coef[m + 1];
        if ((rc = aug_impl(A, &V1, &V0, Z, o, true, s, nullptr, nullptr, nullptr, m == 1 ? X : nullptr))) return rc;
        std::swap(V0, V1);  // (V0, V1) = (v_m, v_m+1)
    }
    return SELL_OK;
}

int sell_cheb_backward(const sell_mat *A, const sell_bv *G, int64_t N, double scale, double c, int64_t K,
                       const void *ckpt, sell_bv *dX, double *dval, void *stream) {
    int rc = check_matrix(A);
    if (rc) return rc;
    if (A->h.nrows != A->h.ncols) return SELL_ERR_SHAPE;
    if (!G || !dX || !ckpt) return SELL_ERR_ARG;
    const int64_t n = A->h.nrows;
    const int b = G->ncols;
    if ((rc = check_block(A, G, n, b)) || (rc = check_block(A, dX, n, b))) return rc;
    if (b > kMaxSliceCols) return SELL_ERR_UNSUPPORTED;
    if (N < 1 || K < 1 || !(scale != 0.0) || !std::isfinite(scale) || !std::isfinite(c)) return SELL_ERR_ARG;
    if (!dval && A->h.nnz > 0) return SELL_ERR_ARG;
    if (n == 0) return SELL_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    try {
        if ((rc = ensure_transpose(A, s)) || (rc = ensure_row_pointers(const_cast<sell_mat *>(A), s))) return rc;
    } catch (const std::bad_alloc &) {
        return SELL_ERR_OOM;
    }
    const sell_mat *AT = A->transpose;
    const int dt = vec_dt_of(A);
    const size_t vb = size_t(n) * b * (dt == SELL_F64 ? 8 : 4);
    const int64_t nseg = (N + K - 1) / K;
    const int64_t seglen = std::min<int64_t>(K, N);
    // outer products per launch: the steps that make up 16 columns. Past that the gradient's own
    // traffic is small beside the gathers, and the adjoint vectors kept for a launch would cost
    // memory: the group's (16 columns, or one vector where it is wider) and the two that the next step
    // reads. Where there is no room for them a launch takes one step.
    int64_t group = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(seglen, N), kGradPairs / b));
    int64_t nw = group + 2;
    Temps T(s);
    void *pw, *pseg = nullptr;
    if (seglen > 2 && (rc = T.alloc(&pseg, vb * size_t(seglen - 2)))) return rc;
    if ((rc = T.alloc(&pw, vb * size_t(nw))) == SELL_ERR_OOM && group > 1) {
        (void)hipGetLastError();
        group = 1;
        nw = 3;
        rc = T.alloc(&pw, vb * size_t(nw));
    }
    if (rc) return rc;
    auto w = [&](int64_t m) { return block(static_cast<char *>(pw) + size_t(m % nw) * vb, n, b, dt); };
    const char *ck = static_cast<const char *>(ckpt);
    GradTarget target;
    const size_t dvb = size_t(A->h.nnz) * sizeof(double);
    if ((rc = target.init(T, dval, size_t(A->h.nnz),
                          !overlap(dval, dvb, ck, 2 * size_t(nseg) * vb) && !overlap(dval, dvb, G->ptr, vb) &&
                              !overlap(dval, dvb, dX->ptr, vb),
                          false)))
        return rc;
    GradPairs pairs;
    pairs.n = 0;
    pairs.scale = (N > 1 ? 2.0 : 1.0) / scale;
    int written = 0;
    auto flush = [&]() -> int {
        if (pairs.n == 0) return SELL_OK;
        const int r = launch_grad(A, pairs, b, b, dt, b, written, target.work, s);
        pairs.n = 0;
        written = 1;
        return r;
    };
    for (int64_t k = nseg - 1; k >= 0; --k) {
        const int64_t lo = k * K, hi = std::min(lo + K - 1, N - 1);
        // v_lo and v_lo+1 are the segment's checkpoint, v_lo+2 .. v_hi are recomputed from it
        auto v = [&](int64_t m) {
            const int64_t i = m - lo;
            return i < 2 ? block(const_cast<char *>(ck) + size_t(2 * k + i) * vb, n, b, dt)
                         : block(static_cast<char *>(pseg) + size_t(i - 2) * vb, n, b, dt);
        };
        for (int64_t m = lo + 2; m <= hi; ++m) {
            sell_bv out = v(m), prev = v(m - 2);
            if ((rc = shifted_product(A, v(m - 1), out, 2.0 / scale, c, &prev, s))) return rc;
        }
        for (int64_t m = hi; m >= lo; --m) {
            // w_m from w_m+1 (w_N = G) and w_m+2 (w_N+1 = 0)
            const sell_bv w1 = m + 1 == N ? *G : w(m + 1), w2 = m + 2 == N ? *G : w(m + 2);
            pairs.g[pairs.n] = w1.ptr;
            pairs.x[pairs.n] = v(m).ptr;
            pairs.c[pairs.n++] = m > 0 || N == 1 ? 1.0 : 0.5;
            if ((pairs.n == group || m == lo) && (rc = flush())) return rc;
            sell_bv out = m == 0 && !overlap(G->ptr, vb, dX->ptr, vb) ? *dX : w(m);
            if ((rc = shifted_product(AT, w1, out, (m > 0 ? 2.0 : 1.0) / scale, c, m + 2 <= N ? &w2 : nullptr, s)))
                return rc;
        }
    }
    if (overlap(G->ptr, vb, dX->ptr, vb)) {
        const sell_bv w0 = w(0);
        if ((rc = launch_copy(dX, &w0, s))) return rc;
    }
    return target.finish();
}

}  // extern "C"
