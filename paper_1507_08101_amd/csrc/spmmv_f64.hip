// spmmv_f64.hip -- instantiations of the product kernels for one value/vector type pair.
#include "spmmv_impl.h"

namespace sellcs {

int prod_f64(ProdArgs &a, bool aug, int path, hipStream_t s) {
    return aug ? dispatch_prod<VK_F64F64, true>(a, s, path) : dispatch_prod<VK_F64F64, false>(a, s, path);
}

int transpose_f64(ProdArgs &a, hipStream_t s) { return dispatch_transpose<VK_F64F64>(a, s); }

const void *batch_kernel_f64(int b, int vpt, bool aug, int path, int ub, int ubw, uint32_t flags, bool keep) {
    return aug ? batch_kernel_for<VK_F64F64, true>(b, vpt, path, ub, ubw, flags, keep)
               : batch_kernel_for<VK_F64F64, false>(b, vpt, path, ub, ubw, 0, keep);
}

const void *batch_mixed_kernel_f64(bool aug) {
    return aug ? batch_mixed_kernel_for<VK_F64F64, true>() : batch_mixed_kernel_for<VK_F64F64, false>();
}

}  // namespace sellcs
