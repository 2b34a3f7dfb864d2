// spmmv_bf16.hip -- instantiations of the product kernels for one value/vector type pair.
#include "spmmv_impl.h"

namespace sellcs {

int prod_bf16(ProdArgs &a, bool aug, int path, hipStream_t s) {
    return aug ? dispatch_prod<VK_BF16F32, true>(a, s, path) : dispatch_prod<VK_BF16F32, false>(a, s, path);
}

int transpose_bf16(ProdArgs &a, hipStream_t s) { return dispatch_transpose<VK_BF16F32>(a, s); }

const void *batch_kernel_bf16(int b, int vpt, bool aug, int path, int ub, int ubw, uint32_t flags, bool keep) {
    return aug ? batch_kernel_for<VK_BF16F32, true>(b, vpt, path, ub, ubw, flags, keep)
               : batch_kernel_for<VK_BF16F32, false>(b, vpt, path, ub, ubw, 0, keep);
}

const void *batch_mixed_kernel_bf16(bool aug) {
    return aug ? batch_mixed_kernel_for<VK_BF16F32, true>() : batch_mixed_kernel_for<VK_BF16F32, false>();
}

}  // namespace sellcs
