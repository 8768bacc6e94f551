// kernels_mfma_wide.hip -- long fp16/bf16 rows as a tiled matrix product.
#include "wide_kernels.hpp"

namespace exemcl {

hipError_t wide_run(int prec, const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    if (x.m0) return hipErrorInvalidValue;
    if (prec == P_FP16) return wide_dispatch<_Float16>(pl, x, st);
    if (prec == P_BF16) return wide_dispatch<__bf16>(pl, x, st);
    return hipErrorInvalidValue;
}

}  // namespace exemcl
