// kernels_mfma_f32.hip -- fp32 instantiations of the kernels in
// mfma_kernels.hpp: d <= 2 (v_mfma_f32_32x32x2_f32: one instruction holds
// both coordinates), and the staging of 16-coordinate blocks for the kernel
// that splits the coordinates (bigd_kernels.hpp).
#include "mfma_kernels.hpp"

namespace exemcl {

hipError_t pack_run_f32(const MfmaPlan &pl, const void *V, int64_t n, int ld, const int32_t *sets, int64_t l,
                        int64_t k, void *tiles, hipStream_t st) {
    return pl.tile == 32 ? pack_launch<float, 32>(pl, V, n, ld, sets, l, k, tiles, st)
                         : pack_launch<float, 16>(pl, V, n, ld, sets, l, k, tiles, st);
}

template <int MODE>
static hipError_t eval_f32(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    if (pl.tile != 32 || pl.nkb != 1 || pl.nks_last != 1) return hipErrorInvalidValue;
    return eval_launch<float, 32, 1, 1, plan_rt(4, 32, 1), plan_waves(4, 32, 1), MODE>(x, st);
}

hipError_t eval_run_f32(const MfmaPlan &pl, int mode, const MfmaArgs &x, hipStream_t st) {
    return mode == MODE_ROWMAX ? eval_f32<MODE_ROWMAX>(pl, x, st) : eval_f32<MODE_SUM>(pl, x, st);
}

}  // namespace exemcl
