// kernels_mfma_split.hip -- fp32 evaluation of sets on the bf16 matrix cores and its staging.
#include "split_kernels.hpp"

namespace exemcl {

hipError_t split_pack_run(const MfmaPlan &pl, const void *V, int64_t n, int ld, const int32_t *sets, int64_t l,
                          int64_t k, void *tiles, hipStream_t st, const int32_t *live, int64_t live0,
                          const int32_t *sets2, int64_t l2, void *tiles2) {
    if (l < 1 || k < 1) return hipErrorInvalidValue;
    switch (split_key(pl.nkb, pl.nt)) {
#define EXEMCL_CASE(NKB, NT) \
    case split_key(NKB, NT): return split_pack_t<NKB, NT>(V, n, ld, pl.d, sets, l, k, tiles, st, live, live0, sets2, l2, tiles2);
        EXEMCL_SPLIT_CASES(EXEMCL_CASE)
#undef EXEMCL_CASE
    }
    return hipErrorInvalidValue;
}

hipError_t split_sum_run(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    switch (split_key(pl.nkb, pl.nt)) {
#define EXEMCL_CASE(NKB, NT) \
    case split_key(NKB, NT): return split_eval_t<NKB, NT, MODE_SUM, false, false>(pl, x, st);
        EXEMCL_SPLIT_CASES(EXEMCL_CASE)
#undef EXEMCL_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace exemcl
