// kernels_mfma_split_rowmax.hip -- the per-point cache g(v) of the fp32 kernels.
#include "split_kernels.hpp"

namespace exemcl {

hipError_t split_rowmax_run(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    switch (split_key(pl.nkb, pl.nt)) {
#define EXEMCL_CASE(NKB, NT) \
    case split_key(NKB, NT): return split_eval_t<NKB, NT, MODE_ROWMAX, true, false>(pl, x, st);
        EXEMCL_SPLIT_CASES(EXEMCL_CASE)
#undef EXEMCL_CASE
    }
    return hipErrorInvalidValue;
}

hipError_t split_rowmax_gather_run(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    switch (split_key(pl.nkb, pl.nt)) {
#define EXEMCL_CASE(NKB, NT) \
    case split_key(NKB, NT): return split_eval_t<NKB, NT, MODE_ROWMAX, true, true>(pl, x, st);
        EXEMCL_SPLIT_CASES(EXEMCL_CASE)
#undef EXEMCL_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace exemcl
