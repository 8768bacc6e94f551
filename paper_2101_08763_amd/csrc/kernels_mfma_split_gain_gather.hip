// kernels_mfma_split_gain_gather.hip -- scoring of S u {c} without staged tiles in memory.
#include "split_kernels.hpp"

namespace exemcl {

hipError_t split_gain_gather_run(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    switch (split_key(pl.nkb, pl.nt)) {
#define EXEMCL_CASE(NKB, NT) \
    case split_key(NKB, NT): return split_eval_t<NKB, NT, MODE_SUM, true, true>(pl, x, st);
        EXEMCL_SPLIT_CASES(EXEMCL_CASE)
#undef EXEMCL_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace exemcl
