// kernels_mfma_split_gather.hip -- fp32 evaluation of sets without staged tiles in memory.
#include "split_kernels.hpp"

namespace exemcl {

hipError_t split_gather_run(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    switch (split_key(pl.nkb, pl.nt)) {
#define EXEMCL_CASE(NKB, NT) \
    case split_key(NKB, NT): return split_eval_t<NKB, NT, MODE_SUM, false, true>(pl, x, st);
        EXEMCL_SPLIT_CASES(EXEMCL_CASE)
#undef EXEMCL_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace exemcl
