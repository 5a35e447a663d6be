// Double-precision matrix-element kernel of g g -> t t~ t t~: the colour-ordered
// recursion of two quark lines with the generated process's colour matrix.
#include "generated/gen_gg_tttt.h"
#include "me_kernel.h"
#include "ordered_kernel.h"

namespace rwgt {

RWGT_PROCESS_TRAITS(gg_tttt, RWGT_PAIRED_COLOUR(gg_tttt))

hipError_t launch_ordered_gg_tttt(const Fp64Call& a, hipStream_t s) {
  return ordered::launch<Proc_gg_tttt, ordered::QuarkPairs>(a, s);
}

hipError_t launch_ordered_rows_gg_tttt(const double* mom, int64_t nevt, const CardPair* cards, int ncards,
                                       const double* w_in, double* w_out, double* me_out, const int32_t* rows,
                                       const unsigned int* nrows, hipStream_t s) {
  return ordered::launch_rows<Proc_gg_tttt, ordered::QuarkPairs>(mom, nevt, cards, ncards, w_in, w_out, me_out, rows, nrows, s);
}

}  // namespace rwgt
