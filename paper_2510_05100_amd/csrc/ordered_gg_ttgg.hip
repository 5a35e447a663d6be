// Double-precision matrix-element kernel of g g -> t t~ g g: the colour-ordered
// recursion with the generated process's colour matrix.
#include "generated/gen_gg_ttgg.h"
#include "me_kernel.h"
#include "ordered_kernel.h"

namespace rwgt {

RWGT_PROCESS_TRAITS(gg_ttgg, RWGT_PAIRED_COLOUR(gg_ttgg))

hipError_t launch_ordered_gg_ttgg(const Fp64Call& a, hipStream_t s) {
  return ordered::launch<Proc_gg_ttgg, ordered::QuarkLine>(a, s);
}

hipError_t launch_ordered_rows_gg_ttgg(const double* mom, int64_t nevt, const CardPair* cards, int ncards,
                                       const double* w_in, double* w_out, double* me_out, const int32_t* rows,
                                       const unsigned int* nrows, hipStream_t s) {
  return ordered::launch_rows<Proc_gg_ttgg, ordered::QuarkLine>(mom, nevt, cards, ncards, w_in, w_out, me_out, rows, nrows, s);
}

}  // namespace rwgt
