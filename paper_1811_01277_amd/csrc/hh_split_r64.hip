// fp64 instances of the two-lane family's path: compact-WY kernels that read
// the reflectors in place (one translation unit per element type, so that the
// kernel variants compile in parallel).
#include "hh_split_impl.h"

namespace ehh {

#define EHH_WYD(NB, K)                                                        \
  {ELPA_PATH_SPLIT, 0, NB, K, 2, &launch_split<WyDirect<NB, K>>,               \
   &launch_split_batched<WyDirect<NB, K>>, &split_workspace<double, NB, K>,    \
   &launch_split_ws<WyDirect<NB, K>>, &prepare_split<WyDirect<NB, K>>}

const StripeEntry* split_table_r64(int* size) {
  static const StripeEntry table[] = {
      EHH_WYD(32, 32), EHH_WYD(32, 64), EHH_WYD(32, 96),
      EHH_WYD(64, 48), EHH_WYD(64, 64), EHH_WYD(64, 80),
  };
  *size = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

}  // namespace ehh
