// Certified FP64 elimination, mask-free build for n_nu 128, screened items.
#include "df_ladder_gjb.hpp"

namespace df {

DF_GJB_BUILD(128, true, true)

}  // namespace df
