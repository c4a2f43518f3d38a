// Certified FP64 elimination, mask-free builds for n_nu 96.
#include "df_ladder_gjb.hpp"

namespace df {

DF_GJB_BUILD(96, true, true)
DF_GJB_BUILD(96, true, false)

}  // namespace df
