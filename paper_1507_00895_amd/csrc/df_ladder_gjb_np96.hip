// Certified FP64 elimination, builds for n_nu padded to 96.
#include "df_ladder_gjb.hpp"

namespace df {

DF_GJB_BUILD(96, false, true)
DF_GJB_BUILD(96, false, false)

}  // namespace df
