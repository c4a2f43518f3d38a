// Certified FP64 elimination, builds for n_nu padded to 64.
#include "df_ladder_gjb.hpp"

namespace df {

DF_GJB_BUILD(64, true, true)
DF_GJB_BUILD(64, true, false)
DF_GJB_BUILD(64, false, true)
DF_GJB_BUILD(64, false, false)
DF_GJB_BUILD_ALL(64)

}  // namespace df
