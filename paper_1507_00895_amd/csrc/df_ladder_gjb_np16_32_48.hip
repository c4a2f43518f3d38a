// Certified FP64 elimination, builds for n_nu padded to 16, 32, 48.
#include "df_ladder_gjb.hpp"

namespace df {

DF_GJB_BUILD(16, true, true)
DF_GJB_BUILD(16, true, false)
DF_GJB_BUILD(16, false, true)
DF_GJB_BUILD(16, false, false)
DF_GJB_BUILD(32, true, true)
DF_GJB_BUILD(32, true, false)
DF_GJB_BUILD(32, false, true)
DF_GJB_BUILD(32, false, false)
DF_GJB_BUILD(48, true, true)
DF_GJB_BUILD(48, true, false)
DF_GJB_BUILD(48, false, true)
DF_GJB_BUILD(48, false, false)
DF_GJB_BUILD_ALL(16)
DF_GJB_BUILD_ALL(32)
DF_GJB_BUILD_ALL(48)

}  // namespace df
