// Certified FP64 elimination, build for n_nu padded to 128.
#include "df_ladder_gjb.hpp"

namespace df {

DF_GJB_BUILD(128, false, false)

}  // namespace df
