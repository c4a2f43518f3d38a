// Certified FP64 elimination, build for n_nu padded to 128, screened items.
#include "df_ladder_gjb.hpp"

namespace df {

DF_GJB_BUILD(128, false, true)

}  // namespace df
