// FP64 ladder of the queued items: sizes, dispatch to the per-size builds.
#include "df_ladder_gjb.hpp"

namespace df {

int ladder_gjb_padded_size(int n_nu) {
    if (n_nu <= 0) return 0;
    if (n_nu <= 16) return 16;
    if (n_nu <= 32) return 32;
    if (n_nu <= 48) return 48;
    if (n_nu <= 64) return 64;
    if (n_nu <= 96) return 96;
    if (n_nu <= 128) return 128;   // 8 waves; spills a little (one work-group per CU)
    return 0;
}

bool ladder_gjb_has_occ3(int n_nu) {
    const int np = ladder_gjb_padded_size(n_nu);
    return np != 0 && np <= 64;
}

hipError_t launch_ladder_rest(const LadderArgs &a, int grid, hipStream_t s) {
    if (grid <= 0 || !a.queue || !a.queue_count) return hipErrorInvalidValue;
    switch (ladder_gjb_padded_size(a.n_nu)) {
        case 16: return launch_rest_16(a, grid, s);
        case 32: return launch_rest_32(a, grid, s);
        case 48: return launch_rest_48(a, grid, s);
        case 64: return launch_rest_64(a, grid, s);
        case 96: return launch_rest_96(a, grid, s);
        case 128: return launch_rest_128(a, grid, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace df
