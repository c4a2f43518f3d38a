// Certified FP64 elimination: sizes, dispatch to the per-size builds.
#include "df_internal.hpp"

namespace df {

// df_ladder_gjb.hpp
template <int NP, bool FULL, bool SCREENED> hipError_t launch_gjb(const LadderArgs &a, bool pivot, hipStream_t s);
template <int NP, bool FULL> hipError_t launch_all(const LadderArgs &a, hipStream_t s);
template <int NP> static hipError_t launch_size(const LadderArgs &a, bool screened, bool pivot, hipStream_t s) {
    if (a.full) return screened ? launch_gjb<NP, true, true>(a, pivot, s) : launch_gjb<NP, true, false>(a, false, s);
    return screened ? launch_gjb<NP, false, true>(a, pivot, s) : launch_gjb<NP, false, false>(a, false, s);
}

int resident_groups(const void *kern, int threads) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, threads, 0) != hipSuccess || per < 1) per = 1;
    (void)hipGetLastError();
    return cus * per;
}

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

static hipError_t launch_sizes(const LadderArgs &a, bool screened, bool pivot, hipStream_t s) {
    switch (ladder_gjb_padded_size(a.n_nu)) {
        case 16: return launch_size<16>(a, screened, pivot, s);
        case 32: return launch_size<32>(a, screened, pivot, s);
        case 48: return launch_size<48>(a, screened, pivot, s);
        case 64: return launch_size<64>(a, screened, pivot, s);
        case 96: return launch_size<96>(a, screened, pivot, s);
        case 128: return launch_size<128>(a, screened, pivot, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_ladder_gjb(const LadderArgs &a, hipStream_t s) {
    if (a.n_items <= 0 || !a.queue || !a.queue_count || !a.near_queue || !a.near_count)
        return hipErrorInvalidValue;
    return launch_sizes(a, false, false, s);
}

hipError_t launch_ladder_all(const LadderArgs &a, hipStream_t s) {
    if (a.n_items <= 0) return hipErrorInvalidValue;
    switch (ladder_gjb_padded_size(a.n_nu)) {
        case 16: return a.full ? launch_all<16, true>(a, s) : launch_all<16, false>(a, s);
        case 32: return a.full ? launch_all<32, true>(a, s) : launch_all<32, false>(a, s);
        case 48: return a.full ? launch_all<48, true>(a, s) : launch_all<48, false>(a, s);
        case 64: return a.full ? launch_all<64, true>(a, s) : launch_all<64, false>(a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_ladder_rest(const LadderArgs &a, hipStream_t s) {
    if (a.n_items <= 0 || !a.queue || !a.queue_count || !a.cert) return hipErrorInvalidValue;
    // The pivoting of a long queue at n_nu 66..96 is a launch of its own, on the thread grid
    // that is best for it alone (256 threads; 384 or 768 here): 6,144 items, half of
    // them uncertified, n_nu 80 / 96 1684 / 1629 us against 1921 / 1847 in one launch; 512
    // items 264 / 282 against 201 / 185, where the two run side by side.
    const bool pivot = ladder_gjb_padded_size(a.n_nu) != 96 || a.n_items <= 2048;
    const hipError_t e = launch_sizes(a, true, pivot, s);
    return e != hipSuccess || pivot ? e : launch_ladder_fp64_queue(a, s);
}

}  // namespace df
