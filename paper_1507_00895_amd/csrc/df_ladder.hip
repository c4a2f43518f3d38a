// FP64 ladder with partial pivoting (df_ladder_pivot.hpp): every item (the tuner's
// "vector" choice), or the queue of the items that the certified kernels leave.
#include "df_ladder_pivot.hpp"

namespace df {

template <int NP, int TR, int TC>
__global__ __launch_bounds__(TR *TC) void k_ladder_fp64(LadderArgs a0) {
    pivot_item<NP, TR, TC>(a0, a0.item0 + xcd_item(blockIdx.x, gridDim.x));
}

// (n_nu 64: 130 registers without the cap, two too many for four waves per SIMD)
template <int NP, int TR, int TC>
__global__ __launch_bounds__(TR *TC) __attribute__((amdgpu_waves_per_eu(NP <= 64 ? 4 : 2)))
void k_ladder_fp64_queue(LadderArgs a0) {
    pivot_queue<NP, TR, TC>(a0, gridDim.x);
}

int ladder_padded_size(int n_nu) {
    if (n_nu <= 0) return 0;
    if (n_nu <= 16) return 16;
    if (n_nu <= 32) return 32;
    if (n_nu <= 48) return 48;
    if (n_nu <= 64) return 64;
    if (n_nu <= 96) return 96;
    if (n_nu <= 128) return 128;
    return 0;
}

template <int NP, int TR, int TC>
static hipError_t launch_one(const LadderArgs &a, hipStream_t s) {
    // split huge batches so gridDim.x stays well inside its limit
    const int chunk = 1 << 30;
    for (int off = 0; off < a.n_items; off += chunk) {
        LadderArgs b = a;
        b.item0 = a.item0 + off;
        const int cnt = (a.n_items - off < chunk) ? a.n_items - off : chunk;
        hipLaunchKernelGGL((k_ladder_fp64<NP, TR, TC>), dim3(cnt), dim3(TR * TC), 0, s, b);
    }
    return hipGetLastError();
}

template <int NP, int TR, int TC>
static hipError_t launch_queue(const LadderArgs &a, hipStream_t s) {
    const int grid = queue_groups(a.n_items, TR * TC);
    hipLaunchKernelGGL((k_ladder_fp64_queue<NP, TR, TC>), dim3(grid), dim3(TR * TC), 0, s, a);
    return hipGetLastError();
}

#define DF_PIVOT_SIZES(LAUNCH)                                                  \
    switch (ladder_padded_size(a.n_nu)) {                                       \
        case 16: return LAUNCH<16, 8, 8>(a, s);                                 \
        case 32: return LAUNCH<32, 8, 8>(a, s);                                 \
        case 48: return LAUNCH<48, 24, 8>(a, s);                                \
        case 64: return LAUNCH<64, 32, 8>(a, s);                                \
        case 96: return LAUNCH<96, 16, 16>(a, s);                               \
        case 128: return LAUNCH<128, 32, 16>(a, s);                             \
        default: return hipErrorInvalidValue;                                   \
    }
hipError_t launch_ladder_fp64(const LadderArgs &a, hipStream_t s) { DF_PIVOT_SIZES(launch_one) }
hipError_t launch_ladder_fp64_queue(const LadderArgs &a, hipStream_t s) {
    if (a.n_items <= 0 || !a.queue || !a.queue_count) return hipErrorInvalidValue;
    DF_PIVOT_SIZES(launch_queue)
}

}  // namespace df
