// Symmetric FP64 ladder: builds for one to eight 16-row blocks, dispatch.
#include "df_ladder_sym.hpp"
#include "df_lattice_ladder.hpp"

namespace df {

// Waves per item and waves per SIMD of the build for NT 16-row blocks.  Two tile
// columns per wave: fewer waves per item leave more items on a CU at the same
// registers, and only one wave of an item works while a pivot block is
// inverted (n_nu 64: four waves of one column 36 ns per item, two of two columns
// 26; n_nu 96: 150 and 82; n_nu 128: 186 and 178).  At NT <= 3 one wave holds the
// whole item, without barriers (n_nu 48: 13 ns; two waves 16, three 18).  At
// NT = 6 three waves per SIMD spill 69 registers a lane and are still faster
// than two without spills (82 against 107 ns).
template <int NT> struct SymBuild;
#define DF_SYM_BUILD(NT, W_, EU_) template <> struct SymBuild<NT> { static constexpr int W = W_, EU = EU_; };
DF_SYM_BUILD(1, 1, 4)
DF_SYM_BUILD(2, 1, 3)
DF_SYM_BUILD(3, 1, 2)
DF_SYM_BUILD(4, 2, 3)
DF_SYM_BUILD(5, 3, 3)
DF_SYM_BUILD(6, 3, 3)
DF_SYM_BUILD(7, 4, 2)
DF_SYM_BUILD(8, 4, 2)

template <int NT, bool FULL>
__global__ __launch_bounds__(64 * SymBuild<NT>::W)
__attribute__((amdgpu_waves_per_eu(SymBuild<NT>::EU, SymBuild<NT>::EU)))
void k_ladder_sym(LadderArgs a0) {
    sym_item<NT, SymBuild<NT>::W, FULL>(a0, a0.item0 + xcd_item(blockIdx.x, gridDim.x));
}

template <int NT> static hipError_t launch_nt(const LadderArgs &a, hipStream_t s) {
    const dim3 grid(a.n_items), block(64 * SymBuild<NT>::W);
    if (a.full_sym) hipLaunchKernelGGL((k_ladder_sym<NT, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_ladder_sym<NT, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_ladder_sym(const LadderArgs &a, hipStream_t s) {
    if (a.n_items <= 0) return hipErrorInvalidValue;
    switch ((a.n_nu + 15) / 16) {
        case 1: return launch_nt<1>(a, s);
        case 2: return launch_nt<2>(a, s);
        case 3: return launch_nt<3>(a, s);
        case 4: return launch_nt<4>(a, s);
        case 5: return launch_nt<5>(a, s);
        case 6: return launch_nt<6>(a, s);
        case 7: return launch_nt<7>(a, s);
        case 8: return launch_nt<8>(a, s);
        default: return hipErrorInvalidValue;
    }
}

// The lattice observables' ladder term (LAT)
template <int NT>
__global__ __launch_bounds__(64 * SymBuild<NT>::W)
__attribute__((amdgpu_waves_per_eu(SymBuild<NT>::EU, SymBuild<NT>::EU)))
void k_lattice_sym(LadderArgs a0, const double *L, double *lad) {
    sym_item<NT, SymBuild<NT>::W, false, true>(a0, xcd_item(blockIdx.x, gridDim.x), L, lad);
}

hipError_t launch_lattice_sym(const LadderArgs &a, const double *L, double *lad, hipStream_t s) {
    if (a.n_items <= 0) return hipErrorInvalidValue;
    switch ((a.n_nu + 15) / 16) {
#define DF_SYM(NT)                                                                                          \
    case NT:                                                                                                \
        hipLaunchKernelGGL(k_lattice_sym<NT>, dim3(a.n_items), dim3(64 * SymBuild<NT>::W), 0, s, a, L, lad); \
        break;
        DF_SYM(1) DF_SYM(2) DF_SYM(3) DF_SYM(4) DF_SYM(5) DF_SYM(6) DF_SYM(7) DF_SYM(8)
#undef DF_SYM
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace df
