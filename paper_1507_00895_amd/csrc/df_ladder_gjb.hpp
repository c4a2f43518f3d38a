// Batched Bethe-Salpeter ladder, FP64 (kernel templates; instantiated per size
// in df_ladder_gjb_np*.hip): certified pivot-free blocked
// Gauss-Jordan inversion on the FP64 matrix cores (df_gj_core.hpp), for the
// quantities of eqs. (dual_ladder), (lin_alg_inv), the radius rule and the
// second-order term Gamma^(2) = gamma chi gamma of eq. (sd).
//
// The kernel serves the items that the symmetric kernel (df_ladder_sym.hpp) and
// the FP32 ones do not, from two device-side queues:
//   near queue   items of vertices that are not symmetric (certified by the
//                screening kernel), and the refined kernel's items near the
//                instability (certified here): Gauss-Jordan
//   queue        uncertified items, and those of the near queue that fail the
//                certificate here: partial pivoting (df_ladder_pivot.hpp)
// One launch for both: each is empty in most calls.
// One work-group of NP/16 waves per item.  A certified item has rho(M) < 1, i.e. it
// is inside the radius.
#pragma once

#include "df_gj_core.hpp"
#include "df_ladder_pivot.hpp"

namespace df {

constexpr int CERT_ITERS = 6;
constexpr double CERT_MAX_F64 = 0.999;

// Returns false, with no results written, for an uncertified item.
template <int NP>
__device__ __forceinline__ bool gjb_item(LadderArgs a0, int gitem) {
    constexpr int NT = NP / 16;
    typedef MT<double>::v4 d4;
    __shared__ GjShared<double, NP> sh;
    __shared__ cd yv[NP];
    __shared__ cd tv[NP];
    __shared__ int s_flag;

    // an opaque copy of the thread index per item (see df_gj_core.hpp)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int w = tid >> 6;
    const int l = tid & 63;
    const int lj = l & 15;
    const int lg = l >> 4;
    LadderArgs a = a0;
    const int item = resolve_item(a, gitem);   // gitem: global item (fused launches)
    const int n_nu = a.n_nu, N = a.N;
    int q, cm;
    item_coords(a, item, &cm, &q);
    const int im = __builtin_amdgcn_readfirstlane(cm % a.n_om);
    const size_t nn = (size_t)n_nu * n_nu;
    const double *gam = a.gdm + 2 * (size_t)cm * nn;
    const double *pm = a.pdm + 2 * (size_t)cm * nn;
    const double *gtr = a.gtr + 2 * (size_t)cm * nn;

    // ---- t_i = (gamma chi gamma)_ii = sum_j (gamma_ij gamma_ji) chi_j, on its own
    // before the D tiles exist, so its loads do not sit beside them.  Per tile
    // column all loads first and without branches (indices clamped into the
    // matrix, the padding masked afterwards), so that they are in flight together.
    const int nm1 = n_nu - 1;
    {
        cd tp[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) tp[r] = {0.0, 0.0};
#pragma unroll
        for (int tc = 0; tc < NT; ++tc) {
            const int j = 16 * tc + lj;
            const cd xj = ld(a.chi, ((size_t)im * n_nu + clamp_nu<false>(j, nm1)) * N + q);
            cd pv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r)
                pv[r] = ld(pm, (size_t)clamp_nu<false>(16 * w + MT<double>::row(lg, r), nm1) * n_nu + clamp_nu<false>(j, nm1));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * w + MT<double>::row(lg, r);
                const bool in = ((i < n_nu) && (j < n_nu));
                tp[r] = fma_c(tp[r], in ? pv[r] : cd{0.0, 0.0}, xj);
            }
        }
        rows16_sum<true>(tp, sh.Xw[w], tv + 16 * w, tid);
    }

    // ---- D = 1 - gamma diag(chi) in accumulator tiles (opaque column index:
    // the chi loads are not shared with the loop above)
    d4 Cr[NT], Ci[NT];
#pragma unroll
    for (int tc = 0; tc < NT; ++tc) {
        int j = 16 * tc + lj;
        asm volatile("" : "+v"(j));
        const cd xj = ld(a.chi, ((size_t)im * n_nu + clamp_nu<false>(j, nm1)) * N + q);
        cd gv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            gv[r] = ld(gam, (size_t)clamp_nu<false>(16 * w + MT<double>::row(lg, r), nm1) * n_nu + clamp_nu<false>(j, nm1));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * w + MT<double>::row(lg, r);
            const bool in = ((i < n_nu) && (j < n_nu));
            const cd x = gv[r] * xj;
            Cr[tc][r] = (((i == j) ? 1.0 : 0.0) - (in ? x.re : 0.0));
            Ci[tc][r] = (in ? -x.im : 0.0);
        }
    }

    if (!a0.screened) {
        const double cw = gj_certify<double, NP, (NP <= 64)>(Cr, Ci, sh, CERT_ITERS, CERT_MAX_F64, tid);
        if (!(cw < CERT_MAX_F64)) return false;   // uniform over the work-group
    }

    gj_sweep<double, NP>(Cr, Ci, sh, tid);

    if (w == 0) {
        cd ldv;
        const int stt = gj_logdet<NP>(sh.pivv, &ldv, tid);
        if (l == 0) {
            s_flag = stt;
            const size_t o = (size_t)cm * N + q;
            if (a.logdet) st(a.logdet, o, ldv);
            if (a.status) a.status[o] = (int8_t)stt;
            if (stt != 0 && a.fallback_count) atomicAdd(a.fallback_count, 1);
        }
    }
    // ---- Gamma_nn = sum_l (D^-1)_nl gamma_ln  (gamma^T read row-wise); loads
    // per tile column without branches (clamped indices, padding masked).
    // Formed by every wave before the radius test is known (the result is
    // used only inside the radius), so that waves 1.. form it while wave 0
    // forms log det, with one barrier fewer
    {
        // an opaque copy of the row base keeps the compiler from sharing these
        // indices with the identical ones of the D build, which would hold them
        // in registers across the sweep
        int row0 = 16 * w, col0 = lj;
        asm volatile("" : "+v"(row0), "+v"(col0));
        cd yp[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) yp[r] = {0.0, 0.0};
#pragma unroll
        for (int tc = 0; tc < NT; ++tc) {
            const int j = 16 * tc + col0;
            cd gv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r)
                gv[r] = ld(gtr, (size_t)clamp_nu<false>(row0 + MT<double>::row(lg, r), nm1) * n_nu + clamp_nu<false>(j, nm1));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = ((row0 + MT<double>::row(lg, r) < n_nu) && (j < n_nu));
                yp[r] = fma_c(yp[r], cd{Cr[tc][r], Ci[tc][r]}, in ? gv[r] : cd{0.0, 0.0});
            }
        }
        rows16_sum<true>(yp, sh.Xw[w], yv + 16 * w, tid);
    }
    __syncthreads();
    const int stt = s_flag;
    for (int n = tid; n < n_nu; n += NP * 4) {
        const cd tt = tv[n];
        cd wv;
        if (stt == 0) {
            const cd y = yv[n];
            wv = {y.re - 0.5 * tt.re, y.im - 0.5 * tt.im};
        } else {
            const cd gnn = ld(gam, (size_t)n * n_nu + n);
            wv = {gnn.re + 0.5 * tt.re, gnn.im + 0.5 * tt.im};
        }
        st(a.w, ((size_t)cm * n_nu + n) * N + q, wv);
    }
    return true;
}

// rows of threads of the pivoting item with NP * 4 threads (TC columns each)
template <int NP> constexpr int pivot_tc() { return NP <= 64 ? 8 : 16; }

// Both queues, grid-stride; uniform over the work-group, which may run several
// items in turn (LDS is reused: a barrier separates them).
template <int NP>
__device__ __forceinline__ void rest_items(const LadderArgs &a0) {
    const int n_near = a0.near_count ? *a0.near_count : 0, n = n_near + *a0.queue_count;
    for (int u = (int)blockIdx.x; u < n; u += (int)gridDim.x) {
        const int item = __builtin_amdgcn_readfirstlane(u < n_near ? a0.near_queue[u] : a0.queue[u - n_near]);
        bool done = false;
        if (u < n_near) done = gjb_item<NP>(a0, item);
        __syncthreads();
        if (!done) {
            pivot_item<NP, NP * 4 / pivot_tc<NP>(), pivot_tc<NP>()>(a0, item);
            __syncthreads();
        }
    }
}

// Register budget: three waves per SIMD up to NP = 64; the compiler's own at 96
// and 128 (at 96 the capped build spills and measured 6-25 % slower).
template <int NP>
__global__ __launch_bounds__(NP * 4) void k_ladder_rest(LadderArgs a0) {
    rest_items<NP>(a0);
}
template <int NP>
__global__ __launch_bounds__(NP * 4) __attribute__((amdgpu_waves_per_eu(3, 3)))
void k_ladder_rest_o3(LadderArgs a0) {
    rest_items<NP>(a0);
}

template <int NP>
static hipError_t launch_rest(const LadderArgs &a, int grid, hipStream_t s) {
    if constexpr (NP <= 64) hipLaunchKernelGGL(k_ladder_rest_o3<NP>, dim3(grid), dim3(NP * 4), 0, s, a);
    else hipLaunchKernelGGL(k_ladder_rest<NP>, dim3(grid), dim3(NP * 4), 0, s, a);
    return hipGetLastError();
}

// per-size builds (df_ladder_gjb_np*.hip)
#define DF_GJB_DECLARE(NP) hipError_t launch_rest_##NP(const LadderArgs &a, int grid, hipStream_t s);
DF_GJB_DECLARE(16)
DF_GJB_DECLARE(32)
DF_GJB_DECLARE(48)
DF_GJB_DECLARE(64)
DF_GJB_DECLARE(96)
DF_GJB_DECLARE(128)

#define DF_GJB_INSTANTIATE(NP)                                                  \
    hipError_t launch_rest_##NP(const LadderArgs &a, int grid, hipStream_t s) {  \
        return launch_rest<NP>(a, grid, s);                                      \
    }

}  // namespace df
