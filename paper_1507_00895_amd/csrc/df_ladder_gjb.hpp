// Batched Bethe-Salpeter ladder, FP64 (kernel templates; instantiated per size
// in df_ladder_gjb_np*.hip): certified pivot-free blocked
// Gauss-Jordan inversion on the FP64 matrix cores (df_gj_core.hpp), for the
// quantities of eqs. (dual_ladder), (lin_alg_inv), the radius rule and the
// second-order term Gamma^(2) = gamma chi gamma of eq. (sd).
//
// The kernel serves the items that the symmetric kernel (df_ladder_sym.hpp) and
// the FP32 ones do not:
//   - certified items of vertices that are not symmetric, marked by the screening
//     kernel, which has formed their certificate and Gamma^(2) (SCREENED);
//   - the refined kernel's items near the instability (its near queue);
//   - every item of a launch too small for the screening to pay.
// A certified item has rho(M) < 1, i.e. it is inside the radius; those that fail the
// certificate here take partial pivoting (df_ladder_pivot.hpp).
// Bound: the SIMDs' issue, as df_ladder_sym.hpp.  Non-symmetric vertex, 14,336 items, all
// launches of a call, us at n_nu 16 / 32 / 48 / 64 / 96 / 128:
//   one loop over one queue, 768 work-groups      128 266 478 767 2830 5435
//   here (n_nu 16: k_ladder_all_o3)                52 165 376 681 2094 4808
//   elimination of every item, no screening        58 165 376 675 2242 5055
// In one loop the kernel held the registers of both paths (n_nu 128 190 spilled, 96
// one work-group per CU), and 768 work-groups are one wave each at n_nu 16.
#pragma once

#include "df_gj_core.hpp"
#include "df_ladder_pivot.hpp"

namespace df {

constexpr int CERT_ITERS = 6;
constexpr double CERT_MAX_F64 = 0.999;

// FULL: n_nu equals the padded size NP, so no index is clamped and no padding is
// masked.  SCREENED: certified by the screening kernel, which left Gamma^(2)_nn in W.
// ITEMS > 1: the work-group holds several items, one per slot of NP / 16 waves; all
// slots take every barrier, so an uncertified item is not left early but carried
// through with its results discarded, and `dummy` marks a slot without an item of its
// own, which computes a copy of the last item and writes nothing.
// Returns false, with no results written, for an uncertified item (ITEMS = 1; a slot of
// several queues it).
template <int NP, bool FULL, bool SCREENED, int ITEMS>
__device__ __forceinline__ bool gjb_item(LadderArgs a0, int gitem, bool dummy) {
    constexpr int NT = NP / 16;
    typedef MT<double>::v4 d4;
    __shared__ GjShared<double, NP> shv[ITEMS];
    __shared__ cd yvv[ITEMS][NP];
    __shared__ cd tvv[ITEMS][NP];
    __shared__ int s_flagv[ITEMS];
    // an opaque copy of the thread index per item (see df_gj_core.hpp); the slot is the
    // same for a whole wave
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int slot = ITEMS > 1 ? __builtin_amdgcn_readfirstlane(tid / (NP * 4)) : 0;
    tid -= slot * (NP * 4);
    GjShared<double, NP> &sh = shv[slot];
    cd *yv = yvv[slot];
    cd *tv = tvv[slot];
    int &s_flag = s_flagv[slot];
    const int w = tid >> 6;
    const int l = tid & 63;
    const int lj = l & 15;
    const int lg = l >> 4;
    LadderArgs a = a0;
    const int item = resolve_item(a, gitem);   // gitem: global item (fused launches)
    bool skip = dummy;   // no results of this slot are written
    const int n_nu = FULL ? NP : a.n_nu, N = a.N;
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
    if constexpr (SCREENED) {
        for (int n = tid; n < n_nu; n += NP * 4) tv[n] = ld(a.w, ((size_t)cm * n_nu + n) * N + q);
    } else {
        cd tp[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) tp[r] = {0.0, 0.0};
#pragma unroll
        for (int tc = 0; tc < NT; ++tc) {
            const int j = 16 * tc + lj;
            const cd xj = ld(a.chi, ((size_t)im * n_nu + clamp_nu<FULL>(j, nm1)) * N + q);
            cd pv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r)
                pv[r] = ld(pm, (size_t)clamp_nu<FULL>(16 * w + MT<double>::row(lg, r), nm1) * n_nu + clamp_nu<FULL>(j, nm1));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * w + MT<double>::row(lg, r);
                const bool in = FULL || ((i < n_nu) && (j < n_nu));
                tp[r] = fma_c(tp[r], in ? pv[r] : cd{0.0, 0.0}, xj);
            }
        }
        rows16_sum<ITEMS == 1>(tp, sh.Xw[w], tv + 16 * w, tid);
    }

    // ---- D = 1 - gamma diag(chi) in accumulator tiles (opaque column index:
    // the chi loads are not shared with the loop above)
    d4 Cr[NT], Ci[NT];
#pragma unroll
    for (int tc = 0; tc < NT; ++tc) {
        int j = 16 * tc + lj;
        asm volatile("" : "+v"(j));
        const cd xj = ld(a.chi, ((size_t)im * n_nu + clamp_nu<FULL>(j, nm1)) * N + q);
        cd gv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            gv[r] = ld(gam, (size_t)clamp_nu<FULL>(16 * w + MT<double>::row(lg, r), nm1) * n_nu + clamp_nu<FULL>(j, nm1));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * w + MT<double>::row(lg, r);
            const bool in = FULL || ((i < n_nu) && (j < n_nu));
            const cd x = gv[r] * xj;
            Cr[tc][r] = (((i == j) ? 1.0 : 0.0) - (in ? x.re : 0.0));
            Ci[tc][r] = (in ? -x.im : 0.0);
        }
    }

    if constexpr (!SCREENED) {
        const double cw = gj_certify<double, NP, (NP <= 64)>(Cr, Ci, sh, CERT_ITERS, CERT_MAX_F64, tid,
                                                 ITEMS > 1 ? shv : nullptr, ITEMS > 1 ? ITEMS : 0);
        if (!(cw < CERT_MAX_F64)) {
            if constexpr (ITEMS == 1) return false;   // uniform: every thread of the work-group leaves here
            if (tid == 0 && !dummy) a.queue[atomicAdd(a.queue_count, 1)] = gitem;
            skip = true;
        }
    }

    gj_sweep<double, NP>(Cr, Ci, sh, tid);

    if (w == 0) {
        cd ldv;
        const int stt = gj_logdet<NP>(sh.pivv, &ldv, tid);
        if (l == 0) {
            s_flag = stt;
            const size_t o = (size_t)cm * N + q;
            if (!skip) {
                if (a.logdet) st(a.logdet, o, ldv);
                if (a.status) a.status[o] = (int8_t)stt;
                if (stt != 0 && a.fallback_count) atomicAdd(a.fallback_count, 1);
            }
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
                gv[r] = ld(gtr, (size_t)clamp_nu<FULL>(row0 + MT<double>::row(lg, r), nm1) * n_nu + clamp_nu<FULL>(j, nm1));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = FULL || ((row0 + MT<double>::row(lg, r) < n_nu) && (j < n_nu));
                yp[r] = fma_c(yp[r], cd{Cr[tc][r], Ci[tc][r]}, in ? gv[r] : cd{0.0, 0.0});
            }
        }
        rows16_sum<ITEMS == 1>(yp, sh.Xw[w], yv + 16 * w, tid);
    }
    __syncthreads();
    const int stt = s_flag;
    if (!skip)
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

// Position of work-group b of G in the round that starts at k0, or -1 beyond it.  The rounds
// are dealt to the XCDs in contiguous ranges: neighbouring momenta share cache lines.
__device__ __forceinline__ int round_group(int k0, int groups, int b, int G) {
    const int left = groups - k0, m = left < G ? left : G;
    return b < m ? k0 + xcd_item(b, m) : -1;
}

// The launch's items (ITEMS per work-group) by work-group b of G, in rounds of G; LDS is
// reused: a barrier separates the items.  Uniform over the work-group.
//   SCREENED: those marked CERT_GENERAL, if near_count says that there are any (most calls
//             end there).  The marks of 64 rounds are read at once, one per lane.
//   else:     the near queue.
template <int NP, bool FULL, bool SCREENED, int ITEMS>
__device__ __forceinline__ void gjb_items(const LadderArgs &a0, int b, int G) {
    const int slot = ITEMS > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / (NP * 4)) : 0;
    const int near = __builtin_amdgcn_readfirstlane(*a0.near_count);
    if (near == 0) return;
    const int n = SCREENED ? a0.n_items : near;
    const int groups = (n + ITEMS - 1) / ITEMS;
    auto run = [&](int g) __attribute__((always_inline)) {
        int u = ITEMS * g + slot;
        bool dummy = ITEMS > 1 && u >= n;
        if (dummy) u = n - 1;
        const int item = __builtin_amdgcn_readfirstlane(SCREENED ? a0.item0 + u : a0.near_queue[u]);
        if (SCREENED && ITEMS > 1)
            dummy = dummy || __builtin_amdgcn_readfirstlane((int)a0.cert[item]) != CERT_GENERAL;
        const bool done = gjb_item<NP, FULL, SCREENED, ITEMS>(a0, item, dummy);
        if (!SCREENED && ITEMS == 1 && !done && threadIdx.x == 0) a0.queue[atomicAdd(a0.queue_count, 1)] = item;
        __syncthreads();
    };
    if constexpr (SCREENED) {
        for (int k0 = 0; k0 < groups; k0 += 64 * G) {
            const int k = k0 + (int)(threadIdx.x & 63) * G;
            const int g = k < groups ? round_group(k, groups, b, G) : -1;
            bool mine = false;
            if (g >= 0)
                for (int x = 0; x < ITEMS; ++x)
                    if (ITEMS * g + x < n) mine = mine || a0.cert[a0.item0 + ITEMS * g + x] == CERT_GENERAL;
            // (the same in every wave of the work-group)
            unsigned long long todo = __ballot(mine);
            while (todo) {
                const int j = __builtin_ctzll(todo);
                todo &= todo - 1;
                run(__builtin_amdgcn_readlane(g, j));
            }
        }
    } else {
        for (int k0 = 0; k0 < groups; k0 += G) {
            const int g = round_group(k0, groups, b, G);
            if (g < 0) break;
            run(g);
        }
    }
}

// The near queue; or, SCREENED, the queue of the uncertified items (complete before the
// launch) by its first work-groups and the certified general items by the others.  One
// launch: both are empty in most calls, and where both have items they run side by
// side.  A work-group has one of the two paths, each with its own copy of the thread
// index: neither holds the other's values.
template <int NP, bool FULL, bool SCREENED, int ITEMS>
__device__ __forceinline__ void gjb_kernel(const LadderArgs &a0) {
    constexpr int TC = NP <= 64 ? 8 : 16;
    const int np = SCREENED ? a0.pivot_groups : 0;
    if constexpr (SCREENED)
        if ((int)blockIdx.x < np) {
            pivot_queue<NP, NP * 4 * ITEMS / TC, TC>(a0, np);
            return;
        }
    gjb_items<NP, FULL, SCREENED, ITEMS>(a0, (int)blockIdx.x - np, (int)gridDim.x - np);
}

// Register budget: three waves per SIMD up to NP = 64; the compiler's own at 96
// and 128 (at 96 the capped one-item build spills and measured 6-25 % slower).
// At NP = 96 an item is six waves, and work-groups of one item ran one per CU (1.5 waves
// per SIMD measured); twelve-wave work-groups of two items fill three per SIMD
// (mask-free launches only: the masked build needs more registers).
template <int NP, bool FULL, bool SCREENED>
__global__ __launch_bounds__(NP * 4) void k_ladder_gjb(LadderArgs a0) {
    gjb_kernel<NP, FULL, SCREENED, 1>(a0);
}
template <int NP, bool FULL, bool SCREENED>
__global__ __launch_bounds__(NP * 4) __attribute__((amdgpu_waves_per_eu(3, 3)))
void k_ladder_gjb_o3(LadderArgs a0) {
    gjb_kernel<NP, FULL, SCREENED, 1>(a0);
}
template <int NP, bool FULL, bool SCREENED>
__global__ __launch_bounds__(NP * 8) void k_ladder_gjb_x2(LadderArgs a0) {
    gjb_kernel<NP, FULL, SCREENED, 2>(a0);
}
// Every item of a small launch: an uncertified one is pivoted where it is, in one chain
// and one launch.
template <int NP, bool FULL>
__global__ __launch_bounds__(NP * 4) __attribute__((amdgpu_waves_per_eu(3, 3)))
void k_ladder_all_o3(LadderArgs a0) {
    const int item = a0.item0 + xcd_item(blockIdx.x, gridDim.x);
    if (gjb_item<NP, FULL, false, 1>(a0, item, false)) return;
    __syncthreads();
    pivot_item<NP, NP / 2, 8>(a0, item);
}

// Work-groups of a launch.  The near queue: kQueueWaves at most.  The screened items: four
// times what the device holds at once - in rounds of exactly that, work-groups that
// start late leave places empty (n_nu 32, 14,336 items 210 us, 172 with one work-group per
// item), and work-groups without an item cost a start each (n_nu 96, 188,416 items of
// symmetric vertices: 0.3 ms of 13.4 with one per item pair).  pivot: the queue too, as
// many work-groups as the device holds.
template <int PER, bool SCREENED, typename K>
static hipError_t launch_items(K kern, int threads, LadderArgs a, bool pivot, hipStream_t s) {
    int grid = (a.n_items + PER - 1) / PER;
    a.pivot_groups = 0;
    if constexpr (SCREENED) {
        static const int resident = resident_groups((const void *)kern, threads);
        if (grid > 4 * resident) grid = 4 * resident;
        if (pivot) a.pivot_groups = a.n_items < resident ? a.n_items : resident;
    } else {
        grid = queue_groups(grid, threads);
    }
    hipLaunchKernelGGL(kern, dim3(grid + a.pivot_groups), dim3(threads), 0, s, a);
    return hipGetLastError();
}

// (explicitly instantiated per size and build in df_ladder_gjb_np*.hip: the large ones
// take minutes to compile)
template <int NP, bool FULL, bool SCREENED>
hipError_t launch_gjb(const LadderArgs &a, bool pivot, hipStream_t s) {
    if constexpr (NP <= 64) return launch_items<1, SCREENED>(k_ladder_gjb_o3<NP, FULL, SCREENED>, NP * 4, a, pivot, s);
    else if constexpr (NP == 96 && FULL)
        return launch_items<2, SCREENED>(k_ladder_gjb_x2<NP, FULL, SCREENED>, NP * 8, a, pivot, s);
    else return launch_items<1, SCREENED>(k_ladder_gjb<NP, FULL, SCREENED>, NP * 4, a, pivot, s);
}
template <int NP, bool FULL> hipError_t launch_all(const LadderArgs &a, hipStream_t s) {
    hipLaunchKernelGGL((k_ladder_all_o3<NP, FULL>), dim3(a.n_items), dim3(NP * 4), 0, s, a);
    return hipGetLastError();
}
#define DF_GJB_BUILD_ALL(NP)                                                                \
    template hipError_t launch_all<NP, true>(const LadderArgs &a, hipStream_t s);           \
    template hipError_t launch_all<NP, false>(const LadderArgs &a, hipStream_t s);
#define DF_GJB_BUILD(NP, FULL, SCREENED) \
    template hipError_t launch_gjb<NP, FULL, SCREENED>(const LadderArgs &a, bool pivot, hipStream_t s);

}  // namespace df
