// Lattice observables of a dual solution (Sec. 2.3, "Resulting observables").
//
//   k_lattice_fields      per (nu, k): G~0, G~ (eqs. gd0, dyson), Sigma_lat (eq. sigma_lat,
//                         denominator 1 + g Sigma~), G_lat (eq. glat, in a form free of
//                         cancellation), frak G = G~ (G~0 + g) / G~0
//   (k_dual_gf / k_bubble of df_fft_kernels.hip turn frak G, G_lat and G~ into
//    L_nu(q), the per-nu lattice bubble and chi~ at Omega = 0, the three in one
//    launch each)
//   ladder term           per (channel, q): sum_{nu nu'} L_nu Gamma_{nu nu'} L_nu' with
//                         Gamma = [1 - gamma chi~]^-1 gamma at Omega = 0: certified items
//                         of symmetric vertices in the block ladder of
//                         df_ladder_sym.hpp, the rest here (k_lattice_rest) by
//                         Gauss-Jordan with partial pivoting of [D | gamma L] in registers
//   k_lattice_chi_sum     chi^{ch/sp}(q) = sum_nu bubble_nu(q) + ladder term
//
// 32x32, n_nu 64, 2,048 items: 95 us per call, of it 62 the block ladder (bound by
// the issue of its pivot inversions, df_ladder_sym.hpp); 1219 us with eliminations of
// all items on matrices in global memory (four launches of 288 us), one transform
// and one bubble launch per field and one thread per momentum in the final sum.
#include "df_lattice_ladder.hpp"
#include "df_ladder_pivot.hpp"

namespace df {

// ------------------------------------------------------------------------
// One block per fermionic frequency n (nu_n = (2n + 1 - n_nu) pi / beta).
// ------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_lattice_fields(LatticeFieldArgs a) {
    const int n = blockIdx.x;
    const cd gn = ld(a.g, n), dn = ld(a.delta, n);
    const cd ginv = recip(gn);
    const double nu = (double)(2 * n + 1 - a.n_nu) * M_PI / a.beta;
    // Sigma^DMFT = i nu + mu - Delta - 1/g
    const cd sdmft = {a.mu - dn.re - ginv.re, nu - dn.im - ginv.im};
    const cd one = {1.0, 0.0};
    for (int k = threadIdx.x; k < a.N; k += blockDim.x) {
        const size_t e = (size_t)n * a.N + k;
        const cd dme = {dn.re - a.eps[k], dn.im};        // Delta - eps
        const cd G0 = recip(ginv + dme) - gn;
        const cd S = a.sigma ? ld(a.sigma, e) : cd{0.0, 0.0};
        const cd G = cdiv(G0, fms(one, G0, S));
        // eq. (glat) with G~ from eqs. (gd0), (dyson) is g (1 + g S) / (1 + g (Delta - eps)(1 + g S)):
        // the same value without the cancellation of its two terms where Delta - eps is small
        const cd h = fma_c(one, gn, S);                   // 1 + g S
        const cd Gl = cdiv(gn * h, fma_c(one, gn * dme, h));
        if (a.sigma_lat) st(a.sigma_lat, e, cdiv(S, fma_c(one, gn, S)) + sdmft);
        if (a.g_lat) st(a.g_lat, e, Gl);
        st(a.gl, e, Gl);
        st(a.gd, e, G);
        st(a.fg, e, cdiv(G * (G0 + gn), G0));
    }
}

// ------------------------------------------------------------------------
// lad = L^T z, D z = y, D = 1 - gamma diag(chi~), y = gamma L (left in W by the
// screening kernel) of the queued items: Gauss-Jordan with partial pivoting as in
// pivot_item (df_ladder_pivot.hpp), the matrix spread cyclically over the
// registers of TR x TC threads, but only the columns right of the pivot are
// updated, and y with them.  Rows are never moved: z_k is y of the row that was
// the pivot of column k, divided by the pivot.
// ------------------------------------------------------------------------
template <int NP, int TR, int TC>
__global__ __launch_bounds__(TR *TC) void k_lattice_rest(LadderArgs a, const double *L, double *lad) {
    constexpr int NT = TR * TC, BR = NP / TR, BC = NP / TC;
    __shared__ cd colbuf[2][NP];
    __shared__ cd rowblk[BR][NP];
    __shared__ cd yv[NP];
    __shared__ int prow[NP];
    __shared__ cd ipv[NP];
    __shared__ cd red[NT / 64];
    const int tid = threadIdx.x, tr = tid / TC, tc = tid % TC, lane = tid & 63;
    const int n = a.n_nu, N = a.N;
    const int n_all = *a.queue_count;
    for (int wi = blockIdx.x; wi < n_all; wi += gridDim.x) {
        const int item = a.queue[wi];
        const int c = item / N, q = item % N;
        // the matrix that the screening kernel took for y = gamma L: with another one here, D and
        // y of a symmetrised vertex differ by its antisymmetric part in first order
        const bool sym = vertex_symmetric(a.symp, n, c, lane);
        const double *gam = (sym ? a.gsym : a.gdm) + 2 * (size_t)c * n * n;
        cd A[BR][BC];
#pragma unroll
        for (int b = 0; b < BC; ++b) {
            const int j = tc + TC * b;
            const cd x = j < n ? ld(a.chi, (size_t)j * N + q) : cd{0.0, 0.0};
#pragma unroll
            for (int ai = 0; ai < BR; ++ai) {
                const int i = tr + TR * ai;
                const double d = (i == j) ? 1.0 : 0.0;
                A[ai][b] = {d, 0.0};
                if (i < n && j < n) {
                    const cd g = ld(gam, (size_t)i * n + j) * x;
                    A[ai][b] = {d - g.re, -g.im};
                }
            }
        }
        for (int i = tid; i < NP; i += NT) yv[i] = i < n ? ld(a.w, ((size_t)c * n + i) * N + q) : cd{0.0, 0.0};
        if (tc == 0) {
#pragma unroll
            for (int ai = 0; ai < BR; ++ai) colbuf[0][tr + TR * ai] = A[ai][0];
        }
        __syncthreads();
        bool used0 = false, used1 = false;
#pragma unroll
        for (int kk = 0; kk < BC; ++kk) {
            for (int tcol = 0; tcol < TC; ++tcol) {
                const int k = kk * TC + tcol;
                if (k >= n) break;
                const cd *col = colbuf[k & 1];
                unsigned key = 0u;
                if (lane < NP && !used0) key = pivot_key(cabs1(col[lane]), lane);
                if (NP > 64 && lane + 64 < NP && !used1) {
                    const unsigned k2 = pivot_key(cabs1(col[lane + 64]), lane + 64);
                    key = k2 > key ? k2 : key;
                }
                const int p = 255 - (int)(__ockl_wfred_max_u32(key) & 255u);
                if (p == lane) used0 = true;
                if (p == lane + 64) used1 = true;
                const cd ip = recip(col[p]);
                if (tr == p % TR) {
#pragma unroll
                    for (int ai = 0; ai < BR; ++ai)
#pragma unroll
                        for (int b = kk; b < BC; ++b) rowblk[ai][tc + TC * b] = A[ai][b];
                }
                if (tid == 0) {
                    prow[k] = p;
                    ipv[k] = ip;
                }
                const cd yp = yv[p] * ip;
                __syncthreads();
                cd f[BR];
#pragma unroll
                for (int ai = 0; ai < BR; ++ai) {
                    const int i = tr + TR * ai;
                    f[ai] = (i == p) ? cd{0.0, 0.0} : col[i] * ip;
                }
#pragma unroll
                for (int b = kk; b < BC; ++b) {
                    const cd r = rowblk[p / TR][tc + TC * b];
#pragma unroll
                    for (int ai = 0; ai < BR; ++ai) A[ai][b] = fms(A[ai][b], f[ai], r);
                }
                // (the pivot row stays as it is, in the matrix and in y)
                for (int i = tid; i < n; i += NT)
                    if (i != p) yv[i] = fms(yv[i], col[i], yp);
                cd *nxt = colbuf[(k + 1) & 1];
                if (tcol + 1 < TC) {
                    if (tc == tcol + 1) {
#pragma unroll
                        for (int ai = 0; ai < BR; ++ai) nxt[tr + TR * ai] = A[ai][kk];
                    }
                } else if (kk + 1 < BC) {
                    if (tc == 0) {
#pragma unroll
                        for (int ai = 0; ai < BR; ++ai) nxt[tr + TR * ai] = A[ai][kk + 1 < BC ? kk + 1 : kk];
                    }
                }
                __syncthreads();
            }
        }
        cd s = {0.0, 0.0};
        for (int k = tid; k < n; k += NT) s = fma_c(s, ld(L, (size_t)k * N + q), yv[prow[k]] * ipv[k]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            s.re += __shfl_xor(s.re, off, 64);
            s.im += __shfl_xor(s.im, off, 64);
        }
        if (lane == 0) red[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) {
            cd r = red[0];
            for (int x = 1; x < NT / 64; ++x) r = r + red[x];
            st(lad, (size_t)c * N + q, r);
        }
        __syncthreads();
    }
}

// chi_c(q) = sum_nu bubble[nu][q] + lad[c][q]; 64 momenta per block, four threads
// each, fixed order.
__global__ __launch_bounds__(256) void k_lattice_chi_sum(LatticeSumArgs a) {
    __shared__ cd red[4][64];
    const int x = threadIdx.x & 63, p = threadIdx.x >> 6;
    const int q = blockIdx.x * 64 + x;
    cd s = {0.0, 0.0};
    if (q < a.N)
        for (int n = p; n < a.n_nu; n += 4) s = s + ld(a.bub, (size_t)n * a.N + q);
    red[p][x] = s;
    __syncthreads();
    if (p != 0 || q >= a.N) return;
    s = (red[0][x] + red[1][x]) + (red[2][x] + red[3][x]);
    if (a.chi_ch) st(a.chi_ch, q, s + ld(a.lad, q));
    if (a.chi_sp) st(a.chi_sp, q, s + ld(a.lad, (size_t)a.N + q));
}

hipError_t launch_lattice_fields(const LatticeFieldArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_lattice_fields, dim3(a.n_nu), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_lattice_rest(const LadderArgs &a, const double *L, double *lad, hipStream_t s) {
    if (a.n_items <= 0 || !a.queue || !a.queue_count) return hipErrorInvalidValue;
#define DF_REST(NP, TR, TC)                                                                              \
    hipLaunchKernelGGL((k_lattice_rest<NP, TR, TC>), dim3(queue_groups(a.n_items, TR * TC)), dim3(TR * TC), 0, s, a, L, lad)
    switch (ladder_padded_size(a.n_nu)) {
        case 16: DF_REST(16, 8, 8); break;
        case 32: DF_REST(32, 8, 8); break;
        case 48: DF_REST(48, 16, 16); break;
        case 64: DF_REST(64, 16, 16); break;
        case 96: DF_REST(96, 32, 16); break;
        case 128: DF_REST(128, 32, 16); break;
        default: return hipErrorInvalidValue;
    }
#undef DF_REST
    return hipGetLastError();
}

hipError_t launch_lattice_chi_sum(const LatticeSumArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_lattice_chi_sum, dim3((a.N + 63) / 64), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace df
