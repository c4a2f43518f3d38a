// Batched Bethe-Salpeter ladder, eqs. (dual_ladder) and (lin_alg_inv), with
// the convergence-radius rule that follows them and the second-order term
// Gamma^(2) = gamma chi gamma of eq. (sd).
//
// One work-group per (channel c, bosonic Om_m, momentum q).  The matrix
// D = 1 - gamma^c_m diag(chi_m(q)) (n_nu x n_nu complex, zero-padded to NP
// with an identity block) lives in registers: thread (tr, tc) of a TR x TC
// grid owns rows tr + TR*a and columns tc + TC*b (cyclic).  D is inverted in
// place by Gauss-Jordan elimination with partial pivoting; rows are never
// moved, the pivot rows are recorded instead.  Each step needs two barriers:
//   1. every wave finds the pivot of column k (held in LDS) by a
//      wave-level arg-max; the owners of the pivot row copy their rows to LDS;
//   2. every thread reads the pivot-row values of its columns and the
//      column-k values of its rows and applies the rank-1 update; the owners
//      of column k+1 publish it for the next step.
// With R the in-place result and sigma(k) the pivot row of step k,
// D^-1[k][sigma(j)] = R[sigma(k)][j], so
//   Gamma_nn = (D^-1 gamma)_nn = sum_j R[sigma(n)][j] gamma[sigma(j)][n].
// log det D = sum_k log(pivot_k) + i pi * parity(sigma).
#pragma once

#include "df_internal.hpp"

extern "C" __device__ __attribute__((const)) unsigned int __ockl_wfred_max_u32(unsigned int);

namespace df {

// Pivot-search key: the magnitude rounded to FP32 (whose bit pattern orders
// like the value for non-negative numbers) with its low 8 bits replaced by
// 255 - row, so that the unsigned maximum picks the largest magnitude and,
// among equal magnitudes, the lowest row.  Rows already pivoted get key 0.
__device__ __forceinline__ unsigned pivot_key(double mag, int row) {
    const unsigned bits = __float_as_uint((float)mag);
    return (bits & 0xFFFFFF00u) | (unsigned)(255 - row);
}

// 1 / z of a pivot.  By the hardware reciprocal of |z|^2 (relative error e below 2^-22) and
// one third-order step, y (1 + e + e^2), error e^3; z is scaled by a power of two first, so
// that |z|^2 neither overflows nor underflows for any finite z (chi and gamma may be of any
// size; only near the radius is the matrix near one).  0, infinite and NaN pivots give
// non-finite values.  (The scaling costs 1-3 % of a launch; behind a branch for
// extreme |z|^2 only, 4-7 %.)
__device__ __forceinline__ cd recip_pivot(cd z) {
    const int s = -__builtin_amdgcn_frexp_exp(fmax(fabs(z.re), fabs(z.im)));
    const double a = __builtin_amdgcn_ldexp(z.re, s), b = __builtin_amdgcn_ldexp(z.im, s);
    const double m = fma(a, a, b * b);
    const double y = __builtin_amdgcn_rcp(m);
    const double e = fma(-m, y, 1.0);
    const double inv = fma(y, fma(e, e, e), y);
    return {__builtin_amdgcn_ldexp(a * inv, s), __builtin_amdgcn_ldexp(-b * inv, s)};
}

// One item (gitem: global item) by the TR * TC threads of the work-group.
// Contains barriers; LDS is free again after the caller's next barrier.
template <int NP, int TR, int TC>
__device__ __forceinline__ void pivot_item(const LadderArgs &a0, int gitem) {
    constexpr int NT = TR * TC;
    constexpr int BR = NP / TR;
    constexpr int BC = NP / TC;
    static_assert(BR * TR == NP && BC * TC == NP, "tile");
    static_assert(NP <= 128, "pivot search covers 128 rows");
    static_assert(TC <= 64 && (64 % TC) == 0, "row groups within a wave");

    __shared__ cd colbuf[2][NP];
    __shared__ cd rowblk[NP];
    __shared__ cd pivv[NP];
    __shared__ int prow[NP];
    __shared__ int rowstep[NP];
    __shared__ cd yv[NP];
    __shared__ cd tv[NP];
    __shared__ int s_status;

    // an opaque copy of the thread index per item: the queue's loop over items would hoist
    // the addresses formed from it and hold them
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int tr = tid / TC, tc = tid % TC;
    const int lane = tid & 63;
    LadderArgs a = a0;
    const int item = resolve_item(a, gitem);
    const int n_nu = a.n_nu, N = a.N;
    int q, cm;
    item_coords(a, item, &cm, &q);
    const int im = cm % a.n_om;
    const size_t nn = (size_t)n_nu * n_nu;
    const double *gam = a.gdm + 2 * (size_t)cm * nn;
    const double *pm = a.pdm + 2 * (size_t)cm * nn;

    // ---- build D = 1 - gamma diag(chi) and t_i = sum_j gamma_ij chi_j gamma_ji
    cd chi_j[BC];
#pragma unroll
    for (int b = 0; b < BC; ++b) {
        const int j = tc + TC * b;
        chi_j[b] = (j < n_nu) ? ld(a.chi, ((size_t)im * n_nu + j) * N + q) : cd{0.0, 0.0};
    }
    cd A[BR][BC];
    cd tpart[BR];
#pragma unroll
    for (int ai = 0; ai < BR; ++ai) {
        const int i = tr + TR * ai;
        tpart[ai] = {0.0, 0.0};
#pragma unroll
        for (int b = 0; b < BC; ++b) {
            const int j = tc + TC * b;
            const double d = (i == j) ? 1.0 : 0.0;
            if (i < n_nu && j < n_nu) {
                const cd gij = ld(gam, (size_t)i * n_nu + j);
                const cd x = gij * chi_j[b];
                A[ai][b] = {d - x.re, -x.im};
                tpart[ai] = fma_c(tpart[ai], ld(pm, (size_t)i * n_nu + j), chi_j[b]);
            } else {
                A[ai][b] = {d, 0.0};
            }
        }
    }
    // t_i: reduce over the TC consecutive lanes that share row i
#pragma unroll
    for (int off = TC / 2; off >= 1; off >>= 1) {
#pragma unroll
        for (int ai = 0; ai < BR; ++ai) {
            tpart[ai].re += __shfl_xor(tpart[ai].re, off, 64);
            tpart[ai].im += __shfl_xor(tpart[ai].im, off, 64);
        }
    }
    if (tc == 0) {
#pragma unroll
        for (int ai = 0; ai < BR; ++ai) {
            colbuf[0][tr + TR * ai] = A[ai][0];
            tv[tr + TR * ai] = tpart[ai];
        }
    }
    // the padding is an identity block: its columns are their own pivots and
    // need no elimination step
    for (int k = n_nu + tid; k < NP; k += NT) {
        prow[k] = k;
        rowstep[k] = k;
        pivv[k] = {1.0, 0.0};
    }
    __syncthreads();

    // ---- Gauss-Jordan with partial pivoting
    bool used0 = false, used1 = false;
#pragma unroll
    for (int kk = 0; kk < BC; ++kk) {
        for (int tcol = 0; tcol < TC; ++tcol) {
            const int k = kk * TC + tcol;
            if (k >= n_nu) break;
            const cd *col = colbuf[k & 1];
            // arg-max of |re| + |im| over rows not yet pivoted (lowest index on
            // ties), as one wave-wide unsigned max of packed (magnitude, index) keys
            unsigned key = 0u;
            if (lane < NP && !used0) key = pivot_key(cabs1(col[lane]), lane);
            if (NP > 64 && lane + 64 < NP && !used1) {
                const unsigned k2 = pivot_key(cabs1(col[lane + 64]), lane + 64);
                key = k2 > key ? k2 : key;
            }
            const int p = __builtin_amdgcn_readfirstlane(255 - (int)(__ockl_wfred_max_u32(key) & 255u));
            if (p == lane) used0 = true;
            if (p == lane + 64) used1 = true;
            const cd piv = col[p];
            const cd ip = recip_pivot(piv);
            const int trp = p % TR;
            const int ap = p / TR;
            if (tr == trp) {
#pragma unroll
                for (int ai = 0; ai < BR; ++ai) {
                    if (ai != ap) continue;       // uniform
#pragma unroll
                    for (int b = 0; b < BC; ++b) rowblk[tc + TC * b] = A[ai][b];
                }
            }
            if (tid == 0) {
                prow[k] = p;
                rowstep[p] = k;
                pivv[k] = piv;
            }
            __syncthreads();

            cd r[BC];
#pragma unroll
            for (int b = 0; b < BC; ++b) r[b] = rowblk[tc + TC * b];
            cd f[BR];
#pragma unroll
            for (int ai = 0; ai < BR; ++ai) {
                const int i = tr + TR * ai;
                const cd cv = col[i];
                f[ai] = (i == p) ? cd{1.0 - ip.re, -ip.im} : cv * ip;
            }
#pragma unroll
            for (int b = 0; b < BC; ++b) {
                if (TC * b >= n_nu) break;        // columns of the padding only
#pragma unroll
                for (int ai = 0; ai < BR; ++ai) A[ai][b] = fms(A[ai][b], f[ai], r[b]);
            }
            if (tc == tcol) {
#pragma unroll
                for (int ai = 0; ai < BR; ++ai) {
                    const int i = tr + TR * ai;
                    A[ai][kk] = (i == p) ? ip : cd{-f[ai].re, -f[ai].im};
                }
            }
            if (k + 1 < NP) {
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
            }
            __syncthreads();
        }
    }

    // ---- log det and the convergence-radius test (wave 0)
    if (tid < 64) {
        double lre = 0.0, lim = 0.0;
        int inv = 0;
        for (int k = lane; k < NP; k += 64) {
            const cd pv = pivv[k];
            lre += log(hypot(pv.re, pv.im));
            lim += atan2(pv.im, pv.re);
            const int pk = prow[k];
            for (int j = 0; j < k; ++j) inv += (prow[j] > pk) ? 1 : 0;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            lre += __shfl_xor(lre, off, 64);
            lim += __shfl_xor(lim, off, 64);
            inv += __shfl_xor(inv, off, 64);
        }
        if (lane == 0) {
            double ph = lim + ((inv & 1) ? M_PI : 0.0);
            ph = remainder(ph, 2.0 * M_PI);
            if (ph <= -M_PI) ph += 2.0 * M_PI;
            int stt;
            if (!isfinite(lre) || !isfinite(ph)) stt = 2;
            else stt = (cos(ph) > 0.0) ? 0 : 1;
            s_status = stt;
            const size_t o = (size_t)cm * N + q;
            if (a.logdet) st(a.logdet, o, cd{lre, ph});
            if (a.status) a.status[o] = (int8_t)stt;
            if (stt != 0 && a.fallback_count) atomicAdd(a.fallback_count, 1);
        }
    }
    __syncthreads();
    const int stt = s_status;

    // ---- Gamma_nn: partial sums over this thread's columns, then a
    //      reduction over the TC consecutive lanes sharing the rows
    cd ypart[BR];
#pragma unroll
    for (int ai = 0; ai < BR; ++ai) {
        ypart[ai] = {0.0, 0.0};
        if (stt == 0) {
            const int i = tr + TR * ai;
            const int n = rowstep[i];
            if (n < n_nu) {
#pragma unroll
                for (int b = 0; b < BC; ++b) {
                    const int l = prow[tc + TC * b];
                    if (l < n_nu) ypart[ai] = fma_c(ypart[ai], A[ai][b], ld(gam, (size_t)l * n_nu + n));
                }
            }
        }
    }
#pragma unroll
    for (int off = TC / 2; off >= 1; off >>= 1) {
#pragma unroll
        for (int ai = 0; ai < BR; ++ai) {
            ypart[ai].re += __shfl_xor(ypart[ai].re, off, 64);
            ypart[ai].im += __shfl_xor(ypart[ai].im, off, 64);
        }
    }
    if (tc == 0) {
#pragma unroll
        for (int ai = 0; ai < BR; ++ai) {
            const int i = tr + TR * ai;
            yv[rowstep[i]] = ypart[ai];
        }
    }
    __syncthreads();
    for (int n = tid; n < n_nu; n += NT) {
        const cd t = tv[n];
        cd w;
        if (stt == 0) {
            const cd y = yv[n];
            w = {y.re - 0.5 * t.re, y.im - 0.5 * t.im};
        } else {
            const cd gnn = ld(gam, (size_t)n * n_nu + n);
            w = {gnn.re + 0.5 * t.re, gnn.im + 0.5 * t.im};
        }
        st(a.w, ((size_t)cm * n_nu + n) * N + q, w);
    }
}

// The queue of the uncertified items by `groups` work-groups from the launch's first, in turn.
template <int NP, int TR, int TC>
__device__ __forceinline__ void pivot_queue(const LadderArgs &a0, int groups) {
    const int n = __builtin_amdgcn_readfirstlane(*a0.queue_count);
    for (int u = (int)blockIdx.x; u < n; u += groups) {
        pivot_item<NP, TR, TC>(a0, __builtin_amdgcn_readfirstlane(a0.queue[u]));
        __syncthreads();
    }
}

}  // namespace df
