// Batched Bethe-Salpeter ladder, FP64, for vertices that are symmetric in
// their two fermionic frequencies (gamma_nn' = gamma_n'n, time reversal;
// checked on the device by k_gamma_prep): eqs. (dual_ladder), (lin_alg_inv).
//
// Instead of inverting D = 1 - gamma chi and contracting D^-1 gamma, the
// ladder is summed block by block of 16 fermionic frequencies: with S^(0) =
// gamma and S^(t+1) the ladder whose internal lines run over blocks 0..t,
//   S^(t+1) = S^(t) + S^(t)_{:,t} K_t S^(t)_{t,:},
//   K_t = Z_t chi_t,  Z_t = (1 - chi_t S^(t)_tt)^-1,
// so S^(NT) = Gamma.  The matrices 1 - chi_t S^(t)_tt are (transposed) the
// pivot blocks of the blocked elimination of D, so det D is the product of
// their determinants, and the certificate that makes pivot-free elimination of
// D stable (rho(|gamma chi|) < 1) does the same here.  What this saves over the
// inversion:
//   - only Gamma_nn is wanted, so a tile (i, j) is updated at step t only while
//     it is still to be a pivot row or column: max(i, j) > t;
//   - every S^(t) is symmetric, so one tile of each pair is kept;
//   - a finished block (j < t) needs only the diagonal of its update, four
//     complex multiplications per lane of operands already in registers, and
//     the pivot block itself diag(S_tt Z_t); its column takes H = K S_tt =
//     Z_t - 1 without a product;
//   - no separate contraction with gamma at the end, and the vertex is read once.
// Complex 16 x 16 x 16 products per item at NT = 4 / 6 / 8 blocks: 32 / 100 /
// 224, where the inversion makes 60 / 210 / 504.
//
// Measured against the inversion of every item (one work-group of NT waves per
// item), screening included: 2D 32x32, n_nu 64, 63,488 items 2.9 -> 1.65 ms;
// 3D 16^3, n_nu 96, 188,416 items 29.2 -> 13.4 ms; n_nu 128, 6,144 items 2.17 ->
// 0.97 ms; n_nu 80 (six blocks' padding before, five now) 197 -> 51 ns per item.
//
// Bound: the SIMDs' issue.  An FP64 matrix instruction (64 cycles) keeps the
// vector ALU of its SIMD from issuing (measured: a wave of matrix and a wave of
// vector instructions on one SIMD take the sum of their times), so every
// vector instruction of the pivot inversions counts beside the products, and
// independent items per CU are what fills the gaps between the barriers.
//
// Work-group: W waves per item; wave w keeps the tile columns j = w + W u, of
// each the tiles (i, j), i = j + d mod NT, d = 0..NT/2 (at even NT the pairs at
// distance NT/2 belong to columns < NT/2).
// FP64 16x16x4 MFMA lane layouts: the accumulator holds C[i][j] at lane
// j + 16 (i % 4), register i / 4, and the B operand of k-slice r takes B[4r + k][j]
// at lane j + 16 k.  These are the same, and so is the A operand of the
// transposed tile: a tile published to LDS in accumulator order is read back
// as B operand (for H = K S_tj) and as A operand of its transpose (for S_it,
// from S_ti) with the same addresses, and H goes from the accumulator of one
// product into the B operand of the next without leaving its registers.
#pragma once

#include "df_gj_core.hpp"

namespace df {

typedef MT<double>::v4 sd4;

template <int NT> struct SymShared {
    cd P[NT][16][17];         // panel of step t: P[x][k][j] = S_tx[k][j]
    cd K[16][17];             // K_t (symmetric up to rounding: read as its transpose)
    cd xv[16 * NT];           // chi of this item, zero beyond n_nu
    cd pivv[16 * NT];         // reciprocal scalar pivots
    int flag;
};
// LAT (below): S L of the unfinished blocks, K_t (S L)_t of the step
template <int NT> struct SymVectors {
    cd u[16 * (NT > 0 ? NT : 1)];
    cd v[16];
};
template <> struct SymVectors<0> {};

// C += A H with A in operand form A[4r + lg][lj], H as accumulators, in three
// real products per complex one (T1 = A_re H_re, T2 = A_im H_im, C_im += (A_re +
// A_im)(H_re + H_im) - T1 - T2): 12 matrix instructions and about 24 additions
// for 16 matrix instructions.
__device__ __forceinline__ void sym_update(sd4 &Cr, sd4 &Ci, const cd (*A)[17], const sd4 &Hr,
                                           const sd4 &Hi, int lj, int lg) {
    sd4 T1 = {0, 0, 0, 0}, T2 = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const cd a = A[4 * r + lg][lj];
        T1 = MT<double>::mma(a.re, Hr[r], T1);
        T2 = MT<double>::mma(a.im, Hi[r], T2);
        Ci = MT<double>::mma(a.re + a.im, Hr[r] + Hi[r], Ci);
    }
    Cr += T1 - T2;
    Ci -= T1 + T2;
}

// v - 1 on one lane of the wave, in place: the execution mask is narrowed to
// the lane (all lanes are active here), so it costs one vector instruction.
// (s_nop: a DPP read of v needs two wait states after the write, which the
// compiler does not count across inline assembly.)
template <int LANE> __device__ __forceinline__ void lane_minus_one(double &v) {
    unsigned long long keep;
    asm volatile("s_mov_b64 %1, exec\n\t"
                 "s_mov_b64 exec, %2\n\t"
                 "v_add_f64 %0, %0, -1.0\n\t"
                 "s_mov_b64 exec, %1\n\t"
                 "s_nop 1"
                 : "+v"(v), "=&s"(keep)
                 : "s"(1ull << LANE));
}

// 1 / |z|^2 by the hardware reciprocal (relative error e below 2^-22) and one
// third-order step: y (1 + e + e^2), error e^3.
__device__ __forceinline__ double recip_m(double m) {
    const double y = __builtin_amdgcn_rcp(m);
    const double e = fma(-m, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// X <- -X^-1 of one 16 x 16 complex tile held by a wave in accumulator layout, by
// 16 sweeps without pivoting.  Sweep s: with p = x_ss, x_ij <- x_ij - c_i r_j / p
// off the pivot row and column, x_sj <- r_j / p, x_is <- c_i / p, x_ss <- -1 / p.
// With x_ss replaced by p - 1 the first formula gives the second and the third,
// and 1 - 1/p at the pivot: two additions on one lane, where treating the pivot
// row and column apart takes about eight instructions per sweep.  The
// reciprocal pivots go to piv (every lane stores the same value).
template <int S> __device__ __forceinline__ void sym_sweep(sd4 &Xr, sd4 &Xi, cd *piv, int lj) {
    constexpr int LS = S & 3, RS = S >> 2, SRC = S + 16 * LS;
    const cd p = {readlane_v(Xr[RS], SRC), readlane_v(Xi[RS], SRC)};
    double xs = Xr[RS];
    lane_minus_one<SRC>(xs);
    Xr[RS] = xs;
    const int from = (lj + 16 * LS) << 2;
    const cd rr = {bperm_v(from, Xr[RS]), bperm_v(from, Xi[RS])};
    const double y = recip_m(fma(p.re, p.re, p.im * p.im));
    const cd ip = {p.re * y, -p.im * y};
    put_split<double>(piv[S], ip.re, ip.im);
    const cd rp = rr * ip;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const cd c = {row_bcast_v(Xr[r], S), row_bcast_v(Xi[r], S)};
        const cd x = fms(cd{Xr[r], Xi[r]}, c, rp);
        Xr[r] = x.re;
        Xi[r] = x.im;
    }
    xs = Xr[RS];
    lane_minus_one<SRC>(xs);
    Xr[RS] = xs;
    if constexpr (S + 1 < 16) sym_sweep<S + 1>(Xr, Xi, piv, lj);
}

// sum over the four lane groups, returned to all of them
__device__ __forceinline__ cd sum_groups(cd v) {
    v.re += __shfl_xor(v.re, 16, 64);
    v.im += __shfl_xor(v.im, 16, 64);
    v.re += __shfl_xor(v.re, 32, 64);
    v.im += __shfl_xor(v.im, 32, 64);
    return v;
}

// The pivot block: S_tt (accumulators C) is published to P, then replaced by
// H = Z - 1, Z = (1 - chi S)^-1; K = Z chi goes to LDS, diag(S Z) is returned
// (this lane's part: column lj, rows lg + 4r).
__device__ __forceinline__ cd sym_pivot(sd4 &Cr, sd4 &Ci, cd (*P)[17], const cd *x, cd (*K)[17],
                                        cd *piv, int l) {
    const int lj = l & 15, lg = l >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const cd s = {Cr[r], Ci[r]};
        put_split<double>(P[lg + 4 * r][lj], s.re, s.im);
        const cd y = x[lg + 4 * r] * s;
        Cr[r] = ((lj == lg + 4 * r) ? 1.0 : 0.0) - y.re;
        Ci[r] = -y.im;
    }
    sym_sweep<0>(Cr, Ci, piv, lj);
    const cd xj = x[lj];
    cd d = {0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const cd z = {-Cr[r], -Ci[r]};
        d = fma_c(d, P[lg + 4 * r][lj], z);
        const cd k = z * xj;
        put_split<double>(K[lg + 4 * r][lj], k.re, k.im);
        Cr[r] = z.re - ((lj == lg + 4 * r) ? 1.0 : 0.0);
        Ci[r] = z.im;
    }
    return d;
}

// W waves, each with NU tile columns of up to ND tiles.  FULL: n_nu = 16 NT.
// LAT: the lattice observables' ladder term instead, lad = L^T Gamma L (n_om = 1).
// With u = S^(t) L it grows by u_t^T K_t u_t per step, and u_i by S_it K_t u_t, so a
// tile is updated only while both its blocks are unfinished.  W holds gamma L.
template <int NT, int W, bool FULL, bool LAT = false>
__device__ __forceinline__ void sym_item(const LadderArgs &a0, int gitem, const double *L = nullptr,
                                         double *lad = nullptr) {
    constexpr int NP = 16 * NT;
    constexpr int NU = (NT + W - 1) / W;
    constexpr int ND = NT / 2 + 1;
    constexpr bool EVEN = (NT % 2) == 0;
    __shared__ SymShared<NT> sh;
    __shared__ SymVectors<LAT ? NT : 0> vec;
    const int tid = threadIdx.x;
    const int w = W > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    const int l0 = tid & 63;
    // screened by k_ladder_screen: other kernels have the rest.  (The place of the test
    // changes the register allocation: LAT is 1.5 us of 57 faster with it here, the
    // masked ladder builds 0.5 of 60 with it below.)
    if (LAT && __builtin_amdgcn_readfirstlane((int)a0.cert[gitem]) != CERT_SYMMETRIC) return;
    LadderArgs a = a0;
    const int item = resolve_item(a, gitem);
    if (!LAT && __builtin_amdgcn_readfirstlane((int)a.cert[gitem]) != CERT_SYMMETRIC) return;
    const int n_nu = FULL ? NP : a.n_nu, N = a.N;
    int q, cm;
    item_coords(a, item, &cm, &q);
    const int im = __builtin_amdgcn_readfirstlane(cm % a.n_om);
    const size_t nn = (size_t)n_nu * n_nu;
    const double *gs = a.gsym + 2 * (size_t)cm * nn;
    const int nm1 = n_nu - 1;
    auto sync = [&]() __attribute__((always_inline)) {
        if constexpr (W > 1) __syncthreads();
        else wave_sync_lds();
        __builtin_amdgcn_sched_barrier(0);
    };
    // tile (u, d) exists for the columns of slot u (of a pair at distance NT/2
    // one tile is kept); its column and row
    auto col = [&](int u) __attribute__((always_inline)) { return w + W * u; };
    auto has = [&](int u, int d) __attribute__((always_inline)) {
        if ((NT / 2) % W == 0) return !(EVEN && 2 * d == NT && W * u >= NT / 2);   // known per slot
        return !(EVEN && 2 * d == NT && col(u) >= NT / 2);
    };
    auto own = [&](int u) __attribute__((always_inline)) { return NT % W == 0 || col(u) < NT; };
    auto row = [&](int u, int d) __attribute__((always_inline)) {
        const int i = col(u) + d;
        return i >= NT ? i - NT : i;
    };

    for (int j = tid; j < NP; j += 64 * W) {
        const cd x = ld(a.chi, ((size_t)im * n_nu + clamp_nu<FULL>(j, nm1)) * N + q);
        sh.xv[j] = (FULL || j < n_nu) ? x : cd{0.0, 0.0};
        if constexpr (LAT) {
            const cd u = ld(a.w, ((size_t)cm * n_nu + clamp_nu<FULL>(j, nm1)) * N + q);
            vec.u[j] = (FULL || j < n_nu) ? u : cd{0.0, 0.0};
        }
    }
    cd lsum = {0.0, 0.0};    // LAT: this lane's part of lad
    if constexpr (LAT)
        for (int j = tid; j < n_nu; j += 64 * W)
            lsum = fma_c(lsum, ld(L, (size_t)j * N + q), ld(a.w, ((size_t)cm * n_nu + j) * N + q));
    sd4 Cr[NU][ND], Ci[NU][ND];
    {
        const int lj = l0 & 15, lg = l0 >> 4;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (!own(u)) continue;
#pragma unroll
            for (int d = 0; d < ND; ++d) {
                if (!has(u, d)) continue;
                const int i0 = 16 * row(u, d);
                const int j = 16 * col(u) + lj;
                cd g[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    g[r] = ld(gs, (size_t)clamp_nu<FULL>(i0 + lg + 4 * r, nm1) * n_nu + clamp_nu<FULL>(j, nm1));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool in = FULL || ((i0 + lg + 4 * r < n_nu) && (j < n_nu));
                    Cr[u][d][r] = in ? g[r].re : 0.0;
                    Ci[u][d][r] = in ? g[r].im : 0.0;
                }
            }
        }
    }
    sync();
    cd dacc[NU];     // Gamma_nn of the finished blocks, this lane's part, per column
#pragma unroll
    for (int u = 0; u < NU; ++u) dacc[u] = {0.0, 0.0};
#pragma unroll
    for (int ut = 0; ut < NU; ++ut)
#pragma unroll 1
    for (int wt = 0; wt < (ut + 1 < NU ? W : NT - W * ut); ++wt) {
        const int t = W * ut + wt;                // pivot block: slot ut of wave wt
        cd (*P)[16][17] = sh.P;
        const cd (*K)[17] = sh.K;
        // an opaque copy of the lane index per step, so that the LDS addresses
        // of the step are formed where they are used instead of being hoisted
        // out of the loop and held in registers
        int l = l0;
        asm volatile("" : "+v"(l));
        const int lj = l & 15, lg = l >> 4;
        // ---- the pivot block, and the rest of the panel S_tx
        if (w == wt)
            dacc[ut] = sym_pivot(Cr[ut][0], Ci[ut][0], P[t], sh.xv + 16 * t, sh.K, sh.pivv + 16 * t, l);
        if constexpr (LAT) {
            if (w == wt) {
                // v = K u_t (column sums of K, symmetric), lad += u_t^T v
                cd v = {0.0, 0.0};
#pragma unroll
                for (int r = 0; r < 4; ++r) v = fma_c(v, K[lg + 4 * r][lj], vec.u[16 * t + lg + 4 * r]);
                v = sum_groups(v);
                if (lg == 0) {
                    vec.v[lj] = v;
                    lsum = fma_c(lsum, vec.u[16 * t + lj], v);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int d = 1; d < ND; ++d) {
                if (!has(u, d) || !own(u)) continue;
                if (u == ut && w == wt) {
                    // the wave holds S_it: transposed
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        put_split<double>(P[row(u, d)][lj][lg + 4 * r], Cr[u][d][r], Ci[u][d][r]);
                } else if (row(u, d) == t) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        put_split<double>(P[col(u)][lg + 4 * r][lj], Cr[u][d][r], Ci[u][d][r]);
                }
            }
        if (NT == 1) break;
        sync();
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (!own(u)) continue;
            const int j = col(u);
            if constexpr (LAT) {
                if (j <= t) continue;             // finished
                cd du = {0.0, 0.0};
#pragma unroll
                for (int r = 0; r < 4; ++r) du = fma_c(du, P[j][4 * r + lg][lj], vec.v[4 * r + lg]);
                du = sum_groups(du);
                if (lg == 0) vec.u[16 * j + lj] = vec.u[16 * j + lj] + du;
            }
            __builtin_amdgcn_sched_barrier(0);
            sd4 Hr, Hi;
            if (u == ut && w == wt) {
                Hr = Cr[u][0];                    // Z - 1
                Hi = Ci[u][0];
            } else {
                // ---- H = K S_tj (three real products per complex one)
                cd b[4];
                sd4 T1 = {0, 0, 0, 0}, T2 = {0, 0, 0, 0}, T3 = {0, 0, 0, 0};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const cd k = K[4 * r + lg][lj];
                    b[r] = P[j][4 * r + lg][lj];
                    T1 = MT<double>::mma(k.re, b[r].re, T1);
                    T2 = MT<double>::mma(k.im, b[r].im, T2);
                    T3 = MT<double>::mma(k.re + k.im, b[r].re + b[r].im, T3);
                }
                Hr = T1 - T2;
                Hi = T3 - T1 - T2;
                if (j < t) {
                    // finished block: the diagonal of S_jt H only
#pragma unroll
                    for (int r = 0; r < 4; ++r) dacc[u] = fma_c(dacc[u], b[r], cd{Hr[r], Hi[r]});
                } else {
                    __builtin_amdgcn_sched_barrier(0);
                    sym_update(Cr[u][0], Ci[u][0], P[j], Hr, Hi, lj, lg);
                }
            }
#pragma unroll
            for (int d = 1; d < ND; ++d) {
                if (!has(u, d)) continue;
                const int i = row(u, d);
                __builtin_amdgcn_sched_barrier(0);   // one tile's operands at a time
                if (LAT ? i > t : (i > t || j > t)) sym_update(Cr[u][d], Ci[u][d], P[i], Hr, Hi, lj, lg);
            }
        }
        if (t + 1 < NT) sync();   // the panel and K are free
    }
    sync();
    if constexpr (LAT) {
        lsum.re = wave_sum(lsum.re);
        lsum.im = wave_sum(lsum.im);
        if (l0 == 0) sh.xv[w] = lsum;
        sync();
        if (tid == 0) {
            cd r = sh.xv[0];
            for (int x = 1; x < W; ++x) r = r + sh.xv[x];
            st(lad, (size_t)cm * N + q, r);
        }
        return;
    }
    // t_n = (gamma chi gamma)_nn was left in W by the screening kernel.  Up to four
    // blocks it is loaded here, to arrive while log det is formed; the larger builds
    // have no registers for it (n_nu 48 13.2 -> 12.6 ns per item, 96 76 -> 81)
    constexpr bool EARLY = NT <= 4;
    cd tn[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int n = 16 * col(u) + (l0 & 15);
        if (EARLY) tn[u] = ld(a.w, ((size_t)cm * n_nu + clamp_nu<false>(n, nm1)) * N + q);
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) dacc[u] = sum_groups(dacc[u]);
    if (w == 0) {
        // det D = 1 / (the product of the reciprocal pivots): the signs of the
        // real parts agree, log and phase change sign (phase kept in (-pi, pi])
        cd ldv;
        const int stt = gj_logdet<NP>(sh.pivv, &ldv, tid);
        if (l0 == 0) {
            sh.flag = stt;
            const size_t o = (size_t)cm * N + q;
            if (a.logdet) st(a.logdet, o, cd{-ldv.re, ldv.im == M_PI ? ldv.im : -ldv.im});
            if (a.status) a.status[o] = (int8_t)stt;
            if (stt != 0 && a.fallback_count) atomicAdd(a.fallback_count, 1);
        }
    }
    sync();
    const int stt = sh.flag;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int n = 16 * col(u) + (l0 & 15);
        if (l0 < 16 && n < n_nu) {
            const size_t o = ((size_t)cm * n_nu + n) * N + q;
            if (!EARLY) tn[u] = ld(a.w, o);
            cd wv = {dacc[u].re - 0.5 * tn[u].re, dacc[u].im - 0.5 * tn[u].im};
            if (stt != 0) {
                const cd gnn = ld(gs, (size_t)n * n_nu + n);
                wv = {gnn.re + 0.5 * tn[u].re, gnn.im + 0.5 * tn[u].im};
            }
            st(a.w, o, wv);
        }
    }
}

}  // namespace df
