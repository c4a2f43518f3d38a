// Bandwidth-bound steps of the ladder dual-fermion iteration:
//   eq. (gd0) + eq. (dyson)     k_dual_gf      (fused with the inverse FFT of G~)
//   eq. (dual_bubble)           k_bubble       (pair product + forward FFT in LDS)
//   eq. (sd)                    k_sigma_part   (inverse FFT of V, reflected product,
//                                               accumulation over a chunk of Om,
//                                               forward FFT)
//   reduction over Om chunks, linear mixing, Frobenius norms (deterministic order)
//   eq. (spin_symm)             k_gamma_prep   (gamma^{d,m} and gamma_ij gamma_ji)
//
// Every FFT works on one N-point array (N = nk^D <= 4096), one work-group per
// array, in register passes with LDS between them (df_fft.hpp); the kernels are
// built per grid shape (D, nk).
#include "df_fft.hpp"
#include "df_internal.hpp"

namespace df {

// ------------------------------------------------------------------------
// G~ = G~0 / (1 - G~0 Sigma~),  G~0 = 1 / (1/g + Delta - eps) - g.
// One block per fermionic frequency n.  Writes gd[n][k] (if gd_out) and
// the inverse FFT gr[n][r] = (1/N) sum_k e^{ikr} G~(k) (if gr_out).
// With from_gd set, G~ is read from gd instead of being computed.
// ------------------------------------------------------------------------
template <typename P>
__global__ __launch_bounds__(P::T) void k_dual_gf(DualGfArgs a) {
    __shared__ cd X[P::LDS_N];
    __shared__ cd tw[P::nk];
    const int n = blockIdx.x;
    cd ginv = {0, 0}, gn = {0, 0}, dn = {0, 0};
    if (!a.from_gd) {
        gn = ld(a.g, n);
        dn = ld(a.delta, n);
        ginv = recip(gn);
    }
    auto value = [&](int k) __attribute__((always_inline)) {
        const size_t e = (size_t)n * P::N + k;
        if (a.from_gd) return ld(a.gd_in, e);
        const cd den = {ginv.re + dn.re - a.eps[k], ginv.im + dn.im};
        const cd G0 = recip(den) - gn;
        cd G = G0;
        if (a.sigma) G = cdiv(G0, fms(cd{1.0, 0.0}, G0, ld(a.sigma, e)));
        if (a.gd_out) st(a.gd_out, e, G);
        return G;
    };
    if (!a.gr_out) {
        for (int k = threadIdx.x; k < P::N; k += P::T) (void)value(k);
        return;
    }
    fft_twiddles<P>(tw);
    constexpr double invN = 1.0 / (double)P::N;
    auto store = [&](int, int, int r, int, cd x) __attribute__((always_inline)) {
        st(a.gr_out, (size_t)n * P::N + r, scale(x, invN));
    };
    if constexpr (P::PASSES == 1) {
        fft_run<P, true>(X, tw, [&](int k, int) __attribute__((always_inline)) { return value(k); }, store);
    } else {
        // G~ by every thread into LDS first: the divisions, one element at a time
        // and thread, instead of a line of them in each of the first pass's threads
        for (int k = threadIdx.x; k < P::N; k += P::T) X[P::pad(k)] = value(k);
        __syncthreads();
        fft_first_lds<P, true>(X, tw);
        fft_middle<P, 1, true>(X, tw);
        fft_last<P, true>(X, store);
    }
}

// Clear the counters of the ladder launches that follow on the stream (one
// work-group of a kernel before them: no launch of its own).
__device__ __forceinline__ void zero_ints(int *p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

// ------------------------------------------------------------------------
// chi_{m,n}(q) = -T FFT_r[ gr_n(-r) gr_{n+m}(r) ](q); zero when n+m leaves
// the window.  One block per (n, m).
// ------------------------------------------------------------------------
template <typename P>
__global__ __launch_bounds__(P::T) void k_bubble(BubbleArgs a) {
    __shared__ cd X[P::LDS_N];
    __shared__ cd tw[P::nk];
    const int n = blockIdx.x, im = blockIdx.y;
    const int m = im - (a.n_om - 1) / 2;
    const int n2 = n + m;
    if (n == 0 && im == 0) zero_ints(a.zero, a.n_zero);
    double *out = a.chi + 2 * ((size_t)im * a.n_nu + n) * P::N;
    if (n2 < 0 || n2 >= a.n_nu) {
        for (int q = threadIdx.x; q < P::N; q += P::T) st(out, q, cd{0.0, 0.0});
        return;
    }
    fft_twiddles<P>(tw);
    if constexpr (P::S == 2) __syncthreads();
    const double *ga = a.gr + 2 * (size_t)n * P::N;
    const double *gb = a.gr + 2 * (size_t)n2 * P::N;
    const double mT = -1.0 / a.beta;
    fft_run<P, false>(X, tw,
                      [&](int r, int rr) __attribute__((always_inline)) { return ld(ga, rr) * ld(gb, r); },
                      [&](int, int, int q, int, cd x) __attribute__((always_inline)) { st(out, q, scale(x, mT)); });
}

// ------------------------------------------------------------------------
// sigma_calc <- s and sigma <- (1 - alpha) sigma + alpha s of one element (each may
// be null); |sigma_new - sigma_old|^2 and |sigma_new|^2 are added to dn, nn.
// ------------------------------------------------------------------------
__device__ __forceinline__ void mix_element(double *sigma_calc, double *sigma, double alpha, size_t e,
                                            cd s, double &dn, double &nn) {
    if (sigma_calc) st(sigma_calc, e, s);
    if (!sigma) return;
    const cd old = ld(sigma, e);
    const cd nw = {(1.0 - alpha) * old.re + alpha * s.re, (1.0 - alpha) * old.im + alpha * s.im};
    st(sigma, e, nw);
    const double dr = nw.re - old.re, di = nw.im - old.im;
    dn += dr * dr + di * di;
    nn += nw.re * nw.re + nw.im * nw.im;
}

// ------------------------------------------------------------------------
// Partial dual self-energy over one chunk of bosonic frequencies:
//   part[chunk][n][k] = (T/2) FFT_r[ sum_{m in chunk} v_{m,n}(-r) gr_{n+m}(r) ](k),
//   v_{m,n} = IFFT_q[ 3 W^m_{m,n} + W^d_{m,n} ].
// One block per (n, chunk).  The accumulator B(r) = sum_m v(r) gr(-r) lives in
// registers where the inverse FFT's last pass leaves v, and FFT_r[B(-r)](k) is the
// transform of B with the other sign, whose first pass takes it from there.
// ALL, one chunk: the block has the whole sum and mixes it itself, without the launch
// and the pass over memory of k_reduce_mix (8 x 8, n_nu 16, n_om 1, an iteration of
// the loop without a graph 58 -> 41 us).
// RED: W of a symmetry-reduced ladder, solved at m index >= im0 and representative
// q only.  The rest is read from there (k_sym_expand's rule) instead of being
// written out and read back in every iteration (32 x 32, n_nu 64, n_om 31: 19.5 us of
// k_sym_expand per iteration, now once per call).
// Each switch is a build of its own: the mixing code in the chunked build cost
// 64 x 64, n_nu 128 88 -> 109 us.
// ------------------------------------------------------------------------
template <typename P, typename Q, bool RED, bool ALL>
__global__ __launch_bounds__(P::T) void k_sigma_part(SigmaArgs a) {
    constexpr int LAST = P::PASSES - 1, V = P::lines_per_thread(LAST), R = 1 << P::bits(LAST);
    __shared__ cd X[P::LDS_N > Q::LDS_N ? P::LDS_N : Q::LDS_N];
    __shared__ cd tw[P::nk];
    __shared__ unsigned short rep[RED ? P::N : 1];
    __shared__ double red[2][P::T / 64];
    const int n = blockIdx.x, chunk = blockIdx.y;
    fft_twiddles<P>(tw);
    if constexpr (RED)
        for (int q = threadIdx.x; q < P::N; q += P::T) rep[q] = (unsigned short)a.qrep[q];
    cd acc[V][R];
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
        for (int i = 0; i < R; ++i) acc[v][i] = {0.0, 0.0};
    const int h = (a.n_om - 1) / 2;
    const int m_lo = chunk * a.chunk_len;
    const int m_hi = min(a.n_om, m_lo + a.chunk_len);
    const size_t plane = (size_t)a.n_om * a.n_nu * P::N;   // one channel of W
    for (int im = m_lo; im < m_hi; ++im) {
        const int n2 = n + im - h;
        if (n2 < 0 || n2 >= a.n_nu) continue;
        const bool flip = RED && im < a.im0;               // conjugate of -Om at -nu
        const int ims = flip ? a.n_om - 1 - im : im, ns = flip ? a.n_nu - 1 - n : n;
        const double sg = flip ? -1.0 : 1.0;
        const double *wd = a.w + 2 * ((size_t)ims * a.n_nu + ns) * P::N, *wm = wd + 2 * plane;
        const double *gb = a.gr + 2 * (size_t)n2 * P::N;
        __syncthreads();
        fft_run<P, true>(X, tw,
                         [&](int q, int) __attribute__((always_inline)) {
                             const int qs = RED ? (int)rep[q] : q;
                             const cd d = ld(wd, qs), m = ld(wm, qs);
                             const cd v = {fma(3.0, m.re, d.re), fma(3.0, m.im, d.im)};
                             return RED ? cd{v.re, sg * v.im} : v;
                         },
                         [&](int v, int i, int, int rr, cd x) __attribute__((always_inline)) {
                             acc[v][i] = fma_c(acc[v][i], x, ld(gb, rr));
                         });
    }
    const double sc = 0.5 / (a.beta * (double)P::N);      // T/2 and the inverse FFT's 1/N
    double dn = 0.0, nn = 0.0;
    double *out = ALL ? nullptr : a.part + 2 * ((size_t)chunk * a.n_nu + n) * P::N;
    auto store = [&](int, int, int k, int, cd x) __attribute__((always_inline)) {
        if constexpr (ALL) mix_element(a.sigma_calc, a.sigma, a.alpha, (size_t)n * P::N + k, scale(x, sc), dn, nn);
        else st(out, k, scale(x, sc));
    };
    if constexpr (P::PASSES == 1) {
        if (threadIdx.x == 0) {
            fft_reg<R, true>(acc[0]);
#pragma unroll
            for (int i = 0; i < R; ++i) store(0, i, i, 0, acc[0][i]);
        }
    } else {
        __syncthreads();
        fft_first_reg<Q, true>(X, tw, acc);
        fft_middle<Q, 1, true>(X, tw);
        fft_last<Q, true>(X, store);
    }
    if (!ALL || !a.sigma) return;
    for (int x = 32; x > 0; x >>= 1) {
        dn += __shfl_xor(dn, x, 64);
        nn += __shfl_xor(nn, x, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = dn;
        red[1][threadIdx.x >> 6] = nn;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int x = 1; x < P::T / 64; ++x) {
            dn += red[0][x];
            nn += red[1][x];
        }
        a.norm_part[2 * n] = dn;
        a.norm_part[2 * n + 1] = nn;
    }
}

// ------------------------------------------------------------------------
// sigma_calc = sum over chunks of part (fixed order); optionally
// sigma <- (1 - alpha) sigma + alpha sigma_calc with per-block partial sums of
// |sigma_new - sigma_old|^2 and |sigma_new|^2.
// ------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_reduce_mix(ReduceMixArgs a) {
    __shared__ double red[2][256];
    double dn = 0.0, nn = 0.0;
    const size_t M = a.count;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < M;
         e += (size_t)gridDim.x * blockDim.x) {
        cd s = ld(a.part, e);
        for (int c = 1; c < a.n_chunks; ++c) s = s + ld(a.part, (size_t)c * M + e);
        mix_element(a.sigma_calc, a.sigma, a.alpha, e, s, dn, nn);
    }
    if (!a.sigma) return;
    red[0][threadIdx.x] = dn;
    red[1][threadIdx.x] = nn;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            red[0][threadIdx.x] += red[0][threadIdx.x + s];
            red[1][threadIdx.x] += red[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.norm_part[2 * blockIdx.x] = red[0][0];
        a.norm_part[2 * blockIdx.x + 1] = red[1][0];
    }
}

// ------------------------------------------------------------------------
// gamma^{d/m} = gamma^uu +- gamma^ud, P^c[i][j] = gamma^c_ij gamma^c_ji and the
// layouts and copies of them that the ladder kernels read.  One block per 256
// elements of a bosonic index, both channels; its partial maxima tell whether
// gamma^c is symmetric.  The symmetric ladder takes the symmetric part S =
// (gamma + gamma^T) / 2: with gamma = S + A, A antisymmetric, the first-order change of
// Gamma_nn is ((1 + Gamma chi) A (1 + chi Gamma))_nn, the diagonal of an
// antisymmetric matrix, i.e. zero; so is that of log det, tr(chi (1 - S chi)^-1 A),
// and Gamma^(2)_nn uses P itself.  Results change by (|A| / |gamma|)^2 at most
// times powers of the condition number: with |A_ij| <= 2^-40 max |gamma| far
// below rounding.  (Rounding of the inputs makes |A| / max |gamma| 1e-16 at half
// filling and up to 4e-14 for the Lehmann vertices at n_nu = 128.)
// ------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_gamma_prep(GammaPrepArgs a) {
    __shared__ float red[4][4];
    if (blockIdx.x == 0 && blockIdx.y == 0) zero_ints(a.zero, a.n_zero);
    const size_t nn = (size_t)a.n_nu * a.n_nu;
    const size_t tot = (size_t)a.n_om * nn;
    const size_t b0 = (size_t)blockIdx.y * nn;
    const size_t u = (size_t)blockIdx.x * 256 + threadIdx.x;
    float big[2] = {0.f, 0.f}, dif[2] = {0.f, 0.f};
    if (u < nn) {
        const int i = (int)(u / a.n_nu), j = (int)(u % a.n_nu);
        const size_t e = b0 + u, et = b0 + (size_t)j * a.n_nu + i;
        const cd uu = ld(a.guu, e), ud = ld(a.gud, e);
        const cd uut = ld(a.guu, et), udt = ld(a.gud, et);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const cd g = c == 0 ? uu + ud : uu - ud;
            const cd gt = c == 0 ? uut + udt : uut - udt;
            const cd p = g * gt;
            const size_t o = c * tot + e;
            st(a.gdm, o, g);
            if (a.pdm) st(a.pdm, o, p);
            st(a.gtr, o, gt);
            if (a.gp32) st4f(a.gp32, o, (float)g.re, (float)g.im, (float)p.re, (float)p.im);
            if (a.gtr32) st2f(a.gtr32, o, (float)gt.re, (float)gt.im);
            st(a.gsym, o, cd{0.5 * (g.re + gt.re), 0.5 * (g.im + gt.im)});
            // |gamma|, transposed (a modulus below the FP32 range counts as its
            // smallest normal value)
            float m = (float)sqrt(fma(gt.re, gt.re, gt.im * gt.im));
            if (m < 1.17549435e-38f && (gt.re != 0.0 || gt.im != 0.0)) m = 1.17549435e-38f;
            a.gabs[o] = m;
            // a NaN makes the maxima NaN, and the comparison of prep_symmetric false
            const float d = (float)(fabs(g.re - gt.re) + fabs(g.im - gt.im));
            big[c] = max_nan(big[c], m);
            dif[c] = max_nan(dif[c], d);
        }
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            big[c] = max_nan(big[c], __shfl_xor(big[c], off, 64));
            dif[c] = max_nan(dif[c], __shfl_xor(dif[c], off, 64));
        }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][w] = big[0];
        red[1][w] = big[1];
        red[2][w] = dif[0];
        red[3][w] = dif[1];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        float m = red[threadIdx.x][0];
        for (int x = 1; x < 4; ++x) m = max_nan(m, red[threadIdx.x][x]);
        a.symp[4 * ((size_t)blockIdx.y * kPrepChunks + blockIdx.x) + threadIdx.x] = m;
    }
}

__global__ void k_zero_ints(int *p, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// ------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------
// the build for the grid's shape (nk^D <= 4096)
#define DF_FFT_SHAPES(F)                                                          \
    F(1, 2) F(1, 3) F(1, 4) F(1, 5) F(1, 6) F(2, 2) F(2, 3) F(2, 4) F(2, 5) F(2, 6) \
    F(3, 2) F(3, 3) F(3, 4) F(4, 2) F(4, 3)
#define DF_FFT_SWITCH(F)                       \
    switch (a.grid.D * 16 + a.grid.lognk) {    \
        DF_FFT_SHAPES(F)                       \
        default: return hipErrorInvalidValue;  \
    }

// (few work-groups, one per frequency, of an element's divisions each: more threads)
template <int D, int LK> using DualFft = Fft<D, LK, false, ((1 << (D * LK)) < 1024 ? ((1 << (D * LK)) < 64 ? 64 : (1 << (D * LK))) : ((1 << (D * LK)) >= 4096 ? 1024 : 512))>;

hipError_t launch_dual_gf(const DualGfArgs &a, hipStream_t s) {
#define DF_CASE(D, LK)                                                                               \
    case D * 16 + LK:                                                                                \
        hipLaunchKernelGGL((k_dual_gf<DualFft<D, LK>>), dim3(a.n_nu), dim3(DualFft<D, LK>::T), 0, s, a); \
        break;
    DF_FFT_SWITCH(DF_CASE)
#undef DF_CASE
    return hipGetLastError();
}

hipError_t launch_bubble(const BubbleArgs &a, hipStream_t s) {
#define DF_CASE(D, LK)                                                                                      \
    case D * 16 + LK:                                                                                       \
        hipLaunchKernelGGL((k_bubble<Fft<D, LK>>), dim3(a.n_nu, a.n_om), dim3(Fft<D, LK>::T), 0, s, a); \
        break;
    DF_FFT_SWITCH(DF_CASE)
#undef DF_CASE
    return hipGetLastError();
}

template <typename P, typename Q> static hipError_t launch_sigma_grid(const SigmaArgs &a, hipStream_t s) {
    const dim3 grid(a.n_nu, a.n_chunks), block(P::T);
    const bool all = a.one_pass != 0;
    if (all && a.n_chunks != 1) return hipErrorInvalidValue;
    if (a.qrep && all) hipLaunchKernelGGL((k_sigma_part<P, Q, true, true>), grid, block, 0, s, a);
    else if (a.qrep) hipLaunchKernelGGL((k_sigma_part<P, Q, true, false>), grid, block, 0, s, a);
    else if (all) hipLaunchKernelGGL((k_sigma_part<P, Q, false, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_sigma_part<P, Q, false, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_sigma_part(const SigmaArgs &a, hipStream_t s) {
#define DF_CASE(D, LK) \
    case D * 16 + LK: return launch_sigma_grid<Fft<D, LK>, Fft<D, LK, true>>(a, s);
    DF_FFT_SWITCH(DF_CASE)
#undef DF_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_reduce_mix(const ReduceMixArgs &a, int blocks, hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_mix, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_zero_ints(int *p, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_ints, dim3(1), dim3(64), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_gamma_prep(const GammaPrepArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_gamma_prep, dim3(prep_chunks(a.n_nu), a.n_om), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace df
