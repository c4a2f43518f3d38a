// FFT over the D-dimensional k-grid of one N-point array (N = nk^D <= 4096), in
// passes of one radix-4, 8 or 16 transform per thread and line, held in
// registers; LDS only carries the array from one pass to the next.
//
// Bound: LDS traffic and the barriers between passes, at two work-groups per CU
// (an N = 4096 array takes 70 KB).  A line of an axis of nk <= 16 points is one
// radix-nk pass (on the 16 x 16 grid two of radix 4), one of 32 or 64 points two (8 x
// 4, 8 x 8): three LDS round trips for 64 x 64 and two for 16^3, where radix-4 passes from and to LDS took six.
// The first pass takes its points from the caller (global memory) and the last
// one hands them over, so input and output add none.  Against radix-4 passes on LDS
// (256 to 1024 threads): bubble at 16^3, n_nu 96, n_om 23 68.6 -> 44.0 us (145 MB of chi
// written, 3.3 TB/s), Schwinger-Dyson at 64 x 64, n_nu 128, n_om 15 99 -> 74 us (252 MB
// of W read, 3.4 TB/s), bubble at 32 x 32, n_nu 64, n_om 31 17.0 -> 10.8 us.
//
// Lines of two passes: with n = n1 RB + n2 the first pass transforms over n1
// (stride RB) and multiplies by w^(n2 k1), the second over n2; the result of
// frequency k1 + RA k2 sits at position k1 RB + k2.  No bit reversal: the last pass
// knows the frequency of what it holds.
#pragma once

#include "df_device.hpp"

namespace df {

// e^{-+ 2 pi i j / 16}, j = 1, 2, 3 (INV: the + sign)
template <bool INV> __device__ __forceinline__ cd mul_i(cd a) {   // times -+ i
    return INV ? cd{-a.im, a.re} : cd{a.im, -a.re};
}
template <bool INV> __device__ __forceinline__ cd tw_const(cd a, double c, double s) {   // times c -+ i s
    return INV ? cd{fma(a.re, c, -a.im * s), fma(a.im, c, a.re * s)}
               : cd{fma(a.re, c, a.im * s), fma(a.im, c, -a.re * s)};
}
template <bool INV> __device__ __forceinline__ void fft4(cd &a, cd &b, cd &c, cd &d) {
    const cd s = a + c, t = a - c, u = b + d, v = mul_i<INV>(b - d);
    a = s + u;
    b = t + v;
    c = s - u;
    d = t - v;
}
// x[0..R-1] in natural order to natural order
template <int R, bool INV> __device__ __forceinline__ void fft_reg(cd (&x)[R]) {
    constexpr double H = 0.70710678118654752440;      // cos(pi / 4)
    constexpr double C1 = 0.92387953251128675613, S1 = 0.38268343236508977173;   // pi / 8
    if constexpr (R == 4) {
        fft4<INV>(x[0], x[1], x[2], x[3]);
    } else if constexpr (R == 8) {
        // 2 x 4: n = 2 n1 + n2, k = k1 + 4 k2
        cd e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
        fft4<INV>(e[0], e[1], e[2], e[3]);
        fft4<INV>(o[0], o[1], o[2], o[3]);
        o[1] = tw_const<INV>(o[1], H, H);
        o[2] = mul_i<INV>(o[2]);
        o[3] = tw_const<INV>(o[3], -H, H);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] = e[k] + o[k];
            x[k + 4] = e[k] - o[k];
        }
    } else {
        static_assert(R == 16, "radix");
        // 4 x 4: n = 4 n1 + n2, k = k1 + 4 k2
#pragma unroll
        for (int n2 = 0; n2 < 4; ++n2) fft4<INV>(x[n2], x[4 + n2], x[8 + n2], x[12 + n2]);
        // x[4 k1 + n2] *= w16^(n2 k1)
        x[5] = tw_const<INV>(x[5], C1, S1);
        x[6] = tw_const<INV>(x[6], H, H);
        x[7] = tw_const<INV>(x[7], S1, C1);
        x[9] = tw_const<INV>(x[9], H, H);
        x[10] = mul_i<INV>(x[10]);
        x[11] = tw_const<INV>(x[11], -H, H);
        x[13] = tw_const<INV>(x[13], S1, C1);
        x[14] = tw_const<INV>(x[14], -H, H);
        x[15] = tw_const<INV>(x[15], -C1, -S1);
        cd y[16];
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            cd a = x[4 * k1], b = x[4 * k1 + 1], c = x[4 * k1 + 2], d = x[4 * k1 + 3];
            fft4<INV>(a, b, c, d);
            y[k1] = a;
            y[k1 + 4] = b;
            y[k1 + 8] = c;
            y[k1 + 12] = d;
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k] = y[k];
    }
}

// The plan of one grid.  REV: the radices of two-pass lines swapped (4 x 8) and the
// axes in the order in which the slowest one comes first, for a transform whose
// input is held in registers as the other plan's last pass left it.
// TMIN: threads of the work-group at least (they all load and store, and a pass with
// fewer lines leaves some idle).
template <int D_, int LK_, bool REV = false, int TMIN = 64> struct Fft {
    static constexpr int D = D_, LK = LK_, nk = 1 << LK, N = 1 << (D * LK);
    // passes per axis; the larger radix.  16 x 16: two radix-4 passes, since one of
    // radix 16 gives work to 16 lanes only (Schwinger-Dyson with the transform of G~,
    // n_nu 48, n_om 7: 16.1 -> 8.3 us; 16^3 has 256 lines and keeps radix 16)
    static constexpr int S = LK > 4 || (LK == 4 && D == 2) ? 2 : 1;
    static constexpr int LMAX = S == 1 ? LK : (LK == 4 ? 2 : 3);
    static constexpr int LA = S == 1 ? LK : (LK == 5 && REV ? 2 : LMAX), LB = S == 1 ? 0 : LK - LA;
    static constexpr int RA = 1 << LA, RB = 1 << LB;
    static constexpr int PASSES = D * S;
    // threads of a work-group: one line of the larger radix each
    static constexpr int T = (N >> LMAX) < TMIN ? TMIN : (N >> LMAX);
    // one complex of padding per 2^PB: the lanes' contiguous lines of axis 0 then
    // fall in different banks
    static constexpr int PB = S == 1 ? LK : LK - LMAX;
    static constexpr int LDS_N = N + (N >> PB);
    static __device__ __forceinline__ int pad(int p) { return p + (p >> PB); }
    // pass i: its axis, whether it is the second of the axis, and the bits of the
    // position that its digit takes
    static constexpr int axis(int i) {
        if (S == 1) {
            if (REV) return i == 0 ? D - 1 : (D == 3 ? (i == 1 ? 0 : 1) : (D == 4 ? (i == 1 ? 2 : i - 2) : 0));
            return D < 3 ? i : (i == 0 ? 1 : (i == 1 ? 0 : i));
        }
        return D == 1 ? 0 : (i == 0 || i == 3 ? 1 : 0);
    }
    static constexpr bool second(int i) { return S == 2 && (D == 1 ? i == 1 : i >= 2); }
    static constexpr int off(int i) { return axis(i) * LK + (S == 2 && !second(i) ? LB : 0); }
    static constexpr int bits(int i) { return S == 1 ? LK : (second(i) ? LB : LA); }
    static constexpr int lines_per_thread(int i) { return (N >> bits(i)) > T ? (N >> bits(i)) / T : 1; }
};

// Position of point 0 of line u of a pass whose digit has B bits at O.
template <int O, int B> __device__ __forceinline__ int line_base(int u) {
    return ((u >> O) << (O + B)) | (u & ((1 << O) - 1));
}

// -r mod nk on every axis but AX (whose field is zero in r)
template <int D, int LK, int AX> __device__ __forceinline__ int reflect_others(int r) {
    constexpr int m = (1 << LK) - 1;
    int out = 0;
#pragma unroll
    for (int a = 0; a < D; ++a)
        if (a != AX) out |= ((-(r >> (a * LK))) & m) << (a * LK);
    return out;
}

// twiddles w^t, w = e^{-2 pi i / nk}, for the two-pass lines
template <typename P> __device__ __forceinline__ void fft_twiddles(cd *tw) {
    if constexpr (P::S == 2)
        for (int t = threadIdx.x; t < P::nk; t += P::T) {
            double s, c;
            sincospi(-2.0 * (double)t / (double)P::nk, &s, &c);
            tw[t] = {c, s};
        }
}

template <typename P, int I, bool INV>
__device__ __forceinline__ void fft_twiddle(cd (&x)[1 << P::bits(I)], int base, const cd *tw) {
    if constexpr (P::S == 2 && !P::second(I)) {
        const int n2 = (base >> (P::axis(I) * P::LK)) & (P::RB - 1);
#pragma unroll
        for (int k = 1; k < P::RA; ++k) {
            const cd w = tw[(n2 * k) & (P::nk - 1)];
            x[k] = x[k] * (INV ? conj(w) : w);
        }
    }
}

template <typename P, int I> __device__ __forceinline__ bool line_in(int u) {
    constexpr int lines = P::N >> P::bits(I);
    return lines >= P::T ? true : u < lines;
}

// First pass: x = load(r, rr), r the position, rr = -r on the grid; into LDS.
template <typename P, bool INV, typename Load>
__device__ __forceinline__ void fft_first(cd *X, const cd *tw, Load &&load) {
    constexpr int O = P::off(0), B = P::bits(0), R = 1 << B, AX = P::axis(0), sh = AX * P::LK;
#pragma unroll
    for (int v = 0; v < P::lines_per_thread(0); ++v) {
        const int u = threadIdx.x + v * P::T;
        if (!line_in<P, 0>(u)) continue;
        const int base = line_base<O, B>(u);
        const int low = (base >> sh) & (P::nk - 1), other = base & ~((P::nk - 1) << sh);
        const int ro = reflect_others<P::D, P::LK, AX>(other);
        cd x[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int c = low + (i << (O - sh));
            x[i] = load(base + (i << O), ro | (((-c) & (P::nk - 1)) << sh));
        }
        fft_reg<R, INV>(x);
        fft_twiddle<P, 0, INV>(x, base, tw);
#pragma unroll
        for (int i = 0; i < R; ++i) X[P::pad(base) + (i << O) + ((i << O) >> P::PB)] = x[i];
    }
}
// First pass from registers: line v of the thread is y[v], ordered as the other
// plan's last pass leaves it (fft_last); its positions are the same.
template <typename P, bool INV, int V, int R>
__device__ __forceinline__ void fft_first_reg(cd *X, const cd *tw, cd (&y)[V][R]) {
    constexpr int O = P::off(0), B = P::bits(0);
    static_assert(R == (1 << B) && V == P::lines_per_thread(0), "lines of the other plan's last pass");
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int u = threadIdx.x + v * P::T;
        if (!line_in<P, 0>(u)) continue;
        const int base = line_base<O, B>(u);
        fft_reg<R, INV>(y[v]);
        fft_twiddle<P, 0, INV>(y[v], base, tw);
#pragma unroll
        for (int i = 0; i < R; ++i) X[P::pad(base) + (i << O) + ((i << O) >> P::PB)] = y[v][i];
    }
}

template <typename P, int I, bool INV> __device__ __forceinline__ void fft_middle(cd *X, const cd *tw) {
    if constexpr (I + 1 < P::PASSES) {
        constexpr int O = P::off(I), B = P::bits(I), R = 1 << B;
        __syncthreads();
#pragma unroll
        for (int v = 0; v < P::lines_per_thread(I); ++v) {
            const int u = threadIdx.x + v * P::T;
            if (!line_in<P, I>(u)) continue;
            const int base = line_base<O, B>(u);
            cd *p = X + P::pad(base);
            cd x[R];
#pragma unroll
            for (int i = 0; i < R; ++i) x[i] = p[(i << O) + ((i << O) >> P::PB)];
            fft_reg<R, INV>(x);
            fft_twiddle<P, I, INV>(x, base, tw);
#pragma unroll
            for (int i = 0; i < R; ++i) p[(i << O) + ((i << O) >> P::PB)] = x[i];
        }
        fft_middle<P, I + 1, INV>(X, tw);
    }
}

// Last pass: store(v, i, k, kk, value) for every point i of line v of the thread, k
// its frequency, kk = -k on the grid.  The lanes take consecutive frequencies of
// axis 0 wherever the last axis is another one.
template <typename P, bool INV, typename Store>
__device__ __forceinline__ void fft_last(const cd *X, Store &&store) {
    constexpr int I = P::PASSES - 1, O = P::off(I), B = P::bits(I), R = 1 << B, AX = P::axis(I), sh = AX * P::LK;
    __syncthreads();
#pragma unroll
    for (int v = 0; v < P::lines_per_thread(I); ++v) {
        const int u = threadIdx.x + v * P::T;
        if (!line_in<P, I>(u)) continue;
        int base, low, others, step;              // position; frequency: axis AX, the others
        if constexpr (P::S == 1) {
            base = line_base<O, B>(u);
            low = 0;
            others = base;
            step = 1;
        } else if constexpr (P::D == 1) {
            base = u << P::LB;
            low = u;
            others = 0;
            step = P::RA;
        } else {
            const int f0 = u & (P::nk - 1), k1 = u >> P::LK;
            base = ((k1 << P::LB) << P::LK) | ((f0 & (P::RA - 1)) << P::LB) | (f0 >> P::LA);
            low = k1;
            others = f0;
            step = P::RA;
        }
        const cd *p = X + P::pad(base);
        cd x[R];
#pragma unroll
        for (int i = 0; i < R; ++i) x[i] = p[(i << O) + ((i << O) >> P::PB)];
        fft_reg<R, INV>(x);
        const int ro = reflect_others<P::D, P::LK, AX>(others);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int c = low + i * step;
            store(v, i, others | (c << sh), ro | (((-c) & (P::nk - 1)) << sh), x[i]);
        }
    }
}

// First pass from LDS, the array in natural order and padded.
template <typename P, bool INV> __device__ __forceinline__ void fft_first_lds(cd *X, const cd *tw) {
    fft_first<P, INV>(X, tw, [&](int r, int) __attribute__((always_inline)) { return X[P::pad(r)]; });
}

// One transform from load to store.  LDS may be in use by an earlier one: a barrier
// comes first when `again`.
template <typename P, bool INV, typename Load, typename Store>
__device__ __forceinline__ void fft_run(cd *X, const cd *tw, Load &&load, Store &&store) {
    if constexpr (P::PASSES == 1) {
        constexpr int R = P::nk;
        if (threadIdx.x == 0) {
            cd x[R];
#pragma unroll
            for (int i = 0; i < R; ++i) x[i] = load(i, (-i) & (P::nk - 1));
            fft_reg<R, INV>(x);
#pragma unroll
            for (int i = 0; i < R; ++i) store(0, i, i, (-i) & (P::nk - 1), x[i]);
        }
    } else {
        fft_first<P, INV>(X, tw, load);
        fft_middle<P, 1, INV>(X, tw);
        fft_last<P, INV>(X, store);
    }
}

}  // namespace df
