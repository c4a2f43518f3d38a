// Screening of the FP64 ladder items, one kernel for 16 momenta at a time: what
// every item needs but the elimination does not have to carry.
//   t_n(q)   = (gamma chi gamma)_nn = sum_n' (gamma_nn' gamma_n'n) chi_n'(q), the
//              second-order term of eq. (sd): a matrix product over q, on the
//              FP64 matrix cores; left in W, where the ladder kernel finds it
//   rho(|M|) <= max_i (B v)_i / v_i, B = |gamma| diag |chi| + eps: the
//              Collatz-Wielandt certificate of the pivot-free elimination
//              (df_gj_core.hpp), with true moduli, by power steps on the FP32
//              matrix cores.
// Work-group: one channel, one bosonic index, 16 momenta; its four waves share
// chi in LDS and take the 16-row blocks in turn, the rows of |gamma| staying in
// registers over the power steps.  Per item the two products are n^2
// operations each; formed inside the ladder kernel, as rows of one item spread
// over a wave, they cost about 1500 vector instructions per item (an eighth of
// the n_nu = 64 elimination), here about 40 matrix instructions.
#include "df_gj_core.hpp"
#include "df_lattice_ladder.hpp"

namespace df {

constexpr int SCREEN_STEPS = 6;
constexpr double SCREEN_MAX = 0.999;

// LAT: the product is gamma L instead (lattice observables' ladder term, n_om = 1).
template <int NT, bool LAT>
__device__ __forceinline__ void screen_body(const LadderArgs &a0, const double *L) {
    constexpr int NP = 16 * NT;
    typedef MT<double>::v4 d4;
    typedef MT<float>::v4 f4;
    __shared__ cd X[NP][16];          // chi[k][q] (LAT: L[k][q])
    __shared__ float xa[NP][16];      // |chi|
    __shared__ float vv[2][NP][16];   // vectors of the power steps
    __shared__ float red[2][4][16];   // per wave and momentum: its largest quotient

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = tid & 63, lj = l & 15, lg = l >> 4;
    LadderArgs a = a0;
    int blk = xcd_item(blockIdx.x, gridDim.x);
    int item0 = a0.item0;
    if (a0.insts) {
        const ConstLadderInstPtr tab = (ConstLadderInstPtr)(const void *)a0.insts;
        int k = 0;
        while (k + 1 < a0.n_insts && tab[k + 1].sblk0 <= blk) ++k;
        const auto &d = tab[k];
        blk -= d.sblk0;
        item0 = d.item0;
        a.pdm = d.pdm;
        a.gabs = d.gabs;
        a.symp = d.symp;
        a.chi = d.chi;
        a.w = d.w;
        a.n_nu = d.n_nu;
        a.n_om = d.n_om;
        a.N = d.N;
        a.qlist = d.qlist;
        a.n_q = d.n_q;
        a.im0 = d.im0;
    }
    const int n = a.n_nu, N = a.N, nm1 = n - 1;
    const int n_q = a.qlist ? a.n_q : N;
    const int m0 = a.qlist ? a.im0 : 0, n_m = a.n_om - m0;
    const int qb = (n_q + 15) / 16;
    // channels next to each other: the second one's chi comes from the L2
    const int c = blk & 1;
    blk >>= 1;
    const int im = m0 + blk / qb;
    const int k0 = 16 * (blk % qb);
    const int kq = k0 + lj;                       // this lane's momentum
    const bool qin = kq < n_q;
    const int kc = qin ? kq : n_q - 1;
    const int q = a.qlist ? a.qlist[kc] : kc;

    constexpr float FMIN = 1.17549435e-38f;
    for (int k = tid >> 4; k < NP; k += 16) {     // (tid & 15 == lj)
        const cd x = ld(a.chi, ((size_t)im * n + (k < nm1 ? k : nm1)) * N + q);
        const cd v = k < n ? x : cd{0.0, 0.0};
        if constexpr (LAT) {
            const cd y = ld(L, (size_t)(k < nm1 ? k : nm1) * N + q);
            X[k][lj] = k < n ? y : cd{0.0, 0.0};
        } else {
            X[k][lj] = v;
        }
        // (a modulus below the FP32 range counts as its smallest normal value:
        // the bound stays an upper bound)
        float m = (float)sqrt(fma(v.re, v.re, v.im * v.im));
        if (m < FMIN && (v.re != 0.0 || v.im != 0.0)) m = FMIN;
        xa[k][lj] = m;
    }

    const int cm = c * a.n_om + im;
    // the matrix of the product, by rows k: P (symmetric); LAT: the symmetric part of
    // gamma where the block ladder takes it, else gamma from its transpose
    const double *pm = a.pdm;
    // (wave 0 needs the answer at the end; asked here, the loads are not waited for alone)
    bool sym = false;
    if (LAT || w == 0) sym = vertex_symmetric(a.symp + 4 * (size_t)im * kPrepChunks, n, c, l);
    if constexpr (LAT) pm = sym ? a.gsym : a.gtr;
    pm += 2 * (size_t)cm * n * n;
    const float *ga = a.gabs + (size_t)cm * n * n;
    // this wave's rows of |gamma| (A operand of every k-slice)
    constexpr int NI = (NT + 3) / 4;
    float gr[NI][4 * NT];
#pragma unroll
    for (int y = 0; y < NI; ++y) {
        const int i = 16 * (w + 4 * y) + lj;
        if (w + 4 * y < NT) {
#pragma unroll
            for (int s = 0; s < 4 * NT; ++s) {
                const int k = 4 * s + lg;
                gr[y][s] = ga[(size_t)(k < nm1 ? k : nm1) * n + (i < nm1 ? i : nm1)];
            }
        }
    }
    __syncthreads();

    // ---- t
#pragma unroll
    for (int y = 0; y < NI; ++y) {
        const int I = w + 4 * y;
        if (I >= NT) continue;
        const int ic = 16 * I + lj < nm1 ? 16 * I + lj : nm1;
        d4 T1 = {0, 0, 0, 0}, T2 = {0, 0, 0, 0}, T3 = {0, 0, 0, 0}, T4 = {0, 0, 0, 0};
#pragma unroll 8
        for (int s = 0; s < 4 * NT; ++s) {
            const int k = 4 * s + lg;
            const cd p = ld(pm, (size_t)(k < nm1 ? k : nm1) * n + ic);
            const cd x = X[k][lj];
            T1 = MT<double>::mma(p.re, x.re, T1);
            T2 = MT<double>::mma(p.im, x.im, T2);
            T3 = MT<double>::mma(p.re, x.im, T3);
            T4 = MT<double>::mma(p.im, x.re, T4);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * I + lg + 4 * r;
            if (qin && i < n) st(a.w, ((size_t)cm * n + i) * N + q, cd{T1[r] - T2[r], T3[r] + T4[r]});
        }
    }
    // ---- certificate: power steps from v = 1 until all 16 momenta pass.  The
    // sums are FP32 over non-negative terms: within (n + 4) 2^-24 of exact
    // with the rounding of the moduli, and the bound is inflated by
    // 1 + 1e-5; eps = 1e-6 keeps v positive.  A NaN never passes.
    bool pass = false;                            // this lane's momentum
    for (int it = 0; it < SCREEN_STEPS; ++it) {
        float ratio = 0.f;
#pragma unroll
        for (int y = 0; y < NI; ++y) {
            const int I = w + 4 * y;
            if (I >= NT) continue;
            f4 U = {0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 4 * NT; ++s) {
                const int k = 4 * s + lg;
                float b = xa[k][lj];
                if (it > 0) b *= vv[it & 1][k][lj];
                U = MT<float>::mma(gr[y][s], b, U);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * I + 4 * lg + r;
                const float vi = it == 0 ? 1.f : vv[it & 1][i][lj];
                const float u = fmaf(1e-6f, vi, U[r]);
                const float rr = u * __builtin_amdgcn_rcpf(vi);
                if (i < n) ratio = max_nan(ratio, rr);
                vv[(it + 1) & 1][i][lj] = i < n ? u : 1.f;
            }
        }
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            const float o = __shfl_xor(ratio, off, 64);
            ratio = max_nan(ratio, o);
        }
        if (lg == 0) red[it & 1][w][lj] = ratio;
        __syncthreads();
        float m = red[it & 1][0][lj];
#pragma unroll
        for (int x = 1; x < 4; ++x) m = max_nan(m, red[it & 1][x][lj]);
        pass = pass || (double)m * (1.0 + 1e-5) < SCREEN_MAX;
        // uniform: every wave holds the same 16 momenta
        if (__all(pass || !qin)) break;
    }
    if (w != 0) return;
    if (lg == 0) {
        const int item = a.qlist ? (c * n_m + (im - m0)) * n_q + kq : cm * N + q;
        if (qin) a.cert[item0 + item] = pass ? (sym ? CERT_SYMMETRIC : CERT_GENERAL) : CERT_NONE;
        // the uncertified ones (the lattice observables' kernel pivots the general
        // vertices' too) are appended to the queue, one counter update per work-group
        const bool put = qin && !(pass && (!LAT || sym));
        const unsigned long long piv = __ballot(put);
        int base = 0;
        if (lj == 0 && piv) base = atomicAdd(a.queue_count, __popcll(piv));
        base = __builtin_amdgcn_readfirstlane(base);
        // (every store writes the same value)
        if (!LAT && __ballot(qin && pass && !sym) && lj == 0) *a.near_count = 1;
        if (put) a.queue[base + __popcll(piv & ((1ull << lj) - 1))] = item0 + item;
    }
}

template <int NT> __global__ __launch_bounds__(256) void k_ladder_screen(LadderArgs a0) {
    screen_body<NT, false>(a0, nullptr);
}
template <int NT> __global__ __launch_bounds__(256) void k_lattice_screen(LadderArgs a0, const double *L) {
    screen_body<NT, true>(a0, L);
}

// work-groups of one instance's screening: channels x bosonic indices x blocks of
// 16 momenta
int ladder_screen_blocks(int n_m, int n_q) {
    return 2 * n_m * ((n_q + 15) / 16);
}

hipError_t launch_ladder_screen(const LadderArgs &a, hipStream_t s) {
    if (a.n_sblk <= 0 || !a.queue || !a.queue_count || !a.near_count) return hipErrorInvalidValue;
    switch ((a.n_nu + 15) / 16) {
#define DF_SCREEN(NT) \
    case NT: hipLaunchKernelGGL(k_ladder_screen<NT>, dim3(a.n_sblk), dim3(256), 0, s, a); break;
        DF_SCREEN(1) DF_SCREEN(2) DF_SCREEN(3) DF_SCREEN(4)
        DF_SCREEN(5) DF_SCREEN(6) DF_SCREEN(7) DF_SCREEN(8)
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_lattice_screen(const LadderArgs &a, const double *L, hipStream_t s) {
    if (a.n_sblk <= 0 || !a.queue || !a.queue_count) return hipErrorInvalidValue;
    switch ((a.n_nu + 15) / 16) {
#define DF_SCREEN_L(NT) \
    case NT: hipLaunchKernelGGL(k_lattice_screen<NT>, dim3(a.n_sblk), dim3(256), 0, s, a, L); break;
        DF_SCREEN_L(1) DF_SCREEN_L(2) DF_SCREEN_L(3) DF_SCREEN_L(4)
        DF_SCREEN_L(5) DF_SCREEN_L(6) DF_SCREEN_L(7) DF_SCREEN_L(8)
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace df
