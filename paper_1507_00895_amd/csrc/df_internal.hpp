// Kernel argument blocks and launcher declarations of libdf (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "df_device.hpp"
#include "df_nan.hpp"

namespace df {

// fermionic index into the vertex and bubble arrays; FULL: n_nu equals the
// padded size and no index leaves the window
template <bool FULL> __device__ __forceinline__ int clamp_nu(int j, int nm1) {
    if constexpr (FULL) return j;
    else return j < nm1 ? j : nm1;
}

struct DualGfArgs {
    Grid grid;
    int n_nu;
    const double *g, *delta, *eps;   // inputs (unused with from_gd)
    const double *sigma;             // may be null (Sigma~ = 0)
    const double *gd_in;             // with from_gd: G~ to transform
    double *gd_out;                  // may be null
    double *gr_out;                  // may be null: [n_nu][N] inverse FFT of G~
    int from_gd;
};

struct BubbleArgs {
    Grid grid;
    int n_nu, n_om;
    double beta;
    const double *gr;                // [n_nu][N]
    double *chi;                     // [n_om][n_nu][N]
    int *zero;                       // counters to clear (may be null)
    int n_zero;
};

struct SigmaArgs {
    Grid grid;
    int n_nu, n_om;
    int chunk_len, n_chunks;
    double beta;
    const double *w;                 // [2][n_om][n_nu][N]
    const double *gr;                // [n_nu][N]
    double *part;                    // [n_chunks][n_nu][N], unless one_pass
    // symmetry-reduced W: only m index >= im0 and q = qrep[q] are read (null: all)
    const int *qrep;
    int im0;
    // one_pass (n_chunks = 1): k_reduce_mix's outputs, norm_part [n_nu][2]
    int one_pass;
    double alpha;
    double *sigma_calc;
    double *sigma;
    double *norm_part;
};

struct ReduceMixArgs {
    size_t count;                    // n_nu * N complex elements
    int n_chunks;
    double alpha;
    const double *part;
    double *sigma_calc;              // may be null
    double *sigma;                   // may be null: no mixing
    double *norm_part;               // [gridDim][2]
};

// Anderson acceleration (df_accel.hip): ring of up to kAccMaxSlots iterates
constexpr int kAccMaxSlots = 9;

struct AccRecordArgs {
    size_t count;                    // n_nu * N complex elements
    const double *x, *fx;            // current iterate, F(iterate)
    double *xh, *rh;                 // rings [kAccMaxSlots][count]
    int slot, n_slots;               // slot written now; slots in use (incl. it)
    double *part;                    // [blocks][kAccMaxSlots] partial dots
    double *dots;                    // [kAccMaxSlots]: Re <r_j, r_slot>
};

struct AccCombineArgs {
    size_t count;
    const double *xh, *rh;
    int n_slots;
    double coef[kAccMaxSlots];       // real weights, summing to one
    double alpha;
    double *x;                       // in: x_k, out: x_{k+1}
    double *norm_part;               // [blocks][2]
};

struct GammaPrepArgs {
    int n_nu, n_om;
    const double *guu, *gud;
    double *gdm;                     // [2][n_om][n_nu][n_nu]
    double *pdm;                     // [2][n_om][n_nu][n_nu] (may be null)
    double *gtr;                     // [2][n_om][n_nu][n_nu]
    float *gp32;                     // [2][n_om][n_nu][n_nu] (gamma, gamma_ij gamma_ji) in FP32, or null
    float *gtr32;                    // [2][n_om][n_nu][n_nu] gamma transposed in FP32, or null
    double *gsym;                    // [2][n_om][n_nu][n_nu] (gamma + gamma^T) / 2
    float *gabs;                     // [2][n_om][n_nu][n_nu] |gamma| transposed, FP32
    float *symp;                     // [n_om][kPrepChunks][4]: partial maxima of its chunks
    int *zero;                       // counters to clear (may be null)
    int n_zero;
};

// Work-groups of k_gamma_prep per bosonic index (256 vertex elements each), and
// what their partial maxima say: {max |gamma^d|, max |gamma^m|, max |gamma^d_ij -
// gamma^d_ji|, the same of gamma^m} of a chunk.  A NaN stays.
constexpr int kPrepChunks = 64;
__host__ __device__ inline int prep_chunks(int n_nu) { return (n_nu * n_nu + 255) / 256; }
// difference within 2^-40 of the largest modulus (an infinite one would pass any)
__device__ inline bool prep_symmetric(float m, float d) {
    return d <= m * 9.094947e-13f && m < 3.0e38f;
}

// Symmetric to rounding (see k_gamma_prep): the largest |gamma_ij - gamma_ji|
// against the largest |gamma|, over the partial maxima of k_gamma_prep.
// One wave, one chunk per lane; uniform result.
__device__ __forceinline__ bool vertex_symmetric(const float *part, int n, int c, int lane) {
    float m = 0.f, d = 0.f;
    if (lane < prep_chunks(n)) {
        m = part[4 * lane + c];
        d = part[4 * lane + 2 + c];
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float om = __shfl_xor(m, off, 64), od = __shfl_xor(d, off, 64);
        m = max_nan(m, om);
        d = max_nan(d, od);
    }
    return prep_symmetric(m, d);
}

// What the screening kernel found of an item: it fails the certificate (and is in the
// queue), or it is certified and its vertex symmetric or not.
enum : uint8_t { CERT_NONE = 0, CERT_SYMMETRIC = 1, CERT_GENERAL = 2 };

// One instance of a fused multi-instance ladder launch (device-side table).
struct LadderInst {
    const double *gdm, *pdm, *gtr, *chi;
    const float *gp32, *gtr32;
    double *w, *logdet;
    int8_t *status;
    int *count;                      // ladders outside the radius (atomic)
    int n_nu, n_om, N;
    int item0;                       // first global item of this instance
    const int *qlist;                // symmetry-reduced launch (else null): solved q
    int n_q, im0;                    // their count; first solved bosonic index
    const double *gsym;              // symmetric part of the vertex, |gamma| and the maxima that tell
    const float *gabs;               // whether it is symmetric (GammaPrepArgs)
    const float *symp;
    int sblk0;                       // first work-group of this instance in a screening launch
};

struct LadderArgs {
    const double *gdm;               // [2][n_om][n_nu][n_nu]
    const double *pdm;               // [2][n_om][n_nu][n_nu]
    const double *chi;               // [n_om][n_nu][N]
    double *w;                       // [2][n_om][n_nu][N]
    double *logdet;                  // [2][n_om][N] or null
    int8_t *status;                  // [2][n_om][N] or null
    int n_nu, n_om, N;
    int item0, n_items;              // items are (c, m, q), q fastest
    int *fallback_count;             // may be null: atomically counts status != 0
    const double *gtr;               // [2][n_om][n_nu][n_nu] gamma transposed (gjb kernel)
    int *queue;                      // certified kernels: uncertified items are appended here
    int *queue_count;                // its length (zeroed before the launch)
    int *near_queue;                 // refined kernel: items whose certificate bound is
    int *near_count;                 // >= CERT_NEAR_MIXED go here for the FP64 kernel; FP64
                                     // screening: 1 if it marked an item CERT_GENERAL
    const LadderInst *insts;         // non-null: fused launch over n_insts instances,
    int n_insts;                     // items are global; the fields above are resolved per item
    const float *gp32;               // FP32 ladder: (gamma, gamma_ij gamma_ji) pairs, FP32
    const float *gtr32;              // FP32 ladder: gamma transposed, FP32
    const int *qlist;                // non-null: symmetry-reduced items (see item_coords)
    int n_q, im0;
    int full;                        // 1: every instance of the launch has n_nu equal to the
                                     // padded size (the mask-free build runs)
    const double *gsym;              // symmetric FP64 ladder and its screening (see LadderInst)
    const float *gabs;
    const float *symp;
    uint8_t *cert;                   // CERT_* of every global item (k_ladder_screen)
    int sblk0, n_sblk;               // work-groups of the screening launch
    int pivot_groups;                // first work-groups of the kernel, which take the queue
    int full_sym;                    // 1: every instance has n_nu equal to the same multiple of 16
};

// Fused launches: find the instance of a global item, fill the per-instance
// fields of a, return the item's index within its instance.  The item is
// uniform over the work-group and the table is read only: it is read through
// the constant address space, so that the instance's fields arrive in scalar
// registers (vector loads would hold them, and the item coordinates built
// from them, in vector registers for the whole item).
typedef __attribute__((address_space(4))) const LadderInst *ConstLadderInstPtr;
__device__ __forceinline__ int resolve_item(LadderArgs &a, int item) {
    if (!a.insts) return item;
    const ConstLadderInstPtr tab = (ConstLadderInstPtr)(const void *)a.insts;
    int k = 0;
    while (k + 1 < a.n_insts && tab[k + 1].item0 <= item) ++k;
    const auto &d = tab[k];
    a.gdm = d.gdm;
    a.pdm = d.pdm;
    a.gtr = d.gtr;
    a.gp32 = d.gp32;
    a.gtr32 = d.gtr32;
    a.chi = d.chi;
    a.w = d.w;
    a.logdet = d.logdet;
    a.status = d.status;
    a.fallback_count = d.count;
    a.n_nu = d.n_nu;
    a.n_om = d.n_om;
    a.N = d.N;
    a.qlist = d.qlist;
    a.n_q = d.n_q;
    a.im0 = d.im0;
    a.gsym = d.gsym;
    return item - d.item0;
}

// An item's (c n_om + m index, q).  Full launches: items are (c, m, q), q
// fastest.  Symmetry-reduced launches (qlist set): items are (c, m index >= im0,
// k < n_q), k fastest, with q = qlist[k] - one q per point-group orbit and the
// bosonic frequencies Omega >= 0; the others follow by symmetry (k_sym_expand).
// The coordinates are uniform over the work-group: readfirstlane puts them
// (and every address built from them) in scalar registers.  Integer division
// is expanded with vector instructions, and without it the quotients stayed in
// vector registers for the whole item.
__device__ __forceinline__ void item_coords(const LadderArgs &a, int item, int *cm, int *q) {
    if (!a.qlist) {
        *q = __builtin_amdgcn_readfirstlane(item % a.N);
        *cm = __builtin_amdgcn_readfirstlane(item / a.N);
        return;
    }
    const int k = item % a.n_q, r = item / a.n_q;
    const int nm = a.n_om - a.im0;
    *q = __builtin_amdgcn_readfirstlane(a.qlist[k]);
    *cm = __builtin_amdgcn_readfirstlane((r / nm) * a.n_om + a.im0 + r % nm);
}

// Representative of q's orbit under the point group of the hypercubic lattice
// (axis permutations and k_a -> -k_a): per axis the smaller of c_a and nk - c_a,
// sorted ascending from axis 0.  Host and device use this same function.
__host__ __device__ inline int canonical_q(int q, int D, int lognk) {
    const int nk = 1 << lognk;
    int r[4] = {0, 0, 0, 0};
    for (int a = 0; a < D; ++a) {
        const int c = (q >> (a * lognk)) & (nk - 1);
        const int m = (nk - c) & (nk - 1);
        r[a] = c < m ? c : m;
    }
    for (int i = 1; i < D; ++i)          // insertion sort of at most four values
        for (int j = i; j > 0 && r[j - 1] > r[j]; --j) {
            const int t = r[j];
            r[j] = r[j - 1];
            r[j - 1] = t;
        }
    int out = 0;
    for (int a = 0; a < D; ++a) out |= r[a] << (a * lognk);
    return out;
}

struct SymTableArgs {
    int D, lognk, N;
    int *qrep;                       // [N]: representative of each q
    int *qlist;                      // [n_irr]: the representatives, ascending
};

struct SymExpandArgs {
    int n_nu, n_om, N, im0;
    const int *qrep;
    double *w;                       // [2][n_om][n_nu][N]
    double *logdet;                  // [2][n_om][N] or null
    int8_t *status;                  // [2][n_om][N] or null
};

// Work-group b of a launch runs on XCD b % 8 (the dispatcher deals work-groups
// round-robin over the eight XCDs, each with its own L2).  Give every XCD one
// contiguous range of the n items instead, so that the neighbouring q of one
// (channel, Om) - which share the cache lines of chi and W - meet in one L2.
constexpr int kXcd = 8;
__device__ __forceinline__ int xcd_item(int b, int n) {
    const int per = n / kXcd, rem = n % kXcd;
    const int x = b % kXcd, i = b / kXcd;
    return x * per + (x < rem ? x : rem) + i;
}

// Lattice observables (df_lattice.hip)
struct LatticeFieldArgs {
    int n_nu, N;
    double beta, mu;
    const double *g, *delta, *eps, *sigma;   // sigma may be null (Sigma~ = 0)
    double *sigma_lat, *g_lat;               // outputs, may be null
    double *gl, *gd, *fg;                    // [n_nu][N] G_lat, G~, frak G
};

struct LatticeSumArgs {
    int n_nu, N;
    const double *bub, *lad;                 // [n_nu][N], [2][N]
    double *chi_ch, *chi_sp;                 // [N], may be null
};

hipError_t launch_dual_gf(const DualGfArgs &a, hipStream_t s);
hipError_t launch_bubble(const BubbleArgs &a, hipStream_t s);
hipError_t launch_sigma_part(const SigmaArgs &a, hipStream_t s);
hipError_t launch_reduce_mix(const ReduceMixArgs &a, int blocks, hipStream_t s);
hipError_t launch_acc_record(const AccRecordArgs &a, int blocks, hipStream_t s);
hipError_t launch_acc_combine(const AccCombineArgs &a, int blocks, hipStream_t s);
hipError_t launch_gamma_prep(const GammaPrepArgs &a, hipStream_t s);

// Work-groups of a launch over a queue of at most `items`, whose length only the device
// knows: three waves per SIMD, further items in rounds.  (The queues are empty in most
// calls, and every work-group costs its start: lattice observables of 32x32, n_nu 64, 768
// work-groups of four waves 93 us, 2048 98.)
constexpr int kQueueWaves = 3072;
inline int queue_groups(int items, int threads) {
    const int most = kQueueWaves / (threads / 64);
    return items < most ? items : most;
}

// padded ladder size for n_nu, 0 if unsupported
int ladder_padded_size(int n_nu);
hipError_t launch_ladder_fp64(const LadderArgs &a, hipStream_t s);
// MFMA blocked Gauss-Jordan variant (n_nu <= 64)
int ladder_mfma_padded_size(int n_nu);
hipError_t launch_ladder_mfma_f64(const LadderArgs &a, hipStream_t s);
// certified pivot-free blocked Gauss-Jordan of the items in near_queue, uncertified ones
// going to queue
int ladder_gjb_padded_size(int n_nu);
bool ladder_gjb_has_occ3(int n_nu);
hipError_t launch_ladder_gjb(const LadderArgs &a, hipStream_t s);
// the same of every item (n_nu <= 64), uncertified ones by partial pivoting
hipError_t launch_ladder_all(const LadderArgs &a, hipStream_t s);
// after the screening: the same elimination of the items marked CERT_GENERAL, Gamma^(2) being
// in W, and the queue by partial pivoting
hipError_t launch_ladder_rest(const LadderArgs &a, hipStream_t s);
// work-groups of the kernel that the device holds at once
int resident_groups(const void *kern, int threads);
// the items in queue by partial pivoting
hipError_t launch_ladder_fp64_queue(const LadderArgs &a, hipStream_t s);
// mixed precision: FP32 certified sweep + one FP64 residual correction, and
// the FP32 sweep alone (n_nu <= 128); occ as above (refined: 0, 3 up to 96,
// 4 up to 64; FP32: 0, and 4, 5 up to 64)
int ladder_mixed_padded_size(int n_nu);
int ladder_fp32_padded_size(int n_nu);
bool ladder_mixed_has_occ(int n_nu, int occ);
bool ladder_fp32_has_occ(int n_nu, int occ);
hipError_t launch_ladder_mixed(const LadderArgs &a, int occ, int grid, hipStream_t s);
hipError_t launch_ladder_fp32(const LadderArgs &a, int occ, int grid, hipStream_t s);
// FP64 ladder of symmetric vertices (n_nu <= 128) behind its screening kernel,
// which leaves t = (gamma chi gamma)_nn in W, marks the certified items by whether their
// vertex is symmetric (cert) and queues the uncertified ones (queue)
int ladder_screen_blocks(int n_m, int n_q);
hipError_t launch_ladder_screen(const LadderArgs &a, hipStream_t s);
hipError_t launch_ladder_sym(const LadderArgs &a, hipStream_t s);
hipError_t launch_zero_ints(int *p, int n, hipStream_t s);
hipError_t launch_sym_tables(const SymTableArgs &a, hipStream_t s);
hipError_t launch_sym_expand(const SymExpandArgs &a, hipStream_t s);
hipError_t launch_lattice_fields(const LatticeFieldArgs &a, hipStream_t s);
hipError_t launch_lattice_chi_sum(const LatticeSumArgs &a, hipStream_t s);

}  // namespace df
