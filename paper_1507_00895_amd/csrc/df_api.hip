// C ABI of libdf: argument validation, workspace layout, launch sequencing,
// the self-consistency loop, its hipGraph capture and the fused
// multi-instance ladder launches.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>
#include <utility>
#include <vector>

#include "../../include/df.h"
#include "../../include/df_lattice.h"
#include "df_internal.hpp"
#include "df_lattice_ladder.hpp"
#include "df_pinned.hpp"
#include "df_tune.hpp"

using namespace df;

namespace {

constexpr size_t kAlign = 256;
constexpr int kMixBlocks = 512;
constexpr int kMaxClasses = 32;
// Layout of the ints region: per kernel class the uncertified-queue length,
// the near-queue length; then per instance the count of its ladders outside the radius.
constexpr int kIntsNear = kMaxClasses;
constexpr int kIntsInst = 2 * kMaxClasses;

size_t align_up(size_t x) { return (x + kAlign - 1) & ~(kAlign - 1); }

int ilog2_exact(int x) {
    if (x <= 0 || (x & (x - 1))) return -1;
    int l = 0;
    while ((1 << l) < x) ++l;
    return l;
}

struct Shape {
    int D, nk, lognk, N, n_nu, n_om;
    int chunk_len, n_chunks;
    int items;                        // 2 n_om N ladder items
    int im0;                          // bosonic index of Omega = 0
    int n_irr;                        // point-group orbits of the q-grid
    int items_sym;                    // 2 (n_om - im0) n_irr: symmetry-reduced ladder items
};

int check_inst(const df_inst_t &p, Shape *s) {
    if (p.D < 1 || p.D > 4) return DF_E_UNSUPPORTED;
    const int l = ilog2_exact(p.nk);
    if (l < 2 || l > 6) return DF_E_UNSUPPORTED;
    long N = 1;
    for (int a = 0; a < p.D; ++a) N *= p.nk;
    if (N > 4096) return DF_E_UNSUPPORTED;
    if (p.n_nu < 2 || (p.n_nu & 1)) return DF_E_INVAL;
    if (p.n_nu > 128) return DF_E_UNSUPPORTED;
    if (p.n_om < 1 || !(p.n_om & 1) || p.n_om > p.n_nu - 1) return DF_E_INVAL;
    if (!(p.beta > 0.0) || !isfinite(p.beta)) return DF_E_INVAL;
    s->D = p.D;
    s->nk = p.nk;
    s->lognk = l;
    s->N = (int)N;
    s->n_nu = p.n_nu;
    s->n_om = p.n_om;
    s->items = 2 * p.n_om * (int)N;
    s->im0 = (p.n_om - 1) / 2;
    // point-group orbits: sorted D-tuples of the nk / 2 + 1 values min(c, nk - c), i.e.
    // binomial(nk / 2 + D, D) (counting them took 20 us of every call at N = 4096)
    s->n_irr = 1;
    for (int a = 1; a <= p.D; ++a) s->n_irr = s->n_irr * (p.nk / 2 + a) / a;
    s->items_sym = 2 * (p.n_om - s->im0) * s->n_irr;
    // work-groups of the Schwinger-Dyson kernel: two N = 4096 arrays fit a CU (512 in
    // all; twice as many chunks cost 18 % at 64 x 64, n_nu 128: 88 -> 106 us with the
    // partial sums), smaller ones run four per CU (32 x 32, n_nu 64, n_om 31: 1024
    // work-groups 30.6 us, 512 34.6, 2048 38.5)
    const int target = s->N >= 4096 ? 512 : 1024;
    int nch = (target + p.n_nu - 1) / p.n_nu;
    if (nch > p.n_om) nch = p.n_om;
    if (nch < 1) nch = 1;
    s->chunk_len = (p.n_om + nch - 1) / nch;
    s->n_chunks = (p.n_om + s->chunk_len - 1) / s->chunk_len;
    return DF_OK;
}

// work-groups (and norm partials) of the mixing and Anderson kernels
int mix_blocks(const Shape &s) {
    const size_t count = (size_t)s.n_nu * s.N;
    int blocks = (int)((count + 255) / 256);
    return blocks > kMixBlocks ? kMixBlocks : blocks;
}

// sigma_calc in W's own memory: then no work-group may write it before all have read W
bool sigma_over_w(const df_inst_t &p, const Shape &s) {
    const uintptr_t a = (uintptr_t)p.sigma_calc, b = (uintptr_t)p.w;
    const size_t fld = (size_t)s.n_nu * s.N * 16;
    return a && b && a < b + 2 * s.n_om * fld && b < a + fld;
}

// The Schwinger-Dyson kernel writes sigma_calc (and mixes) itself: one chunk
bool sigma_one_pass(const df_inst_t &p, const Shape &s) { return s.n_chunks == 1 && !sigma_over_w(p, s); }

// norm partials of one iteration
int norm_parts(const df_inst_t &p, const Shape &s, int accel) {
    return accel > 0 || !sigma_one_pass(p, s) ? mix_blocks(s) : s.n_nu;
}

// Per-instance workspace regions (byte offsets from the instance base).
struct Layout {
    size_t gr, gdm, pdm, gtr, gp32, gtr32, gsym, gabs, symp, part, gd, chi, w;
    size_t qrep, qlist;               // symmetry tables: int[N] each
    size_t fx, xh, rh, accpart;       // Anderson acceleration (0 when unused)
    size_t total;
};

// slots: ring length of the Anderson acceleration, 0 for linear mixing
Layout layout_of(const Shape &s, int slots) {
    Layout L;
    const size_t cdb = 16;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes);
        return at;
    };
    const size_t fld = (size_t)s.n_nu * s.N * cdb;
    const size_t gam = 2 * (size_t)s.n_om * s.n_nu * s.n_nu * cdb;
    L.gr = take(fld);
    L.gdm = take(gam);
    L.pdm = take(gam);
    L.gtr = take(gam);
    L.gp32 = take(gam);              // (gamma, gamma_ij gamma_ji) as 4 floats
    L.gtr32 = take(gam / 2);
    L.gsym = take(gam);
    L.gabs = take(gam / 4);
    L.symp = take((size_t)s.n_om * kPrepChunks * 4 * sizeof(float));
    L.part = take((size_t)s.n_chunks * fld);
    L.gd = take(fld);
    L.chi = take((size_t)s.n_om * fld);
    L.w = take(2 * (size_t)s.n_om * fld);
    L.qrep = take((size_t)s.N * sizeof(int));
    L.qlist = take((size_t)s.N * sizeof(int));
    L.fx = L.xh = L.rh = L.accpart = 0;
    if (slots > 0) {
        L.fx = take(fld);
        L.xh = take((size_t)slots * fld);
        L.rh = take((size_t)slots * fld);
        L.accpart = take((size_t)kMixBlocks * kAccMaxSlots * sizeof(double));
    }
    L.total = o;
    return L;
}

// Workspace regions shared by all instances of a call.
struct Global {
    size_t table;                     // LadderInst[n_inst] (fused launches)
    size_t queue;                     // int[sum of items]: uncertified items
    size_t near;                      // int[sum of items]: refined kernel's items near the instability
    size_t cert;                      // uint8[sum of items]: what the FP64 screening found
    size_t ints;                      // int[kIntsInst + n_inst]: queue lengths, item counters,
                                      // outside counts
    size_t norms;                     // double[sum of mix_blocks][2]: norm partials, right after
                                      // the ints: one readback per iteration
    size_t accdots;                   // double[n_inst][kAccMaxSlots] (Anderson)
    size_t total;
};

struct Plan {
    std::vector<Shape> shape;
    std::vector<Layout> lay;
    std::vector<size_t> base;
    std::vector<size_t> norm0;        // first norm partial of each instance (doubles)
    size_t readback = 0;              // bytes of ints and norm partials
    Global g;
    size_t total = 0;
};

// accel: Anderson history depth of df_iterate (0: linear mixing); it sizes
// the extra workspace regions
int make_plan(const df_inst_t *inst, int32_t n_inst, Plan *P, int accel = 0) {
    if (!inst || n_inst < 1) return DF_E_INVAL;
    P->shape.resize(n_inst);
    P->lay.resize(n_inst);
    P->base.resize(n_inst);
    size_t off = 0;
    size_t items = 0;
    for (int i = 0; i < n_inst; ++i) {
        const int rc = check_inst(inst[i], &P->shape[i]);
        if (rc != DF_OK) return rc;
        P->lay[i] = layout_of(P->shape[i], accel > 0 ? accel + 1 : 0);
        P->base[i] = off;
        off = align_up(off + P->lay[i].total);
        items += (size_t)P->shape[i].items;
    }
    if (items > (size_t)0x7fffffff) return DF_E_UNSUPPORTED;
    Global &g = P->g;
    g.table = off;
    off = align_up(off + (size_t)n_inst * sizeof(LadderInst));
    g.queue = off;
    off = align_up(off + items * sizeof(int));
    g.near = off;
    off = align_up(off + items * sizeof(int));
    g.cert = off;
    off = align_up(off + items);
    g.ints = off;
    off += ((size_t)(kIntsInst + n_inst) * sizeof(int) + 7) & ~(size_t)7;
    g.norms = off;
    size_t norms = 0;
    P->norm0.clear();
    for (int i = 0; i < n_inst; ++i) {
        P->norm0.push_back(norms);
        norms += 2 * (size_t)std::max(mix_blocks(P->shape[i]), P->shape[i].n_nu);
    }
    off += norms * sizeof(double);
    P->readback = off - g.ints;
    off = align_up(off);
    g.accdots = off;
    off = align_up(off + (size_t)n_inst * kAccMaxSlots * sizeof(double));
    g.total = off;
    P->total = off;
    return DF_OK;
}

int check_ws(const Plan &P, void *ws, size_t ws_bytes) {
    if (!ws) return DF_E_WORKSPACE;
    if (((uintptr_t)ws) & (kAlign - 1)) return DF_E_WORKSPACE;
    if (ws_bytes < P.total) return DF_E_WORKSPACE;
    return DF_OK;
}

template <typename T> T *at(void *ws, size_t off) {
    return reinterpret_cast<T *>(static_cast<char *>(ws) + off);
}

Grid grid_of(const Shape &s) {
    Grid g;
    g.D = s.D;
    g.lognk = s.lognk;
    g.nk = s.nk;
    g.N = s.N;
    return g;
}

#define HIPCHK(x)                                  \
    do {                                           \
        hipError_t e_ = (x);                       \
        if (e_ != hipSuccess) return DF_E_HIP;     \
    } while (0)

// ---- ladder kernel choice ---------------------------------------------------
// In order: the variant named by DF_LADDER_KERNEL (any name of the variant
// table) when it serves this n_nu and precision; the autotuner's choice; the
// default, which is the certified pivot-free kernels on the matrix cores (FP64; FP32 +
// FP64 refinement in its three-wave build where there is one; FP32 in its four-wave
// build), whose uncertified items go to partial pivoting.
int env_variant() {
    static int v = -2;
    if (v == -2) {
        const char *e = getenv("DF_LADDER_KERNEL");
        v = e ? variant_from_name(e) : -1;
    }
    return v;
}

int default_variant(int n_nu, int prec) {
    if (prec == DF_FP32_REFINE) {
        if (ladder_mixed_has_occ(n_nu, 3)) return LV_MIXED_O3;
        return LV_MIXED;
    }
    if (prec == DF_FP32) {
        if (ladder_fp32_has_occ(n_nu, 4)) return LV_FP32_O4;
        return LV_FP32;
    }
    if (ladder_gjb_has_occ3(n_nu)) return LV_GJB_O3;
    if (ladder_gjb_padded_size(n_nu) != 0) return LV_GJB;
    return LV_VECTOR;
}

int ladder_variant(int n_nu, int prec) {
    const int e = env_variant();
    if (e >= 0 && variant_supports(e, n_nu, prec)) return e;
    const int t = tuned_variant(prec, n_nu);
    if (t >= 0 && variant_supports(t, n_nu, prec)) return t;
    return default_variant(n_nu, prec);
}

// Instances that share a kernel build, its padded size and launch shape are
// fused in one launch.
// The certified FP64 choices all run the symmetric kernel, built per 16
// frequencies.
bool fp64_certified(int v) { return v == LV_GJB || v == LV_GJB_O3 || v == LV_GJB_O4; }

// Small FP64 launches skip the screening and the symmetric kernel: every item is
// certified and eliminated, or pivoted, in one kernel.  While the items' waves (one per 16
// frequencies) do not fill the SIMDs' three places each, what counts is the chain of a
// launch: screening, block ladder and the rest are three of them.  df_ladder_solve, us,
// symmetric vertex, with the screening / without it:
//   n_nu 16   128 items 19 / 14   2,560 22 / 16   14,336 56 / 53   30,720 89 / 89   122,880 291 / 323
//   n_nu 32   128 items 22 / 14     640 26 / 17    1,152 28 / 23    2,560 36 / 40
//   n_nu 48   128 items 30 / 21     640 41 / 32      896 41 / 36    1,152 42 / 52
//   n_nu 64   128 items 38 / 28     384 46 / 41      640 47 / 49      896 58 / 66
// (general vertices gain up to larger counts: n_nu 64, 896 items 76 / 66; n_nu 80 and above
// gain from the screening at any count: 128 items 59 without, 51 with it)
bool fp64_direct(int n_nu, int items) {
    const int nt = (n_nu + 15) / 16;
    return nt == 1 ? items <= 32768 : nt <= 4 && items * nt <= 2560;
}

int ladder_class(int n_nu, int prec) {
    const int v = ladder_variant(n_nu, prec);
    if (fp64_certified(choice_variant(v))) return LV_GJB * 256 + (n_nu + 15) / 16 * 16;
    return v * 256 + variant_padded_size(v, n_nu);
}

// Queues and counters of one kernel class in the workspace.
struct ClassSlots {
    int *queue, *queue_count;         // uncertified items -> pivoting kernel
    int *near, *near_count;           // refined kernel: items near the instability -> FP64 kernel
    uint8_t *cert;                    // FP64 screening: CERT_* of the items
};

ClassSlots class_slots(void *ws, const Global &g, int cls, size_t queue_off) {
    int *ints = at<int>(ws, g.ints);
    ClassSlots c;
    c.queue = at<int>(ws, g.queue) + queue_off;
    c.near = at<int>(ws, g.near) + queue_off;
    c.cert = at<uint8_t>(ws, g.cert) + queue_off;
    c.queue_count = ints + cls;
    c.near_count = ints + kIntsNear + cls;
    return c;
}

// Launch the ladder for the items in a (single instance, or a fused table)
// with choice c.  The FP32 kernel and the screening of the FP64 class queue their
// uncertified items, the refined kernel its items near the instability too; the certified
// elimination (of those, or of the general vertices' items) and the pivoting follow.  The class's counters must be zero before the call.
int launch_ladder_variant(int c, LadderArgs a, const ClassSlots &q, hipStream_t st) {
    const int v = choice_variant(c);
    switch (v) {
        case LV_VECTOR: HIPCHK(launch_ladder_fp64(a, st)); return DF_OK;
        case LV_MFMA: HIPCHK(launch_ladder_mfma_f64(a, st)); return DF_OK;
        default: break;
    }
    a.queue = q.queue;
    a.queue_count = q.queue_count;
    a.cert = q.cert;
    a.near_count = q.near_count;
    const int grid = a.n_items;
    const bool refined = (v == LV_MIXED || v == LV_MIXED_O3 || v == LV_MIXED_O4);
    if (refined) a.near_queue = q.near;
    switch (v) {
        case LV_FP32: HIPCHK(launch_ladder_fp32(a, 0, grid, st)); break;
        case LV_FP32_O4: HIPCHK(launch_ladder_fp32(a, 4, grid, st)); break;
        case LV_FP32_O5: HIPCHK(launch_ladder_fp32(a, 5, grid, st)); break;
        case LV_MIXED: HIPCHK(launch_ladder_mixed(a, 0, grid, st)); break;
        case LV_MIXED_O3: HIPCHK(launch_ladder_mixed(a, 3, grid, st)); break;
        case LV_MIXED_O4: HIPCHK(launch_ladder_mixed(a, 4, grid, st)); break;
        default:
            if (fp64_direct(a.n_nu, a.n_items)) {
                HIPCHK(launch_ladder_all(a, st));
                return DF_OK;
            }
            // the items are screened (certificate, Gamma^(2)); the certified ones
            // of symmetric vertices run in the symmetric kernel
            HIPCHK(launch_ladder_screen(a, st));
            HIPCHK(launch_ladder_sym(a, st));
            HIPCHK(launch_ladder_rest(a, st));
            return DF_OK;
    }
    if (refined) HIPCHK(launch_ladder_gjb(a, st));
    HIPCHK(launch_ladder_fp64_queue(a, st));
    return DF_OK;
}

// ---- per-instance stages -----------------------------------------------------
int stage_dual_gf(const df_inst_t &p, const Shape &s, const double *sigma, double *gd,
                  double *gr, hipStream_t st) {
    DualGfArgs a{};
    a.grid = grid_of(s);
    a.n_nu = s.n_nu;
    a.g = p.g;
    a.delta = p.delta;
    a.eps = p.eps;
    a.sigma = sigma;
    a.gd_out = gd;
    a.gr_out = gr;
    a.from_gd = 0;
    HIPCHK(launch_dual_gf(a, st));
    return DF_OK;
}

int stage_transform_gd(const Shape &s, const double *gd, double *gr, hipStream_t st) {
    DualGfArgs a{};
    a.grid = grid_of(s);
    a.n_nu = s.n_nu;
    a.gd_in = gd;
    a.gr_out = gr;
    a.from_gd = 1;
    HIPCHK(launch_dual_gf(a, st));
    return DF_OK;
}

int stage_bubble(const df_inst_t &p, const Shape &s, const double *gr, double *chi,
                 int *zero, int n_zero, hipStream_t st) {
    BubbleArgs a{};
    a.grid = grid_of(s);
    a.n_nu = s.n_nu;
    a.n_om = s.n_om;
    a.beta = p.beta;
    a.gr = gr;
    a.chi = chi;
    a.zero = zero;
    a.n_zero = n_zero;
    HIPCHK(launch_bubble(a, st));
    return DF_OK;
}

// zero: the call's counters are cleared too (the ladder launches follow on the stream)
int stage_gamma_prep(const df_inst_t &p, const Plan &P, int i, void *ws, bool zero, hipStream_t st) {
    const Shape &s = P.shape[i];
    const Layout &L = P.lay[i];
    const size_t base = P.base[i];
    GammaPrepArgs a{};
    a.n_nu = s.n_nu;
    a.n_om = s.n_om;
    a.guu = p.gamma_uu;
    a.gud = p.gamma_ud;
    a.gdm = at<double>(ws, base + L.gdm);
    a.pdm = at<double>(ws, base + L.pdm);
    a.gtr = at<double>(ws, base + L.gtr);
    a.gp32 = at<float>(ws, base + L.gp32);
    a.gtr32 = at<float>(ws, base + L.gtr32);
    a.gsym = at<double>(ws, base + L.gsym);
    a.gabs = at<float>(ws, base + L.gabs);
    a.symp = at<float>(ws, base + L.symp);
    if (zero) {
        a.zero = at<int>(ws, P.g.ints);
        a.n_zero = kIntsInst + (int)P.shape.size();
    }
    HIPCHK(launch_gamma_prep(a, st));
    return DF_OK;
}

// Sigma~ from W: sigma_calc and, with sigma given, the mixing step and its norm
// partials.  One launch, or two where the bosonic frequencies are split into chunks.
// sym: only the symmetry-reduced entries of W are valid (its tables in the workspace).
int stage_sigma(const df_inst_t &p, const Shape &s, void *ws, size_t base, const Layout &L,
                const double *w, bool sym, double *sigma_calc, double *sigma, double alpha,
                double *norm, hipStream_t st) {
    SigmaArgs a{};
    a.grid = grid_of(s);
    a.n_nu = s.n_nu;
    a.n_om = s.n_om;
    a.chunk_len = s.chunk_len;
    a.n_chunks = s.n_chunks;
    a.beta = p.beta;
    a.w = w;
    a.gr = at<double>(ws, base + L.gr);
    a.part = at<double>(ws, base + L.part);
    if (sym) a.qrep = at<int>(ws, base + L.qrep);
    a.im0 = s.im0;
    a.alpha = alpha;
    a.sigma_calc = sigma_calc;
    a.sigma = sigma;
    a.norm_part = norm;
    a.one_pass = sigma_one_pass(p, s);
    HIPCHK(launch_sigma_part(a, st));
    if (a.one_pass) return DF_OK;
    ReduceMixArgs r{};
    r.count = (size_t)s.n_nu * s.N;
    r.n_chunks = s.n_chunks;
    r.alpha = alpha;
    r.part = a.part;
    r.sigma_calc = sigma_calc;
    r.sigma = sigma;
    r.norm_part = norm;
    HIPCHK(launch_reduce_mix(r, mix_blocks(s), st));
    return DF_OK;
}

double *norm_part(const Plan &P, void *ws, int i) { return at<double>(ws, P.g.norms) + P.norm0[i]; }

// diff = sqrt(sum |new - old|^2 / sum |new|^2) from the n block partials of the
// mixing kernels, in a fixed order; false if a sum is not finite.  (On the host: the
// partials are read back with the counters, a launch less per iteration.)
bool norm_diff(const double *part, int n, double *diff) {
    double d[256] = {}, m[256] = {};
    for (int i = 0; i < n; ++i) {
        d[i % 256] += part[2 * i];
        m[i % 256] += part[2 * i + 1];
    }
    for (int s = 128; s > 0; s >>= 1)
        for (int i = 0; i < s; ++i) {
            d[i] += d[i + s];
            m[i] += m[i + s];
        }
    if (m[0] == 0.0) *diff = d[0] == 0.0 ? 0.0 : INFINITY;
    else *diff = sqrt(d[0] / m[0]);
    return isfinite(d[0]) && isfinite(m[0]);
}

// Page-locked host memory for one call's readbacks (into pageable memory the runtime
// stages every copy: two of them took 25 us of an 87 us iteration), leased from a bounded
// pool.  Without page-locked memory the lease falls back to ordinary memory.
void *pinned_alloc(size_t bytes) {
    void *p = nullptr;
    if (hipHostMalloc(&p, bytes, hipHostMallocPortable) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}
void pinned_release(void *p) { (void)hipHostFree(p); }
PinnedPool g_pinned(pinned_alloc, pinned_release);

class PinnedLease {
public:
    explicit PinnedLease(size_t bytes) {
        p_ = g_pinned.take(bytes, &cap_);
        if (!p_) plain_.resize(bytes);
    }
    ~PinnedLease() {
        // (after a failed call a copy may still be on its way into the buffer: it is
        // given up)
        if (p_ && idle_) g_pinned.give(p_, cap_);
    }
    PinnedLease(const PinnedLease &) = delete;
    PinnedLease &operator=(const PinnedLease &) = delete;
    char *data() { return p_ ? static_cast<char *>(p_) : plain_.data(); }
    // n bytes from device memory to offset off, and the wait for it
    bool read(size_t off, const void *dev, size_t n, hipStream_t st) {
        idle_ = false;
        if (hipMemcpyAsync(data() + off, dev, n, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return false;
        idle_ = true;
        return true;
    }

private:
    void *p_ = nullptr;
    size_t cap_ = 0;
    bool idle_ = true;
    std::vector<char> plain_;
};

bool ladder_prec(int prec) { return prec == DF_FP64 || prec == DF_FP32_REFINE || prec == DF_FP32; }

// need_loop: df_iterate's fields are checked too; adaptive: DF_ADAPTIVE allowed
constexpr int kMaxGraphUnroll = 64;

int check_opts(const df_opts_t *o, bool need_loop, bool adaptive) {
    if (!o) return need_loop ? DF_E_INVAL : DF_OK;
    if (!ladder_prec(o->prec) && !(adaptive && o->prec == DF_ADAPTIVE)) return DF_E_INVAL;
    if (o->accel < 0 || o->accel > kAccMaxSlots - 1 || !isfinite(o->switch_tol)) return DF_E_INVAL;
    if (o->symmetry != 0 && o->symmetry != 1) return DF_E_INVAL;
    if (o->graph_unroll < 0 || o->graph_unroll > kMaxGraphUnroll) return DF_E_INVAL;
    if (need_loop) {
        if (!(o->mix > 0.0 && o->mix <= 1.0)) return DF_E_INVAL;
        if (o->max_iter < 1) return DF_E_INVAL;
        if (!isfinite(o->tol)) return DF_E_INVAL;
    }
    return DF_OK;
}

// ---- symmetry reduction ---------------------------------------------------------
int stage_sym_tables(const Shape &s, void *ws, size_t base, const Layout &L, hipStream_t st) {
    SymTableArgs a{};
    a.D = s.D;
    a.lognk = s.lognk;
    a.N = s.N;
    a.qrep = at<int>(ws, base + L.qrep);
    a.qlist = at<int>(ws, base + L.qlist);
    HIPCHK(launch_sym_tables(a, st));
    return DF_OK;
}

int stage_sym_expand(const Shape &s, void *ws, size_t base, const Layout &L, double *w,
                     double *logdet, int8_t *status, hipStream_t st) {
    SymExpandArgs a{};
    a.n_nu = s.n_nu;
    a.n_om = s.n_om;
    a.N = s.N;
    a.im0 = s.im0;
    a.qrep = at<int>(ws, base + L.qrep);
    a.w = w;
    a.logdet = logdet;
    a.status = status;
    HIPCHK(launch_sym_expand(a, st));
    return DF_OK;
}

// ---- the fused multi-instance iteration --------------------------------------
struct FusedClass {
    int variant;
    int n_nu;                         // any member's n_nu (same padded size)
    int t0, t1;                       // table range
    int items;                        // total items of the class
    int sblocks;                      // work-groups of its screening launch
    size_t queue_off;                 // first queue slot (ints)
    int full;                         // every member's n_nu equals the padded size
    int full_sym;                     // every member's n_nu is the class's multiple of 16
};

struct Fused {
    std::vector<int> active;          // instance indices, in table order
    std::vector<FusedClass> cls;
    std::vector<LadderInst> table;    // host copy of the device table
};

// One entry of the device table: the instance's ladder inputs in the workspace,
// its outputs, and its position in the launch (items, screening work-groups).
LadderInst table_entry(const Plan &P, int i, void *ws, bool sym, const double *chi, double *w,
                       double *logdet, int8_t *status, int *items, int *sblocks) {
    const Shape &s = P.shape[i];
    const Layout &L = P.lay[i];
    const size_t b = P.base[i];
    LadderInst d{};
    d.gdm = at<double>(ws, b + L.gdm);
    d.pdm = at<double>(ws, b + L.pdm);
    d.gtr = at<double>(ws, b + L.gtr);
    d.gp32 = at<float>(ws, b + L.gp32);
    d.gtr32 = at<float>(ws, b + L.gtr32);
    d.gsym = at<double>(ws, b + L.gsym);
    d.gabs = at<float>(ws, b + L.gabs);
    d.symp = at<float>(ws, b + L.symp);
    d.chi = chi;
    d.w = w;
    d.logdet = logdet;
    d.status = status;
    d.count = at<int>(ws, P.g.ints) + kIntsInst + i;
    d.n_nu = s.n_nu;
    d.n_om = s.n_om;
    d.N = s.N;
    d.item0 = *items;
    d.sblk0 = *sblocks;
    if (sym) {
        d.qlist = at<int>(ws, b + L.qlist);
        d.n_q = s.n_irr;
        d.im0 = s.im0;
    }
    *items += sym ? s.items_sym : s.items;
    *sblocks += ladder_screen_blocks(s.n_om - (sym ? s.im0 : 0), sym ? s.n_irr : s.N);
    return d;
}

// Group the active instances by ladder class and write the device table.
// Ordinary (not captured) stream work, synchronised before returning.
int build_fused(const df_inst_t *inst, const Plan &P, const std::vector<int> &act,
                const std::vector<int> &prec, bool sym, void *ws, Fused *F, hipStream_t st) {
    F->active.clear();
    F->cls.clear();
    F->table.clear();
    std::vector<int> keys;
    for (int i : act) {
        const int key = ladder_class(P.shape[i].n_nu, prec[i]);
        bool seen = false;
        for (int k : keys) seen = seen || (k == key);
        if (!seen) keys.push_back(key);
    }
    if ((int)keys.size() > kMaxClasses) return DF_E_UNSUPPORTED;
    size_t qoff = 0;
    for (int key : keys) {
        FusedClass c{};
        c.t0 = (int)F->table.size();
        c.items = 0;
        c.sblocks = 0;
        c.queue_off = qoff;
        c.full = 1;
        c.full_sym = 1;
        for (int i : act) {
            if (ladder_class(P.shape[i].n_nu, prec[i]) != key) continue;
            const Shape &s = P.shape[i];
            const Layout &L = P.lay[i];
            const size_t b = P.base[i];
            F->table.push_back(table_entry(P, i, ws, sym,
                                           inst[i].chi ? inst[i].chi : at<double>(ws, b + L.chi),
                                           inst[i].w ? inst[i].w : at<double>(ws, b + L.w),
                                           inst[i].logdet, inst[i].status, &c.items, &c.sblocks));
            c.n_nu = s.n_nu;
            if (s.n_nu != ladder_gjb_padded_size(s.n_nu)) c.full = 0;
            if (s.n_nu % 16) c.full_sym = 0;
            c.variant = ladder_variant(s.n_nu, prec[i]);
            F->active.push_back(i);
        }
        c.t1 = (int)F->table.size();
        qoff += (size_t)c.items;
        F->cls.push_back(c);
    }
    HIPCHK(hipMemcpyAsync(at<LadderInst>(ws, P.g.table), F->table.data(),
                          F->table.size() * sizeof(LadderInst), hipMemcpyHostToDevice, st));
    HIPCHK(hipStreamSynchronize(st));
    return DF_OK;
}

// Queue one outer iteration of the active instances (capturable).
int queue_fused_iteration(const df_inst_t *inst, const Plan &P, const Fused &F,
                          const df_opts_t &o, void *ws, hipStream_t st) {
    int rc;
    for (int i : F.active) {
        const Shape &s = P.shape[i];
        const Layout &L = P.lay[i];
        const size_t b = P.base[i];
        double *gr = at<double>(ws, b + L.gr);
        double *gd = inst[i].gd ? inst[i].gd : at<double>(ws, b + L.gd);
        double *chi = inst[i].chi ? inst[i].chi : at<double>(ws, b + L.chi);
        rc = stage_dual_gf(inst[i], s, inst[i].sigma, gd, gr, st);
        if (rc != DF_OK) return rc;
        // (the first bubble also clears the counters of the ladder launches)
        const bool first = i == F.active[0];
        rc = stage_bubble(inst[i], s, gr, chi, first ? at<int>(ws, P.g.ints) : nullptr,
                          first ? kIntsInst + (int)P.shape.size() : 0, st);
        if (rc != DF_OK) return rc;
    }
    for (size_t c = 0; c < F.cls.size(); ++c) {
        const FusedClass &k = F.cls[c];
        LadderArgs a{};
        a.insts = at<LadderInst>(ws, P.g.table) + k.t0;
        a.n_insts = k.t1 - k.t0;
        a.n_nu = k.n_nu;
        a.full = k.full;
        a.full_sym = k.full_sym;
        a.item0 = 0;
        a.n_items = k.items;
        a.n_sblk = k.sblocks;
        rc = launch_ladder_variant(k.variant, a, class_slots(ws, P.g, (int)c, k.queue_off), st);
        if (rc != DF_OK) return rc;
    }
    for (int i : F.active) {
        const Shape &s = P.shape[i];
        const Layout &L = P.lay[i];
        const size_t b = P.base[i];
        const double *w = inst[i].w ? inst[i].w : at<double>(ws, b + L.w);
        bool sym = o.symmetry != 0;
        if (sym && sigma_over_w(inst[i], s)) {
            // sigma_calc lies over W: W is completed first, not after the loop
            rc = stage_sym_expand(s, ws, b, L, inst[i].w, inst[i].logdet, inst[i].status, st);
            if (rc != DF_OK) return rc;
            sym = false;
        }
        // (accelerated: F(x) only, the step follows outside this sequence)
        if (o.accel > 0)
            rc = stage_sigma(inst[i], s, ws, b, L, w, sym, at<double>(ws, b + L.fx), nullptr,
                             0.0, nullptr, st);
        else
            rc = stage_sigma(inst[i], s, ws, b, L, w, sym, inst[i].sigma_calc, inst[i].sigma,
                             o.mix, norm_part(P, ws, i), st);
        if (rc != DF_OK) return rc;
    }
    return DF_OK;
}

// ---- Anderson acceleration, host side -----------------------------------------
// State of one instance: how many residuals are recorded since the last
// reset (slots fill 0, 1, ... and then wrap), and the Gram matrix of the
// recorded residuals, Re <r_i, r_j>, indexed by slot.
struct AccState {
    int recorded = 0;
    std::vector<double> gram;
};

// Solve the n x n system A y = b in place (partial pivoting); false if singular.
bool small_solve(std::vector<double> &A, std::vector<double> &b, int n) {
    for (int c = 0; c < n; ++c) {
        int piv = c;
        for (int r = c + 1; r < n; ++r)
            if (fabs(A[r * n + c]) > fabs(A[piv * n + c])) piv = r;
        if (!(fabs(A[piv * n + c]) > 0.0) || !isfinite(A[piv * n + c])) return false;
        if (piv != c) {
            for (int k = 0; k < n; ++k) std::swap(A[c * n + k], A[piv * n + k]);
            std::swap(b[c], b[piv]);
        }
        for (int r = c + 1; r < n; ++r) {
            const double f = A[r * n + c] / A[c * n + c];
            for (int k = c; k < n; ++k) A[r * n + k] -= f * A[c * n + k];
            b[r] -= f * b[c];
        }
    }
    for (int c = n - 1; c >= 0; --c) {
        double v = b[c];
        for (int k = c + 1; k < n; ++k) v -= A[c * n + k] * b[k];
        b[c] = v / A[c * n + c];
        if (!isfinite(b[c])) return false;
    }
    return true;
}

// Weights c_j of the accelerated iterate x' = sum_j c_j (x_j + alpha r_j) over
// the recorded slots: least squares of the newest residual against the
// differences of consecutive residuals (real coefficients).  Returns false
// (and the plain mixing step) when the system is singular.
bool acc_weights(const AccState &S, int slots, int newest, double *coef) {
    const int h = S.recorded < slots ? S.recorded : slots;   // slots in use
    for (int j = 0; j < kAccMaxSlots; ++j) coef[j] = 0.0;
    coef[newest] = 1.0;
    if (h < 2) return true;
    std::vector<int> ord(h);                                  // oldest .. newest
    for (int a = 0; a < h; ++a) ord[a] = ((newest - (h - 1 - a)) % slots + slots) % slots;
    const int n = h - 1;
    auto G = [&](int i, int j) { return S.gram[ord[i] * slots + ord[j]]; };
    std::vector<double> A((size_t)n * n), rhs(n);
    double tr = 0.0;
    for (int a = 0; a < n; ++a) {
        for (int c = 0; c < n; ++c)
            A[a * n + c] = G(a + 1, c + 1) - G(a + 1, c) - G(a, c + 1) + G(a, c);
        rhs[a] = G(a + 1, h - 1) - G(a, h - 1);
        tr += A[a * n + a];
    }
    const double lam = 1e-12 * (tr > 0.0 ? tr / n : 1.0);
    for (int a = 0; a < n; ++a) A[a * n + a] += lam;
    if (!small_solve(A, rhs, n)) return false;
    // x' = x_newest - sum_a y_a (x_{a+1} - x_a), same weights for r
    coef[newest] = 0.0;
    for (int a = 0; a < h; ++a) {
        double c = 0.0;
        if (a < n) c += rhs[a];
        if (a > 0) c -= rhs[a - 1];
        if (a == h - 1) c += 1.0;
        coef[ord[a]] = c;
    }
    return true;
}

// ---- lattice observables (df_lattice.h) ---------------------------------------
struct LatticeLayout {
    size_t fields, gr;                // [3][n_nu][N] each: G~, frak G, G_lat; their transforms
    size_t bub;                       // [3][n_nu][N]: their chi~, L, bubble
    size_t w;                         // gamma L [2][n_nu][N]
    size_t gdm, gtr, gsym, gabs, symp;   // vertex at Omega = 0
    size_t cert, queue, count, lad;
    size_t total;
};

// The size is what the interface has always asked for, seven fields, [2][N] and up to 512
// n_nu x (n_nu + 1) matrices: a workspace of that size stays good.  Where it is too small for
// regions of their own, the bubbles take the place of the fields and gamma L that of the
// transforms, which are not needed any more (32x32, n_nu 64: 1.7 us slower).
LatticeLayout lattice_layout_of(const Shape &s) {
    const size_t fld = (size_t)s.n_nu * s.N * 16, gam = 2 * (size_t)s.n_nu * s.n_nu * 16;
    size_t asked = 0;
    for (int f = 0; f < 7; ++f) asked += align_up(fld);
    asked += align_up(2 * (size_t)s.N * 16);
    const size_t matrices = 2 * s.N < 512 ? 2 * (size_t)s.N : 512;
    asked += align_up(matrices * s.n_nu * (s.n_nu + 1) * 16);
    LatticeLayout L;
    for (const bool apart : {true, false}) {
        size_t o = 0;
        auto take = [&](size_t bytes) {
            size_t at = o;
            o = (o + bytes + 15) & ~(size_t)15;
            return at;
        };
        L.fields = take(3 * fld);
        L.gr = take(3 * fld);
        L.bub = apart ? take(3 * fld) : L.fields;
        L.w = apart ? take(2 * fld) : L.gr;
        L.gdm = take(gam);
        L.gtr = take(gam);
        L.gsym = take(gam);
        L.gabs = take(gam / 4);
        L.symp = take((size_t)prep_chunks(s.n_nu) * 4 * sizeof(float));
        L.queue = take(2 * (size_t)s.N * sizeof(int));
        L.cert = take(2 * (size_t)s.N);
        L.count = take(sizeof(int));
        L.lad = take(2 * (size_t)s.N * 16);
        L.total = o > asked ? o : asked;
        if (o <= asked) break;
    }
    return L;
}

}  // namespace

extern "C" {

int df_version(void) { return 100; }

const char *df_strerror(int code) {
    switch (code) {
        case DF_OK: return "success";
        case DF_E_INVAL: return "invalid argument";
        case DF_E_UNSUPPORTED: return "unsupported shape (D in 1..4, nk power of two in [4,64], nk^D <= 4096, n_nu <= 128)";
        case DF_E_WORKSPACE: return "workspace missing, misaligned (256 B) or too small";
        case DF_E_HIP: return "HIP runtime error";
        case DF_E_NONFINITE: return "dual self-energy became non-finite";
        case DF_E_NOT_CONVERGED: return "iteration limit reached before the tolerance";
        case DF_W_FALLBACK: return "success; some ladders were outside the convergence radius";
        default: return "unknown status code";
    }
}

int df_workspace_size(const df_inst_t *inst, int32_t n_inst, const df_opts_t *opts, size_t *bytes) {
    if (!bytes) return DF_E_INVAL;
    int rc = check_opts(opts, false, true);
    if (rc != DF_OK) return rc;
    Plan P;
    rc = make_plan(inst, n_inst, &P, opts ? opts->accel : 0);
    if (rc != DF_OK) return rc;
    *bytes = P.total;
    return DF_OK;
}

int df_dual_gf(const df_inst_t *inst, int32_t n_inst, void *ws, size_t ws_bytes, df_stream_t stream) {
    Plan P;
    int rc = make_plan(inst, n_inst, &P);
    if (rc != DF_OK) return rc;
    rc = check_ws(P, ws, ws_bytes);
    if (rc != DF_OK) return rc;
    for (int i = 0; i < n_inst; ++i)
        if (!inst[i].g || !inst[i].delta || !inst[i].eps || !inst[i].gd) return DF_E_INVAL;
    hipStream_t st = (hipStream_t)stream;
    for (int i = 0; i < n_inst; ++i) {
        rc = stage_dual_gf(inst[i], P.shape[i], inst[i].sigma, inst[i].gd, nullptr, st);
        if (rc != DF_OK) return rc;
    }
    return DF_OK;
}

int df_bubble(const df_inst_t *inst, int32_t n_inst, void *ws, size_t ws_bytes, df_stream_t stream) {
    Plan P;
    int rc = make_plan(inst, n_inst, &P);
    if (rc != DF_OK) return rc;
    rc = check_ws(P, ws, ws_bytes);
    if (rc != DF_OK) return rc;
    for (int i = 0; i < n_inst; ++i)
        if (!inst[i].gd || !inst[i].chi) return DF_E_INVAL;
    hipStream_t st = (hipStream_t)stream;
    for (int i = 0; i < n_inst; ++i) {
        const Shape &s = P.shape[i];
        double *gr = at<double>(ws, P.base[i] + P.lay[i].gr);
        rc = stage_transform_gd(s, inst[i].gd, gr, st);
        if (rc != DF_OK) return rc;
        rc = stage_bubble(inst[i], s, gr, inst[i].chi, nullptr, 0, st);
        if (rc != DF_OK) return rc;
    }
    return DF_OK;
}

}  // extern "C"

// ---- df_bubble without a workspace --------------------------------------------
// The one scratch buffer of df_bubble, G~(r) of one instance ([n_nu][N]
// complex), lives in a file-scope device array: 8 MiB, the size at n_nu = 128
// and N = 4096, so every supported shape fits.  Each device holds its own copy
// for the life of the process; host code reaches it only through the address
// hipGetSymbolAddress returns for that device.
namespace {

constexpr size_t kBubbleScratchBytes = (size_t)128 * 4096 * 16;
__device__ __align__(256) unsigned char scratch[kBubbleScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_addr[kMaxDevices] = {};

// The scratch array's address on the current device, looked up once per device.
int scratch_address(void **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return DF_E_HIP;
    if (dev < 0 || dev >= kMaxDevices) return DF_E_UNSUPPORTED;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DF_E_HIP;
        g_scratch_addr[dev] = p;
    }
    *out = g_scratch_addr[dev];
    return DF_OK;
}

}  // namespace

extern "C" {

int df_bubble_noalloc(const df_inst_t *inst, int32_t n_inst, df_stream_t stream) {
    if (!inst || n_inst < 1) return DF_E_INVAL;
    for (int i = 0; i < n_inst; ++i) {
        Shape s;
        const int rc = check_inst(inst[i], &s);
        if (rc != DF_OK) return rc;
        if (!inst[i].gd || !inst[i].chi) return DF_E_INVAL;
        if ((size_t)s.n_nu * s.N * 16 > kBubbleScratchBytes) return DF_E_WORKSPACE;
    }
    void *scr = nullptr;
    int rc = scratch_address(&scr);
    if (rc != DF_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    double *gr = static_cast<double *>(scr);
    // instances in turn on one stream: each overwrites the whole G~(r) it reads
    for (int i = 0; i < n_inst; ++i) {
        Shape s;
        (void)check_inst(inst[i], &s);
        rc = stage_transform_gd(s, inst[i].gd, gr, st);
        if (rc != DF_OK) return rc;
        rc = stage_bubble(inst[i], s, gr, inst[i].chi, nullptr, 0, st);
        if (rc != DF_OK) return rc;
    }
    return DF_OK;
}

int df_ladder_solve(const df_inst_t *inst, int32_t n_inst, const df_opts_t *opts, void *ws,
                    size_t ws_bytes, df_stream_t stream) {
    int rc = check_opts(opts, false, false);
    if (rc != DF_OK) return rc;
    Plan P;
    rc = make_plan(inst, n_inst, &P);
    if (rc != DF_OK) return rc;
    rc = check_ws(P, ws, ws_bytes);
    if (rc != DF_OK) return rc;
    for (int i = 0; i < n_inst; ++i)
        if (!inst[i].gamma_uu || !inst[i].gamma_ud || !inst[i].chi || !inst[i].w) return DF_E_INVAL;
    hipStream_t st = (hipStream_t)stream;
    const int prec = opts ? opts->prec : DF_FP64;
    const bool sym = opts && opts->symmetry;
    int *ints = at<int>(ws, P.g.ints);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) return DF_E_HIP;
    if (n_inst > 1 && cap == hipStreamCaptureStatusNone) {
        // several instances, not captured: the fused launches of df_iterate (one
        // per kernel class over a device table of the instances)
        std::vector<int> act(n_inst), pr(n_inst, prec);
        for (int i = 0; i < n_inst; ++i) {
            act[i] = i;
            rc = stage_gamma_prep(inst[i], P, i, ws, i == 0, st);
            if (rc == DF_OK && sym) rc = stage_sym_tables(P.shape[i], ws, P.base[i], P.lay[i], st);
            if (rc != DF_OK) return rc;
        }
        Fused F;
        rc = build_fused(inst, P, act, pr, sym, ws, &F, st);
        if (rc != DF_OK) return rc;
        for (size_t c = 0; c < F.cls.size(); ++c) {
            const FusedClass &k = F.cls[c];
            LadderArgs a{};
            a.insts = at<LadderInst>(ws, P.g.table) + k.t0;
            a.n_insts = k.t1 - k.t0;
            a.n_nu = k.n_nu;
            a.full = k.full;
            a.full_sym = k.full_sym;
            a.item0 = 0;
            a.n_items = k.items;
            a.n_sblk = k.sblocks;
            rc = launch_ladder_variant(k.variant, a, class_slots(ws, P.g, (int)c, k.queue_off), st);
            if (rc != DF_OK) return rc;
        }
        if (sym)
            for (int i = 0; i < n_inst; ++i) {
                rc = stage_sym_expand(P.shape[i], ws, P.base[i], P.lay[i], inst[i].w, inst[i].logdet,
                                      inst[i].status, st);
                if (rc != DF_OK) return rc;
            }
        return DF_OK;
    }
    // one launch per instance with plain kernel arguments (capturable)
    for (int i = 0; i < n_inst; ++i) {
        const Shape &s = P.shape[i];
        const Layout &L = P.lay[i];
        const size_t b = P.base[i];
        rc = stage_gamma_prep(inst[i], P, i, ws, true, st);
        if (rc != DF_OK) return rc;
        LadderArgs a{};
        a.gdm = at<double>(ws, b + L.gdm);
        a.pdm = at<double>(ws, b + L.pdm);
        a.gtr = at<double>(ws, b + L.gtr);
        a.gp32 = at<float>(ws, b + L.gp32);
        a.gtr32 = at<float>(ws, b + L.gtr32);
        a.gsym = at<double>(ws, b + L.gsym);
        a.gabs = at<float>(ws, b + L.gabs);
        a.symp = at<float>(ws, b + L.symp);
        a.n_sblk = ladder_screen_blocks(s.n_om - (sym ? s.im0 : 0), sym ? s.n_irr : s.N);
        a.chi = inst[i].chi;
        a.w = inst[i].w;
        a.logdet = inst[i].logdet;
        a.status = inst[i].status;
        a.fallback_count = ints + kIntsInst + i;
        a.n_nu = s.n_nu;
        a.n_om = s.n_om;
        a.N = s.N;
        a.full = s.n_nu == ladder_gjb_padded_size(s.n_nu);
        a.full_sym = s.n_nu % 16 == 0;
        a.item0 = 0;
        a.n_items = s.items;
        if (sym) {
            rc = stage_sym_tables(s, ws, b, L, st);
            if (rc != DF_OK) return rc;
            a.qlist = at<int>(ws, b + L.qlist);
            a.n_q = s.n_irr;
            a.im0 = s.im0;
            a.n_items = s.items_sym;
        }
        rc = launch_ladder_variant(ladder_variant(s.n_nu, prec), a, class_slots(ws, P.g, 0, 0), st);
        if (rc != DF_OK) return rc;
        if (sym) {
            rc = stage_sym_expand(s, ws, b, L, inst[i].w, inst[i].logdet, inst[i].status, st);
            if (rc != DF_OK) return rc;
        }
    }
    return DF_OK;
}

int df_sigma(const df_inst_t *inst, int32_t n_inst, void *ws, size_t ws_bytes, df_stream_t stream) {
    Plan P;
    int rc = make_plan(inst, n_inst, &P);
    if (rc != DF_OK) return rc;
    rc = check_ws(P, ws, ws_bytes);
    if (rc != DF_OK) return rc;
    for (int i = 0; i < n_inst; ++i)
        if (!inst[i].w || !inst[i].gd || !inst[i].sigma_calc) return DF_E_INVAL;
    hipStream_t st = (hipStream_t)stream;
    for (int i = 0; i < n_inst; ++i) {
        const Shape &s = P.shape[i];
        const Layout &L = P.lay[i];
        const size_t b = P.base[i];
        double *gr = at<double>(ws, b + L.gr);
        rc = stage_transform_gd(s, inst[i].gd, gr, st);
        if (rc != DF_OK) return rc;
        rc = stage_sigma(inst[i], s, ws, b, L, inst[i].w, false, inst[i].sigma_calc, nullptr, 0.0, nullptr,
                         st);
        if (rc != DF_OK) return rc;
    }
    return DF_OK;
}

int df_iterate(const df_inst_t *inst, int32_t n_inst, const df_opts_t *opts, int32_t *iters_out,
               double *diff_out, void *ws, size_t ws_bytes, df_stream_t stream) {
    int rc = check_opts(opts, true, true);
    if (rc != DF_OK) return rc;
    Plan P;
    rc = make_plan(inst, n_inst, &P, opts->accel);
    if (rc != DF_OK) return rc;
    rc = check_ws(P, ws, ws_bytes);
    if (rc != DF_OK) return rc;
    for (int i = 0; i < n_inst; ++i) {
        const df_inst_t &p = inst[i];
        if (!p.g || !p.delta || !p.eps || !p.gamma_uu || !p.gamma_ud || !p.sigma) return DF_E_INVAL;
    }
    const int slots = opts->accel > 0 ? opts->accel + 1 : 0;
    std::vector<AccState> acc(slots > 0 ? n_inst : 0);
    for (auto &S : acc) S.gram.assign((size_t)slots * slots, 0.0);
    hipStream_t st = (hipStream_t)stream;
    const bool graph = opts->use_graph != 0 && st != nullptr;
    // iterations per captured graph: the host step of Anderson acceleration
    // and of the adaptive precision switch needs every iteration's measure
    const int unroll = (graph && slots == 0 && opts->prec != DF_ADAPTIVE && opts->graph_unroll > 1)
                           ? opts->graph_unroll : 1;

    for (int i = 0; i < n_inst; ++i) {
        rc = stage_gamma_prep(inst[i], P, i, ws, false, st);
        if (rc != DF_OK) return rc;
        if (opts->symmetry) {
            rc = stage_sym_tables(P.shape[i], ws, P.base[i], P.lay[i], st);
            if (rc != DF_OK) return rc;
        }
    }

    hipGraphExec_t exec = nullptr;
    auto cleanup = [&]() {
        if (exec) (void)hipGraphExecDestroy(exec);
        exec = nullptr;
    };
    std::vector<int> act;
    for (int i = 0; i < n_inst; ++i) act.push_back(i);
    std::vector<double> last(n_inst, INFINITY);
    // host side of the readbacks: counters and norm partials, dots
    const size_t dots_bytes = slots > 0 ? (size_t)n_inst * kAccMaxSlots * sizeof(double) : 0;
    PinnedLease lease(P.readback + dots_bytes);
    const int *hints = reinterpret_cast<const int *>(lease.data());
    const double *hnorms = reinterpret_cast<const double *>(lease.data() + (P.g.norms - P.g.ints));
    const double *hdots = reinterpret_cast<const double *>(lease.data() + P.readback);
    // ladder precision of each instance; DF_ADAPTIVE starts in FP32 and moves
    // an instance to FP64 (for good) once its diff falls below switch_tol
    const bool adaptive = opts->prec == DF_ADAPTIVE;
    const double switch_tol = opts->switch_tol > 0.0 ? opts->switch_tol : 1e-4;
    std::vector<int> cur(n_inst, adaptive ? DF_FP32 : opts->prec);
    std::vector<double> last_prev(n_inst, INFINITY);
    Fused F;
    bool rebuild = true;
    int it = 0;
    int result = DF_OK;
    // per instance: some ladder of its own last iteration fell back
    std::vector<char> fell_back(n_inst, 0);
    while (it < opts->max_iter && !act.empty()) {
        if (rebuild) {
            cleanup();
            rc = build_fused(inst, P, act, cur, opts->symmetry != 0, ws, &F, st);
            if (rc != DF_OK) return rc;
            if (graph) {
                hipGraph_t g = nullptr;
                if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess)
                    return DF_E_HIP;
                rc = DF_OK;
                for (int u = 0; u < unroll && rc == DF_OK; ++u)
                    rc = queue_fused_iteration(inst, P, F, *opts, ws, st);
                const hipError_t e = hipStreamEndCapture(st, &g);
                if (rc != DF_OK || e != hipSuccess) {
                    if (g) (void)hipGraphDestroy(g);
                    return rc != DF_OK ? rc : DF_E_HIP;
                }
                const hipError_t e2 = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
                (void)hipGraphDestroy(g);
                if (e2 != hipSuccess) return DF_E_HIP;
            }
            rebuild = false;
        }
        if (graph && opts->max_iter - it >= unroll) {
            if (hipGraphLaunch(exec, st) != hipSuccess) {
                cleanup();
                return DF_E_HIP;
            }
            it += unroll;
        } else {
            // without a graph, or the iterations left are fewer than one
            // graph's: queued one by one
            const int n = graph ? opts->max_iter - it : 1;
            for (int u = 0; u < n; ++u) {
                rc = queue_fused_iteration(inst, P, F, *opts, ws, st);
                if (rc != DF_OK) {
                    cleanup();
                    return rc;
                }
            }
            it += n;
        }
        if (slots > 0) {
            // record x_k, r_k and their dots; weights on the host; the step
            for (int i : act) {
                const Shape &sh = P.shape[i];
                const Layout &L = P.lay[i];
                const size_t b = P.base[i];
                AccRecordArgs ra{};
                ra.count = (size_t)sh.n_nu * sh.N;
                ra.x = inst[i].sigma;
                ra.fx = at<double>(ws, b + L.fx);
                ra.xh = at<double>(ws, b + L.xh);
                ra.rh = at<double>(ws, b + L.rh);
                ra.slot = acc[i].recorded % slots;
                ra.n_slots = acc[i].recorded + 1 < slots ? acc[i].recorded + 1 : slots;
                ra.part = at<double>(ws, b + L.accpart);
                ra.dots = at<double>(ws, P.g.accdots) + (size_t)i * kAccMaxSlots;
                if (launch_acc_record(ra, mix_blocks(sh), st) != hipSuccess) {
                    cleanup();
                    return DF_E_HIP;
                }
            }
            if (!lease.read(P.readback, at<double>(ws, P.g.accdots), dots_bytes, st)) {
                cleanup();
                return DF_E_HIP;
            }
            for (int i : act) {
                AccState &S = acc[i];
                const int slot = S.recorded % slots;
                const int nv = S.recorded + 1 < slots ? S.recorded + 1 : slots;
                for (int j = 0; j < nv; ++j) {
                    const double d = hdots[(size_t)i * kAccMaxSlots + j];
                    S.gram[slot * slots + j] = d;
                    S.gram[j * slots + slot] = d;
                }
                ++S.recorded;
                AccCombineArgs ca{};
                const bool ok = acc_weights(S, slots, slot, ca.coef);
                if (!ok) {
                    // plain mixing step; the history restarts from this iterate
                    for (int j = 0; j < kAccMaxSlots; ++j) ca.coef[j] = (j == slot) ? 1.0 : 0.0;
                }
                const Shape &sh = P.shape[i];
                const Layout &L = P.lay[i];
                const size_t b = P.base[i];
                ca.count = (size_t)sh.n_nu * sh.N;
                ca.xh = at<double>(ws, b + L.xh);
                ca.rh = at<double>(ws, b + L.rh);
                ca.n_slots = nv;
                ca.alpha = opts->mix;
                ca.x = inst[i].sigma;
                ca.norm_part = norm_part(P, ws, i);
                if (launch_acc_combine(ca, mix_blocks(sh), st) != hipSuccess) {
                    cleanup();
                    return DF_E_HIP;
                }
                if (!ok) S.recorded = 0;
            }
        }
        if (!lease.read(0, at<int>(ws, P.g.ints), P.readback, st)) {
            cleanup();
            return DF_E_HIP;
        }
        std::vector<int> next;
        for (int i : act) {
            double diff = 0.0;
            const bool finite = norm_diff(hnorms + P.norm0[i], norm_parts(inst[i], P.shape[i], opts->accel), &diff);
            last[i] = diff;
            fell_back[i] = hints[kIntsInst + i] != 0;
            if (!finite || !isfinite(diff)) {
                result = DF_E_NONFINITE;
                continue;
            }
            // move to FP64 below switch_tol, at tol (an instance converges
            // only on FP64 ladders), or when the FP32 iteration stops
            // contracting (its rounding floor)
            const double prev = last_prev[i];
            last_prev[i] = diff;
            if (adaptive && cur[i] == DF_FP32 &&
                (diff < switch_tol || (opts->tol > 0.0 && diff < opts->tol) ||
                 diff > 0.95 * prev)) {
                cur[i] = DF_FP64;
                rebuild = true;
                if (slots > 0) acc[i].recorded = 0;   // FP32 residuals leave the history
                next.push_back(i);
                continue;
            }
            if (opts->tol > 0.0 && diff < opts->tol) continue;
            next.push_back(i);
        }
        if (result == DF_E_NONFINITE) break;
        if (next.size() != act.size()) rebuild = true;
        act.swap(next);
    }
    cleanup();
    if (opts->symmetry) {
        // the entries of the outputs that the reduced ladders leave out
        bool any = false;
        for (int i = 0; i < n_inst; ++i) {
            if (!inst[i].w && !inst[i].logdet && !inst[i].status) continue;
            if (sigma_over_w(inst[i], P.shape[i])) continue;   // (done in the loop)
            const Layout &L = P.lay[i];
            double *w = inst[i].w ? inst[i].w : at<double>(ws, P.base[i] + L.w);
            rc = stage_sym_expand(P.shape[i], ws, P.base[i], L, w, inst[i].logdet, inst[i].status, st);
            if (rc != DF_OK) return rc;
            any = true;
        }
        if (any && hipStreamSynchronize(st) != hipSuccess) return DF_E_HIP;
    }
    if (slots > 0) {
        // sigma_calc (F of the last iterate) where the caller asked for it
        for (int i = 0; i < n_inst; ++i) {
            if (!inst[i].sigma_calc) continue;
            const Shape &sh = P.shape[i];
            if (hipMemcpyAsync(inst[i].sigma_calc, at<double>(ws, P.base[i] + P.lay[i].fx),
                               (size_t)sh.n_nu * sh.N * 16, hipMemcpyDeviceToDevice, st) != hipSuccess)
                return DF_E_HIP;
        }
        if (hipStreamSynchronize(st) != hipSuccess) return DF_E_HIP;
    }
    if (iters_out) *iters_out = it;
    if (diff_out)
        for (int i = 0; i < n_inst; ++i) diff_out[i] = last[i];
    if (result != DF_OK) return result;
    if (opts->tol > 0.0) {
        for (int i = 0; i < n_inst; ++i)
            if (!(last[i] < opts->tol)) return DF_E_NOT_CONVERGED;
    }
    for (int i = 0; i < n_inst; ++i)
        if (fell_back[i]) return DF_W_FALLBACK;
    return DF_OK;
}

int df_autotune(const df_inst_t *inst, int32_t n_inst, const df_opts_t *opts, void *ws,
                size_t ws_bytes, df_stream_t stream) {
    int rc = check_opts(opts, false, true);
    if (rc != DF_OK) return rc;
    Plan P;
    rc = make_plan(inst, n_inst, &P);
    if (rc != DF_OK) return rc;
    rc = check_ws(P, ws, ws_bytes);
    if (rc != DF_OK) return rc;
    for (int i = 0; i < n_inst; ++i) {
        const df_inst_t &p = inst[i];
        if (!p.g || !p.delta || !p.eps || !p.gamma_uu || !p.gamma_ud) return DF_E_INVAL;
    }
    hipStream_t st = (hipStream_t)stream;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) return DF_E_HIP;
    if (cap != hipStreamCaptureStatusNone) return DF_E_INVAL;   // timing needs synchronisation
    std::vector<int> precs;
    if (opts && opts->prec == DF_ADAPTIVE) precs = {DF_FP32, DF_FP64};
    else precs = {opts ? opts->prec : DF_FP64};
    int *ints = at<int>(ws, P.g.ints);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return DF_E_HIP;
    }
    // One group per distinct n_nu: every instance of the group gets its ladder
    // inputs in the workspace (G~ from sigma, NULL = zero, and chi), and the
    // variants are timed on one fused launch over the whole group - the launch
    // df_iterate makes - writing only workspace outputs.
    std::vector<int> done;
    for (int i0 = 0; i0 < n_inst && rc == DF_OK; ++i0) {
        const int n_nu = P.shape[i0].n_nu;
        bool seen = false;
        for (int n : done) seen = seen || (n == n_nu);
        if (seen) continue;
        done.push_back(n_nu);
        std::vector<LadderInst> table;
        int items = 0, sblocks = 0;
        for (int i = i0; i < n_inst && rc == DF_OK; ++i) {
            const Shape &s = P.shape[i];
            if (s.n_nu != n_nu) continue;
            const Layout &L = P.lay[i];
            const size_t b = P.base[i];
            double *gr = at<double>(ws, b + L.gr);
            double *gd = at<double>(ws, b + L.gd);
            double *chi = at<double>(ws, b + L.chi);
            rc = stage_gamma_prep(inst[i], P, i, ws, false, st);
            if (rc == DF_OK) rc = stage_dual_gf(inst[i], s, inst[i].sigma, gd, gr, st);
            if (rc == DF_OK) rc = stage_bubble(inst[i], s, gr, chi, nullptr, 0, st);
            table.push_back(table_entry(P, i, ws, false, chi, at<double>(ws, b + L.w), nullptr, nullptr,
                                        &items, &sblocks));
        }
        if (rc != DF_OK) break;
        if (hipMemcpyAsync(at<LadderInst>(ws, P.g.table), table.data(),
                           table.size() * sizeof(LadderInst), hipMemcpyHostToDevice, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess) {
            rc = DF_E_HIP;
            break;
        }
        LadderArgs a{};
        a.insts = at<LadderInst>(ws, P.g.table);
        a.n_insts = (int)table.size();
        a.n_nu = n_nu;
        a.full = n_nu == ladder_gjb_padded_size(n_nu);
        a.full_sym = n_nu % 16 == 0;
        a.item0 = 0;
        a.n_items = items;
        a.n_sblk = sblocks;
        for (int prec : precs) {
        // two passes over the candidates, each variant keeping its faster
        // pass: a variant timed right after the slow pivoting kernels (or
        // while clocks settle) is not ranked on that pass alone
        float vms[kChoices];
        for (int v = 0; v < kChoices; ++v) vms[v] = -1.f;
        for (int pass = 0; pass < 2 && rc == DF_OK; ++pass)
        for (int v = 0; v < kChoices && rc == DF_OK; ++v) {
            if (!variant_supports(v, n_nu, prec)) continue;
            // (the certified FP64 choices run the same kernels: the default stands for them)
            if (fp64_certified(choice_variant(v)) && v != default_variant(n_nu, prec)) continue;
            constexpr int kReps = 3;
            float ms = 0.f;
            for (int r = 0; r <= kReps && rc == DF_OK; ++r) {   // r = 0: untimed first launch
                if (r == 1 && hipEventRecord(e0, st) != hipSuccess) rc = DF_E_HIP;
                if (rc == DF_OK && launch_zero_ints(ints, kIntsInst + n_inst, st) != hipSuccess)
                    rc = DF_E_HIP;
                if (rc == DF_OK) rc = launch_ladder_variant(v, a, class_slots(ws, P.g, 0, 0), st);
            }
            if (rc == DF_OK && (hipEventRecord(e1, st) != hipSuccess ||
                                hipEventSynchronize(e1) != hipSuccess ||
                                hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
                rc = DF_E_HIP;
            if (rc == DF_OK && (vms[v] < 0.f || ms < vms[v])) vms[v] = ms;
        }
        int best = -1;
        for (int v = 0; v < kChoices; ++v)
            if (vms[v] >= 0.f && (best < 0 || vms[v] < vms[best])) best = v;
        if (rc == DF_OK && best >= 0) set_tuned_variant(prec, n_nu, best);
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != DF_OK) return rc;
    if (hipStreamSynchronize(st) != hipSuccess) return DF_E_HIP;
    return save_tune_cache() == 0 ? DF_OK : DF_E_INVAL;
}

int df_ladder_variant(int32_t n_nu, int32_t prec, char *name, size_t name_len) {
    if (!name || name_len == 0) return DF_E_INVAL;
    if (!ladder_prec(prec)) return DF_E_INVAL;
    if (n_nu < 2 || (n_nu & 1) || n_nu > 128) return DF_E_UNSUPPORTED;
    const char *v = variant_name(ladder_variant(n_nu, prec));
    if (strlen(v) + 1 > name_len) return DF_E_INVAL;
    strcpy(name, v);
    return DF_OK;
}

int df_ladder_set_variant(int32_t n_nu, int32_t prec, const char *name) {
    if (!ladder_prec(prec)) return DF_E_INVAL;
    if (n_nu < 2 || (n_nu & 1) || n_nu > 128) return DF_E_UNSUPPORTED;
    const int v = variant_from_name(name);
    if (v < 0) return DF_E_INVAL;
    if (!variant_supports(v, n_nu, prec)) return DF_E_UNSUPPORTED;
    set_tuned_variant(prec, n_nu, v);
    return DF_OK;
}

int df_autotune_reset(void) {
    clear_tuned();
    return DF_OK;
}

int df_lattice_workspace_size(const df_inst_t *inst, size_t *bytes) {
    if (!inst || !bytes) return DF_E_INVAL;
    Shape s;
    const int rc = check_inst(*inst, &s);
    if (rc != DF_OK) return rc;
    *bytes = lattice_layout_of(s).total;
    return DF_OK;
}

int df_lattice(const df_inst_t *inst, double mu, double *sigma_lat, double *g_lat, double *chi_ch,
               double *chi_sp, void *ws, size_t ws_bytes, df_stream_t stream) {
    if (!inst) return DF_E_INVAL;
    const df_inst_t &p = *inst;
    Shape s;
    int rc = check_inst(p, &s);
    if (rc != DF_OK) return rc;
    if (!isfinite(mu)) return DF_E_INVAL;
    if (!p.g || !p.delta || !p.eps) return DF_E_INVAL;
    const bool want_chi = chi_ch || chi_sp;
    if (want_chi && (!p.gamma_uu || !p.gamma_ud)) return DF_E_INVAL;
    const LatticeLayout L = lattice_layout_of(s);
    if (!ws || (((uintptr_t)ws) & (kAlign - 1)) || ws_bytes < L.total) return DF_E_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;

    LatticeFieldArgs f{};
    f.n_nu = s.n_nu;
    f.N = s.N;
    f.beta = p.beta;
    f.mu = mu;
    f.g = p.g;
    f.delta = p.delta;
    f.eps = p.eps;
    f.sigma = p.sigma;
    f.sigma_lat = sigma_lat;
    f.g_lat = g_lat;
    // the three fields next to each other: one transform and one bubble launch
    const size_t fld = 2 * (size_t)s.n_nu * s.N;         // doubles of one field
    f.gd = at<double>(ws, L.fields);
    f.fg = f.gd + fld;
    f.gl = f.gd + 2 * fld;
    HIPCHK(launch_lattice_fields(f, st));
    if (!want_chi) return DF_OK;

    // chi~, L and the per-nu lattice bubble at Omega = 0: the iteration's FFT bubble
    // with a one-frequency bosonic window
    Shape s3 = s;
    s3.n_om = 1;
    s3.n_nu = 3 * s.n_nu;
    rc = stage_transform_gd(s3, f.gd, at<double>(ws, L.gr), st);
    if (rc == DF_OK) rc = stage_bubble(p, s3, at<double>(ws, L.gr), at<double>(ws, L.bub), nullptr, 0, st);
    if (rc != DF_OK) return rc;
    const double *chi0 = at<double>(ws, L.bub), *Lq = chi0 + fld, *bub = chi0 + 2 * fld;

    // the ladder term with the ladder kernels on the vertex at Omega = 0
    GammaPrepArgs g{};
    g.n_nu = s.n_nu;
    g.n_om = 1;
    const size_t v0 = 2 * (size_t)((s.n_om - 1) / 2) * s.n_nu * s.n_nu;
    g.guu = p.gamma_uu + v0;
    g.gud = p.gamma_ud + v0;
    g.gdm = at<double>(ws, L.gdm);
    g.gtr = at<double>(ws, L.gtr);
    g.gsym = at<double>(ws, L.gsym);
    g.gabs = at<float>(ws, L.gabs);
    g.symp = at<float>(ws, L.symp);
    g.zero = at<int>(ws, L.count);
    g.n_zero = 1;
    HIPCHK(launch_gamma_prep(g, st));
    LadderArgs c{};
    c.gdm = g.gdm;
    c.gtr = g.gtr;
    c.gsym = g.gsym;
    c.gabs = g.gabs;
    c.symp = g.symp;
    c.cert = at<uint8_t>(ws, L.cert);
    c.chi = chi0;
    c.w = at<double>(ws, L.w);
    c.n_nu = s.n_nu;
    c.n_om = 1;
    c.N = s.N;
    c.n_items = 2 * s.N;
    c.n_sblk = ladder_screen_blocks(1, s.N);
    c.queue = at<int>(ws, L.queue);
    c.queue_count = g.zero;
    double *lad = at<double>(ws, L.lad);
    HIPCHK(launch_lattice_screen(c, Lq, st));
    HIPCHK(launch_lattice_sym(c, Lq, lad, st));
    HIPCHK(launch_lattice_rest(c, Lq, lad, st));
    LatticeSumArgs m{};
    m.n_nu = s.n_nu;
    m.N = s.N;
    m.bub = bub;
    m.lad = lad;
    m.chi_ch = chi_ch;
    m.chi_sp = chi_sp;
    HIPCHK(launch_lattice_chi_sum(m, st));
    return DF_OK;
}

}  // extern "C"
