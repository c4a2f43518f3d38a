// Learned warm start: forward, backward and Adam kernels of a small MLP on the
// FP32 matrix cores, behind the C ABI of include/df_mlp.h.
//
// GEMM: C[M x N] = op(A)[M x K] op(B)[K x N], one T x T tile per work-group of four
// waves (quadrants of v_mfma_f32_16x16x4f32 tiles), T = 64, or 32 where 64 would
// leave the CUs with too few work-groups.  At these sizes (batch 1024-4096, width
// 256) a launch is a few hundred work-groups of 8-16 K chunks: it is bound by
// the latency of its loads, so a chunk is 32 deep and the next one's operands
// are in flight, as 16-byte loads into registers, while this one's products
// run.  Fused epilogues: bias, SiLU with the pre-activation saved, the mean
// squared error with its gradient (last layer), multiplication by SiLU'(Z) of
// the previous layer (backward), column sums of A (the bias gradient), split-K
// partial sums reduced in a fixed order by a second kernel.  Batch 4096, widths
// 132-256-256-256-96: loss and gradients 101 us; 1219 us with 16-deep chunks of scalar
// loads (a product 30 us) and a column-sum kernel of one work-group per 64 columns
// (four of 217 us).
#include <math.h>

#include "../../include/df_mlp.h"
#include "df_internal.hpp"

namespace df {

typedef float f4 __attribute__((ext_vector_type(4)));

struct GemmArgs {
    int M, N, K;
    const float *A;
    int lda;
    const float *B;
    int ldb;
    float *C;
    int ldc;
    const float *bias;        // [N] or null
    float *Zout;              // pre-activation store (ldc layout) or null
    int act;                  // 1: SiLU
    const float *T;           // target [M][ldc] or null: C = 2 (v - T) / (M N), lpart the
    float *lpart;             // work-group's sum of (v - T)^2
    const float *dz;          // backward: multiply by SiLU'(dz[m ldc + n]) or null
    float *asum;              // [M] sums of A over K (work-groups of the first tile column), or null
    float *part;              // split-K: partial sums [gridDim.z][M][N], then [gridDim.z][M] of asum
    int kchunk;               // K range per split (multiple of 16)
};

__device__ __forceinline__ float sigm(float z) { return 1.0f / (1.0f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }
__device__ __forceinline__ float dsilu(float z) {
    const float s = sigm(z);
    return s * (1.0f + z * (1.0f - s));
}

// One operand tile of a K chunk: T rows (m or n) x KC.  KMAJOR = false: row-major
// in memory with K contiguous, kept so in LDS (stride 36: the 16 rows x 4 k of an
// MFMA operand fall in 64 different banks); true: rows contiguous for each k,
// LDS [k][row] with stride T + 16 (same).  VEC: 16-byte loads (base and leading
// dimension aligned); elements outside the matrix or the K range are zero.
constexpr int KC = 32;
template <int T, bool KMAJOR> struct TileLds {
    static constexpr int LD = KMAJOR ? T + 16 : KC + 4;
    float x[KMAJOR ? KC * LD : T * LD];
    __device__ __forceinline__ float at(int row, int k) const { return KMAJOR ? x[k * LD + row] : x[row * LD + k]; }
};
template <int T, bool KMAJOR, bool VEC> struct TileLoad {
    static constexpr int NV = T * KC / 4 / 256;   // float4 per thread
    f4 v[NV];
    static __device__ __forceinline__ void where(int e, int *row, int *k) {
        if (KMAJOR) { *k = e / (T / 4); *row = 4 * (e % (T / 4)); }
        else { *row = e / (KC / 4); *k = 4 * (e % (KC / 4)); }
    }
    __device__ __forceinline__ void load(const float *p, int ld, int row0, int rows, int k0, int kend) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            int r, k;
            where((int)threadIdx.x + 256 * i, &r, &k);
            r += row0;
            k += k0;
            f4 t = {0.f, 0.f, 0.f, 0.f};
            const float *q = KMAJOR ? p + (size_t)k * ld + r : p + (size_t)r * ld + k;
            if (KMAJOR ? (k < kend) : (r < rows)) {
                const int left = KMAJOR ? rows - r : kend - k;
                if (VEC && left >= 4) t = *reinterpret_cast<const f4 *>(q);
                else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (j < left) t[j] = q[j];
                }
            }
            v[i] = t;
        }
    }
    __device__ __forceinline__ void store(TileLds<T, KMAJOR> &s) const {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            int r, k;
            where((int)threadIdx.x + 256 * i, &r, &k);
            *reinterpret_cast<f4 *>(&s.x[KMAJOR ? k * s.LD + r : r * s.LD + k]) = v[i];
        }
    }
};

// AT / BT: the operand is k-major in memory (A(m, k) = A[k lda + m], B(k, n) =
// B[k ldb + n]); else A[m lda + k], B[n ldb + k].
// Work-group (bx, by) of the tiles of split bz of nz.
template <int T, bool AT, bool BT, bool VEC>
__device__ __forceinline__ void gemm_item(const GemmArgs &g, int bx, int by, int bz, int nz, int n_loss) {
    constexpr int F = T / 32;                      // MFMA tiles per wave and direction
    __shared__ __align__(16) TileLds<T, AT> As;
    __shared__ __align__(16) TileLds<T, BT> Bs;
    __shared__ float red[4][64];
    const int tid = threadIdx.x;
    const int w = tid >> 6, l = tid & 63, lj = l & 15, lg = l >> 4;
    const int wm = (w >> 1) * (T / 2), wn = (w & 1) * (T / 2);
    const int m0 = by * T, n0 = bx * T;
    const int kbeg = bz * g.kchunk;
    const int kend = min(g.K, kbeg + g.kchunk);
    const bool sums = g.asum && bx == 0;
    f4 acc[F][F];
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    float asum = 0.f;                              // row tid % T, a quarter or an eighth of the k

    TileLoad<T, AT, VEC> la;
    TileLoad<T, BT, VEC> lb;
    la.load(g.A, g.lda, m0, g.M, kbeg, kend);
    lb.load(g.B, g.ldb, n0, g.N, kbeg, kend);
    for (int k0 = kbeg; k0 < kend; k0 += KC) {
        __syncthreads();
        la.store(As);
        lb.store(Bs);
        __syncthreads();
        if (k0 + KC < kend) {
            la.load(g.A, g.lda, m0, g.M, k0 + KC, kend);
            lb.load(g.B, g.ldb, n0, g.N, k0 + KC, kend);
        }
#pragma unroll
        for (int k4 = 0; k4 < KC / 4; ++k4) {
            float av[F], bv[F];
#pragma unroll
            for (int i = 0; i < F; ++i) av[i] = As.at(wm + 16 * i + lj, 4 * k4 + lg);
#pragma unroll
            for (int j = 0; j < F; ++j) bv[j] = Bs.at(wn + 16 * j + lj, 4 * k4 + lg);
#pragma unroll
            for (int i = 0; i < F; ++i)
#pragma unroll
                for (int j = 0; j < F; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
        if (sums) {
            constexpr int PART = KC * T / 256;
#pragma unroll
            for (int k = 0; k < PART; ++k) asum += As.at(tid % T, (tid / T) * PART + k);
        }
    }
    if (sums) {
        // the 256 / T parts of a row, in order
        __syncthreads();
        float *r = &As.x[0];
        r[tid] = asum;
        __syncthreads();
        if (tid < T && m0 + tid < g.M) {
            float s = 0.f;
            for (int p = 0; p < 256 / T; ++p) s += r[p * T + tid];
            if (nz > 1) g.part[(size_t)nz * g.M * g.N + (size_t)bz * g.M + m0 + tid] = s;
            else g.asum[m0 + tid] = s;
        }
    }

    const float sc = g.T ? 2.0f / ((float)g.M * (float)g.N) : 0.f;
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + 16 * i + 4 * lg + r;
                const int n = n0 + wn + 16 * j + lj;
                if (m >= g.M || n >= g.N) continue;
                float v = acc[i][j][r];
                if (nz > 1) {
                    g.part[((size_t)bz * g.M + m) * g.N + n] = v;
                    continue;
                }
                const size_t o = (size_t)m * g.ldc + n;
                if (g.bias) v += g.bias[n];
                if (g.dz) v *= dsilu(g.dz[o]);
                if (g.Zout) g.Zout[o] = v;
                if (g.act) v = silu(v);
                if (g.T) {
                    const float d = v - g.T[o];
                    sq += d * d;
                    v = sc * d;
                }
                g.C[o] = v;
            }
    if (g.T) {
        // fixed order: within the lanes, then the waves
        for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
        if (l == 0) red[w][0] = sq;
        __syncthreads();
        if (tid == 0)
            g.lpart[n_loss] = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
    }
}

template <int T, bool AT, bool BT, bool VEC>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmArgs g) {
    gemm_item<T, AT, BT, VEC>(g, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.z,
                              blockIdx.y * gridDim.x + blockIdx.x);
}

// The weight gradients of several layers in one launch (A and B k-major): one alone
// is too few work-groups to fill the chip to its end.  Batch 4096, widths
// 132-256-256-256-96: four launches and their four sums 64 us, one
// and one 32 us.
struct GemmGroup {
    GemmArgs p[DF_MLP_MAX_LAYERS];
    int tx[DF_MLP_MAX_LAYERS], ty[DF_MLP_MAX_LAYERS];   // tiles per split
    int wg0[DF_MLP_MAX_LAYERS + 1];                     // first work-group of each
    int n, splits;
};
template <int T, bool VEC>
__global__ __launch_bounds__(256) void k_gemm_group(GemmGroup a) {
    int i = 0;
    while (i + 1 < a.n && (int)blockIdx.x >= a.wg0[i + 1]) ++i;
    const int u = (int)blockIdx.x - a.wg0[i], bx = u % a.tx[i], r = u / a.tx[i];
    gemm_item<T, true, true, VEC>(a.p[i], bx, r % a.ty[i], r / a.ty[i], a.splits, 0);
}

// Per layer C[m][n] = sum over splits of part[s][m][n], in split order, and the same
// for the column sums db [M].  Block 0 also finishes the loss (n_loss block partials,
// count elements) where wanted.
struct SumSplitsArgs {
    const float *part[DF_MLP_MAX_LAYERS];
    int M[DF_MLP_MAX_LAYERS], N[DF_MLP_MAX_LAYERS];
    float *C[DF_MLP_MAX_LAYERS];                        // rows of N
    float *db[DF_MLP_MAX_LAYERS];
    int wg0[DF_MLP_MAX_LAYERS + 1];                     // first work-group of each layer
    int n, splits;
    const float *lpart;
    int n_loss;
    float count;
    float *loss;
};
__device__ __forceinline__ void finish_loss(const float *part, int n, float count, float *loss) {
    __shared__ float red[256];
    float s = 0.f;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = red[0] / count;
}
__global__ __launch_bounds__(256) void k_sum_splits(SumSplitsArgs a) {
    int i = 0;
    while (i + 1 < a.n && (int)blockIdx.x >= a.wg0[i + 1]) ++i;
    const size_t tot = (size_t)a.M[i] * a.N[i];
    const size_t e = (size_t)(blockIdx.x - a.wg0[i]) * 256 + threadIdx.x;
    const float *part = a.part[i];
    // the weights, then the bias
    if (e < tot) {
        float s = 0.f;
#pragma unroll 8
        for (int z = 0; z < a.splits; ++z) s += part[(size_t)z * tot + e];
        a.C[i][e] = s;
    } else if (e < tot + a.M[i]) {
        const size_t m = e - tot;
        float s = 0.f;
#pragma unroll 8
        for (int z = 0; z < a.splits; ++z) s += part[a.splits * tot + (size_t)z * a.M[i] + m];
        a.db[i][m] = s;
    }
    if (a.loss && blockIdx.x == 0) finish_loss(a.lpart, a.n_loss, a.count, a.loss);
}
__global__ __launch_bounds__(256) void k_loss(const float *part, int n, float count, float *loss) {
    finish_loss(part, n, count, loss);
}

__global__ __launch_bounds__(256) void k_adam(size_t count, float *p, const float *g, float *m, float *v,
                                              float lr, float c1, float c2) {
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
         e += (size_t)gridDim.x * blockDim.x) {
        const float gg = g[e];
        const float mm = 0.9f * m[e] + 0.1f * gg;
        const float vv = 0.999f * v[e] + 0.001f * gg * gg;
        m[e] = mm;
        v[e] = vv;
        p[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + 1e-8f);
    }
}

}  // namespace df

using namespace df;

namespace {

constexpr size_t kAl = 256;
size_t alup(size_t x) { return (x + kAl - 1) & ~(kAl - 1); }
int check_net(int32_t n_layers, const int32_t *dims) {
    if (n_layers < 1 || n_layers > DF_MLP_MAX_LAYERS || !dims) return DF_E_INVAL;
    for (int i = 0; i <= n_layers; ++i)
        if (dims[i] < 1 || dims[i] > DF_MLP_MAX_WIDTH) return DF_E_INVAL;
    return DF_OK;
}

size_t n_params(int32_t L, const int32_t *d) {
    size_t c = 0;
    for (int l = 0; l < L; ++l) c += (size_t)d[l + 1] * d[l] + d[l + 1];
    return c;
}

int splits_for(int K) {
    int s = (K + 255) / 256;
    return s < 1 ? 1 : (s > 64 ? 64 : s);
}

// workspace: Z[l], Y[l] for l = 1..L (batch x d_l; the backward pass leaves dZ_l in Z_l),
// split partials of every layer, loss partials
struct MlpWs {
    size_t z[DF_MLP_MAX_LAYERS + 1], y[DF_MLP_MAX_LAYERS + 1], part, lpart, total;
};

MlpWs mlp_ws(int32_t L, const int32_t *d, int32_t batch) {
    MlpWs w{};
    size_t o = 0;
    for (int l = 1; l <= L; ++l) {
        w.z[l] = o;
        o = alup(o + (size_t)batch * d[l] * sizeof(float));
        w.y[l] = o;
        o = alup(o + (size_t)batch * d[l] * sizeof(float));
    }
    w.part = o;
    o = alup(o + (size_t)splits_for(batch) * n_params(L, d) * sizeof(float));
    w.lpart = o;
    o = alup(o + (size_t)((batch + 31) / 32) * ((d[L] + 31) / 32) * sizeof(float));
    w.total = o;
    return w;
}

template <typename T> T *wsp(void *ws, size_t off) {
    return reinterpret_cast<T *>(static_cast<char *>(ws) + off);
}

// The tile: 64, unless that gives fewer than four work-groups per CU (of 256), where
// the loads of too few waves are in flight - then 32.  Batch 4096, width 256, loss
// and gradients (a launch per product): 162 us with 64 x 64 tiles (256 work-groups), 137
// with 32 x 32;
// batch 1024 forward: 64 work-groups of 64 x 64, 256 of 32 x 32 (28 us).
int gemm_tile(int M, int N, int splits) {
    return (long)((M + 63) / 64) * ((N + 63) / 64) * splits >= 1024 ? 64 : 32;
}

int gemm_splits(int K, int wanted, int *kchunk) {
    *kchunk = ((K + wanted - 1) / wanted + 15) / 16 * 16;
    if (*kchunk < 16) *kchunk = 16;
    const int s = (K + *kchunk - 1) / *kchunk;
    return s < 1 ? 1 : s;
}

bool aligned16(const float *p, int ld) { return ((uintptr_t)p & 15) == 0 && ld % 4 == 0; }

template <int T, bool AT, bool BT>
void launch_gemm_t(const GemmArgs &g, int splits, hipStream_t st) {
    const dim3 grid((g.N + T - 1) / T, (g.M + T - 1) / T, splits);
    // 16-byte loads need aligned rows (a layer's weights start wherever the
    // previous layers' parameters end)
    if (aligned16(g.A, g.lda) && aligned16(g.B, g.ldb))
        hipLaunchKernelGGL((k_gemm_f32<T, AT, BT, true>), grid, dim3(256), 0, st, g);
    else hipLaunchKernelGGL((k_gemm_f32<T, AT, BT, false>), grid, dim3(256), 0, st, g);
}

template <bool AT, bool BT>
hipError_t gemm(GemmArgs g, hipStream_t st, int splits = 1) {
    splits = gemm_splits(g.K, splits, &g.kchunk);
    if (gemm_tile(g.M, g.N, splits) == 64) launch_gemm_t<64, AT, BT>(g, splits, st);
    else launch_gemm_t<32, AT, BT>(g, splits, st);
    return hipGetLastError();
}

// T (targets) set: the last layer leaves dZ_L = 2 (Y - T) / count in Z_L's place and
// the partial sums of the loss in the workspace
int forward_impl(int32_t L, const int32_t *d, const float *params, const float *X, int32_t batch,
                 float *Yout, const float *T, void *ws, const MlpWs &w, hipStream_t st) {
    const float *in = X;
    size_t po = 0;
    for (int l = 0; l < L; ++l) {
        const float *W = params + po;
        const float *b = W + (size_t)d[l + 1] * d[l];
        po += (size_t)d[l + 1] * d[l] + d[l + 1];
        const bool last = (l == L - 1);
        GemmArgs g{};
        g.M = batch;
        g.N = d[l + 1];
        g.K = d[l];
        g.A = in;
        g.lda = d[l];
        g.B = W;
        g.ldb = d[l];
        g.ldc = d[l + 1];
        g.bias = b;
        // (pre-activations are kept for the backward pass)
        g.Zout = Yout || last ? nullptr : wsp<float>(ws, w.z[l + 1]);
        g.act = last ? 0 : 1;
        g.C = (last && Yout) ? Yout : wsp<float>(ws, w.y[l + 1]);
        if (last && T) {
            g.T = T;
            g.lpart = wsp<float>(ws, w.lpart);
            g.C = wsp<float>(ws, w.z[L]);
        }
        if (gemm<false, false>(g, st) != hipSuccess) return DF_E_HIP;
        in = g.C;
    }
    return DF_OK;
}

}  // namespace

extern "C" {

int df_mlp_param_count(int32_t n_layers, const int32_t *dims, size_t *count) {
    if (!count) return DF_E_INVAL;
    const int rc = check_net(n_layers, dims);
    if (rc != DF_OK) return rc;
    *count = n_params(n_layers, dims);
    return DF_OK;
}

int df_mlp_workspace_size(int32_t n_layers, const int32_t *dims, int32_t batch, size_t *bytes) {
    if (!bytes || batch < 1) return DF_E_INVAL;
    const int rc = check_net(n_layers, dims);
    if (rc != DF_OK) return rc;
    *bytes = mlp_ws(n_layers, dims, batch).total;
    return DF_OK;
}

int df_mlp_forward(int32_t n_layers, const int32_t *dims, const float *params, const float *X,
                   int32_t batch, float *Y, void *ws, size_t ws_bytes, df_stream_t stream) {
    int rc = check_net(n_layers, dims);
    if (rc != DF_OK) return rc;
    if (!params || !X || !Y || batch < 1) return DF_E_INVAL;
    const MlpWs w = mlp_ws(n_layers, dims, batch);
    if (!ws || ((uintptr_t)ws & (kAl - 1)) || ws_bytes < w.total) return DF_E_WORKSPACE;
    return forward_impl(n_layers, dims, params, X, batch, Y, nullptr, ws, w, (hipStream_t)stream);
}

int df_mlp_loss_grad(int32_t n_layers, const int32_t *dims, const float *params, const float *X,
                     const float *T, int32_t batch, float *grads, float *loss, void *ws,
                     size_t ws_bytes, df_stream_t stream) {
    int rc = check_net(n_layers, dims);
    if (rc != DF_OK) return rc;
    if (!params || !X || !T || !grads || batch < 1) return DF_E_INVAL;
    const int32_t L = n_layers;
    const int32_t *d = dims;
    const MlpWs w = mlp_ws(L, d, batch);
    if (!ws || ((uintptr_t)ws & (kAl - 1)) || ws_bytes < w.total) return DF_E_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    // forward; dZ_L = 2 (Y - T) / count (last layer has no activation)
    rc = forward_impl(L, d, params, X, batch, nullptr, T, ws, w, st);
    if (rc != DF_OK) return rc;
    const int tile = gemm_tile(batch, d[L], 1);
    const int n_loss = ((batch + tile - 1) / tile) * ((d[L] + tile - 1) / tile);
    const float count = (float)batch * (float)d[L];

    // parameter offsets
    size_t off[DF_MLP_MAX_LAYERS + 1];
    off[0] = 0;
    for (int l = 0; l < L; ++l) off[l + 1] = off[l] + (size_t)d[l + 1] * d[l] + d[l + 1];

    // dZ_l = (dZ_{l+1} W_l) * SiLU'(Z_l), in the place of Z_l
    for (int l = L - 1; l >= 1; --l) {
        GemmArgs h{};
        h.M = batch;
        h.N = d[l];
        h.K = d[l + 1];
        h.A = wsp<float>(ws, w.z[l + 1]);
        h.lda = d[l + 1];
        h.B = params + off[l];
        h.ldb = d[l];
        h.C = wsp<float>(ws, w.z[l]);
        h.ldc = d[l];
        h.dz = h.C;
        if (gemm<false, true>(h, st) != hipSuccess) return DF_E_HIP;
    }
    // dW_l = dZ^T X_l (split over the batch), db_l = column sums of dZ: the layers of one
    // tile size and alignment in one launch
    int kchunk;
    const int splits = gemm_splits(batch, splits_for(batch), &kchunk);
    for (int kind = 0; kind < 4; ++kind) {
        const int t = kind & 1 ? 64 : 32;
        const bool vec = (kind & 2) != 0;
        GemmGroup G{};
        G.splits = splits;
        for (int l = 0; l < L; ++l) {
            GemmArgs g{};
            g.M = d[l + 1];
            g.N = d[l];
            g.K = batch;
            g.A = wsp<float>(ws, w.z[l + 1]);
            g.lda = d[l + 1];
            g.B = l == 0 ? X : wsp<float>(ws, w.y[l]);
            g.ldb = d[l];
            g.C = grads + off[l];
            g.ldc = d[l];
            g.asum = g.C + (size_t)d[l + 1] * d[l];
            g.part = wsp<float>(ws, w.part) + (size_t)splits * off[l];
            g.kchunk = kchunk;
            if (gemm_tile(g.M, g.N, splits) != t) continue;
            if ((aligned16(g.A, g.lda) && aligned16(g.B, g.ldb)) != vec) continue;
            G.p[G.n] = g;
            G.tx[G.n] = (g.N + t - 1) / t;
            G.ty[G.n] = (g.M + t - 1) / t;
            G.wg0[G.n + 1] = G.wg0[G.n] + G.tx[G.n] * G.ty[G.n] * splits;
            ++G.n;
        }
        if (G.n == 0) continue;
        const dim3 grid(G.wg0[G.n]);
        if (t == 64 && vec) hipLaunchKernelGGL((k_gemm_group<64, true>), grid, dim3(256), 0, st, G);
        else if (t == 64) hipLaunchKernelGGL((k_gemm_group<64, false>), grid, dim3(256), 0, st, G);
        else if (vec) hipLaunchKernelGGL((k_gemm_group<32, true>), grid, dim3(256), 0, st, G);
        else hipLaunchKernelGGL((k_gemm_group<32, false>), grid, dim3(256), 0, st, G);
        if (hipGetLastError() != hipSuccess) return DF_E_HIP;
    }
    if (splits > 1) {
        SumSplitsArgs r{};
        r.n = L;
        r.splits = splits;
        for (int l = 0; l < L; ++l) {
            r.M[l] = d[l + 1];
            r.N[l] = d[l];
            r.C[l] = grads + off[l];
            r.db[l] = r.C[l] + (size_t)d[l + 1] * d[l];
            r.part[l] = wsp<float>(ws, w.part) + (size_t)splits * off[l];
            r.wg0[l + 1] = r.wg0[l] + (int)((off[l + 1] - off[l] + 255) / 256);
        }
        r.lpart = wsp<float>(ws, w.lpart);
        r.n_loss = n_loss;
        r.count = count;
        r.loss = loss;
        hipLaunchKernelGGL(k_sum_splits, dim3(r.wg0[L]), dim3(256), 0, st, r);
    } else if (loss) {
        hipLaunchKernelGGL(k_loss, dim3(1), dim3(256), 0, st, wsp<float>(ws, w.lpart), n_loss, count, loss);
    }
    if (hipGetLastError() != hipSuccess) return DF_E_HIP;
    return DF_OK;
}

int df_mlp_adam(size_t count, float *params, const float *grads, float *m, float *v, int32_t step,
                float lr, df_stream_t stream) {
    if (!params || !grads || !m || !v || step < 1 || count == 0 || !(lr > 0.f)) return DF_E_INVAL;
    const float c1 = 1.0f - powf(0.9f, (float)step);
    const float c2 = 1.0f - powf(0.999f, (float)step);
    int blocks = (int)((count + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_adam, dim3(blocks), dim3(256), 0, (hipStream_t)stream, count, params, grads,
                       m, v, lr, c1, c2);
    return hipGetLastError() == hipSuccess ? DF_OK : DF_E_HIP;
}

}  // extern "C"
