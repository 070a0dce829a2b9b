// Term-pruning MLP: forward, backward and Adam kernels (FP32, gfx950).
//
// A small fully connected network reads per-term features (slot positions,
// singular values, light-cone sizes, gate neighbourhoods, level-1 magnitudes,
// weight) and predicts log X of a level-2/3 term.  It is trained on the term
// values the estimate itself produces.  Layout of the state buffer (floats):
//   [ mean[n_in] | inv_std[n_in] | params P | grads P | adam m P | adam v P ]
// params: per layer l, W_l (out_l x in_l, row-major) then b_l (out_l); layers
// n_in -> width (ReLU) -> ... -> width (ReLU) -> 1 (linear).
// All reductions run in a fixed order (no atomics), so results are
// deterministic.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <random>
#include <string>
#include <type_traits>
#include <vector>

#include "tn_internal.h"
#include "tn_mlp.h"

namespace tn {

#define HIPCHK_M(x)                                                                        \
    do {                                                                                   \
        hipError_t e_ = (x);                                                               \
        if (e_ != hipSuccess) fail(TN_EHIP, std::string(#x) + ": " + hipGetErrorString(e_)); \
    } while (0)

struct MlpLayout {
    int n_in, width, depth, n_layers;
    std::vector<int> din, dout;
    std::vector<int64_t> w_off, b_off;   // offsets inside params
    int64_t P;                           // parameter count
    int64_t norm_off, params_off, grads_off, m_off, v_off, total;
};

static MlpLayout layout_of(const tn_mlp_shape* s) {
    if (!s || s->n_in < 1 || s->n_in > 4096 || s->width < 1 || s->width > 4096 || s->depth < 1 || s->depth > 16)
        fail(TN_EINVAL, "bad MLP shape");
    MlpLayout L;
    L.n_in = s->n_in;
    L.width = s->width;
    L.depth = s->depth;
    L.n_layers = s->depth + 1;
    int64_t off = 0;
    for (int l = 0; l < L.n_layers; ++l) {
        const int din = l == 0 ? s->n_in : s->width;
        const int dout = l == L.n_layers - 1 ? 1 : s->width;
        L.din.push_back(din);
        L.dout.push_back(dout);
        L.w_off.push_back(off);
        off += (int64_t)din * dout;
        L.b_off.push_back(off);
        off += dout;
    }
    L.P = off;
    L.norm_off = 0;
    L.params_off = 2 * (int64_t)s->n_in;
    L.grads_off = L.params_off + L.P;
    L.m_off = L.grads_off + L.P;
    L.v_off = L.m_off + L.P;
    L.total = L.v_off + L.P;
    return L;
}

// The fused launch serves networks whose layers a block's eight waves hold in
// registers (up to 256 columns) and whose rows fit 64 KB of LDS; others go
// layer by layer.  Rows per block: 64 for the most reuse of a block's weight
// reads, fewer while that leaves CUs without a block.  Returns the LDS bytes of
// a block of 16 rt rows, 0 if the shape is not served.
static size_t fused_lds(const MlpLayout& L, int rt, bool train, int* pitch) {
    const int cols = (std::max(L.n_in, L.width) + 15) / 16 * 16;
    *pitch = cols + 4;      // rows start 4 LDS banks apart: conflict-free 16-byte reads
    const size_t b = (size_t)16 * rt * *pitch * 4 * (train ? L.depth + 1 : 1);
    return cols <= 256 && b <= 60 * 1024 ? b : 0;
}

// Output tiles of a weight-gradient launch (64 x 64 weights each; of all layers,
// layer < 0, or of one) and the number of row ranges a batch of n is split over:
// enough blocks for two per CU, at least 64 rows each.  One range writes the
// gradients directly, more write FP64 partials that the reduction adds in range
// order.
constexpr int kGradTile = 64;
static int64_t grad_tiles(const MlpLayout& L, int layer) {
    int64_t t = 0;
    for (int l = 0; l < L.n_layers; ++l)
        if (layer < 0 || l == layer)
            t += (int64_t)((L.dout[l] + kGradTile - 1) / kGradTile) * ((L.din[l] + kGradTile - 1) / kGradTile);
    return t;
}
static int64_t grad_splits(const MlpLayout& L, int64_t n, int layer) {
    const int64_t s = std::max<int64_t>(1, std::min<int64_t>(512 / grad_tiles(L, layer), n / 64));
    return s >= 8 ? s & ~int64_t(7) : s;     // as many ranges on each XCD
}
static int64_t layer_params(const MlpLayout& L, int l) { return (int64_t)L.dout[l] * (L.din[l] + 1); }

// Layer by layer, the pre-activations' gradients of more hidden layers than two
// are kept for one weight-gradient launch over all layers while they take up to
// 256 MB more than two would.  Above that a layer's weight gradients are formed
// before its inputs' gradients, which then take the place of its inputs (16
// hidden layers of 1024, 65536 rows: 8.6 GB of workspace, 4.3 GB so).  Below, the
// launches per layer are not worth it (6 hidden layers of 272, 16000 rows, a step
// 2993 us kept, 3058 in place; 5 of 1024, 8192 rows 13615 and 13053).
constexpr int64_t kKeptGradFloats = 64 << 20;
static int64_t in_place_from(const MlpLayout& L) {      // smallest such batch
    int pitch;
    if (L.depth <= 2 || fused_lds(L, 1, true, &pitch)) return INT64_MAX;
    return kKeptGradFloats / ((int64_t)(L.depth - 2) * L.width) + 1;
}

// Workspace of a batch of n (float offsets): normalized input, activations of
// the hidden layers, output, its gradient, gradients of the hidden layers'
// pre-activations, FP64 loss partials (a block's rows each) and FP64 gradient
// partials.
struct MlpWs {
    int64_t xn, acts, y, dy, dz, part, grad, total;
};
static MlpWs ws_layout(const MlpLayout& L, int64_t n) {
    MlpWs w;
    auto up = [](int64_t v) { return (v + 63) / 64 * 64; };
    w.xn = 0;
    w.acts = up(n * L.n_in);
    w.y = up(w.acts + (int64_t)L.depth * n * L.width);
    w.dy = up(w.y + n);
    w.dz = up(w.dy + n);
    const bool in_place = n >= in_place_from(L);
    if (in_place) w.dz = w.acts;
    w.part = in_place ? up(w.dy + n) : up(w.dz + (int64_t)L.depth * n * L.width);
    w.grad = up(w.part + 2 * ((n + 15) / 16));
    int64_t partials = 0;                               // FP64, of the ranges that run together
    for (int l = in_place ? 0 : -1; l < (in_place ? L.n_layers : 0); ++l) {
        const int64_t S = grad_splits(L, n, l);
        if (S > 1) partials = std::max(partials, S * (l < 0 ? L.P : layer_params(L, l)));
    }
    w.total = up(w.grad + 2 * partials);
    return w;
}
// floats that hold every batch up to n
static int64_t ws_floats(const MlpLayout& L, int64_t n) {
    const int64_t m = in_place_from(L) - 1;
    return std::max(ws_layout(L, n).total, n > m ? ws_layout(L, m).total : 0);
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
__global__ void k_fill(float* p, int64_t n, float v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// column mean and 1/std of x (n x d); one block per column, FP64 accumulation
__global__ __launch_bounds__(256) void k_col_stats(const float* x, int64_t n, int d, float* mean, float* istd) {
    __shared__ double s1[256], s2[256];
    const int c = blockIdx.x;
    double a = 0, b = 0;
    for (int64_t r = threadIdx.x; r < n; r += 256) {
        const double v = x[r * d + c];
        a += v;
        b += v * v;
    }
    s1[threadIdx.x] = a;
    s2[threadIdx.x] = b;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            s1[threadIdx.x] += s1[threadIdx.x + w];
            s2[threadIdx.x] += s2[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double m = s1[0] / (double)n;
        const double var = s2[0] / (double)n - m * m;
        mean[c] = (float)m;
        istd[c] = var > 1e-12 ? (float)(1.0 / sqrt(var)) : 1.0f;
    }
}

__global__ void k_normalize(const float* x, const float* mean, const float* istd, float* y, int64_t n, int d) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * d) return;
    const int c = (int)(i % d);
    y[i] = (x[i] - mean[c]) * istd[c];
}

// Y[n x out] = act(X[n x in] W^T + b); 64 x 64 output tile, 256 threads with
// 4 x 4 outputs each, inputs staged through LDS in chunks of 16
__global__ __launch_bounds__(256) void k_linear_fwd(const float* __restrict__ X, const float* __restrict__ W,
                                                    const float* __restrict__ b, float* __restrict__ Y, int64_t n,
                                                    int din, int dout, int relu) {
    __shared__ float Xs[16][64 + 1];
    __shared__ float Ws[16][64 + 1];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int o0 = blockIdx.y * 64;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < din; k0 += 16) {
        for (int e = threadIdx.x; e < 16 * 64; e += 256) {
            const int kk = e & 15, rr = e >> 4;
            const int64_t r = r0 + rr;
            const int o = o0 + rr;
            Xs[kk][rr] = (r < n && k0 + kk < din) ? X[r * din + k0 + kk] : 0.0f;
            Ws[kk][rr] = (o < dout && k0 + kk < din) ? W[(int64_t)o * din + k0 + kk] : 0.0f;
        }
        __syncthreads();
        for (int kk = 0; kk < 16; ++kk) {
            float xv[4], wv[4];
            for (int i = 0; i < 4; ++i) xv[i] = Xs[kk][ty + 16 * i];
            for (int j = 0; j < 4; ++j) wv[j] = Ws[kk][tx + 16 * j];
            for (int i = 0; i < 4; ++i)
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(xv[i], wv[j], acc[i][j]);
        }
        __syncthreads();
    }
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) {
            const int64_t r = r0 + ty + 16 * i;
            const int o = o0 + tx + 16 * j;
            if (r < n && o < dout) {
                float v = acc[i][j] + b[o];
                if (relu) v = v > 0.0f ? v : 0.0f;
                Y[r * dout + o] = v;
            }
        }
}

// squared-error gradient: dY = 2 w (y - t) / n; per-block partial losses (FP64)
__global__ __launch_bounds__(256) void k_loss_grad(const float* y, const float* t, const float* w, float* dy,
                                                   double* part, int64_t n) {
    __shared__ double red[256];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double l = 0;
    if (i < n) {
        const float wi = w ? w[i] : 1.0f;
        const float d = y[i] - t[i];
        dy[i] = 2.0f * wi * d / (float)n;
        l = (double)wi * (double)d * (double)d;
    }
    red[threadIdx.x] = l;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// dX[n x din] = (dZ[n x dout] W) * (A_prev > 0): gradient through a layer and
// the previous layer's ReLU (A_prev is that layer's output; dX may replace it)
__global__ __launch_bounds__(256) void k_linear_bwd_data(const float* __restrict__ dZ, const float* __restrict__ W,
                                                         const float* Aprev, float* dX,
                                                         int64_t n, int din, int dout) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * din) return;
    const int64_t r = idx / din;
    const int i = (int)(idx - r * din);
    float s = 0.0f;
    for (int o = 0; o < dout; ++o) s = fmaf(dZ[r * dout + o], W[(int64_t)o * din + i], s);
    dX[idx] = Aprev[idx] > 0.0f ? s : 0.0f;
}

struct AdamArgs {
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(float* p, float gi, float* m, float* v, int64_t i, const AdamArgs& a) {
    const float mi = a.b1 * m[i] + (1.0f - a.b1) * gi;
    const float vi = a.b2 * v[i] + (1.0f - a.b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}

__global__ void k_adam(float* p, const float* g, float* m, float* v, int64_t P, AdamArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < P) adam_update(p, g[i], m, v, i, a);
}

__global__ void k_log_targets(const double* x, float* t, int64_t n, double floor_v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) t[i] = (float)log(x[i] > floor_v ? x[i] : floor_v);
}

static unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

static AdamArgs adam_args(float lr, int step) {
    AdamArgs a{lr, 0.9f, 0.999f, 1e-8f, 0, 0};
    a.c1 = 1.0f - std::pow(a.b1, (float)step);
    a.c2 = 1.0f - std::pow(a.b2, (float)step);
    return a;
}

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_u __attribute__((ext_vector_type(4), aligned(4)));   // 4 floats at any float's alignment
typedef double v4d __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// The whole network of a block of 16 RT rows in one launch: normalized rows
// and activations stay in LDS, eight waves take 16 CT output columns each, and
// the products run on the FP32 matrix cores (v_mfma_f32_16x16x4f32, which adds
// its four products one after another like a chain of fmaf).  Every sum runs over
// ascending inner indices, as in the kernels of one layer each, so both routes
// give the same bits: instruction q of a group of 16 takes indices 4 q + lane / 16.
// In LDS the 16 are stored 4 x 4 transposed, so a lane reads its four with one
// 16-byte load; weights are transposed in registers (four lane swaps).
//   TRAIN = false: the output column only, layers in place in one LDS buffer.
//   TRAIN = true: also the loss partial of the block, dL/dy, and the gradients
//     through the layers (the same products against W instead of W^T), each
//     written over its layer's activations in LDS; normalized rows,
//     activations and gradients go to the workspace for the weight gradients.
// Bound: the matrix cores for many rows; for a mini-batch (4096 rows: 256
// blocks, one per CU) the chain of 2 depth layers, each its weights from L2
// (150 KB per block at 36 -> 128 x 3 -> 1) and its MFMAs.  36 -> 128 x 3 -> 1:
// scores of 32490 rows 112 us with a launch per layer (64 x 64 FMA tiles), 31 us
// with this one; the training step below.
// ---------------------------------------------------------------------------
struct MlpArgs {
    const float *x, *t, *w, *mean, *istd, *params;
    float *y, *xn, *acts, *dy, *dz;
    double* part;
    int64_t n;
    int n_in, width, depth, pitch;
};

// LDS position of column c of a row: 4 x 4 transposed within its group of 16
__device__ __forceinline__ int lds_col(int c) { return (c & ~15) | (c & 3) << 2 | (c >> 2 & 3); }

// lane group g's element q becomes lane group q's element g (groups of 16 lanes)
__device__ __forceinline__ v4f transpose_groups(v4f x) {
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    uint32_t u[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] = __float_as_uint(x[q]);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const v2u t = __builtin_amdgcn_permlane32_swap(u[q], u[q + 2], false, false);
        u[q] = t[0];
        u[q + 2] = t[1];
    }
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
        const v2u t = __builtin_amdgcn_permlane16_swap(u[q], u[q + 1], false, false);
        u[q] = t[0];
        u[q + 1] = t[1];
    }
    return v4f{__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]), __uint_as_float(u[3])};
}

// (128 registers where two blocks share a CU: four waves per SIMD)
template <int RT, int CT, bool TRAIN>
__global__ __launch_bounds__(512, CT == 1 && !TRAIN ? 4 : 2) void k_mlp_fused(MlpArgs a) {
    constexpr int R = 16 * RT;
    extern __shared__ __align__(16) float lds[];
    __shared__ __align__(16) float wo[256];
    __shared__ float dys[R];
    __shared__ double ls[R];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane & 15, grp = lane >> 4;
    const int pitch = a.pitch, W = a.width, D = a.n_in;
    const int64_t r0 = (int64_t)blockIdx.x * R;
    const int64_t bufsz = (int64_t)R * pitch;
    const int64_t lsz = (int64_t)W * W + W;                  // parameters of a hidden layer past the first
    const float* p1 = a.params + (int64_t)D * W + W;         // second layer
    const int c0 = wave * 16 * CT;                           // this wave's first column
    constexpr int G = 8;                                     // groups of 16 inner indices in registers
    v4f acc[RT][CT], w[CT][G], wt[CT];
    float bias[CT];
    // w = the whole inner groups g0 .. g0 + G of a layer's weights, wt = the ragged
    // group behind its last whole one (bwd = false: Wt is W x K, the lane's column is
    // a row of it; true: Wt is K x W).  Columns past W repeat the last one: their
    // results are not used.  The code is kept short: a block runs each part of the
    // kernel once or twice, so it waits for instructions as much as for data.
    auto weights = [&](const float* Wt, int K, int g0, auto bwd) {
        constexpr bool BWD = decltype(bwd)::value;
        const int nf = K >> 4;
        uint32_t at[CT];
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int c = c0 + 16 * j + sub, col = c < W ? c : W - 1;
            at[j] = BWD ? grp * W + col : col * K + 4 * grp;
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (g0 + g >= nf) break;
            const float* p = Wt + 16 * (g0 + g) * (BWD ? W : 1);
#pragma unroll
            for (int j = 0; j < CT; ++j)
                if constexpr (BWD) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) w[j][g][q] = (p + 4 * q * W)[at[j]];
                } else {
                    w[j][g] = *(const v4f_u*)(p + at[j]);
                }
        }
        if ((K & 15) && nf <= g0 + G) {
            const float* p = Wt + 16 * nf * (BWD ? W : 1);
#pragma unroll
            for (int j = 0; j < CT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    wt[j][q] = 0.0f;
                    if (16 * nf + 4 * q + grp < K) wt[j][q] = p[at[j] + (BWD ? 4 * q * W : 4 * q - 3 * grp)];
                }
        }
    };
    // acc = In Wt^T or In Wt, K <= 256 inner indices; w and wt hold the first groups
    auto product = [&](const float* in, const float* Wt, int K, auto bwd) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) acc[i][j] = v4f{0, 0, 0, 0};
        const int nf = K >> 4;
        auto group = [&](int at, const v4f* wg, int step) {
            v4f x[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i) x[i] = *(const v4f*)&in[(16 * i + sub) * pitch + 16 * at + 4 * grp];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int j = 0; j < CT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i][q], wg[j * step][q], acc[i][j], 0, 0, 0);
        };
        for (int g0 = 0; g0 < nf || g0 == 0; g0 += G) {
            if (g0 > 0) weights(Wt, K, g0, bwd);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (g0 + g >= nf) break;
                if constexpr (!decltype(bwd)::value) {
#pragma unroll
                    for (int j = 0; j < CT; ++j) w[j][g] = transpose_groups(w[j][g]);
                }
                group(g0 + g, &w[0][g], G);
            }
        }
        if (K & 15) group(nf, wt, 1);
    };
    constexpr std::integral_constant<bool, false> fwd{};
    constexpr std::integral_constant<bool, true> back{};
    // a layer's biases and weights, the biases first (loads arrive in order)
    auto layer = [&](const float* Wl, int K) {
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int col = c0 + 16 * j + sub;
            bias[j] = Wl[(int64_t)K * W + (col < W ? col : W - 1)];
        }
        weights(Wl, K, 0, fwd);
    };
    // rows of an LDS buffer to global memory, a wave a row
    auto save = [&](const float* from, float* to, int cols) {
        for (int r = wave; r < R && r0 + r < a.n; r += 8)
            for (int c = lane; c < cols; c += 64) to[(r0 + r) * cols + c] = from[r * pitch + lds_col(c)];
    };
    const int din16 = (D + 15) & ~15, w16 = (W + 15) & ~15;
    const float* Wo = p1 + (int64_t)(a.depth - 1) * lsz;     // output layer
    const int orl = 16 * wave + 4 * grp + sub;               // this thread's row there, if it has one
    const bool orv = wave < RT && sub < 4;
    const int64_t orow = r0 + orl;
    float tr = 0.0f, wr = 1.0f;
    if (TRAIN && orv && orow < a.n) {
        tr = a.t[orow];
        if (a.w) wr = a.w[orow];
    }
    if (tid < 256) wo[lds_col(tid)] = tid < W ? Wo[tid] : 0.0f;
    const float bo = Wo[W];
    if (c0 < w16) layer(a.params, D);
    // rows in, normalized; inner columns up to a multiple of 16 are zero
    for (int c = lane; c < din16; c += 64) {
        const float m = c < D ? a.mean[c] : 0.0f, is = c < D ? a.istd[c] : 0.0f;
        for (int r = wave; r < R; r += 8)
            lds[r * pitch + lds_col(c)] = c < D && r0 + r < a.n ? (a.x[(r0 + r) * D + c] - m) * is : 0.0f;
    }
    __syncthreads();
    if (TRAIN) save(lds, a.xn, D);
    // element e of a lane's result is row 4 grp + e of its block
    float* cur = lds;
    for (int l = 0; l < a.depth; ++l) {
        const float* Wl = l == 0 ? a.params : p1 + (l - 1) * lsz;
        float* nxt = TRAIN ? cur + bufsz : cur;
        float bl[CT];
        if (c0 < w16) {
            product(cur, Wl, l == 0 ? D : W, fwd);
#pragma unroll
            for (int j = 0; j < CT; ++j) bl[j] = bias[j];
            // the next product's weights arrive during this layer's end
            if (l + 1 < a.depth) layer(p1 + l * lsz, W);
            else if (TRAIN && l > 0) weights(p1 + (l - 1) * lsz, W, 0, back);
        }
        if (!TRAIN) __syncthreads();                         // every wave has read the rows it overwrites
        if (c0 < w16) {
#pragma unroll
            for (int j = 0; j < CT; ++j) {
                const int col = c0 + 16 * j + sub, pos = lds_col(col);
                if (col >= w16) continue;
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float s = acc[i][j][e] + bl[j];
                        nxt[(16 * i + 4 * grp + e) * pitch + pos] = col < W && s > 0.0f ? s : 0.0f;
                    }
            }
        }
        cur = nxt;
        __syncthreads();
    }
    // output layer: a wave per 16 rows (all 16 columns of the product are the one)
    if (wave < RT) {
        v4f o = v4f{0, 0, 0, 0};
        for (int g = 0; g < w16; g += 16) {
            const v4f x = *(const v4f*)&cur[(16 * wave + sub) * pitch + g + 4 * grp], y = *(const v4f*)&wo[g + 4 * grp];
#pragma unroll
            for (int q = 0; q < 4; ++q) o = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q], y[q], o, 0, 0, 0);
        }
        const float y = (sub == 0 ? o[0] : sub == 1 ? o[1] : sub == 2 ? o[2] : o[3]) + bo;
        if (orv) {
            if (!TRAIN) {
                if (orow < a.n) a.y[orow] = y;
            } else {
                float dy = 0.0f;
                double l = 0.0;
                if (orow < a.n) {
                    const float d = y - tr;
                    dy = 2.0f * wr * d / (float)a.n;
                    l = (double)wr * (double)d * (double)d;
                    a.dy[orow] = dy;
                }
                dys[orl] = dy;
                ls[orl] = l;
            }
        }
    }
    if constexpr (TRAIN) {
        for (int l = 0; l < a.depth; ++l) save(lds + (l + 1) * bufsz, a.acts + (int64_t)l * a.n * W, W);
        __syncthreads();
        if (tid == 0) {
            double l = 0.0;
            for (int r = 0; r < R; ++r) l += ls[r];
            a.part[blockIdx.x] = l;
        }
        // gradient of the last hidden layer's pre-activations, over its activations
        for (int r = wave; r < R; r += 8)
            for (int c = lane; c < w16; c += 64) cur[r * pitch + c] = cur[r * pitch + c] > 0.0f ? dys[r] * wo[c] : 0.0f;
        __syncthreads();
        for (int l = a.depth - 1; l > 0; --l) {
            float* prev = cur - bufsz;                       // activations below layer l, then their gradients
            if (c0 < w16) {
                product(cur, p1 + (l - 1) * lsz, W, back);
                if (l > 1) weights(p1 + (l - 2) * lsz, W, 0, back);
#pragma unroll
                for (int j = 0; j < CT; ++j) {
                    if (c0 + 16 * j >= w16) continue;
                    float* at = prev + 4 * grp * pitch + lds_col(c0 + 16 * j + sub);
#pragma unroll
                    for (int i = 0; i < RT; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float& v = at[(16 * i + e) * pitch];
                            v = v > 0.0f ? acc[i][j][e] : 0.0f;
                        }
                }
            }
            cur = prev;
            __syncthreads();
        }
        for (int l = 0; l < a.depth; ++l) save(lds + (l + 1) * bufsz, a.dz + (int64_t)l * a.n * W, W);
    }
}

// Weight and bias gradients of all layers: dW[o][i] = sum_r dZ[r][o] A[r][i],
// db[o] = sum_r dZ[r][o], accumulated in FP64 on the matrix cores
// (v_mfma_f64_16x16x4f64; products of two floats are exact).  Block (tile,
// split): 64 x 64 weights over one range of rows, a wave 32 x 32 of them read
// straight from the row-major operands (64-byte runs), the next rows' loads in
// flight during these rows' products.  Bound: the FP64 pipes (half as many blocks
// of twice the rows take the same time).  A training step of 4096 rows,
// 36 -> 128 x 3 -> 1: 6137 us with one thread per weight summing all rows, 50 us
// with this launch (21 us of it; 27.7 with conditional loads that were waited for
// one by one) and the fused one (three launches instead of 15).
struct GradArgs {
    const float *xn, *acts, *dy, *dz;      // acts, dz: hidden layers after one another
    int n_in, width, depth, splits;
    int layer;                             // the one layer of this launch, -1: all
    int64_t n, rows, P;                    // rows: rows of a split; P: parameters of the launch
    float* grads;                          // splits == 1: written here
    double* part;                          // else: partials [split][P]
};

__global__ __launch_bounds__(256) void k_mlp_wgrad(GradArgs a) {
    // The tiles of a row range run on one of the eight XCDs (blocks go to them in
    // turn), so its rows come from memory once.
    const int b = blockIdx.x, per = (int)gridDim.x / a.splits;
    const bool by8 = a.splits % 8 == 0;
    const int split = by8 ? (b >> 3) / per * 8 + (b & 7) : b / per;
    int t = by8 ? (b >> 3) % per : b % per;
    // layers in order: n_in -> width, the hidden ones, width -> 1
    const int W = a.width, tw = (W + kGradTile - 1) / kGradTile, ti = (a.n_in + kGradTile - 1) / kGradTile;
    int l = a.layer < 0 ? 0 : a.layer;
    if (a.layer < 0 && t >= tw * ti) {
        t -= tw * ti;
        l = 1 + t / (tw * tw) < a.depth ? 1 + t / (tw * tw) : a.depth;
        t -= (l - 1) * tw * tw;
    }
    const int din = l == 0 ? a.n_in : W, dout = l == a.depth ? 1 : W;
    const int64_t w_off =
        l == 0 || a.layer >= 0 ? 0 : (int64_t)W * (a.n_in + 1) + (int64_t)(l - 1) * W * (W + 1);
    const int64_t b_off = w_off + (int64_t)din * dout;
    const int ti_n = l == 0 ? ti : tw;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int o0 = t / ti_n * kGradTile + 32 * (wave >> 1), i0 = t % ti_n * kGradTile + 32 * (wave & 1);
    if (o0 >= dout || i0 >= din) return;
    const int sub = lane & 15, grp = lane >> 4;
    const int64_t rb = (int64_t)split * a.rows;
    const int64_t re = rb + a.rows < a.n ? rb + a.rows : a.n;
    const float* __restrict__ dz = l == a.depth ? a.dy : a.dz + l * a.n * W;
    const float* __restrict__ act = l == 0 ? a.xn : a.acts + (l - 1) * a.n * W;
    const bool ov[2] = {o0 + sub < dout, o0 + 16 + sub < dout};
    const bool iv[2] = {i0 + sub < din, i0 + 16 + sub < din};
    // every lane loads (conditional loads were waited for one by one): columns past
    // the layer repeat its last one, rows past the range its first
    const int oc[2] = {o0 + sub < dout ? o0 + sub : dout - 1, o0 + 16 + sub < dout ? o0 + 16 + sub : dout - 1};
    const int ic[2] = {i0 + sub < din ? i0 + sub : din - 1, i0 + 16 + sub < din ? i0 + 16 + sub : din - 1};
    const bool two_o = o0 + 16 < dout, two_i = i0 + 16 < din;
    v4d acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = v4d{0, 0, 0, 0};
    double bs[2] = {0.0, 0.0};
    constexpr int U = 8;           // row groups of 4 whose loads are in flight together
    auto load = [&](int64_t r, float (&x)[U][2], float (&y)[U][2]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t at = r + 4 * u + grp, row = at < re ? at : rb;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                x[u][q] = dz[row * dout + oc[q]];
                y[u][q] = act[row * din + ic[q]];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int64_t r, const float (&x)[U][2], const float (&y)[U][2]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r + 4 * u >= re) break;
            // (columns past the layer are not written: only rows past the range are zeroed)
            const bool rv = r + 4 * u + grp < re;
            const double xd[2] = {rv ? (double)x[u][0] : 0.0, rv ? (double)x[u][1] : 0.0};
            const double yd[2] = {rv ? (double)y[u][0] : 0.0, rv ? (double)y[u][1] : 0.0};
            bs[0] += xd[0];
            bs[1] += xd[1];
            acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(xd[0], yd[0], acc[0][0], 0, 0, 0);
            if (two_i) acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(xd[0], yd[1], acc[0][1], 0, 0, 0);
            if (two_o) acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(xd[1], yd[0], acc[1][0], 0, 0, 0);
            if (two_o && two_i) acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(xd[1], yd[1], acc[1][1], 0, 0, 0);
        }
    };
    // the next 4 U rows are loaded during the products of these
    float x0[U][2], y0[U][2], x1[U][2], y1[U][2];
    if (rb < re) load(rb, x0, y0);
    for (int64_t r = rb; r < re; r += 8 * U) {
        load(r + 4 * U, x1, y1);
        multiply(r, x0, y0);
        load(r + 8 * U, x0, y0);
        multiply(r + 4 * U, x1, y1);
    }
    double* part = a.part + (int64_t)split * a.P;
    auto put = [&](int64_t at, double v) {
        if (a.splits == 1) a.grads[at] = (float)v;
        else part[at] = v;
    };
    // element e of a lane's result is row grp + 4 e of its block
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = o0 + 16 * i + grp + 4 * e;
                if (o < dout && iv[j]) put(w_off + (int64_t)o * din + i0 + 16 * j + sub, acc[i][j][e]);
            }
    if (i0 == 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            bs[i] += __shfl_xor(bs[i], 16);
            bs[i] += __shfl_xor(bs[i], 32);
            if (grp == 0 && ov[i]) put(b_off + o0 + 16 * i + sub, bs[i]);
        }
    }
}

// Gradient partials added in range order, the Adam update of the same weight
// (adam != 0), and the loss (the launch's last block; loss null: none).
__global__ __launch_bounds__(256) void k_mlp_reduce(const double* part, int splits, int64_t P, float* g, float* p,
                                                    float* m, float* v, int adam, AdamArgs aa, const double* lpart,
                                                    int nb, int64_t n, float* loss) {
    if (loss && blockIdx.x == gridDim.x - 1) {
        __shared__ double red[256];
        double s = 0;
        for (int i = threadIdx.x; i < nb; i += 256) s += lpart[i];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss = (float)(red[0] / (double)n);
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= P) return;
    float gi;
    if (splits > 1) {
        double s = 0.0;
#pragma unroll 8
        for (int q = 0; q < splits; ++q) s += part[q * P + i];
        gi = (float)s;
        g[i] = gi;
    } else {
        gi = g[i];
    }
    if (adam) adam_update(p, gi, m, v, i, aa);
}

template <int RT, bool TRAIN>
static void launch_fused_rt(const MlpArgs& a, size_t lds, hipStream_t s) {
    const dim3 grid(nblk(a.n, 16 * RT));
    if (a.width <= 128) hipLaunchKernelGGL((k_mlp_fused<RT, 1, TRAIN>), grid, dim3(512), lds, s, a);
    else hipLaunchKernelGGL((k_mlp_fused<RT, 2, TRAIN>), grid, dim3(512), lds, s, a);
}

// launches the fused kernel; returns its row blocks, 0 if the shape is not served
template <bool TRAIN>
static int64_t launch_fused(const MlpLayout& L, MlpArgs a, hipStream_t s) {
    int rt = TRAIN ? 2 : 4;
    while (rt > 1 && (a.n < (int64_t)16 * rt * 256 || !fused_lds(L, rt, TRAIN, &a.pitch))) rt /= 2;
    const size_t lds = fused_lds(L, rt, TRAIN, &a.pitch);
    if (!lds) return 0;
    if (rt == 1) launch_fused_rt<1, TRAIN>(a, lds, s);
    else if (rt == 2) launch_fused_rt<2, TRAIN>(a, lds, s);
    else if constexpr (!TRAIN) launch_fused_rt<4, TRAIN>(a, lds, s);
    return nblk(a.n, 16 * rt);
}

static MlpArgs mlp_args(const MlpLayout& L, const float* state, const float* x, int64_t n) {
    MlpArgs a{};
    a.x = x;
    a.mean = state + L.norm_off;
    a.istd = a.mean + L.n_in;
    a.params = state + L.params_off;
    a.n = n;
    a.n_in = L.n_in;
    a.width = L.width;
    a.depth = L.depth;
    return a;
}

// layer by layer, activations kept in the workspace
static void forward_layers(const MlpLayout& L, const float* state, const float* x, int64_t n, float* ws, float* y,
                           hipStream_t s) {
    const MlpWs o = ws_layout(L, n);
    hipLaunchKernelGGL(k_normalize, dim3(nblk(n * L.n_in, 256)), dim3(256), 0, s, x, state + L.norm_off,
                       state + L.norm_off + L.n_in, ws + o.xn, n, L.n_in);
    const float* in = ws + o.xn;
    const float* params = state + L.params_off;
    for (int l = 0; l < L.n_layers; ++l) {
        const bool last = l == L.n_layers - 1;
        float* out = last ? y : ws + o.acts + (int64_t)l * n * L.width;
        dim3 grid(nblk(n, 64), nblk(L.dout[l], 64));
        hipLaunchKernelGGL(k_linear_fwd, grid, dim3(256), 0, s, in, params + L.w_off[l], params + L.b_off[l], out, n,
                           L.din[l], L.dout[l], last ? 0 : 1);
        in = out;
    }
}

static bool overlap(const float* a, int64_t na, const float* b, int64_t nb) {
    const uintptr_t pa = (uintptr_t)a, pb = (uintptr_t)b;
    return pa < pb + 4 * (uintptr_t)nb && pb < pa + 4 * (uintptr_t)na;
}

// A block writes its outputs while others still read their rows, the weights or
// (layer by layer) the last activations: outputs that lie over any of these are
// formed in the workspace and copied once every block is done.
static void forward(const MlpLayout& L, const float* state, const float* x, int64_t n, float* ws, float* y,
                    hipStream_t s) {
    const MlpWs o = ws_layout(L, n);
    const bool over = overlap(y, n, x, n * L.n_in) || overlap(y, n, state, L.total) || overlap(y, n, ws, o.total);
    // (the normalized rows are not read any more when the last layer runs)
    float* out = !over ? y : ws + (overlap(y, n, ws + o.y, n) ? o.xn : o.y);
    MlpArgs a = mlp_args(L, state, x, n);
    a.y = out;
    if (!launch_fused<false>(L, a, s)) forward_layers(L, state, x, n, ws, out, s);
    if (over) HIPCHK_M(hipMemcpyAsync(y, out, n * 4, hipMemcpyDeviceToDevice, s));
}

// loss and gradients, and with `adam` the update of the parameters
static void gradients(const MlpLayout& L, float* state, const float* x, const float* t, const float* w, int64_t n,
                      float* ws, float* loss, const AdamArgs* adam, hipStream_t s) {
    const MlpWs o = ws_layout(L, n);
    double* lpart = (double*)(ws + o.part);
    float* params = state + L.params_off;
    MlpArgs a = mlp_args(L, state, x, n);
    a.t = t;
    a.w = w;
    a.xn = ws + o.xn;
    a.acts = ws + o.acts;
    a.dy = ws + o.dy;
    a.dz = ws + o.dz;
    a.part = lpart;
    GradArgs g{};
    g.xn = a.xn;
    g.acts = a.acts;
    g.dy = a.dy;
    g.dz = a.dz;
    g.n_in = L.n_in;
    g.width = L.width;
    g.depth = L.depth;
    g.n = n;
    g.part = (double*)(ws + o.grad);
    int64_t nb = launch_fused<true>(L, a, s);
    // weight gradients of one layer or (layer < 0) of all
    auto wgrad = [&](int layer) {
        g.layer = layer;
        g.splits = (int)grad_splits(L, n, layer);
        g.rows = (n + g.splits - 1) / g.splits;
        g.P = layer < 0 ? L.P : layer_params(L, layer);
        g.grads = state + L.grads_off + (layer < 0 ? 0 : L.w_off[layer]);
        hipLaunchKernelGGL(k_mlp_wgrad, dim3((unsigned)(grad_tiles(L, layer) * g.splits)), dim3(256), 0, s, g);
    };
    // ... added up, and the update; the loss with the first launch
    auto reduce = [&](bool with_loss) {
        const int64_t at = g.grads - state - L.grads_off;
        hipLaunchKernelGGL(k_mlp_reduce, dim3(nblk(g.P, 256) + (with_loss ? 1 : 0)), dim3(256), 0, s, g.part, g.splits,
                           g.P, g.grads, params + at, state + L.m_off + at, state + L.v_off + at, adam ? 1 : 0,
                           adam ? *adam : AdamArgs{}, lpart, (int)nb, n, with_loss ? loss : nullptr);
    };
    if (!nb) {
        const bool in_place = o.dz == o.acts;
        forward_layers(L, state, x, n, ws, ws + o.y, s);
        nb = nblk(n, 256);
        hipLaunchKernelGGL(k_loss_grad, dim3((unsigned)nb), dim3(256), 0, s, ws + o.y, t, w, a.dy, lpart, n);
        const float* dz = a.dy;
        for (int l = L.n_layers - 1; l >= 0; --l) {
            if (in_place) wgrad(l);
            if (l > 0) {
                float* below = a.dz + (int64_t)(l - 1) * n * L.width;
                hipLaunchKernelGGL(k_linear_bwd_data, dim3(nblk(n * L.din[l], 256)), dim3(256), 0, s, dz,
                                   params + L.w_off[l], a.acts + (int64_t)(l - 1) * n * L.width, below, n, L.din[l],
                                   L.dout[l]);
                dz = below;
            }
            if (in_place) reduce(l == L.n_layers - 1);
        }
        if (in_place) return;
    }
    wgrad(-1);
    reduce(true);
}

}  // namespace tn

using namespace tn;

template <class F>
static int mguard(F&& f) {
    try {
        f();
        set_last_error("");
        return TN_OK;
    } catch (const Error& e) {
        set_last_error(e.msg);
        return e.code;
    } catch (const std::exception& e) {
        set_last_error(e.what());
        return TN_EINVAL;
    }
}

extern "C" {

int tn_mlp_sizes(const tn_mlp_shape* s, int64_t batch, int64_t* n_params, size_t* state_bytes, size_t* ws_bytes) {
    return mguard([&] {
        MlpLayout L = layout_of(s);
        if (n_params) *n_params = L.P;
        if (state_bytes) *state_bytes = (size_t)L.total * 4;
        if (ws_bytes) *ws_bytes = (size_t)ws_floats(L, std::max<int64_t>(1, batch)) * 4;
    });
}

int tn_mlp_init(const tn_mlp_shape* s, uint64_t seed, void* d_state, void* stream) {
    return mguard([&] {
        MlpLayout L = layout_of(s);
        if (!d_state) fail(TN_EINVAL, "null state");
        std::vector<float> h(L.total, 0.0f);
        for (int i = 0; i < L.n_in; ++i) h[L.norm_off + L.n_in + i] = 1.0f;   // identity normalizer
        std::mt19937_64 rng(seed ? seed : 2211170280ULL);
        for (int l = 0; l < L.n_layers; ++l) {
            std::normal_distribution<double> nd(0.0, std::sqrt(2.0 / L.din[l]));   // He initialisation
            for (int64_t k = 0; k < (int64_t)L.din[l] * L.dout[l]; ++k) h[L.params_off + L.w_off[l] + k] = (float)nd(rng);
        }
        hipStream_t st = (hipStream_t)stream;
        HIPCHK_M(hipMemcpyAsync(d_state, h.data(), h.size() * 4, hipMemcpyHostToDevice, st));
        HIPCHK_M(hipStreamSynchronize(st));
    });
}

int tn_mlp_fit_normalizer(const tn_mlp_shape* s, void* d_state, const float* d_x, int64_t n, void* stream) {
    return mguard([&] {
        MlpLayout L = layout_of(s);
        if (!d_state || !d_x || n < 1) fail(TN_EINVAL, "bad normalizer arguments");
        float* st = (float*)d_state;
        hipLaunchKernelGGL(k_col_stats, dim3(L.n_in), dim3(256), 0, (hipStream_t)stream, d_x, n, L.n_in,
                           st + L.norm_off, st + L.norm_off + L.n_in);
        HIPCHK_M(hipGetLastError());
    });
}

int tn_mlp_forward(const tn_mlp_shape* s, const void* d_state, const float* d_x, int64_t n, float* d_y, void* d_ws,
                   void* stream) {
    return mguard([&] {
        MlpLayout L = layout_of(s);
        if (!d_state || !d_x || !d_y || !d_ws || n < 1) fail(TN_EINVAL, "bad forward arguments");
        forward(L, (const float*)d_state, d_x, n, (float*)d_ws, d_y, (hipStream_t)stream);
        HIPCHK_M(hipGetLastError());
    });
}

int tn_mlp_gradients(const tn_mlp_shape* s, void* d_state, const float* d_x, const float* d_t, const float* d_w,
                     int64_t n, void* d_ws, float* d_loss, void* stream) {
    return mguard([&] {
        MlpLayout L = layout_of(s);
        if (!d_state || !d_x || !d_t || !d_ws || !d_loss || n < 1) fail(TN_EINVAL, "bad gradient arguments");
        gradients(L, (float*)d_state, d_x, d_t, d_w, n, (float*)d_ws, d_loss, nullptr, (hipStream_t)stream);
        HIPCHK_M(hipGetLastError());
    });
}

int tn_mlp_adam(const tn_mlp_shape* s, void* d_state, float lr, int32_t step, void* stream) {
    return mguard([&] {
        MlpLayout L = layout_of(s);
        if (!d_state || step < 1) fail(TN_EINVAL, "bad adam arguments");
        float* st = (float*)d_state;
        hipLaunchKernelGGL(k_adam, dim3(nblk(L.P, 256)), dim3(256), 0, (hipStream_t)stream, st + L.params_off,
                           st + L.grads_off, st + L.m_off, st + L.v_off, L.P, adam_args(lr, step));
        HIPCHK_M(hipGetLastError());
    });
}

int tn_mlp_log_targets(const double* d_x, float* d_t, int64_t n, double floor_v, void* stream) {
    return mguard([&] {
        if (!d_x || !d_t || n < 0 || !(floor_v > 0)) fail(TN_EINVAL, "bad target arguments");
        if (n == 0) return;
        hipLaunchKernelGGL(k_log_targets, dim3(nblk(n, 256)), dim3(256), 0, (hipStream_t)stream, d_x, d_t, n, floor_v);
        HIPCHK_M(hipGetLastError());
    });
}

int tn_mlp_train_step(const tn_mlp_shape* s, void* d_state, const float* d_x, const float* d_t, const float* d_w,
                      int64_t n, float lr, int32_t step, void* d_ws, float* d_loss, void* stream) {
    return mguard([&] {
        MlpLayout L = layout_of(s);
        if (!d_state || !d_x || !d_t || !d_ws || !d_loss || n < 1) fail(TN_EINVAL, "bad gradient arguments");
        // as two calls: with a bad step the gradients are still computed
        const AdamArgs a = adam_args(lr, std::max(step, 1));
        gradients(L, (float*)d_state, d_x, d_t, d_w, n, (float*)d_ws, d_loss, step < 1 ? nullptr : &a,
                  (hipStream_t)stream);
        HIPCHK_M(hipGetLastError());
        if (step < 1) fail(TN_EINVAL, "bad adam arguments");
    });
}

int tn_pruner_train_step(const tn_mlp_shape* s, void* d_state, const float* d_x, const float* d_t,
                         const float* d_w, int64_t n, float lr, int32_t step, void* d_ws, float* d_loss,
                         void* stream) {
    return tn_mlp_train_step(s, d_state, d_x, d_t, d_w, n, lr, step, d_ws, d_loss, stream);
}

// saved model: header {magic, n_in, width, depth, P} then normalizer and parameters
static const char kPrunerMagic[8] = {'T', 'N', 'P', 'R', 'U', 'N', 'E', '1'};

int tn_pruner_save(const tn_mlp_shape* s, const void* d_state, void* h_buf, size_t buf_bytes, size_t* need_bytes,
                   void* stream) {
    return mguard([&] {
        MlpLayout L = layout_of(s);
        const size_t body = (size_t)(L.params_off + L.P) * 4;
        const size_t need = TN_PRUNER_HEADER_BYTES + body;
        if (need_bytes) *need_bytes = need;
        if (!h_buf) return;
        if (!d_state) fail(TN_EINVAL, "null state");
        if (buf_bytes < need) fail(TN_ENOMEM, "buffer smaller than the saved model");
        unsigned char* h = (unsigned char*)h_buf;
        std::memset(h, 0, TN_PRUNER_HEADER_BYTES);
        std::memcpy(h, kPrunerMagic, 8);
        const int32_t dims[3] = {s->n_in, s->width, s->depth};
        std::memcpy(h + 8, dims, sizeof(dims));
        const int64_t P = L.P;
        std::memcpy(h + 24, &P, 8);
        hipStream_t st = (hipStream_t)stream;
        HIPCHK_M(hipMemcpyAsync(h + TN_PRUNER_HEADER_BYTES, d_state, body, hipMemcpyDeviceToHost, st));
        HIPCHK_M(hipStreamSynchronize(st));
    });
}

int tn_pruner_load(const tn_mlp_shape* s, void* d_state, const void* h_buf, size_t buf_bytes, void* stream) {
    return mguard([&] {
        MlpLayout L = layout_of(s);
        const size_t body = (size_t)(L.params_off + L.P) * 4;
        if (!d_state || !h_buf) fail(TN_EINVAL, "null pointer");
        if (buf_bytes < TN_PRUNER_HEADER_BYTES + body) fail(TN_EINVAL, "buffer shorter than the saved model");
        const unsigned char* h = (const unsigned char*)h_buf;
        int32_t dims[3];
        int64_t P;
        std::memcpy(dims, h + 8, sizeof(dims));
        std::memcpy(&P, h + 24, 8);
        if (std::memcmp(h, kPrunerMagic, 8) != 0) fail(TN_EINVAL, "not a saved pruner model");
        if (dims[0] != s->n_in || dims[1] != s->width || dims[2] != s->depth || P != L.P)
            fail(TN_EINVAL, "saved model has another shape");
        hipStream_t st = (hipStream_t)stream;
        // normalizer and parameters; gradients and Adam moments start from zero
        std::vector<float> zeros((size_t)(L.total - L.grads_off), 0.0f);
        HIPCHK_M(hipMemcpyAsync(d_state, h + TN_PRUNER_HEADER_BYTES, body, hipMemcpyHostToDevice, st));
        HIPCHK_M(hipMemcpyAsync((float*)d_state + L.grads_off, zeros.data(), zeros.size() * 4,
                                hipMemcpyHostToDevice, st));
        HIPCHK_M(hipStreamSynchronize(st));
    });
}

}  // extern "C"
