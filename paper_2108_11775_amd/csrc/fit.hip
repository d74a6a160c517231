// fit.hip -- occupancy fit (Sec. 3.1: binary cross-entropy, gradient-descent and Adam
// optimisers) and the hand-written backward of the occupancy.
//
// Loss, full batch:  L(w, beta) = (1/n) sum_i BCE(sigma(s_i), y_i) + (l2/2) |w|^2.
// Gradient:          dL/dw_j = (1/n) sum_i r_i phi_ij + l2 w_j,  dL/dbeta = (1/n) sum_i r_i,
//                    r_i = sigma(s_i) - y_i.
// Backward of s(x; w, beta) for an upstream g:  grad_w = Phi^T g, grad_beta = sum g,
//                    grad_x_i = g_i grad s(x_i)   (with s_fwd: g_i sigma'(s_i) grad s(x_i)).
//
// Phi^T g is the same RBF sum as the forward with the roles of points and hinges
// exchanged (phi depends only on |x_i - h_j|), so it runs on the forward kernel:
// the data points become the LDS-staged weighted set, the hinges the lanes.  The
// point set is split into ranges of at most one LDS tile; each range writes a
// partial row and the rows are summed in a fixed order.  Every reduction here is
// fixed-order (block-range sums, then one block), so results are deterministic.
#include <algorithm>

#include "pdmp_common.h"
#include "rbf_split.h"

namespace pdmp {

constexpr int kRedBlock = 256;
constexpr int kRedMaxBlocks = 1024;

// Blocks of a sum over n: a thread per element as far as the partial sums go (10^5 points
// of the BCE in blocks of 2,048: 6.9 us, the chip mostly idle; of 256: 3.3 us).
static int red_blocks(int64_t n) {
    const int64_t b = (n + kRedBlock - 1) / kRedBlock;
    return b < 1 ? 1 : b > kRedMaxBlocks ? kRedMaxBlocks : (int)b;
}

// The sum of v over the block's threads (fixed order), in every thread.
__device__ __forceinline__ double block_sum(double v, double (&sh)[kRedBlock / 64]) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// Per block: contiguous range, thread-strided sequential sums, then the block's.
__global__ void __launch_bounds__(kRedBlock)
k_sum_partial(const float *__restrict__ x, int64_t n, double *parts) {
    __shared__ double sh[kRedBlock / 64];
    const int64_t per = (n + gridDim.x - 1) / gridDim.x;
    const int64_t b0 = (int64_t)blockIdx.x * per;
    const int64_t b1 = b0 + per < n ? b0 + per : n;
    double acc = 0.0;
    for (int64_t i = b0 + threadIdx.x; i < b1; i += kRedBlock) acc += (double)x[i];
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) parts[blockIdx.x] = acc;
}

// BCE on logits: g_i = (sigma(s_i) - y_i) inv_n [g_scale], each block's sums of g (g_part)
// and of the BCE max(s,0) - y s + log(1 + exp(-|s|)) (bce_part); each output is optional.
// With wsq, one block past those of the points writes |w|^2 over M entries.
__global__ void __launch_bounds__(kRedBlock)
k_bce(const float *__restrict__ s, const uint8_t *__restrict__ y, int64_t n, float inv_n,
      const float *__restrict__ g_scale, int blocks, float *__restrict__ g_out,
      double *__restrict__ g_part, double *__restrict__ bce_part, const float *__restrict__ w,
      int M, double *__restrict__ wsq) {
    __shared__ double sh[kRedBlock / 64];
    if ((int)blockIdx.x == blocks) {
        double acc = 0.0;
#pragma unroll 4
        for (int j = threadIdx.x; j < M; j += kRedBlock) acc += (double)w[j] * (double)w[j];
        acc = block_sum(acc, sh);
        if (threadIdx.x == 0) *wsq = acc;
        return;
    }
    const int64_t per = (n + blocks - 1) / blocks;
    const int64_t b0 = (int64_t)blockIdx.x * per;
    const int64_t b1 = b0 + per < n ? b0 + per : n;
    double acc = 0.0, gacc = 0.0;
    const float gsc = g_scale ? *g_scale : 1.0f;
    for (int64_t i = b0 + threadIdx.x; i < b1; i += kRedBlock) {
        const float sv = s[i];
        const float yv = y[i] ? 1.0f : 0.0f;
        float c, sp;
        sigmoid_and_slope(sv, c, sp);
        float g = (c - yv) * inv_n;
        if (g_scale) g *= gsc;
        if (g_out) g_out[i] = g;
        gacc += g;
        if (bce_part) {
            const float e = exp2_fast(-fabsf(sv) * kLog2e);
            acc += (double)(fmaxf(sv, 0.0f) - yv * sv) + (double)log1pf(e);
        }
    }
    if (g_part) {
        gacc = block_sum(gacc, sh);
        if (threadIdx.x == 0) g_part[blockIdx.x] = gacc;
    }
    if (bce_part) {
        acc = block_sum(acc, sh);
        if (threadIdx.x == 0) bce_part[blockIdx.x] = acc;
    }
}

// out = scale * sum(a[0..na)), fixed order, one block.
__global__ void __launch_bounds__(kRedBlock)
k_final(const double *__restrict__ a, int na, double scale, float *out) {
    __shared__ double sh[kRedBlock / 64];
    double acc = 0.0;
    for (int i = threadIdx.x; i < na; i += kRedBlock) acc += a[i];
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) *out = (float)(scale * acc);
}

// The sum over rows of column j = 64 block + lane of part [rows][m] (valid in wave 0).  A
// block owns 64 columns; its sixteen waves sum the rows r = wave (mod 16) in increasing
// order, issuing the loads four at a time (the adds keep the order), and the sixteen sums
// are added in a fixed order.  With few columns (4096 weights: 64 blocks) each thread's
// chain of loads is short.
constexpr int kSumPh = 16;

__device__ __forceinline__ double row_sum(const float *__restrict__ part, int rows, int64_t m,
                                          int64_t j, double (&sh)[kSumPh][64]) {
    const int cl = threadIdx.x & 63, ph = threadIdx.x >> 6;
    double acc = 0.0;
    if (j < m) {
        int r = ph;
        for (; r + 3 * kSumPh < rows; r += 4 * kSumPh) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = part[(size_t)(r + u * kSumPh) * m + j];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc += v[u];
        }
        for (; r < rows; r += kSumPh) acc += part[(size_t)r * m + j];
    }
    sh[ph][cl] = acc;
    __syncthreads();
    double t = sh[0][cl];
#pragma unroll
    for (int q = 1; q < kSumPh; ++q) t += sh[q][cl];
    return t;
}

// The sum of v over the block's 64 kSumPh threads (fixed order), in thread 0.
__device__ __forceinline__ double wide_sum(double v, double (&sh)[64]) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = sh[0];
#pragma unroll
    for (int q = 1; q < kSumPh; ++q) t += sh[q];
    return t;
}

// out[0..m) = the sums over rows of part, out[m] = the sum of the np partial sums gp, or of
// g[0..n) itself where gp is null (the first block).
__global__ void __launch_bounds__(64 * kSumPh)
k_bwd_sum(const float *__restrict__ part, int rows, int m, const float *__restrict__ g, int64_t n,
          const double *__restrict__ gp, int np, float *out) {
    __shared__ double sh[kSumPh][64];
    if (blockIdx.x == 0) {
        double acc = 0.0;
        if (gp) {
            if ((int)threadIdx.x < np) acc = gp[threadIdx.x];
        } else {
            constexpr int kStep = 64 * kSumPh;
            int64_t i = threadIdx.x;
            for (; i + 7 * kStep < n; i += 8 * kStep) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = g[i + u * kStep];
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += v[u];
            }
            for (; i < n; i += kStep) acc += g[i];
        }
        acc = wide_sum(acc, sh[0]);
        if (threadIdx.x == 0) out[m] = (float)acc;
        return;
    }
    const int64_t j = (int64_t)(blockIdx.x - 1) * 64 + (threadIdx.x & 63);
    const double t = row_sum(part, rows, m, j, sh);
    if (threadIdx.x < 64 && j < m) out[j] = (float)t;
}

// g_eff[i] = g[i] * sigma'(s[i])
__global__ void __launch_bounds__(256)
k_chain_sigmoid(const float *__restrict__ g, const float *__restrict__ s, int64_t n, float *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float c, sp;
    sigmoid_and_slope(s[i], c, sp);
    out[i] = g[i] * sp;
}

// Adam (Kingma & Ba 2015, Algorithm 1); the first n_decay entries get l2 * p added to
// their gradient.  bc1 = 1/(1 - beta1^t), bc2 = 1/(1 - beta2^t).
__global__ void __launch_bounds__(256)
k_adam(float *p, const float *__restrict__ g, float *m, float *v, int64_t n, int64_t n_decay,
       float lr, float b1, float b2, float eps, float bc1, float bc2, float l2) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    float gk = g[k];
    if (k < n_decay) gk = fmaf(l2, p[k], gk);
    const float mk = b1 * m[k] + (1.0f - b1) * gk;
    const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    const float mh = mk * bc1, vh = vk * bc2;
    p[k] = p[k] - lr * mh / (sqrtf(vh) + eps);
}

// ---------------------------------------------------------------- fit step ---
//
// A step of the fit is four launches: the forward, k_bce, the weight gradient's partial
// rows and k_fit_update (nine, with the sums, the loss, the gradient's reduction and the
// update in kernels of their own).  At 10^4 points and hinges in the hundreds a step is
// launches more than work: 1.4x to 1.9x per fit there; 2^20 points and 16^3 hinges:
// 178 -> 150 us per step, the forward and the weight gradient (49 + 91 us) the rest.

// One optimiser step's coefficients; m == nullptr: gradient descent (lr on w, lr_b on the
// bias), else Adam (bc1 = 1/(1 - beta1^t), bc2 = 1/(1 - beta2^t)).
struct FitStep {
    float lr, lr_b, l2;
    float *m, *v;
    float b1, b2, eps, bc1, bc2;
};

// Gradient descent, w -= lr (g + l2 w) and beta -= lr_b g, or the update of k_adam, for
// entry j of [w (M), beta] from its gradient g.
__device__ __forceinline__ void fit_apply(float *w, int64_t j, bool bias, float g,
                                          const FitStep &o) {
    const float p = w[j];
    if (!o.m) {
        w[j] = bias ? p - o.lr_b * g : p - o.lr * fmaf(o.l2, p, g);
        return;
    }
    const float gk = bias ? g : fmaf(o.l2, p, g);
    const float mk = o.b1 * o.m[j] + (1.0f - o.b1) * gk;
    const float vk = o.b2 * o.v[j] + (1.0f - o.b2) * gk * gk;
    o.m[j] = mk;
    o.v[j] = vk;
    const float mh = mk * o.bc1, vh = vk * o.bc2;
    w[j] = p - o.lr * mh / (sqrtf(vh) + o.eps);
}

// Sums the partial rows of Phi^T g and updates the weights; the last block sums g for the
// bias, updates it, and writes the loss inv_n sum BCE + (l2/2) |w|^2 (|w|^2 from k_bce,
// before any update).
__global__ void __launch_bounds__(64 * kSumPh)
k_fit_update(const float *__restrict__ part, int rows, int M, float *w, FitStep o,
             const double *__restrict__ g_part, const double *__restrict__ bce_part, int nb,
             double inv_n, const double *__restrict__ wsq, float *__restrict__ loss) {
    __shared__ double sh[kSumPh][64];
    if (blockIdx.x == gridDim.x - 1) {
        static_assert(kRedMaxBlocks <= 64 * kSumPh, "a thread per partial sum");
        const bool in = (int)threadIdx.x < nb;
        const double g = wide_sum(in ? g_part[threadIdx.x] : 0.0, sh[0]);
        const double b = loss ? wide_sum(in ? bce_part[threadIdx.x] : 0.0, sh[1]) : 0.0;
        if (threadIdx.x != 0) return;
        fit_apply(w, M, true, (float)g, o);
        if (loss) *loss = (float)(inv_n * b + 0.5 * (double)o.l2 * *wsq);
        return;
    }
    const int64_t j = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const double t = row_sum(part, rows, M, j, sh);
    if (threadIdx.x < 64 && j < M) fit_apply(w, j, false, (float)t, o);
}

// ------------------------------------------------------------------ host ---

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Splits of the point set for Phi^T g: each range within one LDS tile, and enough block
// rows (256 or 512 hinges each) to fill the chip, as far as the workspace's rows go.
static int64_t range_tile(int dim) { return dim == 2 ? tile_chunks<2>() : tile_chunks<3>(); }
static int bwd_splits(int dim, int M, int64_t n, int64_t hinges_per_block) {
    const int64_t nch = (n + 3) / 4;
    const int64_t tile = range_tile(dim);
    int64_t s = (nch + tile - 1) / tile;
    const int64_t hb = (M + hinges_per_block - 1) / hinges_per_block;
    const int64_t want = (1024 + hb - 1) / hb;
    if (s < want) s = want;
    if (s > nch) s = nch;
    if (s < 1) s = 1;
    return (int)s;
}

// Hinges per block of the pairwise weight gradient, lanes being hinges.  Two per lane halve the
// LDS reads that bind it (3-D, 600,000 points, 1,500 hinges: 0.78 of the time with one), but
// pay from 1,500 hinges and 65,536 points on (1,000 hinges, 200,000 points: 1.23), where the
// last block of 512 idles for at most an eighth of the work, and where the launch fills its
// rounds of as many blocks as the LDS holds no worse (3-D, 6,000 hinges, 300,000 points: 1,032
// blocks on 512 slots against 1,776: 1.13).
static int wgrad_hinges_per_block(int dim, int64_t M, int64_t n) {
    const int64_t two = (M + 511) / 512 * 512, one = (M + 255) / 256 * 256;
    if (M < 1500 || n < 65536 || 8 * two > 9 * one) return 256;
    auto fill = [&](int64_t per) {
        const int64_t s = bwd_splits(dim, (int)M, n, per), blocks = (M + per - 1) / per * s;
        const int64_t lds = ((n + 3) / 4 + s - 1) / s * 16 * (dim + 1);
        const int64_t slots = 256 * std::min<int64_t>(8, (int64_t)160 * 1024 / lds);
        return (double)blocks / (double)((blocks + slots - 1) / slots * slots);
    };
    return fill(512) >= fill(256) ? 512 : 256;
}

// Partial rows of a workspace: for the pairwise splits and for the grid kernels.
static size_t bwd_rows(int dim, int M, int64_t n) {
    const size_t a = (size_t)bwd_splits(dim, M, n, 256), b = wgrad_rows_max(n);
    return a > b ? a : b;
}

size_t bwd_ws_bytes(int dim, int M, int64_t n) {
    return align256(bwd_rows(dim, M, n) * M * sizeof(float)) + align256((size_t)n * sizeof(float)) +
           align256(kRedMaxBlocks * sizeof(double));
}

// Phi^T g by the pairwise kernel with the roles exchanged: the data points are the
// weighted set and the hinges the lanes; S ranges of points give S partial rows.
static int32_t launch_pairwise_wgrad(int dim, const float *hinges, int M, float kappa,
                                     float gscale, const float *x, int64_t n, const float *gw,
                                     float *part, int S, int per, hipStream_t st) {
    RbfArgs a;
    a.hinges = x;
    a.weights = gw;
    a.M = (int)n;
    a.bias = nullptr;
    a.kappa = kappa;
    a.gscale = gscale;
    a.x_in = hinges;
    a.n = M;
    a.s_out = part;
    a.splits = S;
    return S > 1 ? launch_rbf_wgrad(dim, a, per, st) : launch_rbf(dim, kEval, a, st);
}

size_t bce_ws_bytes(int64_t) { return align256(kRedMaxBlocks * sizeof(double)); }

size_t fit_ws_bytes(int dim, int M, int64_t n) {
    return bwd_ws_bytes(dim, M, n) + 2 * align256((size_t)n * sizeof(float)) +
           align256((size_t)(M + 1) * sizeof(float)) + 2 * align256(kRedMaxBlocks * sizeof(double));
}

// Partial rows of Phi^T g into part (bwd_rows of them at most), S their number: on the grid
// kernels where the grid fits them, else pairwise.
static int32_t launch_wgrad_rows(int dim, const float *hinges, int M, const int *grid, float kappa,
                                 float gscale, const float *x, int64_t n, const float *gw,
                                 float *part, int &S, hipStream_t st) {
    const int32_t e = launch_grid_wgrad(dim, hinges, M, grid, kappa, x, n, gw, part, &S, st);
    if (e != PDMP_EUNSUPPORTED) return e;
    const int64_t most = (int64_t)bwd_rows(dim, M, n);
    const int per = wgrad_hinges_per_block(dim, M, n);
    S = bwd_splits(dim, M, n, per);
    if (S > most) S = (int)most;
    return launch_pairwise_wgrad(dim, hinges, M, kappa, gscale, x, n, gw, part, S, per, st);
}

// Up to this many points one block sums g beside the blocks that sum the rows (10^5: 7.1 us,
// in launches of their own 4.6 + 4.2 + 2.9 us and two more gaps); beyond, partial sums of a
// launch of their own first.
constexpr int64_t kBiasDirect = (int64_t)1 << 17;

// Backward of the logit: grad_w[0..M) = Phi^T g_eff, grad_w[M] = sum g_eff,
// grad_x = g (sigma'(s))? grad s.  `ws` holds partial rows, g_eff and reduce parts.
int32_t launch_logit_bwd(int dim, const float *hinges, const float *weights, int M,
                         const int *grid, float ell, const float *x, int64_t n, const float *g,
                         const float *s_fwd, float *grad_w, float *grad_x, void *ws,
                         hipStream_t st) {
    float kappa, gscale;
    derive_scales(ell, kappa, gscale);
    char *p = (char *)ws;
    float *part = (float *)p;
    p += align256(bwd_rows(dim, M, n) * M * sizeof(float));
    float *geff = (float *)p;
    p += align256((size_t)n * sizeof(float));
    double *rparts = (double *)p;

    const float *gw = g;
    if (s_fwd) {
        if (int32_t e = grid_guard((n + 255) / 256, 256, "k_chain_sigmoid")) return e;
        hipLaunchKernelGGL(k_chain_sigmoid, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g,
                           s_fwd, n, geff);
        if (int32_t e = check_launch("k_chain_sigmoid")) return e;
        gw = geff;
    }
    if (grad_w) {
        int S = 0;
        if (int32_t e = launch_wgrad_rows(dim, hinges, M, grid, kappa, gscale, x, n, gw, part, S, st))
            return e;
        const bool direct = n <= kBiasDirect;
        const int nb = direct ? 0 : red_blocks(n);
        if (!direct)
            hipLaunchKernelGGL(k_sum_partial, dim3(nb), dim3(kRedBlock), 0, st, gw, n, rparts);
        hipLaunchKernelGGL(k_bwd_sum, dim3((unsigned)((M + 63) / 64 + 1)), dim3(64 * kSumPh), 0, st,
                           part, S, M, gw, n, direct ? nullptr : rparts, nb, grad_w);
        if (int32_t e2 = check_launch("k_bwd_sum")) return e2;
    }
    if (grad_x) {
        RbfArgs a;
        a.hinges = hinges;
        a.weights = weights;
        a.M = M;
        a.bias = weights + M;
        a.kappa = kappa;
        a.gscale = gscale;
        a.x_in = x;
        a.n = n;
        a.g_out = grad_x;
        a.g_in = g;
        a.chain = s_fwd ? 1 : 0;
        if (int32_t e = launch_rbf(dim, kGradBwd, a, st)) return e;
    }
    return PDMP_OK;
}

int32_t launch_bce(const float *s, const uint8_t *y, int64_t n, const float *g_scale, float *loss,
                   float *g_out, double *parts, hipStream_t st) {
    const int nb = red_blocks(n);
    hipLaunchKernelGGL(k_bce, dim3(nb), dim3(kRedBlock), 0, st, s, y, n, (float)(1.0 / (double)n),
                       g_scale, nb, g_out, (double *)nullptr, loss ? parts : nullptr,
                       (const float *)nullptr, 0, (double *)nullptr);
    if (loss)
        hipLaunchKernelGGL(k_final, dim3(1), dim3(kRedBlock), 0, st, parts, nb, 1.0 / (double)n,
                           loss);
    return check_launch("k_bce");
}

int32_t launch_adam(float *p, const float *g, float *m, float *v, int64_t n, int64_t n_decay,
                    int t, float lr, float b1, float b2, float eps, float l2, hipStream_t st) {
    const double bc1 = 1.0 / (1.0 - std::pow((double)b1, (double)t));
    const double bc2 = 1.0 / (1.0 - std::pow((double)b2, (double)t));
    if (int32_t e = grid_guard((n + 255) / 256, 256, "k_adam")) return e;
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, g, m, v, n,
                       n_decay, lr, b1, b2, eps, (float)bc1, (float)bc2, l2);
    return check_launch("k_adam");
}

// One full-batch fit: `steps` iterations of forward, BCE, backward and update.
int32_t launch_fit(int dim, const float *hinges, int M, const int *grid, float ell, float *wb,
                   const float *pts, const uint8_t *y, int64_t n, const pdmp_fit_opts &o,
                   float *loss_out, void *ws, hipStream_t st) {
    float kappa, gscale;
    derive_scales(ell, kappa, gscale);
    char *p = (char *)ws;
    float *part = (float *)p;
    p += bwd_ws_bytes(dim, M, n);
    float *s = (float *)p;
    p += align256((size_t)n * sizeof(float));
    float *g = (float *)p;
    p += align256((size_t)n * sizeof(float));
    double *wsq = (double *)p;
    p += align256((size_t)(M + 1) * sizeof(float));
    double *bparts = (double *)p;
    p += align256(kRedMaxBlocks * sizeof(double));
    double *gparts = (double *)p;

    const int nb = red_blocks(n);
    for (int t = 0; t < o.steps; ++t) {
        RbfArgs a;
        a.hinges = hinges;
        a.weights = wb;
        a.M = M;
        a.bias = wb + M;
        a.kappa = kappa;
        a.gscale = gscale;
        a.x_in = pts;
        a.n = n;
        a.s_out = s;
        if (int32_t e = launch_occ_any(dim, kEval, a, grid, st)) return e;
        hipLaunchKernelGGL(k_bce, dim3(nb + (loss_out ? 1 : 0)), dim3(kRedBlock), 0, st, s, y, n,
                           (float)(1.0 / (double)n), (const float *)nullptr, nb, g, gparts,
                           loss_out ? bparts : nullptr, wb, M, loss_out ? wsq : nullptr);
        if (int32_t e = check_launch("k_bce")) return e;
        int S = 0;
        if (int32_t e = launch_wgrad_rows(dim, hinges, M, grid, kappa, gscale, pts, n, g, part, S, st))
            return e;
        FitStep f{o.lr, o.lr_bias, o.l2, nullptr, nullptr, o.beta1, o.beta2, o.eps, 0.0f, 0.0f};
        if (o.optimizer != 0) {
            f.m = o.adam_m;
            f.v = o.adam_v;
            f.bc1 = (float)(1.0 / (1.0 - std::pow((double)o.beta1, (double)(o.t0 + t + 1))));
            f.bc2 = (float)(1.0 / (1.0 - std::pow((double)o.beta2, (double)(o.t0 + t + 1))));
        }
        hipLaunchKernelGGL(k_fit_update, dim3((unsigned)((M + 63) / 64 + 1)), dim3(64 * kSumPh), 0,
                           st, part, S, M, wb, f, gparts, bparts, nb, 1.0 / (double)n, wsq,
                           loss_out ? loss_out + t : nullptr);
        if (int32_t e = check_launch("k_fit_update")) return e;
    }
    return PDMP_OK;
}

}  // namespace pdmp
