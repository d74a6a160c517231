// mlp.hip -- residual MLP of the amortised morph on BF16 MFMA with FP32 accumulation.
//
// q_hat = q + f(q),  f = W_L SiLU(... SiLU(W_1 q + b_1) ...) + b_L, trained by MSE
// against plain-morph targets.  Weights and activations are BF16, products are
// accumulated in FP32 (v_mfma_f32_32x32x16_bf16), biases, the residual and the
// optimiser state are FP32.
//
// The layers' products are
//   forward      Z[b][o]  = sum_i H[b][i] W[o][i]        (+ bias, SiLU)
//   data grad    dH[b][i] = sum_o dZ[b][o] W[o][i]        (x SiLU'(Z_prev))
//   weight grad  dW[o][i] = sum_b dZ[b][o] H[b][i]        (split over b, fixed-order sum)
// Hidden widths that are multiples of 32 up to 256 run the forward (k_mlp_fused) and the
// whole chain of data gradients (k_mlp_chain) as one kernel each, activations in registers;
// other widths run them layer by layer as tiled GEMMs (k_gemm: block tile 64 x 64, four
// waves each owning a 32 x 32 MFMA tile, K staged through LDS 32 at a time).  Both sum
// k in the same order, so a training step's activations and vectors are the same bits on
// either.  The weight gradients of all layers are one kernel (k_mlp_wgrad).  The network's
// BF16 input and output gradient are rows of 16.  The layered path keeps its activations and
// backward vectors sample-major [B][ld], ld the width rounded up to 8; the fused kernels
// keep theirs in the order their lanes hold them, in blocks of 32 samples, so that every
// store and load of a wave is one contiguous kilobyte:
//   Z  (FP32): block, 32-column tile t, quad v of it, lane, 4 columns 32t + 8v + 4(lane/32) ..
//   H, dZ (BF16): block, 16-column step s, lane, 8 columns 16s + 8(lane/32) ..
// with lane%32 the sample in the block.
#include "pdmp_common.h"

#include <algorithm>
#include <type_traits>

namespace pdmp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;

__host__ __device__ inline uint16_t f32_to_bf16(float f) {
    // round to nearest even; NaN stays NaN
    uint32_t u;
    __builtin_memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
    uint32_t u = (uint32_t)h << 16;
    float f;
    __builtin_memcpy(&f, &u, 4);
    return f;
}

__device__ __forceinline__ float silu_f(float z) {
    float c, sp;
    sigmoid_and_slope(z, c, sp);
    return z * c;
}

__device__ __forceinline__ float silu_grad_f(float z) {
    float c, sp;
    sigmoid_and_slope(z, c, sp);
    return c + z * sp;  // sigma (1 + z (1 - sigma))
}

// 16 bytes of the caller's memory, which is aligned to its elements only (activations and
// workspaces to 4 bytes, parameters to 2; still one access each).
template <class V, class E>
__device__ __forceinline__ V load16(const E *p) {
    V v;
    __builtin_memcpy(&v, p, 16);
    return v;
}
template <class V, class E>
__device__ __forceinline__ void store16(E *p, const V &v) {
    __builtin_memcpy(p, &v, 16);
}

enum GemmEpi { kEpiHidden = 1, kEpiOut = 2, kEpiDSilu = 3 };

struct GemmArgs {
    int M = 0, N = 0, K = 0;
    const uint16_t *A = nullptr;
    int64_t a_sm = 0, a_sk = 0;
    const uint16_t *B = nullptr;
    int64_t b_sn = 0, b_sk = 0;
    // epilogues
    const float *bias = nullptr; // kEpiHidden/kEpiOut: bias[n]
    float *zsave = nullptr;      // kEpiHidden: z[m*N + n] (nullable)
    uint16_t *hout = nullptr;    // kEpiHidden: bf16 silu(z)[m*ldh + n]; kEpiDSilu: bf16 out
    int64_t ldh = 0;
    const float *qin = nullptr;  // kEpiOut: residual input [N][ldq] (SoA)
    float *qout = nullptr;       // kEpiOut: q + f, [N][ldq]
    int64_t ldq = 0;
    const float *zprev = nullptr; // kEpiDSilu: z of the layer below, [m*N + n]
};

constexpr int kGT = 64;      // block tile (M and N)
constexpr int kGK = 32;      // K per LDS stage
constexpr int kGPad = 8;     // row padding (bf16) against bank conflicts
constexpr int kGRow = kGK + kGPad;

// Stage a 64 x 32 (rows x k) tile of X(row, k) = X[row*s_row + k*s_k] into T[row][k]
// (row stride kGRow).  A k-contiguous operand (k_vec) uses 16-byte loads, zeros past its
// rows and, with ke a multiple of 8, past its end; a row-contiguous one when the whole tile is
// in range; anything else goes element by element (a batch of one sample spent most of each
// round on that: forward of six layers of 1,024 units 150 -> 99 us, backward 263 -> 196).
__device__ __forceinline__ void stage_tile(const uint16_t *__restrict__ X, int64_t s_row,
                                           int64_t s_k, int rows, int r0, int k0, int ke,
                                           bool k_vec, bool r_vec, int lrow, int lseg, int kr,
                                           int rseg, uint16_t *T) {
    const bool full = r0 + kGT <= rows && k0 + kGK <= ke;
    if (k_vec && (k0 + kGK <= ke || (ke & 7) == 0)) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (r0 + lrow < rows && k0 + lseg < ke)
            v = *reinterpret_cast<const uint4 *>(X + (int64_t)(r0 + lrow) * s_row + k0 + lseg);
        *reinterpret_cast<uint4 *>(&T[lrow * kGRow + lseg]) = v;
        return;
    }
    if (full && r_vec) {
        const uint4 v = *reinterpret_cast<const uint4 *>(X + (int64_t)(k0 + kr) * s_k + r0 + rseg);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            T[(rseg + 2 * j) * kGRow + kr] = (uint16_t)(w[j] & 0xffffu);
            T[(rseg + 2 * j + 1) * kGRow + kr] = (uint16_t)(w[j] >> 16);
        }
        return;
    }
    const int r = r0 + lrow;
    uint16_t v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = k0 + lseg + j;
        v[j] = (k < ke && r < rows) ? X[(int64_t)r * s_row + (int64_t)k * s_k] : (uint16_t)0;
    }
    uint4 p;
    p.x = v[0] | ((uint32_t)v[1] << 16);
    p.y = v[2] | ((uint32_t)v[3] << 16);
    p.z = v[4] | ((uint32_t)v[5] << 16);
    p.w = v[6] | ((uint32_t)v[7] << 16);
    *reinterpret_cast<uint4 *>(&T[lrow * kGRow + lseg]) = p;
}

template <int EPI>
__global__ void __launch_bounds__(256) k_gemm(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) uint16_t As[kGT * kGRow];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[kGT * kGRow];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int m0 = blockIdx.x * kGT, n0 = blockIdx.y * kGT;

    floatx16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;

    const int lrow = tid >> 2;        // 0..63: tile row this thread stages
    const int lseg = (tid & 3) * 8;   // 8 consecutive k
    const int kr = tid >> 3;          // 0..31: k this thread stages (row-contiguous operands)
    const int rseg = (tid & 7) * 8;   // 8 consecutive rows
    // 16-byte loads when an operand is contiguous along k or along its rows
    const bool a_k = g.a_sk == 1 && (g.a_sm & 7) == 0 && ((uintptr_t)g.A & 15) == 0;
    const bool b_k = g.b_sk == 1 && (g.b_sn & 7) == 0 && ((uintptr_t)g.B & 15) == 0;
    const bool b_r = g.b_sn == 1 && (g.b_sk & 7) == 0 && ((uintptr_t)g.B & 15) == 0;
    for (int kt = 0; kt < g.K; kt += kGK) {
        int k0 = kt;  // opaque: the staging's addresses formed anew, not kept in 28 registers
        asm volatile("" : "+s"(k0));
        stage_tile(g.A, g.a_sm, g.a_sk, g.M, m0, k0, g.K, a_k, false, lrow, lseg, kr, rseg, As);
        stage_tile(g.B, g.b_sn, g.b_sk, g.N, n0, k0, g.K, b_k, b_r, lrow, lseg, kr, rseg, Bs);
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kGK; kk += 16) {
            const int ka = kk + 8 * (lane >> 5);
            const uint4 ra = *reinterpret_cast<const uint4 *>(&As[(wm * 32 + (lane & 31)) * kGRow + ka]);
            const uint4 rb = *reinterpret_cast<const uint4 *>(&Bs[(wn * 32 + (lane & 31)) * kGRow + ka]);
            bf16x8_t fa, fb;
            __builtin_memcpy(&fa, &ra, 16);
            __builtin_memcpy(&fb, &rb, 16);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc, 0, 0, 0);
        }
        __syncthreads();
    }

    const int n = n0 + wn * 32 + (lane & 31);
    // one product of the lane's row with each row length; the 16 rows are uniform steps from it
    // (65,536 x 7-288-7 forward 45.2 -> 44.2 us)
    const int mb = m0 + wm * 32 + 4 * (lane >> 5);
    const int64_t cb = (int64_t)mb * g.N + n, hb = (int64_t)mb * g.ldh + n;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = 8 * (v >> 2) + (v & 3), m = mb + r;
        if (m >= g.M || n >= g.N) continue;
        const float a = acc[v];
        const int64_t mn = cb + (int64_t)r * g.N;
        if (EPI == kEpiHidden) {
            const float z = a + g.bias[n];
            if (g.zsave) g.zsave[mn] = z;
            g.hout[hb + (int64_t)r * g.ldh] = f32_to_bf16(silu_f(z));
        } else if (EPI == kEpiOut) {
            const int64_t o = (int64_t)n * g.ldq + m;  // SoA [n_out][B], m = sample
            g.qout[o] = g.qin[o] + (a + g.bias[n]);
        } else {
            g.hout[hb + (int64_t)r * g.ldh] = f32_to_bf16(a * silu_grad_f(g.zprev[mn]));
        }
    }
}

template <int EPI>
static int32_t launch_gemm(const GemmArgs &g, hipStream_t st) {
    if (int32_t e = grid_guard(((int64_t)g.M + kGT - 1) / kGT, 256, "k_gemm")) return e;
    dim3 grid((g.M + kGT - 1) / kGT, (g.N + kGT - 1) / kGT);
    hipLaunchKernelGGL(k_gemm<EPI>, grid, dim3(256), 0, st, g);
    return check_launch("k_gemm");
}

// ---------------------------------------------------------- small kernels ---

constexpr int kIoLd = 16;  // row length of the BF16 input and output-gradient arrays

// q [n_in][B] FP32 (SoA) -> H0 [B][16] BF16, zero past n_in; a thread per half row
__global__ void k_q_to_bf16(const float *__restrict__ q, int n_in, int64_t B, uint16_t *h0) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int c = 8 * blockIdx.y;
    if (b >= B) return;
    uint16_t u[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
        u[i] = c + i < n_in ? f32_to_bf16(q[(int64_t)(c + i) * B + b]) : (uint16_t)0;
    store16(h0 + b * kIoLd + c, u);
}

// the same, rows of n_in; a thread per entry
__global__ void k_q_rows(const float *__restrict__ q, int n_in, int64_t B, uint16_t *h0) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= B * n_in) return;
    const int64_t b = t / n_in;
    h0[t] = f32_to_bf16(q[(t - b * n_in) * B + b]);
}

__global__ void k_f32_to_bf16(const float *__restrict__ x, int64_t n, uint16_t *y) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) y[t] = f32_to_bf16(x[t]);
}

// MSE: dF[b][k] = bf16(2 u_b (q_hat - t) / (n_out B)) (rows of 16, zero past n_out), per-block sums of
// u_b (q_hat - t)^2, with sample weight u_b = hard_w where hard[b] != 0, else 1 (hard
// NULL: the plain MSE).
__global__ void __launch_bounds__(256)
k_mse(const float *__restrict__ qhat, const float *__restrict__ tgt, int n_out, int64_t B,
      float scale, const uint8_t *__restrict__ hard, float hard_w, uint16_t *dF, double *parts) {
    __shared__ double sh[256];
    const int64_t total = B * kIoLd;
    const int64_t per = (total + gridDim.x - 1) / gridDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * per;
    const int64_t t1 = t0 + per < total ? t0 + per : total;
    double acc = 0.0;
    for (int64_t t = t0 + threadIdx.x; t < t1; t += 256) {
        const int64_t b = t / kIoLd;
        const int k = (int)(t - b * kIoLd);
        if (k >= n_out) {
            dF[t] = 0;
            continue;
        }
        const int64_t o = (int64_t)k * B + b;
        const float e = qhat[o] - tgt[o];
        const float u = (hard && hard[b]) ? hard_w : 1.0f;
        acc += (double)u * ((double)e * (double)e);
        dF[t] = f32_to_bf16(2.0f * scale * u * e);
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (unsigned off = 128; off >= 1; off >>= 1) {
        if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) parts[blockIdx.x] = sh[0];
}

// out[j] = sum_{s < S} part[s * MN + j], fixed order; the loads go out eight at a
// time (the adds keep the order), so the sum is not a chain of dependent loads.  With loss,
// one block past those of the entries writes it, scale sum parts[0..np) (a launch of its own
// was 3 us of a training step).
__global__ void __launch_bounds__(256)
k_sum_splits(const float *__restrict__ part, int S, int64_t MN, float *out,
             const double *__restrict__ parts, int np, double scale, float *loss) {
    if ((int64_t)blockIdx.x * 256 >= MN) {
        __shared__ double sh[256];
        double acc = 0.0;
        for (int i = threadIdx.x; i < np; i += 256) acc += parts[i];
        sh[threadIdx.x] = acc;
        __syncthreads();
        for (unsigned off = 128; off >= 1; off >>= 1) {
            if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss = (float)(sh[0] * scale);
        return;
    }
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= MN) return;
    double acc = 0.0;
    int s = 0;
    for (; s + 8 <= S; s += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(s + u) * MN + j];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; s < S; ++s) acc += part[(int64_t)s * MN + j];
    out[j] = (float)acc;
}

// ------------------------------------------------------------ fused forward ---
//
// The forward of the whole network in one kernel: a block of four waves
// takes 128 samples through every layer, each wave its own 32, with the activations
// in registers.  A layer is C = W H^T on v_mfma_f32_32x32x16_bf16 (A = W rows, B =
// the samples' activations, k = input feature), so a wave's output tiles leave lane
// l holding features o = 32t + 8(v/4) + 4(l/32) + v%4 of sample l%32.  The next
// layer takes them as its B operand where they lie: its k-step s reads slot
// (s, l/32, j) as feature pi(16s + 8(l/32) + j) = 16s + 8(j/4) + 4(l/32) + j%4, which
// is accumulator value v = 8(s%2) + j of tile s/2, and its A operand reads W's
// columns in the same permuted order -- a permutation of the contraction index, so
// the sum is the same.  Every layer's BF16 weights are staged per block in LDS (rows
// padded against bank conflicts; a hidden layer of more than 4 tiles in two passes of
// output tiles, so that two blocks share a CU and one stages while the other
// computes).  Numerics as the layered path: BF16 inputs
// and activations, FP32 accumulation, bias, SiLU and residual in FP32.
//
// The training forward (TRAIN) also stores each layer's Z (FP32) and H (BF16), and keeps the
// contraction index in its natural order, so that every Z is the layered path's bits: a
// lane's two quads of a 16-column block lie 8 columns apart, and one v_permlane32_swap
// per register exchanges them with the other half's into 8 consecutive columns (the operand
// and a 16-byte store).  HBM writes bound it: 302 MB at 65,536 x 256 x 3.  Samples past the
// batch repeat the last one and store into the arrays' padding (whole blocks of 128).
// At 65,536 x (7-256-256-256-7): 68 us; one GEMM per layer took 120 us.
constexpr int kMlpFB = 256;  // 4 waves, 128 samples; two blocks per CU

// Slot of column x (0..15) of a 16-column block in the A fragments: lane half h reads
// slots 8h .. 8h + 7, which must hold columns pi(8h + j) = 8(j/4) + 4h + j%4, so the
// block's quads (4 columns) sit in the order 0, 2, 1, 3.
__device__ __forceinline__ int mlp_slot(int x) { return ((x >> 2) & 1) * 8 + (x >> 3) * 4 + (x & 3); }

// Per-layer arrays of a training pass (h0: the BF16 input rows; h[l], z[l] of layer l).
constexpr int kMlpMaxHidden = 6;
struct MlpActs {
    uint16_t *h0;
    float *z[kMlpMaxHidden];
    uint16_t *h[kMlpMaxHidden];
};

// Two floats to BF16, nearest even, packed.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = {a, b};
    const bf2 h = __builtin_convertvector(v, bf2);
    return __builtin_bit_cast(uint32_t, h);
}

// The lane's packed quads of columns 4h .. (lo) and 8 + 4h .. (hi) of a 16-column block
// into its 8 consecutive columns 8h .. 8h + 7, h = lane/32.
__device__ __forceinline__ uint4 natural_order(uint2 lo, uint2 hi) {
    const auto x = __builtin_amdgcn_permlane32_swap(lo.x, hi.x, false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(lo.y, hi.y, false, false);
    return make_uint4(x[0], y[0], x[1], y[1]);
}

template <int TH, bool TRAIN>
__global__ void __launch_bounds__(kMlpFB) __attribute__((amdgpu_waves_per_eu(2)))
k_mlp_fused(const uint16_t *__restrict__ wbf, const float *__restrict__ par, int n_in, int L,
            const float *__restrict__ q, int64_t B, float *__restrict__ qhat, MlpActs acts) {
    constexpr int H = 32 * TH, KH = 2 * TH, LROW = H + 8;
    // hidden layers in passes of TP output tiles, so that two blocks fit in a CU's LDS
    constexpr int TP = TH > 4 ? (TH + 1) / 2 : TH;
    constexpr int WROWS = 32 * TP > 16 ? 32 * TP : 16;
    static_assert(WROWS * LROW >= 16 * H, "room for the first layer's weights");
    __shared__ __attribute__((aligned(16))) uint16_t Ws[WROWS * LROW];
    __shared__ __attribute__((aligned(16))) float bs[H];  // the layer's bias
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6, hh = lane >> 5, r = lane & 31;
    const int64_t n = (int64_t)blockIdx.x * (kMlpFB / 2) + wv * 32 + r;
    const bool live = n < B;
    // layout offsets (as the host's): layer 0 [H][n_in] + H, hidden [H][H] + H, last
    // [n_in][H] + n_in
    const int64_t w1 = (int64_t)H * n_in + H;
    auto woff = [&](int l) -> int64_t {
        return l == 0 ? 0 : w1 + (int64_t)(l - 1) * ((int64_t)H * H + H);
    };
    auto boff = [&](int l) -> int64_t {
        return woff(l) + (l == 0 ? (int64_t)H * n_in : (l == L - 1 ? (int64_t)n_in * H : (int64_t)H * H));
    };
    auto frag = [&](int row, int sk) {  // the A fragment of row, k-step sk, this lane's half
        bf16x8_t a;
        const uint4 w4 = *reinterpret_cast<const uint4 *>(&Ws[row * LROW + 16 * sk + 8 * hh]);
        __builtin_memcpy(&a, &w4, 16);
        return a;
    };
    // layer 0: W_0 [H][n_in] into rows of 16 (zero past n_in), k = column directly
    for (int e = tid; e < H * 16; e += kMlpFB) {
        const int row = e >> 4, c = e & 15;
        Ws[row * 16 + c] = c < n_in ? wbf[(int64_t)row * n_in + c] : (uint16_t)0;
    }
    for (int e = tid; e < H; e += kMlpFB) bs[e] = par[boff(0) + e];
    // its B operand: bf16(q[8hh + j][n]), zero past n_in
    bf16x8_t b0;
    {
        uint16_t u[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int f = 8 * hh + j;
            u[j] = f < n_in ? f32_to_bf16(q[(int64_t)f * B + (live ? n : B - 1)]) : (uint16_t)0;
        }
        __builtin_memcpy(&b0, u, 16);
        if (TRAIN) __builtin_memcpy(acts.h0 + n * kIoLd + 8 * hh, u, 16);
    }
    __syncthreads();
    floatx16_t acc[TH];
#pragma unroll
    for (int t = 0; t < TH; ++t) {
        bf16x8_t a;
        const uint4 w4 = *reinterpret_cast<const uint4 *>(&Ws[(32 * t + r) * 16 + 8 * hh]);
        __builtin_memcpy(&a, &w4, 16);
        floatx16_t z = {};
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b0, z, 0, 0, 0);
    }
    bf16x8_t hb[KH];
    // bias (from bs) + SiLU, into the next layer's B operands (slot j of k-step
    // 2t + v/8 = v%8); biases o .. o + 3 of a quad are one 16-byte LDS read
    auto epilogue = [&](int l) {
#pragma unroll
        for (int t = 0; t < TH; ++t)
#pragma unroll
            for (int u8 = 0; u8 < 2; ++u8) {
                uint2 quad[2];
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const int v0 = 8 * u8 + 4 * g, o = 32 * t + 8 * (v0 >> 2) + 4 * hh;
                    const float4 b4 = *reinterpret_cast<const float4 *>(&bs[o]);
                    const float4 z = make_float4(acc[t][v0] + b4.x, acc[t][v0 + 1] + b4.y,
                                                 acc[t][v0 + 2] + b4.z, acc[t][v0 + 3] + b4.w);
                    if (TRAIN)
                        store16(acts.z[l] + ((n >> 5) * TH + t) * 1024 + (v0 >> 2) * 256 + lane * 4,
                                z);
                    quad[g] = make_uint2(pack_bf16(silu_f(z.x), silu_f(z.y)),
                                         pack_bf16(silu_f(z.z), silu_f(z.w)));
                }
                uint4 w = make_uint4(quad[0].x, quad[0].y, quad[1].x, quad[1].y);
                if (TRAIN) {
                    w = natural_order(quad[0], quad[1]);
                    store16(acts.h[l] + ((n >> 5) * KH + 2 * t + u8) * 512 + lane * 8, w);
                }
                __builtin_memcpy(&hb[2 * t + u8], &w, 16);
            }
    };
    epilogue(0);
    // stage rows [0, rows) of a row-major [rows][H] weight matrix with each 16-column
    // block's quads in the order the activations come in (8-byte moves)
    auto stage = [&](const uint16_t *__restrict__ W, int rows, const float *__restrict__ bias) {
        __syncthreads();  // every wave is done with the previous contents
        if (bias)
            for (int e = tid; e < H; e += kMlpFB) bs[e] = bias[e];
        const int nq = rows * (H / 4);
#pragma unroll 8
        for (int e = tid; e < nq; e += kMlpFB) {
            const int row = e / (H / 4), q4 = e - row * (H / 4);
            const int col = 4 * q4;
            uint2 v;  // the parameters' alignment is the caller's
            __builtin_memcpy(&v, W + (int64_t)row * H + col, 8);
            const int slot = TRAIN ? (col & 15) : mlp_slot(col & 15);
            *reinterpret_cast<uint2 *>(&Ws[row * LROW + (col & ~15) + slot]) = v;
        }
        __syncthreads();
    };
    for (int l = 1; l < L - 1; ++l) {
#pragma unroll
        for (int t = 0; t < TH; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
#pragma unroll
        for (int t0 = 0; t0 < TH; t0 += TP) {
            const int nt = TH - t0 < TP ? TH - t0 : TP;
            stage(wbf + woff(l) + (int64_t)32 * t0 * H, 32 * nt, t0 == 0 ? par + boff(l) : nullptr);
#pragma unroll
            for (int sk = 0; sk < KH; ++sk)
#pragma unroll
                for (int t = t0; t < t0 + TP && t < TH; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        frag(32 * (t - t0) + r, sk), hb[sk], acc[t], 0, 0, 0);
        }
        epilogue(l);
    }
    // last layer: W_L [n_in][H] (rows past n_in read as zero)
    stage(wbf + woff(L - 1), n_in, nullptr);
    floatx16_t out = {};
    const bf16x8_t zero8 = {};
#pragma unroll
    for (int sk = 0; sk < KH; ++sk)
        out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r < n_in ? frag(r, sk) : zero8, hb[sk], out,
                                                      0, 0, 0);
    if (!live) return;
    const float *bL = par + boff(L - 1);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int f = 8 * (v >> 2) + 4 * hh + (v & 3);
        if (f < n_in) {
            const int64_t o = (int64_t)f * B + n;
            qhat[o] = q[o] + (out[v] + bL[f]);
        }
    }
}

// ------------------------------------------- transposed fragments from LDS ---
//
// An MFMA operand wants 8 consecutive k of one row per lane; an array whose rows run along
// the other index ([k][column], k outermost) gives them through ds_read_tr16_b64: of each 16
// lanes, lane i names 4 consecutive elements of row k = i/4, and receives element i of
// the 16 columns for k = 0..3.  The rows are 128 columns in eight groups of 16, group c
// of row k stored at place c ^ kTrSwz(k): the four rows (and two groups) of a 32-lane read
// and the eight rows of a 16-byte store down a column fall in different banks.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
constexpr int kTrRow = 128;  // elements

__device__ __forceinline__ int tr_swz(int k) { return 2 * (k & 3) + ((k >> 2) & 1); }
__device__ __forceinline__ int tr_at(int k, int c) {
    return k * kTrRow + (((c >> 4) ^ tr_swz(k)) << 4) + (c & 15);
}

// The lane's offsets of fragment columns c0 .. c0 + 31 (lane%32; c0 a multiple of 32), for
// rows 8(lane/32) + (0..3) and + (4..7); k0 further rows (a multiple of 16) on by tr_frag.
struct TrOff {
    int lo, hi;
};
__device__ __forceinline__ TrOff tr_off(int c0, int lane) {
    const int k = 8 * (lane >> 5) + ((lane & 15) >> 2);
    const int c = c0 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    return TrOff{tr_at(k, c), tr_at(k + 4, c)};
}
__device__ __forceinline__ bf16x8_t tr_frag(const uint16_t *T, int k0, TrOff o) {
    typedef __attribute__((address_space(3))) s16x4_t lds_t;
    const s16x4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t *)(T + k0 * kTrRow + o.lo));
    const s16x4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t *)(T + k0 * kTrRow + o.hi));
    bf16x8_t f;
    __builtin_memcpy(&f, &a, 8);
    __builtin_memcpy(reinterpret_cast<char *>(&f) + 8, &b, 8);
    return f;
}

// -------------------------------------------------- chain of data gradients ---
//
// dZ_{l-1}[b][i] = (sum_o dZ_l[b][o] W_l[o][i]) SiLU'(Z_{l-1}[b][i]) for l = hi .. lo (L-1 .. 1,
// or a layer at a time, where dz[hi] may be dz[hi - 1]: a wave's vectors are read before
// they are written) in one kernel, from dF (the output's gradient, rows of 16, zero past n_in).  Blocks and
// accumulator layout as k_mlp_fused (C = W^T dZ^T, a wave its own 32 samples), the
// contraction in natural order as its training form; W_l is staged row-major in passes of
// TP column tiles and read transposed.  The vectors go from layer to layer in registers;
// each is stored once for the weight gradients.  HBM bound: Z read, dZ written (302 MB at
// 65,536 x 256 x 3), where one GEMM per layer also read every dZ back: 64 us against 160 us.
struct MlpChain {
    const float *z[kMlpMaxHidden];
    uint16_t *dz[kMlpMaxHidden];
};

template <int TH>
__global__ void __launch_bounds__(kMlpFB) __attribute__((amdgpu_waves_per_eu(2)))
k_mlp_chain(const uint16_t *__restrict__ wbf, int n_in, int L, const uint16_t *dF, int64_t B,
            MlpChain ch, int hi, int lo) {
    constexpr int H = 32 * TH, KH = 2 * TH;
    constexpr int TP = TH > 4 ? (TH + 1) / 2 : TH, CW = 32 * TP;
    static_assert(CW <= kTrRow, "a pass fits a staged row");
    __shared__ __attribute__((aligned(16))) uint16_t Ws[H * kTrRow];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6, hh = lane >> 5, r = lane & 31;
    const int64_t n = (int64_t)blockIdx.x * (kMlpFB / 2) + wv * 32 + r;
    const int64_t nc = n < B ? n : B - 1;
    bf16x8_t dz[KH], nd[KH];
    if (hi == L - 1) {
        dz[0] = load16<bf16x8_t>(dF + nc * kIoLd + 8 * hh);
    } else {
#pragma unroll
        for (int s = 0; s < KH; ++s)
            dz[s] = load16<bf16x8_t>(ch.dz[hi] + ((n >> 5) * KH + s) * 512 + lane * 8);
    }
    const int64_t w1 = (int64_t)H * n_in + H;
    // stage rows [0, rows) of columns [0, 8 c8) of W, every load of a batch in flight
    auto stage = [&](const uint16_t *__restrict__ W, int rows, auto c8) {
        constexpr int per = decltype(c8)::value;
#pragma unroll 8
        for (int e = tid; e < rows * per; e += kMlpFB) {
            const int row = e / per, c = 8 * (e - row * per);
            uint4 v;  // the parameters' alignment is the caller's
            __builtin_memcpy(&v, W + (int64_t)row * H + c, 16);
            *reinterpret_cast<uint4 *>(&Ws[tr_at(row, c)]) = v;
        }
    };
    TrOff off[TP];
#pragma unroll
    for (int t = 0; t < TP; ++t) off[t] = tr_off(32 * t, lane);
#pragma unroll 1
    for (int l = hi; l >= lo; --l) {
        const bool last = l == L - 1;
        const uint16_t *W = wbf + w1 + (int64_t)(l - 1) * ((int64_t)H * H + H);
        const float *zl = ch.z[l - 1] + (n >> 5) * TH * 1024 + lane * 4;
        uint16_t *dl = ch.dz[l - 1] + (n >> 5) * KH * 512 + lane * 8;
#pragma unroll
        for (int t0 = 0; t0 < TH; t0 += TP) {
            constexpr int kTail = TH % TP == 0 ? TP : TH % TP;
            const bool tail = t0 + TP >= TH;  // the last pass may hold fewer tiles
            __syncthreads();  // every wave is done with the previous contents
            if (last) {
                for (int e = tid; e < (16 - n_in) * (CW / 8); e += kMlpFB)
                    *reinterpret_cast<uint4 *>(&Ws[tr_at(n_in + e / (CW / 8), 8 * (e % (CW / 8)))]) =
                        make_uint4(0, 0, 0, 0);
            }
            if (tail) stage(W + 32 * t0, last ? n_in : H, std::integral_constant<int, 4 * kTail>());
            else stage(W + 32 * t0, last ? n_in : H, std::integral_constant<int, 4 * TP>());
            __syncthreads();
            floatx16_t acc[TP];
#pragma unroll
            for (int t = 0; t < TP; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
            float4 z[4], zn[4];  // the tile's and the next tile's Z
            auto load_z = [&](float4(&d)[4], int t) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    d[v] = load16<float4>(zl + t * 1024 + v * 256);
            };
            load_z(zn, t0);
            if (last) {
#pragma unroll
                for (int t = 0; t < TP && t0 + t < TH; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        tr_frag(Ws, 0, off[t]), dz[0], acc[t], 0, 0, 0);
            } else {
#pragma unroll
                for (int sk = 0; sk < KH; ++sk)
#pragma unroll
                    for (int t = 0; t < TP && t0 + t < TH; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            tr_frag(Ws, 16 * sk, off[t]), dz[sk], acc[t], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < TP && t0 + t < TH; ++t) {
#pragma unroll
                for (int v = 0; v < 4; ++v) z[v] = zn[v];
                if (t + 1 < TP && t0 + t + 1 < TH) load_z(zn, t0 + t + 1);
#pragma unroll
                for (int u8 = 0; u8 < 2; ++u8) {
                    uint2 quad[2];
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
                        const int v0 = 8 * u8 + 4 * g;
                        const float4 zz = z[2 * u8 + g];
                        quad[g] = make_uint2(pack_bf16(acc[t][v0] * silu_grad_f(zz.x),
                                                       acc[t][v0 + 1] * silu_grad_f(zz.y)),
                                             pack_bf16(acc[t][v0 + 2] * silu_grad_f(zz.z),
                                                       acc[t][v0 + 3] * silu_grad_f(zz.w)));
                    }
                    const uint4 w = natural_order(quad[0], quad[1]);
                    store16(dl + (2 * (t0 + t) + u8) * 512, w);
                    __builtin_memcpy(&nd[2 * (t0 + t) + u8], &w, 16);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < KH; ++i) dz[i] = nd[i];
    }
}

// --------------------------------------------------------- weight gradients ---
//
// dW_l[o][i] = sum_b dZ_l[b][o] H_{l-1}[b][i] and db_l[o] = sum_b dZ_l[b][o] of every layer in
// one launch over the layers' 128 x 128 output tiles and the ranges of `per` samples, each of
// which writes one row of partials in the parameters' own layout (k_sum_splits adds the
// rows).  Blocks go to the eight XCDs in turn, so block b takes a range congruent to b mod 8
// and all tiles of a range follow each other on one XCD: the tiles that share columns of dZ
// or H find them in its L2.  Both operands have the contraction index outermost: 64
// samples x 128 columns of each are staged row-major (16-byte moves, the next two rounds'
// loads in flight during a round's products, two buffers) and read transposed.  Four waves own
// 64 x 64 outputs each.  The bias sums come from the dZ rows as they are staged (FP32 over
// a thread's two rows of a round, FP64 across rounds and threads, fixed order).
// At 65,536 x (7-256-256-256-7): 67 us, 205 MB read and 22 MB written (46 us at the rate of a
// plain copy); one GEMM per layer with 2-byte transposing stores, the row sums and the column
// sums took 370 us.  A round's LDS traffic and barrier bind it, not HBM.
constexpr int kWgSamples = 256, kWgSlots = 512;  // samples per partial row; blocks at once
constexpr int kWgT = 128, kWgK = 64;
static_assert(kWgT == kTrRow, "a staged row is the tile");

struct MlpWgLayer {
    const uint16_t *dz, *h;
    int ldz, ldh, O, I;      // ldz, ldh: row lengths
    int zblk, hblk;          // 1: in the fused kernels' blocks, 0: sample-major
    int64_t woff, boff;
    int tile0, tiles_i;  // first tile of the layer; tiles along i
};
struct MlpWg {
    MlpWgLayer layer[kMlpMaxHidden + 1];
    int L, tiles;
};

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_mlp_wgrad(MlpWg g, int64_t B, int64_t per, int64_t np, float *__restrict__ part) {
    __shared__ __attribute__((aligned(16))) uint16_t S[2][2][kWgK * kTrRow];  // [buffer][dz, h]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t range = (int64_t)(blockIdx.x >> 3) / g.tiles * 8 + (blockIdx.x & 7);
    const int gt = (blockIdx.x >> 3) % g.tiles;
    const int64_t b0 = range * per, b1 = min(B, b0 + per);
    if (b0 >= B) return;  // the ranges are padded to a multiple of eight
    int l = 0;
    while (l + 1 < g.L && gt >= g.layer[l + 1].tile0) ++l;
    const MlpWgLayer &y = g.layer[l];
    const int tile = gt - y.tile0;
    const int o0 = tile / y.tiles_i * kWgT, i0 = tile % y.tiles_i * kWgT;
    const bool bias = i0 == 0;

    // a thread stages 8 columns at cc, cc + 64 of rows rr, rr + 32; columns past a row's end
    // and rows past the range are stored as zero (a select at the loads would wait for them)
    const int rr = tid & 31, cc = 8 * (tid >> 5);
    const int ldz = y.ldz, ldh = y.ldh, O = y.O, I = y.I;
    const bool zb = y.zblk != 0, hb = y.hblk != 0;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 vz[2][4], vh[2][4];  // two rounds in flight: [round parity][2 (row step) + column step]
    // element offsets of a thread's loads: 64 samples, 32 samples, 64 columns on
    const int64_t sz = 64 * ldz, sh = 64 * ldh, rz = sz / 2, rh = sh / 2;
    const int cz = o0 + cc + 64 < ldz ? (zb ? 4 * 512 : 64) : 0;
    const int ch = i0 + cc + 64 < ldh ? (hb ? 4 * 512 : 64) : 0;
    auto base = [&](bool blk, int ld, int c0) -> int64_t {
        const int64_t row = b0 + rr;
        const int c = c0 + cc < ld ? c0 + cc : 0;
        return blk ? ((row >> 5) * (ld >> 4) + (c >> 4)) * 512 + ((c >> 3) & 1) * 256 + (row & 31) * 8
                   : row * ld + c;
    };
    const uint16_t *pz = y.dz + base(zb, ldz, o0), *ph = y.h + base(hb, ldh, i0);
    auto load = [&](u32x4(&z)[4], u32x4(&h)[4]) {  // whole rounds lie inside the arrays
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            z[u] = load16<u32x4>(pz + (u >> 1) * rz + (u & 1) * cz);
            h[u] = load16<u32x4>(ph + (u >> 1) * rh + (u & 1) * ch);
        }
        pz += sz;
        ph += sh;
    };
    double db[2][8];  // bias sums of the two column steps
#pragma unroll
    for (int j = 0; j < 8; ++j) db[0][j] = db[1][j] = 0.0;

    const int wu = __builtin_amdgcn_readfirstlane(wave);
    const int wo = 64 * (wu & 1), wi = 64 * (wu >> 1);
    floatx16_t acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][c][v] = 0.0f;
    const bool work = o0 + wo < O && i0 + wi < I;  // the wave's part holds outputs
    const TrOff oz[2] = {tr_off(wo, lane), tr_off(wo + 32, lane)};
    const TrOff oh[2] = {tr_off(wi, lane), tr_off(wi + 32, lane)};
    // one round of 64 samples from b: store, request the round after next, multiply
    auto round = [&](int64_t b, u32x4(&z)[4], u32x4(&h)[4], uint16_t *SZ, uint16_t *SH) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = b + rr + 32 * (u >> 1) < b1;
            const int c = cc + 64 * (u & 1), at_lds = tr_at(rr + 32 * (u >> 1), c);
            z[u] &= in && o0 + c < ldz ? 0xffffffffu : 0u;
            h[u] &= in && i0 + c < ldh ? 0xffffffffu : 0u;
            *reinterpret_cast<u32x4 *>(&SZ[at_lds]) = z[u];
            *reinterpret_cast<u32x4 *>(&SH[at_lds]) = h[u];
        }
        if (bias) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t a = z[q][j >> 1], c = z[2 + q][j >> 1];
                    const float fa = __uint_as_float(j & 1 ? a & 0xffff0000u : a << 16);
                    const float fc = __uint_as_float(j & 1 ? c & 0xffff0000u : c << 16);
                    db[q][j] += fa + fc;
                }
        }
        __syncthreads();
        if (b + 2 * kWgK < b1) load(z, h);
        if (work) {
#pragma unroll
            for (int k = 0; k < kWgK; k += 16) {
                const bf16x8_t z0 = tr_frag(SZ, k, oz[0]), z1 = tr_frag(SZ, k, oz[1]);
                const bf16x8_t h0 = tr_frag(SH, k, oh[0]), h1 = tr_frag(SH, k, oh[1]);
                acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(z0, h0, acc[0][0], 0, 0, 0);
                acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(z1, h0, acc[1][0], 0, 0, 0);
                acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(z0, h1, acc[0][1], 0, 0, 0);
                acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(z1, h1, acc[1][1], 0, 0, 0);
            }
        }
    };
    load(vz[0], vh[0]);
    if (b0 + kWgK < b1) load(vz[1], vh[1]);
    for (int64_t b = b0; b < b1; b += 2 * kWgK) {
        round(b, vz[0], vh[0], S[0][0], S[0][1]);
        if (b + kWgK < b1) round(b + kWgK, vz[1], vh[1], S[1][0], S[1][1]);
    }
    float *out = part + range * np;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int i = i0 + wi + 32 * c + (lane & 31);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int o = o0 + wo + 32 * a + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (o < O && i < I) out[y.woff + (int64_t)o * I + i] = acc[a][c][v];
            }
        }
    if (!bias) return;
    __syncthreads();
    double *red = reinterpret_cast<double *>(&S[0][0][0]);  // [32 rows][128 columns]
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < 8; ++j) red[rr * kWgT + cc + 64 * q + j] = db[q][j];
    __syncthreads();
    if (tid < kWgT && o0 + tid < O) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < 32; ++q) t += red[q * kWgT + tid];
        out[y.boff + o0 + tid] = (float)t;
    }
}

// ------------------------------------------------------------------ host ---

static size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

struct MlpLayout {
    int L, n_in, H;
    int in(int l) const { return l == 0 ? n_in : H; }
    int out(int l) const { return l == L - 1 ? n_in : H; }
    int64_t woff(int l) const {
        int64_t o = 0;
        for (int k = 0; k < l; ++k) o += (int64_t)out(k) * in(k) + out(k);
        return o;
    }
    int64_t boff(int l) const { return woff(l) + (int64_t)out(l) * in(l); }
    int64_t nparams() const { return woff(L); }
};

static MlpLayout layout_of(const pdmp_mlp &m) { return MlpLayout{m.n_hidden + 1, m.n_in, m.hidden}; }

int64_t mlp_nparams(const pdmp_mlp &m) { return layout_of(m).nparams(); }

// Row length of the BF16 activations and backward vectors of a hidden layer.
static int mlp_ld(int H) { return (H + 7) & ~7; }

// Shapes the fused kernels take (by the shape alone: a training forward and its backward
// must agree on the activations' layout).
static bool mlp_fused_shape(const pdmp_mlp &m) { return m.hidden % 32 == 0 && m.hidden <= 256; }

// Rows of a batch's arrays: whole blocks of the fused kernels.
static int64_t mlp_rows(int64_t B) { return (B + 127) / 128 * 128; }

// Activations kept by a training forward: H0 bf16 [rows][16]; for l < L-1:
// Z_l f32 [rows][H] and H_l bf16 [rows][ld] (layouts above).
size_t mlp_acts_bytes(const pdmp_mlp &m, int64_t B) {
    const MlpLayout ly = layout_of(m);
    B = mlp_rows(B);
    size_t b = al256((size_t)B * kIoLd * 2);
    for (int l = 0; l < ly.L - 1; ++l)
        b += al256((size_t)B * ly.H * 4) + al256((size_t)B * mlp_ld(ly.H) * 2);
    return b;
}

static MlpActs act_ptrs(const MlpLayout &ly, void *acts, int64_t B) {
    B = mlp_rows(B);
    MlpActs p{};
    char *c = (char *)acts;
    p.h0 = (uint16_t *)c;
    c += al256((size_t)B * kIoLd * 2);
    for (int l = 0; l < ly.L - 1; ++l) {
        p.z[l] = (float *)c;
        c += al256((size_t)B * ly.H * 4);
        p.h[l] = (uint16_t *)c;
        c += al256((size_t)B * mlp_ld(ly.H) * 2);
    }
    return p;
}

// Inference-only forward keeps the BF16 input and two BF16 activation buffers in rows of mlp_ld,
// whose operands are 16-byte loads; in a smaller workspace rows of H.
static size_t mlp_fwd_ws(const pdmp_mlp &m, int64_t B, int ld) {
    return al256((size_t)B * m.n_in * 2) + 2 * al256((size_t)B * ld * 2);
}
size_t mlp_fwd_ws_bytes(const pdmp_mlp &m, int64_t B) { return mlp_fwd_ws(m, B, mlp_ld(m.hidden)); }
size_t mlp_fwd_ws_least(const pdmp_mlp &m, int64_t B) { return mlp_fwd_ws(m, B, m.hidden); }

template <bool TRAIN>
static int32_t launch_mlp_fused(const pdmp_mlp &m, int L, const float *q, int64_t B, float *qhat,
                                const MlpActs &a, hipStream_t st) {
    const int64_t blocks = (B + kMlpFB / 2 - 1) / (kMlpFB / 2);
    if (int32_t e = grid_guard(blocks, kMlpFB, "k_mlp_fused")) return e;
    switch (m.hidden / 32) {
#define PDMP_FUSED(TH)                                                                           \
    case TH:                                                                                     \
        hipLaunchKernelGGL((k_mlp_fused<TH, TRAIN>), dim3((unsigned)blocks), dim3(kMlpFB), 0, st, \
                           m.params_bf16, m.params, m.n_in, L, q, B, qhat, a);                   \
        break;
        PDMP_FUSED(1) PDMP_FUSED(2) PDMP_FUSED(3) PDMP_FUSED(4)
        PDMP_FUSED(5) PDMP_FUSED(6) PDMP_FUSED(7) PDMP_FUSED(8)
#undef PDMP_FUSED
    }
    return check_launch("k_mlp_fused");
}

int32_t launch_mlp_forward(const pdmp_mlp &m, const float *q, int64_t B, float *qhat, void *acts,
                           void *ws, size_t ws_bytes, hipStream_t st) {
    const MlpLayout ly = layout_of(m);
    if (mlp_fused_shape(m) && (acts || ((uintptr_t)m.params_bf16 & 15) == 0)) {
        if (!acts) return launch_mlp_fused<false>(m, ly.L, q, B, qhat, MlpActs{}, st);
        return launch_mlp_fused<true>(m, ly.L, q, B, qhat, act_ptrs(ly, acts, B), st);
    }
    const int ld = acts || ws_bytes >= mlp_fwd_ws_bytes(m, B) ? mlp_ld(ly.H) : ly.H;
    const int ld0 = acts ? kIoLd : ly.n_in;
    MlpActs p{};
    if (acts) {
        p = act_ptrs(ly, acts, B);
        if (int32_t e = grid_guard((B + 255) / 256, 256, "k_q_to_bf16")) return e;
        hipLaunchKernelGGL(k_q_to_bf16, dim3((unsigned)((B + 255) / 256), kIoLd / 8), dim3(256), 0, st,
                           q, ly.n_in, B, p.h0);
        if (int32_t e = check_launch("k_q_to_bf16")) return e;
    } else {
        char *c = (char *)ws;
        p.h0 = (uint16_t *)c;
        c += al256((size_t)B * ld0 * 2);
        for (int l = 0; l < ly.L - 1; ++l)
            p.h[l] = (uint16_t *)(c + (l & 1) * al256((size_t)B * ld * 2));
        const int64_t blocks = (B * ly.n_in + 255) / 256;
        if (int32_t e = grid_guard(blocks, 256, "k_q_rows")) return e;
        hipLaunchKernelGGL(k_q_rows, dim3((unsigned)blocks), dim3(256), 0, st, q, ly.n_in, B, p.h0);
        if (int32_t e = check_launch("k_q_rows")) return e;
    }
    for (int l = 0; l < ly.L; ++l) {
        GemmArgs g;
        g.M = (int)B;
        g.N = ly.out(l);
        g.K = ly.in(l);
        g.A = l == 0 ? p.h0 : p.h[l - 1];
        g.a_sm = l == 0 ? ld0 : ld;
        g.a_sk = 1;
        g.B = m.params_bf16 + ly.woff(l);
        g.b_sn = ly.in(l);
        g.b_sk = 1;
        g.bias = m.params + ly.boff(l);
        int32_t e;
        if (l < ly.L - 1) {
            g.zsave = p.z[l];
            g.hout = p.h[l];
            g.ldh = ld;
            e = launch_gemm<kEpiHidden>(g, st);
        } else {
            g.qin = q;
            g.qout = qhat;
            g.ldq = B;
            e = launch_gemm<kEpiOut>(g, st);
        }
        if (e) return e;
    }
    return PDMP_OK;
}

// ---- backward: sizes ----
//
// With the whole workspace all layers' vectors are kept and all weight gradients are one
// launch.  In a smaller one the vectors of one layer are kept at a time, in rows of H where the
// kernels' layouts leave it open, and each layer's weight gradient is a launch of its own:
// 65,536 x 7-256-256-256-7 in 76 MB instead of 125.

// Ranges of samples of a weight gradient of `tiles` output tiles: each writes a row of partial
// sums.  At least 256 samples (four rounds) each, and no more ranges (in eights, one per XCD) than
// fill the 512 block slots once -- but ranges of 2,048 samples and more as far as 64 go, whatever
// the tiles: one FP32 accumulator sums a range.
static int64_t wgrad_ranges(int tiles, int64_t B) {
    int64_t most = kWgSlots / tiles / 8 * 8;
    most = most < 8 ? 8 : (most > 64 ? 64 : most);
    const int64_t least = std::min<int64_t>(std::max<int64_t>(B / 2048, 1), 64);
    return std::max(std::min((B + kWgSamples - 1) / kWgSamples, most), least);
}
// Samples per range (whole rounds), and the rows that there are then (wgrad_ranges at most).
static int64_t wgrad_per(int64_t ranges, int64_t B) {
    return ((B + ranges - 1) / ranges + kWgK - 1) / kWgK * kWgK;
}
static int64_t wgrad_rows(int64_t ranges, int64_t B) {
    const int64_t per = wgrad_per(ranges, B);
    return (B + per - 1) / per;
}
static int layer_tiles(const MlpLayout &ly, int l) {
    return (ly.out(l) + kWgT - 1) / kWgT * ((ly.in(l) + kWgT - 1) / kWgT);
}
static int wgrad_tiles(const MlpLayout &ly) {
    int t = 0;
    for (int l = 0; l < ly.L; ++l) t += layer_tiles(ly, l);
    return t;
}

// A backward's workspace: dF, the layers' vectors, partial rows, partial losses.
struct MlpBwd {
    bool layered;         // a layer at a time
    bool one;             // its vectors in one buffer (fused kernels), else two in turn
    int64_t rows;         // rows of dF and of a buffer
    int ld, bufs;         // row length and number of the vectors' buffers
    bool dF_in_buf;       // dF lies in the second buffer
    int64_t ranges, part; // partial rows and entries of one (no rows: the gradient itself)
    int nb;               // blocks of the loss
    size_t bytes;
};

static MlpBwd mlp_bwd_plan(const pdmp_mlp &m, int64_t B, bool layered) {
    const MlpLayout ly = layout_of(m);
    const bool fused = mlp_fused_shape(m);
    MlpBwd p{};
    p.layered = layered;
    p.ld = fused || !layered ? mlp_ld(ly.H) : ly.H;
    p.one = layered && fused;
    p.bufs = !layered ? ly.L - 1 : fused ? 1 : 2;
    p.dF_in_buf = layered && !fused && p.ld >= kIoLd;
    p.ranges = layered ? std::min<int64_t>(std::max<int64_t>(B / 2048, 1), 64)
                       : wgrad_ranges(wgrad_tiles(ly), B);
    // a weight gradient reads whole rounds of rows and eights of columns (and drops what lies past
    // the batch and the row): past the vectors, where those are rows of the batch alone, into what
    // follows them
    p.rows = fused || !layered ? mlp_rows(B) : (p.ranges > 1 ? B : (B + kWgK - 1) / kWgK * kWgK);
    p.part = ly.nparams();
    if (layered) {
        p.part = 0;
        for (int l = 0; l < ly.L && p.ranges > 1; ++l)
            p.part = std::max(p.part, (int64_t)ly.out(l) * ly.in(l) + ly.out(l));
    }
    p.nb = layered ? (int)std::min<int64_t>(256, (B * kIoLd + 255) / 256) : 1024;
    p.bytes = (p.dF_in_buf ? 0 : al256((size_t)p.rows * kIoLd * 2)) +
              p.bufs * al256((size_t)p.rows * p.ld * 2) +
              std::max(al256((size_t)p.ranges * p.part * 4) + al256(p.nb * sizeof(double)),
                       p.rows == B ? al256((size_t)kWgK * p.ld * 2 + 16) : 0);
    return p;
}

size_t mlp_bwd_ws_bytes(const pdmp_mlp &m, int64_t B) { return mlp_bwd_plan(m, B, false).bytes; }
size_t mlp_bwd_ws_least(const pdmp_mlp &m, int64_t B) {
    return std::min(mlp_bwd_plan(m, B, true).bytes, mlp_bwd_ws_bytes(m, B));
}

static int32_t launch_mlp_chain(const pdmp_mlp &m, const MlpLayout &ly, const uint16_t *dF, int64_t B,
                                const MlpChain &ch, int hi, int lo, hipStream_t st) {
    const int64_t blocks = (B + kMlpFB / 2 - 1) / (kMlpFB / 2);
    if (int32_t e = grid_guard(blocks, kMlpFB, "k_mlp_chain")) return e;
    switch (ly.H / 32) {
#define PDMP_CHAIN(TH)                                                                        \
    case TH:                                                                                  \
        hipLaunchKernelGGL(k_mlp_chain<TH>, dim3((unsigned)blocks), dim3(kMlpFB), 0, st,      \
                           m.params_bf16, ly.n_in, ly.L, dF, B, ch, hi, lo);                  \
        break;
        PDMP_CHAIN(1) PDMP_CHAIN(2) PDMP_CHAIN(3) PDMP_CHAIN(4)
        PDMP_CHAIN(5) PDMP_CHAIN(6) PDMP_CHAIN(7) PDMP_CHAIN(8)
#undef PDMP_CHAIN
    }
    return check_launch("k_mlp_chain");
}

// Backward of the MSE loss through the whole network from saved activations.
// grad: FP32 [nparams] in the flat layout; loss (nullable): device [1].
int32_t launch_mlp_backward(const pdmp_mlp &m, const float *qhat, const float *target, int64_t B,
                            void *acts, float *grad, float *loss, void *ws, size_t ws_bytes,
                            hipStream_t st, const uint8_t *hard, float hard_w) {
    const MlpLayout ly = layout_of(m);
    const MlpActs ap = act_ptrs(ly, acts, B);
    const bool fused = mlp_fused_shape(m);
    const MlpBwd pl = mlp_bwd_plan(m, B, ws_bytes < mlp_bwd_ws_bytes(m, B));
    char *c = (char *)ws;
    uint16_t *dF = (uint16_t *)c;
    if (!pl.dF_in_buf) c += al256((size_t)pl.rows * kIoLd * 2);
    const size_t buf = al256((size_t)pl.rows * pl.ld * 2);
    MlpChain ch{};
    for (int l = 0; l < ly.L - 1; ++l) {
        ch.z[l] = ap.z[l];
        // layer by layer in two buffers: the last hidden layer's vectors in the first, dF, which
        // they are formed from, in the second
        ch.dz[l] = (uint16_t *)(c + (!pl.layered ? l : pl.one ? 0 : (ly.L - l) & 1) * buf);
    }
    if (pl.dF_in_buf) dF = (uint16_t *)(c + buf);
    c += pl.bufs * buf;
    float *part = (float *)c;
    c += al256((size_t)pl.ranges * pl.part * 4);
    double *rparts = (double *)c;
    const double scale = 1.0 / ((double)ly.n_in * (double)B);

    hipLaunchKernelGGL(k_mse, dim3(pl.nb), dim3(256), 0, st, qhat, target, ly.n_in, B, (float)scale,
                       hard, hard_w, dF, rparts);
    if (int32_t e = check_launch("k_mse")) return e;

    // dZ_{l-1}[b][i] = (sum_o dZ[b][o] W_l[o][i]) * SiLU'(Z_{l-1}[b][i]) for l = hi .. lo
    auto data_grad = [&](int hi, int lo) -> int32_t {
        if (fused) return launch_mlp_chain(m, ly, dF, B, ch, hi, lo, st);
        for (int l = hi; l >= lo; --l) {
            GemmArgs gd;
            gd.M = (int)B;
            gd.N = ly.in(l);
            gd.K = ly.out(l);
            gd.A = l == ly.L - 1 ? dF : ch.dz[l];
            gd.a_sm = l == ly.L - 1 ? kIoLd : pl.ld;
            gd.a_sk = 1;
            gd.B = m.params_bf16 + ly.woff(l);
            gd.b_sn = 1;
            gd.b_sk = ly.in(l);
            gd.hout = ch.dz[l - 1];
            gd.ldh = pl.ld;
            gd.zprev = ap.z[l - 1];
            if (int32_t e = launch_gemm<kEpiDSilu>(gd, st)) return e;
        }
        return PDMP_OK;
    };
    // The gradients of layers [lo, hi] into grad from its entry woff(lo) on: by partial rows of
    // np entries, or, of one range, at once.
    auto weight_grad = [&](int lo, int hi, int64_t np, float *loss) -> int32_t {
        MlpWg wg{};
        const int64_t base = ly.woff(lo);
        for (int l = lo; l <= hi; ++l) {
            MlpWgLayer &y = wg.layer[wg.L++];
            const bool last = l == ly.L - 1;
            y.dz = last ? dF : ch.dz[l];
            y.ldz = last ? kIoLd : pl.ld;
            y.h = l == 0 ? ap.h0 : ap.h[l - 1];
            y.ldh = l == 0 ? kIoLd : mlp_ld(ly.H);
            y.zblk = !last && fused;
            y.hblk = l > 0 && fused;
            y.O = ly.out(l);
            y.I = ly.in(l);
            y.woff = ly.woff(l) - base;
            y.boff = ly.boff(l) - base;
            y.tile0 = wg.tiles;
            y.tiles_i = (y.I + kWgT - 1) / kWgT;
            wg.tiles += layer_tiles(ly, l);
        }
        const int64_t per = wgrad_per(pl.ranges, B), S = wgrad_rows(pl.ranges, B);
        hipLaunchKernelGGL(k_mlp_wgrad, dim3((unsigned)(wg.tiles * ((S + 7) / 8 * 8))), dim3(256), 0,
                           st, wg, B, per, np, pl.part ? part : grad + base);
        const int64_t sum = pl.part ? np : 0;
        if (sum || loss)
            hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((sum + 255) / 256 + (loss ? 1 : 0))),
                               dim3(256), 0, st, part, (int)S, sum, grad + base, rparts, pl.nb, scale,
                               loss);
        return check_launch("mlp wgrad");
    };
    if (!pl.layered) {
        if (int32_t e = data_grad(ly.L - 1, 1)) return e;
        return weight_grad(0, ly.L - 1, ly.nparams(), loss);
    }
    for (int l = ly.L - 1; l >= 0; --l) {
        if (int32_t e = weight_grad(l, l, (int64_t)ly.out(l) * ly.in(l) + ly.out(l),
                                    l == 0 ? loss : nullptr))
            return e;
        if (l > 0)
            if (int32_t e = data_grad(l, l)) return e;
    }
    return PDMP_OK;
}

int32_t launch_f32_to_bf16(const float *x, int64_t n, uint16_t *y, hipStream_t st) {
    if (int32_t e = grid_guard((n + 255) / 256, 256, "k_f32_to_bf16")) return e;
    hipLaunchKernelGGL(k_f32_to_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x, n, y);
    return check_launch("k_f32_to_bf16");
}

}  // namespace pdmp
