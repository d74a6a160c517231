// tanh_net.hip -- the paper's occupancy network (Sec. 3.1): a fully connected network
// with tanh between hidden layers and a sigmoid output, c(x) = sigma(s(x)), its input
// gradient by the chain rule, and the T-step Euler morph of Eq. 1 on top of it.
//
//   a_1 = tanh(W_0 x + b_0),  a_{l+1} = tanh(W_l a_l + b_l),  s = v . a_L + b_o
//   e_L = v * (1 - a_L^2),   e_l = (1 - a_l^2) * (W_l^T e_{l+1}),  grad s = W_0^T e_1
//
// One wave carries 16 points (four lanes per point) through the whole network.  The
// hidden-to-hidden products, forward (W_l a) and backward (W_l^T e), run on the matrix
// cores with the points as the 16 columns.  The accumulator of a 16-row tile t gives
// lane l the units 16t + 4(l/16) + v (v = 0..3) of point l%16; the contraction of the
// next product is ordered to match, so each lane feeds its own accumulator entries
// back as the B operand -- activations never leave the registers.  The matching
// permutation is applied once to the weights when they are staged in LDS in
// fragment order.  The morph, value and gradient kernel runs the products on BF16
// MFMA at FP32 accuracy (v_mfma_f32_16x16x32_bf16, three-way bf16 splits, six
// leading products: mfma_split.h); a 32-wide k-block takes tiles 2kb and 2kb + 1,
// lane l supplying units 16(2kb + j/4) + 4(l/16) + j%4, j < 8.  The fit kernels stay
// on FP32 MFMA (v_mfma_f32_16x16x4_f32, step (t, v) takes units 16t + 4k + v).  The input layer
// (K = dim) and the output dot product are VALU work; the four lanes of a point are
// summed by xor-16 and xor-32 exchanges (the same sum in all four).  Widths up to 64
// run as 1, 2 or 4 tiles of 16, padded units having zero weights (tanh(0) = 0, so
// they add nothing).
#include <type_traits>

#include "mfma_split.h"
#include "pdmp_common.h"

namespace pdmp {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_tn;

constexpr int kTnBlock = 256;   // 4 waves, 16 points each (fit)
constexpr int kTnMorphBlock = 512;  // 8 waves share one LDS copy of the weights (morph)
constexpr int kTnPts = 16;      // points per wave

// tanh(z) and its slope 1 - tanh^2 from e = exp(-2|z|) in (0, 1]:
// tanh = sign(z) (1 - e)/(1 + e), slope = 4e/(1 + e)^2 (no cancellation near +-1).
__device__ __forceinline__ void tanh_slope(float z, float &a, float &d) {
    const float e = exp2_fast(-2.0f * kLog2e * fabsf(z));
    const float r = __builtin_amdgcn_rcpf(1.0f + e);
    a = copysignf((1.0f - e) * r, z);
    d = 4.0f * e * (r * r);
}

// The same from a pre-activation held scaled by 2^zs, k = -2 log2(e) 2^-zs, returning
// as tanh (as a power of two): with r2 = 2/(1 + e) the factors 2 and 4 are taken before the
// rounding, by exact scalings, so a / as and d are the bits tanh_slope gives for z 2^-zs, in
// nine instructions.
__device__ __forceinline__ void tanh_slope_sc(float z, float k, float as, float &a, float &d) {
    const float e = exp2_fast(k * fabsf(z));
    const float r2 = __builtin_amdgcn_rcpf(fmaf(e, 0.5f, 0.5f));
    a = copysignf(fmaf(-e, 0.5f * as, 0.5f * as) * r2, z);
    d = e * (r2 * r2);
}

// Offset of W_l in the flat parameter vector (l = L gives v).
__device__ __forceinline__ int64_t tn_w_off(int l, int dim, int H) {
    return l == 0 ? 0 : (int64_t)H * dim + H + (int64_t)(l - 1) * (H * H + H);
}

__device__ __forceinline__ float4 tn_ld4(const float *p) {
    return *reinterpret_cast<const float4 *>(p);
}

// Sum over the four lanes of a point (the same value in all four), the same bits either way:
// by row swaps, or (LDS) by the LDS's permute.
template <bool LDS = false>
__device__ __forceinline__ float tn_sum4(float p) {
    if (LDS) {
        p = p + __shfl_xor(p, 16, 64);
        return p + __shfl_xor(p, 32, 64);
    }
    auto add = [](float a, float b) { return a + b; };
    return join32(join16(p, add), add);
}

// ---- BF16-MFMA form (morph, value, gradient) ----

// The forward hidden products' scheme (the block's choice from the weights, every
// block alike): FP16 parts when each hidden-to-hidden W_l is finite with every nonzero
// |w| at least 2^-19 of its largest -- then 2^fsw W_l, largest in [2^14, 2^15), has
// two FP16 parts of 11 bits each and three products carry a multiply-add at FP32
// accuracy (mfma_split.h) -- and the layer's scale 2^(fsw + kTnAct) lies in [1, 2^100]
// with the scaled bias at most 2^120 (the accumulator starts from it: nothing is lost
// or overflows in scaling); three-way BF16 splits and six products otherwise.  The
// backward products stay on BF16 parts: their vectors e_l have no bound to scale by.
struct TnFwd {
    int fwh;          // 1: FP16 forward products
    int fsw[4];       // per hidden-to-hidden layer l (index l - 1): the scale exponent
    uint32_t wmx[4], wmn[4], bmx[4];  // largest, smallest nonzero |w|; largest |b| (bits)
};

// Activations enter the FP16 forward products as 2^kTnAct a (|a| <= 1): FP16 keeps 11
// bits of every |a| >= 2^-28 and the products stay below 2^29 in the FP32 accumulator.
constexpr int kTnAct = 14;

// The choice in three parts, every thread of the block calling each: begin, each wave's
// extremes of W_l and b_l noted, end (the scheme is in F; the block is synchronised).
__device__ __forceinline__ void tn_scheme_begin(TnFwd &F) {
    if (threadIdx.x < 4) {
        F.wmx[threadIdx.x] = 0u;
        F.wmn[threadIdx.x] = 0xffffffffu;
        F.bmx[threadIdx.x] = 0u;
    }
    __syncthreads();
}

__device__ __forceinline__ void tn_scheme_note(TnFwd &F, int l, uint32_t mx, uint32_t mn,
                                               uint32_t bm) {
    auto larger = [](float a, float b) {
        return __uint_as_float(max(__float_as_uint(a), __float_as_uint(b)));
    };
    auto smaller = [](float a, float b) {
        return __uint_as_float(min(__float_as_uint(a), __float_as_uint(b)));
    };
    mx = __float_as_uint(wave_all(__uint_as_float(mx), larger));
    mn = __float_as_uint(wave_all(__uint_as_float(mn), smaller));
    bm = __float_as_uint(wave_all(__uint_as_float(bm), larger));
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&F.wmx[l - 1], mx);
        atomicMin(&F.wmn[l - 1], mn);
        atomicMax(&F.bmx[l - 1], bm);
    }
}

template <int L>
__device__ void tn_scheme_end(TnFwd &F) {
    __syncthreads();
    if (threadIdx.x == 0) {
        int ok = L > 1;
        for (int l = 0; l < L - 1; ++l) {
            const uint32_t mx = F.wmx[l], mn = F.wmn[l], bm = F.bmx[l];
            int e = 0;
            if (mx >= 0x7f800000u || bm >= 0x7f800000u) {
                ok = 0;  // Inf or NaN
            } else if (mx != 0u) {
                frexpf(__uint_as_float(mx), &e);  // largest = m 2^e, m in [0.5, 1)
                if (__uint_as_float(mn) < ldexpf(__uint_as_float(mx), -19)) ok = 0;
            }
            const int fsw = mx != 0u ? 15 - e : 0;
            if (fsw + kTnAct < 0 || fsw + kTnAct > 100 ||
                ldexpf(__uint_as_float(bm), fsw + kTnAct) > 0x1p120f)
                ok = 0;
            F.fsw[l] = fsw;
        }
        F.fwh = ok;
    }
    __syncthreads();
}

// From the parameters in memory, eight loads of a thread in flight.
template <int L>
__device__ void tn_forward_scheme(TnFwd &F, const float *__restrict__ P, int dim, int H) {
    tn_scheme_begin(F);
    for (int l = 1; l < L; ++l) {
        const float *W = P + tn_w_off(l, dim, H);  // W_l (H x H), then b_l (H)
        uint32_t mx = 0u, mn = 0xffffffffu, bm = 0u;
        for (int e0 = threadIdx.x; e0 < H * H; e0 += 8 * blockDim.x) {
            uint32_t u[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                u[k] = __float_as_uint(W[min(e0 + k * (int)blockDim.x, H * H - 1)]) & 0x7fffffffu;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                mx = max(mx, u[k]);
                if (u[k] != 0u) mn = min(mn, u[k]);
            }
        }
        for (int e = threadIdx.x; e < H; e += blockDim.x)
            bm = max(bm, __float_as_uint(W[(int64_t)H * H + e]) & 0x7fffffffu);
        tn_scheme_note(F, l, mx, mn, bm);
    }
    tn_scheme_end<L>(F);
}

template <int L>
__global__ void __launch_bounds__(256) k_tanh_scheme(const float *__restrict__ P, int dim, int H,
                                                     int32_t *out) {
    __shared__ TnFwd F;
    tn_forward_scheme<L>(F, P, dim, H);
    if (threadIdx.x == 0) *out = F.fwh ? 2 : 1;
}

// The forward scheme the morph, value and gradient kernel takes: 2 (FP16 parts) or 1.
int32_t launch_tanh_scheme(const pdmp_tanh_net &net, int32_t *out, hipStream_t st) {
#define PDMP_TS(L)                                                                         \
    hipLaunchKernelGGL(k_tanh_scheme<L>, dim3(1), dim3(256), 0, st, net.params, net.dim, \
                       net.hidden, out)
    switch (net.n_hidden) {
        case 1: PDMP_TS(1); break;
        case 2: PDMP_TS(2); break;
        case 3: PDMP_TS(3); break;
        default: PDMP_TS(4); break;
    }
#undef PDMP_TS
    return check_launch("k_tanh_scheme");
}

template <int DIM, int NT, int L>
struct TnLdsX6 {
    static constexpr int HP = 16 * NT;
    static constexpr int KB = (NT + 1) / 2;                      // 32-wide k-blocks
    static constexpr int NF = (L - 1) * NT * KB * 3 * 64;        // bf16x8 fragments per direction
    // fw[((l-1) NT + to) KB + kb][p][lane] = part p of W_l[16to + lane%16][unit(kb, lane, j)]
    // bw[((l-1) NT + ti) KB + kb][p][lane] = part p of W_l[unit(kb, lane, j)][16ti + lane%16]
    // with unit(kb, lane, j) = 16(2kb + j/4) + 4(lane/16) + j%4, j < 8
    bf16x8_t fw[NF > 0 ? NF : 1];
    bf16x8_t bw[NF > 0 ? NF : 1];
    float w0t[DIM][HP];  // W_0 transposed
    float bias[L][HP];
    float vo[HP];
    float bo;
    TnFwd F;  // the forward products' scheme
};

template <int DIM, int NT, int L>
__device__ void tn_stage_x6(TnLdsX6<DIM, NT, L> &S, const float *__restrict__ P, int H) {
    using LD = TnLdsX6<DIM, NT, L>;
    tn_forward_scheme<L>(S.F, P, DIM, H);
    const bool fh = S.F.fwh != 0;
    for (int idx = threadIdx.x; idx < LD::NF / 3; idx += blockDim.x) {
        const int ln = idx & 63, q = idx >> 6;  // q = ((l-1) NT + first) KB + kb
        const int kb = q % LD::KB, first = (q / LD::KB) % NT, l = 1 + q / (LD::KB * NT);
        const float *W = P + tn_w_off(l, DIM, H);
        float vf[8], vb[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int t = 2 * kb + j / 4;
            const int unit = 16 * t + 4 * (ln >> 4) + (j & 3);
            const int other = 16 * first + (ln & 15);
            const bool ok = t < NT && unit < H && other < H;
            vf[j] = ok ? W[(int64_t)other * H + unit] : 0.0f;  // forward: row other, col unit
            vb[j] = ok ? W[(int64_t)unit * H + other] : 0.0f;  // backward: W^T
        }
        bf16x8_t f1, f2, f3, b1, b2, b3;
        const int base = q * 3 * 64 + ln;
        if (fh) {
#pragma unroll
            for (int j = 0; j < 8; ++j) vf[j] = ldexpf(vf[j], S.F.fsw[l - 1]);
            f16x8_t h1, h2;
            split2h(vf, h1, h2);
            reinterpret_cast<f16x8_t *>(S.fw)[base] = h1;
            reinterpret_cast<f16x8_t *>(S.fw)[base + 64] = h2;
        } else {
            split3(vf, f1, f2, f3);
            S.fw[base] = f1;
            S.fw[base + 64] = f2;
            S.fw[base + 128] = f3;
        }
        split3(vb, b1, b2, b3);
        S.bw[base] = b1;
        S.bw[base + 64] = b2;
        S.bw[base + 128] = b3;
    }
    for (int idx = threadIdx.x; idx < LD::HP; idx += blockDim.x) {
        const bool ok = idx < H;
#pragma unroll
        for (int k = 0; k < DIM; ++k) S.w0t[k][idx] = ok ? P[(int64_t)idx * DIM + k] : 0.0f;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const int64_t bo = tn_w_off(l, DIM, H) + (int64_t)H * (l == 0 ? DIM : H);
            // FP16 forward: the hidden biases enter the accumulator as 2^(fsw + kTnAct) b
            const float b = ok ? P[bo + idx] : 0.0f;
            S.bias[l][idx] = fh && l > 0 ? ldexpf(b, S.F.fsw[l - 1] + kTnAct) : b;
        }
        S.vo[idx] = ok ? P[tn_w_off(L, DIM, H) + idx] : 0.0f;
    }
    if (threadIdx.x == 0) S.bo = P[tn_w_off(L, DIM, H) + H];
}

// The lane's B operand of k-block kb from its accumulator-layout values v[t][0..3],
// split into three bf16 parts.
template <int NT>
__device__ __forceinline__ void tn_kblock(const f32x4_tn (&v)[NT], int kb, bf16x8_t &p1,
                                          bf16x8_t &p2, bf16x8_t &p3) {
    float b[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int t = 2 * kb + j / 4;
        b[j] = t < NT ? v[t < NT ? t : 0][j & 3] : 0.0f;
    }
    split3(b, p1, p2, p3);
}

// s (all four lanes of the point) and, with GRAD, grad_x s at the point x; with FH
// the forward hidden products on the FP16 parts (the block's scheme, S.fwh).
template <int DIM, int NT, int L, bool GRAD, bool FH>
__device__ __forceinline__ void tn_point_x6(const TnLdsX6<DIM, NT, L> &S, const float (&x)[DIM],
                                            float &s, float (&g)[DIM]) {
    using LD = TnLdsX6<DIM, NT, L>;
    const int lane0 = threadIdx.x & 63, u4 = 4 * (lane0 >> 4);
    // The weight fragments are the same on every call; an opaque copy of the lane
    // index keeps the compiler from hoisting their LDS reads out of the step loop
    // into registers (which would not fit).
    int lane = lane0;
    asm volatile("" : "+v"(lane));
    f32x4_tn a[NT];
    f32x4_tn d[L][NT];
    // input layer: z = b_0 + W_0 x
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int u0 = 16 * t + u4;
        const float4 bb = tn_ld4(&S.bias[0][u0]);
        float z[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            const float4 w = tn_ld4(&S.w0t[k][u0]);
            z[0] = fmaf(w.x, x[k], z[0]);
            z[1] = fmaf(w.y, x[k], z[1]);
            z[2] = fmaf(w.z, x[k], z[2]);
            z[3] = fmaf(w.w, x[k], z[3]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float av, dv;
            // FP16 forward: the activations feeding a hidden product are held as 2^kTnAct a
            tanh_slope_sc(z[v], -2.0f * kLog2e, FH ? (float)(1 << kTnAct) : 1.0f, av, dv);
            a[t][v] = av;
            d[0][t][v] = dv;
        }
    }
    // hidden layers: z = b_l + W_l a  (the bias preloaded in the accumulator)
#pragma unroll
    for (int l = 1; l < L; ++l) {
        f32x4_tn z[NT];
        // FP16 products accumulate 2^(fsw + kTnAct) (W a + b) from the bias staged at
        // that scale; the tanh below takes the unscaling in its exponent (exact)
        const float kz = FH ? ldexpf(-2.0f * kLog2e, -(S.F.fsw[l - 1] + kTnAct)) : -2.0f * kLog2e;
#pragma unroll
        for (int to = 0; to < NT; ++to) {
            const float4 bb = tn_ld4(&S.bias[l][16 * to + u4]);
            z[to][0] = bb.x;
            z[to][1] = bb.y;
            z[to][2] = bb.z;
            z[to][3] = bb.w;
        }
#pragma unroll
        for (int kb = 0; kb < LD::KB; ++kb) {
            if (FH) {
                float bv[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int t = 2 * kb + j / 4;
                    bv[j] = t < NT ? a[t < NT ? t : 0][j & 3] : 0.0f;  // 2^kTnAct a
                }
                f16x8_t h1, h2;
                split2h(bv, h1, h2);
#pragma unroll
                for (int to = 0; to < NT; ++to) {
                    const f16x8_t *f = reinterpret_cast<const f16x8_t *>(S.fw) +
                                       (((l - 1) * NT + to) * LD::KB + kb) * 3 * 64 + lane;
                    z[to] = mfma16_h3(f[0], f[64], h1, h2, z[to]);
                }
            } else {
                bf16x8_t b1, b2, b3;
                tn_kblock<NT>(a, kb, b1, b2, b3);
#pragma unroll
                for (int to = 0; to < NT; ++to) {
                    const bf16x8_t *f = S.fw + (((l - 1) * NT + to) * LD::KB + kb) * 3 * 64 + lane;
                    z[to] = mfma16_x6(f[0], f[64], f[128], b1, b2, b3, z[to]);
                }
            }
        }
#pragma unroll
        for (int to = 0; to < NT; ++to)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float av, dv;
                // scaled by 2^kTnAct again where the next hidden product takes it
                tanh_slope_sc(z[to][v], kz, FH && l + 1 < L ? (float)(1 << kTnAct) : 1.0f, av,
                              dv);
                a[to][v] = av;
                d[l][to][v] = dv;
            }
    }
    // output: s = v . a_L + b_o
    float p = 0.0f;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const float4 vv = tn_ld4(&S.vo[16 * t + u4]);
        p = fmaf(vv.x, a[t][0], p);
        p = fmaf(vv.y, a[t][1], p);
        p = fmaf(vv.z, a[t][2], p);
        p = fmaf(vv.w, a[t][3], p);
    }
    // one hidden layer has no products to wait for: its waves are bound by the vector unit,
    // and the LDS is free for the sums (200,000 points, H = 5, 10 steps: 25.4 us, by swaps 27)
    s = tn_sum4<L == 1>(p) + S.bo;
    if (!GRAD) return;
    // reverse order: e_L = v * d_L, e_l = d_l * (W_l^T e_{l+1}), grad s = W_0^T e_1
    f32x4_tn e[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const float4 vv = tn_ld4(&S.vo[16 * t + u4]);
        e[t][0] = vv.x * d[L - 1][t][0];
        e[t][1] = vv.y * d[L - 1][t][1];
        e[t][2] = vv.z * d[L - 1][t][2];
        e[t][3] = vv.w * d[L - 1][t][3];
    }
#pragma unroll
    for (int l = L - 1; l >= 1; --l) {
        f32x4_tn G[NT];
        const f32x4_tn zero = {};  // the first k-block starts from the zero accumulator
#pragma unroll
        for (int kb = 0; kb < LD::KB; ++kb) {
            bf16x8_t b1, b2, b3;
            tn_kblock<NT>(e, kb, b1, b2, b3);
#pragma unroll
            for (int ti = 0; ti < NT; ++ti) {
                const bf16x8_t *f = S.bw + (((l - 1) * NT + ti) * LD::KB + kb) * 3 * 64 + lane;
                G[ti] = mfma16_x6(f[0], f[64], f[128], b1, b2, b3, kb == 0 ? zero : G[ti]);
            }
        }
#pragma unroll
        for (int ti = 0; ti < NT; ++ti)
#pragma unroll
            for (int v = 0; v < 4; ++v) e[ti][v] = G[ti][v] * d[l - 1][ti][v];
    }
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        float q = 0.0f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float4 w = tn_ld4(&S.w0t[k][16 * t + u4]);
            q = fmaf(w.x, e[t][0], q);
            q = fmaf(w.y, e[t][1], q);
            q = fmaf(w.z, e[t][2], q);
            q = fmaf(w.w, e[t][3], q);
        }
        g[k] = tn_sum4<L == 1>(q);
    }
}

template <int DIM, int NT, int L, int MODE>
__global__ void __launch_bounds__(kTnMorphBlock)
k_tanh_net(const float *__restrict__ P, int H, const float *x_in, int64_t n, int T, float eta,
           float *c_out, float *s_out, float *g_out, float *x_out) {
    __shared__ __attribute__((aligned(16))) TnLdsX6<DIM, NT, L> S;
    tn_stage_x6<DIM, NT, L>(S, P, H);
    __syncthreads();
    const int lane = threadIdx.x & 63, quad = lane >> 4;
    const int64_t tiles = (n + kTnPts - 1) / kTnPts;
    const int64_t wstride = (int64_t)gridDim.x * (kTnMorphBlock / 64);
    for (int64_t tile = (int64_t)blockIdx.x * (kTnMorphBlock / 64) + (threadIdx.x >> 6); tile < tiles;
         tile += wstride) {
        const int64_t i = tile * kTnPts + (lane & 15);
        const int64_t ic = i < n ? i : n - 1;
        float x[DIM], g[DIM], s = 0.0f;
#pragma unroll
        for (int k = 0; k < DIM; ++k) x[k] = x_in[(size_t)k * n + ic];
        const int steps = MODE == kMorph ? T : 1;
        for (int st = 0; st < steps; ++st) {
            if (S.F.fwh)
                tn_point_x6<DIM, NT, L, MODE != kEval, true>(S, x, s, g);
            else
                tn_point_x6<DIM, NT, L, MODE != kEval, false>(S, x, s, g);
            if (MODE == kMorph) {
                float c, sp;
                sigmoid_and_slope(s, c, sp);
                const float step = eta * sp;
#pragma unroll
                for (int k = 0; k < DIM; ++k) x[k] = fmaf(-step, g[k], x[k]);
            }
        }
        if (quad != 0 || i >= n) continue;
        if (MODE == kMorph) {
#pragma unroll
            for (int k = 0; k < DIM; ++k) x_out[(size_t)k * n + i] = x[k];
        } else {
            float c, sp;
            sigmoid_and_slope(s, c, sp);
            if (c_out) c_out[i] = c;
            if (MODE == kEval) {
                if (s_out) s_out[i] = s;
            } else {
#pragma unroll
                for (int k = 0; k < DIM; ++k) g_out[(size_t)k * n + i] = sp * g[k];
            }
        }
    }
}

// ---- small batches: a wave per tile of 16 units ----
//
// A block of NT waves takes 16 points at a time, wave w the units 16w .. 16w + 15 of every
// layer: its rows of W_l (forward) and of W_l^T (reverse) stay in registers as split
// fragments over all points and steps, in the order of the contraction index
//   unit(kb, lane, j) = 16(2kb + j/4) + 4(lane/16) + j%4, j < 8,
// so that a layer's accumulators, split where they lie, are the next layer's B operands:
// the waves pass them on through LDS (two buffers, one barrier per layer), and every wave
// forms the output sum and the gradient of its points from all units' values.  The same bits
// as k_tanh_net, whose waves take a tile's 64 units alone, eight to a block: few points leave
// most CUs idle there, and a step is one wave's latency.  20 steps of up to 4,096 points: 64
// x 2 units 69 -> 35 us, 64 x 3 110 -> 49, 64 x 4 169 -> 68, 32 x 3 49 -> 33; of 8,192 points
// 70 -> 44, 111 -> 63, 173 -> 89, 50 -> 40.  The waves' exchanges (2 per layer) cost too much
// where the other kernel fills the chip: 65,536 points, 64 x 3: 266 us there, 398 here.
// The parts of four values (a lane's units of a tile), as split2h and split3 give them.
__device__ __forceinline__ void tn_split2h(const float (&v)[4], uint2 &p1, uint2 &p2) {
    const float w[8] = {v[0], v[1], v[2], v[3], 0.0f, 0.0f, 0.0f, 0.0f};
    f16x8_t h1, h2;
    split2h(w, h1, h2);
    __builtin_memcpy(&p1, &h1, 8);
    __builtin_memcpy(&p2, &h2, 8);
}
__device__ __forceinline__ void tn_split3(const float (&v)[4], uint2 &p1, uint2 &p2, uint2 &p3) {
    const float w[8] = {v[0], v[1], v[2], v[3], 0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8_t b1, b2, b3;
    split3(w, b1, b2, b3);
    __builtin_memcpy(&p1, &b1, 8);
    __builtin_memcpy(&p2, &b2, 8);
    __builtin_memcpy(&p3, &b3, 8);
}

template <int DIM, int NT, int L>
struct TnSmallLds {
    static constexpr int HP = 16 * NT;
    uint2 xb[2][3 * NT * 64];  // [part][tile][lane], or float4 [tile][lane]
    float w0t[DIM][HP], vo[HP];
    TnFwd F;  // the forward products' scheme
};

// A wave's share of the parameters, requested at once: its rows of W_l, of W_l^T, its units'
// biases, W_0 rows and v (padded units zero).
template <int DIM, int NT, int L, bool GRAD>
struct TnSmallRaw {
    static constexpr int KB = (NT + 1) / 2, LH = L > 1 ? L - 1 : 1;
    float f[LH][KB][8], b[GRAD ? LH : 1][KB][8], bias[L][4], w0[DIM][4], v[4], bo;

    __device__ __forceinline__ void load(const float *__restrict__ P, int H) {
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, u4 = 4 * (lane >> 4);
        const int own = 16 * wv + (lane & 15);
#pragma unroll
        for (int l = 1; l < L; ++l) {
            const float *W = P + tn_w_off(l, DIM, H);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int unit = 16 * (2 * kb + j / 4) + u4 + (j & 3);
                    const bool ok = unit < H && own < H;
                    f[l - 1][kb][j] = W[ok ? own * H + unit : 0];
                    if (GRAD) b[l - 1][kb][j] = W[ok ? unit * H + own : 0];
                }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int u = 16 * wv + u4 + k, uc = u < H ? u : 0;
#pragma unroll
            for (int j = 0; j < DIM; ++j) w0[j][k] = P[(int64_t)uc * DIM + j];
#pragma unroll
            for (int l = 0; l < L; ++l)
                bias[l][k] = P[tn_w_off(l, DIM, H) + (int64_t)H * (l == 0 ? DIM : H) + uc];
            v[k] = P[tn_w_off(L, DIM, H) + uc];
        }
        bo = P[tn_w_off(L, DIM, H) + H];
#pragma unroll
        for (int l = 1; l < L; ++l)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool ok = 16 * (2 * kb + j / 4) + u4 + (j & 3) < H && own < H;
                    if (!ok) f[l - 1][kb][j] = 0.0f;
                    if (GRAD && !ok) b[l - 1][kb][j] = 0.0f;
                }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (16 * wv + u4 + k < H) continue;
#pragma unroll
            for (int j = 0; j < DIM; ++j) w0[j][k] = 0.0f;
#pragma unroll
            for (int l = 0; l < L; ++l) bias[l][k] = 0.0f;
            v[k] = 0.0f;
        }
    }

    // The forward scheme from the values at hand (the waves' rows are all of every W_l).
    __device__ __forceinline__ void scheme(TnFwd &F) const {
        tn_scheme_begin(F);
#pragma unroll
        for (int l = 1; l < L; ++l) {
            uint32_t mx = 0u, mn = 0xffffffffu, bm = 0u;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t u = __float_as_uint(f[l - 1][kb][j]) & 0x7fffffffu;
                    mx = max(mx, u);
                    if (u != 0u) mn = min(mn, u);
                }
#pragma unroll
            for (int k = 0; k < 4; ++k) bm = max(bm, __float_as_uint(bias[l][k]) & 0x7fffffffu);
            tn_scheme_note(F, l, mx, mn, bm);
        }
        tn_scheme_end<L>(F);
    }
};

template <int DIM, int NT, int L, int MODE, bool FH>
__device__ __forceinline__ void tn_small_body(TnSmallLds<DIM, NT, L> &S,
                                              const TnSmallRaw<DIM, NT, L, MODE != kEval> &R,
                                              const float *x_in, int64_t n, int T, float eta,
                                              float *c_out, float *s_out, float *g_out,
                                              float *x_out) {
    constexpr int KB = (NT + 1) / 2, LH = L > 1 ? L - 1 : 1, FP = FH ? 2 : 3;
    constexpr bool GRAD = MODE != kEval;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, u4 = 4 * (lane >> 4);
    uint4 fw[LH][KB][FP], bw[GRAD ? LH : 1][KB][3];
    float bias[L][4], kz[L];
#pragma unroll
    for (int l = 1; l < L; ++l)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            if constexpr (FH) {
                float vf[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) vf[j] = ldexpf(R.f[l - 1][kb][j], S.F.fsw[l - 1]);
                f16x8_t p[2];
                split2h(vf, p[0], p[1]);
                __builtin_memcpy(fw[l - 1][kb], p, 32);
            } else {
                bf16x8_t p[3];
                split3(R.f[l - 1][kb], p[0], p[1], p[2]);
                __builtin_memcpy(fw[l - 1][kb], p, 48);
            }
            if constexpr (GRAD) {
                bf16x8_t p[3];
                split3(R.b[l - 1][kb], p[0], p[1], p[2]);
                __builtin_memcpy(bw[l - 1][kb], p, 48);
            }
        }
    // FP16 forward: the hidden biases enter the accumulator as 2^(fsw + kTnAct) b, and the
    // tanh takes the unscaling in its exponent (exact)
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const int sc = FH && l > 0 ? S.F.fsw[l > 0 ? l - 1 : 0] + kTnAct : 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) bias[l][v] = ldexpf(R.bias[l][v], sc);
        kz[l] = ldexpf(-2.0f * kLog2e, -sc);
    }

    int buf = 0;
    // all tiles' values of the lane's units, FP32
    auto share = [&](const float (&v)[4], float4 (&all)[NT]) {
        float4 *x = reinterpret_cast<float4 *>(S.xb[buf]);
        x[wv * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t) all[t] = x[t * 64 + lane];
        buf ^= 1;
    };
    // part p of the B operand of k-block kb, after the waves wrote theirs
    auto operand = [&](const uint2 *x, int p, int kb) {
        const uint2 lo = x[(p * NT + 2 * kb) * 64 + lane];
        const uint2 hi = 2 * kb + 1 < NT ? x[(p * NT + (2 * kb + 1 < NT ? 2 * kb + 1 : 0)) * 64 + lane]
                                         : make_uint2(0u, 0u);
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
    };
    auto f16 = [](const uint4 &v) {
        f16x8_t r;
        __builtin_memcpy(&r, &v, 16);
        return r;
    };
    auto b16 = [](const uint4 &v) {
        bf16x8_t r;
        __builtin_memcpy(&r, &v, 16);
        return r;
    };
    // acc + this wave's rows (split fragments f, three BF16 parts) times all units' v
    auto products3 = [&](const uint4 (&f)[KB][3], const float (&v)[4], f32x4_tn acc) {
        uint2 *x = S.xb[buf], p1, p2, p3;
        tn_split3(v, p1, p2, p3);
        x[(0 * NT + wv) * 64 + lane] = p1;
        x[(1 * NT + wv) * 64 + lane] = p2;
        x[(2 * NT + wv) * 64 + lane] = p3;
        __syncthreads();
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
            acc = mfma16_x6(b16(f[kb][0]), b16(f[kb][1]), b16(f[kb][2]), b16(operand(x, 0, kb)),
                            b16(operand(x, 1, kb)), b16(operand(x, 2, kb)), acc);
        buf ^= 1;
        return acc;
    };
    auto products2 = [&](const uint4 (&f)[KB][2], const float (&v)[4], f32x4_tn acc) {
        uint2 *x = S.xb[buf], p1, p2;
        tn_split2h(v, p1, p2);
        x[(0 * NT + wv) * 64 + lane] = p1;
        x[(1 * NT + wv) * 64 + lane] = p2;
        __syncthreads();
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
            acc = mfma16_h3(f16(f[kb][0]), f16(f[kb][1]), f16(operand(x, 0, kb)),
                            f16(operand(x, 1, kb)), acc);
        buf ^= 1;
        return acc;
    };

    const int64_t tiles = (n + kTnPts - 1) / kTnPts;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t i = tile * kTnPts + (lane & 15);
        const int64_t ic = i < n ? i : n - 1;
        float x[DIM], g[DIM], s = 0.0f;
#pragma unroll
        for (int k = 0; k < DIM; ++k) x[k] = x_in[(size_t)k * n + ic];
        const int steps = MODE == kMorph ? T : 1;
        for (int st = 0; st < steps; ++st) {
            float a[4], d[L][4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float z = bias[0][v];
#pragma unroll
                for (int k = 0; k < DIM; ++k) z = fmaf(R.w0[k][v], x[k], z);
                // the activations feeding an FP16 product are held as 2^kTnAct a
                tanh_slope_sc(z, kz[0], FH ? (float)(1 << kTnAct) : 1.0f, a[v], d[0][v]);
            }
#pragma unroll
            for (int l = 1; l < L; ++l) {
                f32x4_tn z = {bias[l][0], bias[l][1], bias[l][2], bias[l][3]};
                if constexpr (FH) z = products2(fw[l - 1], a, z);
                else z = products3(fw[l - 1], a, z);
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    tanh_slope_sc(z[v], kz[l], FH && l + 1 < L ? (float)(1 << kTnAct) : 1.0f, a[v],
                                  d[l][v]);
            }
            float4 all[NT];
            share(a, all);
            float p = 0.0f;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const float4 vv = tn_ld4(&S.vo[16 * t + u4]);
                p = fmaf(vv.x, all[t].x, p);
                p = fmaf(vv.y, all[t].y, p);
                p = fmaf(vv.z, all[t].z, p);
                p = fmaf(vv.w, all[t].w, p);
            }
            s = tn_sum4(p) + R.bo;
            if constexpr (GRAD) {
                // e_L = v d_L, e_l = d_l (W_l^T e_{l+1}), grad s = W_0^T e_1
                float e[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) e[v] = R.v[v] * d[L - 1][v];
#pragma unroll
                for (int l = L - 1; l >= 1; --l) {
                    const f32x4_tn zero = {};
                    const f32x4_tn G = products3(bw[l - 1], e, zero);
#pragma unroll
                    for (int v = 0; v < 4; ++v) e[v] = G[v] * d[l - 1][v];
                }
                share(e, all);
#pragma unroll
                for (int k = 0; k < DIM; ++k) {
                    float q = 0.0f;
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const float4 w = tn_ld4(&S.w0t[k][16 * t + u4]);
                        q = fmaf(w.x, all[t].x, q);
                        q = fmaf(w.y, all[t].y, q);
                        q = fmaf(w.z, all[t].z, q);
                        q = fmaf(w.w, all[t].w, q);
                    }
                    g[k] = tn_sum4(q);
                }
            }
            if (MODE == kMorph) {
                float c, sp;
                sigmoid_and_slope(s, c, sp);
                const float step = eta * sp;
#pragma unroll
                for (int k = 0; k < DIM; ++k) x[k] = fmaf(-step, g[k], x[k]);
            }
        }
        if (wv != 0 || lane >= 16 || i >= n) continue;
        if (MODE == kMorph) {
#pragma unroll
            for (int k = 0; k < DIM; ++k) x_out[(size_t)k * n + i] = x[k];
        } else {
            float c, sp;
            sigmoid_and_slope(s, c, sp);
            if (c_out) c_out[i] = c;
            if (MODE == kEval) {
                if (s_out) s_out[i] = s;
            } else {
#pragma unroll
                for (int k = 0; k < DIM; ++k) g_out[(size_t)k * n + i] = sp * g[k];
            }
        }
    }
}

template <int DIM, int NT, int L, int MODE>
__global__ void __launch_bounds__(64 * NT) __attribute__((amdgpu_waves_per_eu(2)))
k_tanh_small(const float *__restrict__ P, int H, const float *x_in, int64_t n, int T, float eta,
           float *c_out, float *s_out, float *g_out, float *x_out) {
    __shared__ __attribute__((aligned(16))) TnSmallLds<DIM, NT, L> S;
    TnSmallRaw<DIM, NT, L, MODE != kEval> R;
    R.load(P, H);
    // every unit's W_0 and v, for the sums over all units
    const int lane = threadIdx.x & 63, u = 16 * (threadIdx.x >> 6) + 4 * (lane >> 4);
    if ((lane & 15) == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int j = 0; j < DIM; ++j) S.w0t[j][u + k] = R.w0[j][k];
            S.vo[u + k] = R.v[k];
        }
    }
    R.scheme(S.F);
    if (S.F.fwh)
        tn_small_body<DIM, NT, L, MODE, true>(S, R, x_in, n, T, eta, c_out, s_out, g_out, x_out);
    else
        tn_small_body<DIM, NT, L, MODE, false>(S, R, x_in, n, T, eta, c_out, s_out, g_out, x_out);
}

// Batches of at most this many points (a block of four waves per CU) take k_tanh_small, and
// morphs of twice as many where the steps outweigh the staging of W: at 8,192 points, 64 x 4
// units, a single gradient takes 27.5 us there against 21.5, each further step 3.2 against
// 8.0.
constexpr int64_t kTnSmallBatch = 4096;

template <int DIM, int NT, int L>
static void tn_launch(int mode, const pdmp_tanh_net &net, const float *x, int64_t n, int T,
                      float eta, float *c, float *s, float *g, float *xo, hipStream_t st) {
    const int64_t tiles = (n + kTnPts - 1) / kTnPts;
    if (n <= kTnSmallBatch || (mode == kMorph && T >= 4 && n <= 2 * kTnSmallBatch)) {
        const dim3 grid((unsigned)tiles), blk(64 * NT);
        if (mode == kEval)
            hipLaunchKernelGGL((k_tanh_small<DIM, NT, L, kEval>), grid, blk, 0, st, net.params,
                               net.hidden, x, n, T, eta, c, s, g, xo);
        else if (mode == kGrad)
            hipLaunchKernelGGL((k_tanh_small<DIM, NT, L, kGrad>), grid, blk, 0, st, net.params,
                               net.hidden, x, n, T, eta, c, s, g, xo);
        else
            hipLaunchKernelGGL((k_tanh_small<DIM, NT, L, kMorph>), grid, blk, 0, st, net.params,
                               net.hidden, x, n, T, eta, c, s, g, xo);
        return;
    }
    constexpr int wpb = kTnMorphBlock / 64;
    int64_t blocks = (tiles + wpb - 1) / wpb;
    if (blocks > 512) blocks = 512;
    const dim3 grid((unsigned)blocks), blk(kTnMorphBlock);
    if (mode == kEval)
        hipLaunchKernelGGL((k_tanh_net<DIM, NT, L, kEval>), grid, blk, 0, st, net.params,
                           net.hidden, x, n, T, eta, c, s, g, xo);
    else if (mode == kGrad)
        hipLaunchKernelGGL((k_tanh_net<DIM, NT, L, kGrad>), grid, blk, 0, st, net.params,
                           net.hidden, x, n, T, eta, c, s, g, xo);
    else
        hipLaunchKernelGGL((k_tanh_net<DIM, NT, L, kMorph>), grid, blk, 0, st, net.params,
                           net.hidden, x, n, T, eta, c, s, g, xo);
}

template <int DIM, int NT>
static void tn_by_depth(int mode, const pdmp_tanh_net &net, const float *x, int64_t n, int T,
                        float eta, float *c, float *s, float *g, float *xo, hipStream_t st) {
    switch (net.n_hidden) {
        case 1: tn_launch<DIM, NT, 1>(mode, net, x, n, T, eta, c, s, g, xo, st); break;
        case 2: tn_launch<DIM, NT, 2>(mode, net, x, n, T, eta, c, s, g, xo, st); break;
        case 3: tn_launch<DIM, NT, 3>(mode, net, x, n, T, eta, c, s, g, xo, st); break;
        default: tn_launch<DIM, NT, 4>(mode, net, x, n, T, eta, c, s, g, xo, st); break;
    }
}

// The caller has validated net (dim 2 or 3, 1 <= hidden <= 64, 1 <= n_hidden <= 4)
// and n >= 1.
int32_t launch_tanh_net(const pdmp_tanh_net &net, int mode, const float *x, int64_t n, int T,
                        float eta, float *c_out, float *s_out, float *g_out, float *x_out,
                        hipStream_t st) {
    const int h = net.hidden;
#define PDMP_TN(D)                                                                          \
    if (h <= 16) tn_by_depth<D, 1>(mode, net, x, n, T, eta, c_out, s_out, g_out, x_out, st); \
    else if (h <= 32) tn_by_depth<D, 2>(mode, net, x, n, T, eta, c_out, s_out, g_out, x_out, st); \
    else tn_by_depth<D, 4>(mode, net, x, n, T, eta, c_out, s_out, g_out, x_out, st)
    if (net.dim == 2) {
        PDMP_TN(2);
    } else {
        PDMP_TN(3);
    }
#undef PDMP_TN
    return check_launch("k_tanh_net");
}


// ------------------------------------------------------------------ fit ---
//
// BCE fit of the network (Sec. 3.1), full batch over n labelled points.  One step:
//   k_tanh_fit     per point: forward, r = (sigma(s) - y)/n, its part of the loss, the
//                  reverse pass e_L = r v (1 - a_L^2), e_l = (1 - a_l^2) W_l^T e_{l+1}, and the
//                  gradient dW_l = sum_i e_{l+1,i} [a_{l,i}; 1]^T of the block's points ->
//                  one partial row per block;
//   k_tanh_sum     fixed-order sum of the partial rows, + l2 w on the weight entries (not
//                  the biases), and the Adam step (fit) or the gradient alone; one more
//                  block adds the blocks' parts of the loss when it is asked for.
//
// k_tanh_fit: a block of four waves takes 64 points at a time (16 per wave), a layer's
// activations and reverse vectors stay in registers from the forward to the gradient.
// The hidden matrices lie in LDS once, row-major with rows of HP + 4 floats: the forward
// reads 16 bytes down a row per lane, the backward four rows of 16 neighbours, both
// clear of bank conflicts.  For dW_l the block's 64 points of e_{l+1} and a_l meet in LDS,
// and wave w multiplies rows 16w .. of it on FP32 MFMA (16 products of four points per
// tile, as the contraction is over the points); biases, W_0 and v take a multiply-add per
// lane and point instead, summed over the lanes at the end.  A batch of 10^4 points is
// 157 blocks of one wave per SIMD: latency binds it, 5 us of FP32 MFMA the largest part.  The
// first points, all weights and biases are requested before the first wait, and the sums of
// the per-lane gradients over the lanes halve the values held in each round (18.7 -> 16.2 us
// at 10^4 points, 64 x 3 units; 27 -> 18.4 at 16,384, where the loss's block past 256 others
// was a second round).  A step was 44.6 us as two kernels with the activations and vectors
// stored and read back in between and the loss and the sums in kernels of their own, now 22.

constexpr int kTnPtRow = 65;  // floats per unit of the 64 points in LDS (odd: no conflicts)

template <int DIM, int NT, int L>
struct TnFitLds {
    static constexpr int HP = 16 * NT, WS = HP + 4;
    float w[L > 1 ? L - 1 : 1][HP * WS];  // W_l, l = 1 .. L-1
    float w0t[DIM][HP];                   // W_0 transposed
    float bias[L][HP];
    float vo[HP];
    float bo;
    float xs[HP * kTnPtRow], ys[HP * kTnPtRow];  // e_{l+1} and a_l of the block's points
    float cross[4][(DIM + 1 + L) * HP + 1];      // per wave: sums of the per-lane gradients
    double rb[4];
};

// All loads unconditional (a padded entry reads entry 0) and out before the first wait.
// With sq, the thread's part of the weights' sum of squares (each weight in one thread).
template <int DIM, int NT, int L>
__device__ double tn_fit_stage(TnFitLds<DIM, NT, L> &S, const float *__restrict__ P, int H,
                               bool sq) {
    constexpr int HP = 16 * NT, WS = HP + 4, PER = HP * HP / kTnBlock, LH = L > 1 ? L - 1 : 1;
    static_assert(HP * HP % kTnBlock == 0, "whole batches");
    float v[LH][PER];
#pragma unroll
    for (int l = 1; l < L; ++l) {
        const float *W = P + tn_w_off(l, DIM, H);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = u * kTnBlock + threadIdx.x, row = e / HP, col = e % HP;
            v[l - 1][u] = W[row < H && col < H ? row * H + col : 0];
        }
    }
    const int idx = threadIdx.x % HP;
    const bool ok = idx < H, mine = (int)threadIdx.x < HP;
    float w0[DIM], bias[L];
#pragma unroll
    for (int k = 0; k < DIM; ++k) w0[k] = P[ok ? (int64_t)idx * DIM + k : 0];
#pragma unroll
    for (int l = 0; l < L; ++l)
        bias[l] = P[tn_w_off(l, DIM, H) + (int64_t)H * (l == 0 ? DIM : H) + (ok ? idx : 0)];
    const int64_t vo_off = tn_w_off(L, DIM, H);
    const float vo = P[vo_off + (ok ? idx : 0)], bo = P[vo_off + H];
#pragma unroll
    for (int l = 1; l < L; ++l)
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = u * kTnBlock + threadIdx.x, row = e / HP, col = e % HP;
            v[l - 1][u] = row < H && col < H ? v[l - 1][u] : 0.0f;
            S.w[l - 1][row * WS + col] = v[l - 1][u];
        }
    if (mine) {
#pragma unroll
        for (int k = 0; k < DIM; ++k) S.w0t[k][idx] = ok ? w0[k] : 0.0f;
#pragma unroll
        for (int l = 0; l < L; ++l) S.bias[l][idx] = ok ? bias[l] : 0.0f;
        S.vo[idx] = ok ? vo : 0.0f;
    }
    if (threadIdx.x == 0) S.bo = bo;
    double t = 0.0;
    if (sq) {
#pragma unroll
        for (int l = 1; l < L; ++l)
#pragma unroll
            for (int u = 0; u < PER; ++u) t = fma((double)v[l - 1][u], (double)v[l - 1][u], t);
        if (mine && ok) {
#pragma unroll
            for (int k = 0; k < DIM; ++k) t = fma((double)w0[k], (double)w0[k], t);
            t = fma((double)vo, (double)vo, t);
        }
    }
    return t;
}

// Sum over the 16 lanes of a row, the same value in each (DPP moves).
template <int CTRL>
__device__ __forceinline__ float tn_dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL,
                                                              0xf, 0xf, true));
}
__device__ __forceinline__ float tn_sum16(float v) {
    v += tn_dpp<0xB1>(v);
    v += tn_dpp<0x4E>(v);
    v += tn_dpp<0x141>(v);
    return v + tn_dpp<0x140>(v);
}

// The sums over the 16 lanes of a row of NV values (NV <= 16, a power of two), value k in the
// lanes c16 of c16 / (16 / NV) == k: each round halves the values a lane holds and doubles
// the lanes summed, 15 exchanges for 16 values where tn_sum16 of each takes 64.
template <int NV>
__device__ __forceinline__ float tn_scatter16(float (&w)[NV], int c16) {
    auto fold = [&](auto ctrl, int bit, int held) {
        constexpr int C = decltype(ctrl)::value;
        if (held < 2) {
            w[0] += tn_dpp<C>(w[0]);
            return;
        }
        const bool up = c16 & bit;
#pragma unroll
        for (int j = 0; j < NV / 2; ++j) {
            if (j >= held / 2) break;
            const float send = up ? w[j] : w[j + held / 2];
            w[j] = (up ? w[j + held / 2] : w[j]) + tn_dpp<C>(send);
        }
    };
    fold(std::integral_constant<int, 0x140>{}, 8, NV);      // row_mirror
    fold(std::integral_constant<int, 0x141>{}, 4, NV / 2);  // row_half_mirror
    fold(std::integral_constant<int, 0x4E>{}, 2, NV / 4);   // quad_perm [2,3,0,1]
    fold(std::integral_constant<int, 0xB1>{}, 1, NV / 8);   // quad_perm [1,0,3,2]
    return w[0];
}

// Index j of the flat parameters is a weight: in W_0, in the H x H part of a hidden layer,
// or in v.
__device__ __forceinline__ bool tn_is_weight(int64_t j, int dim, int H, int L) {
    const int64_t hl = (int64_t)H * H + H, k = j - ((int64_t)H * dim + H);
    if (k < 0) return j < (int64_t)H * dim;
    return k < (L - 1) * hl ? k % hl < (int64_t)H * H : k - (L - 1) * hl < H;
}

template <int DIM, int NT, int L>
__global__ void __launch_bounds__(kTnBlock)
k_tanh_fit(const float *__restrict__ P, int H, const float *__restrict__ x,
           const uint8_t *__restrict__ y, int64_t n, float inv_n, int64_t np, float half_l2,
           float *__restrict__ part, double *__restrict__ loss_part) {
    constexpr int HP = 16 * NT, WS = HP + 4;
    __shared__ __attribute__((aligned(16))) TnFitLds<DIM, NT, L> S;
    const int blocks = gridDim.x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, q = lane >> 4, c16 = lane & 15;
    const int u4 = 4 * q;
    // the next group's point of this lane, requested a group ahead (the first before W)
    float xn[DIM];
    bool yn;
    auto request = [&](int64_t g) {
        const int64_t i = g * 64 + wv * kTnPts + c16, ic = i < n ? i : n - 1;
#pragma unroll
        for (int k = 0; k < DIM; ++k) xn[k] = x[(size_t)k * n + ic];
        yn = i < n && y[ic];
    };
    request(blockIdx.x);
    // this thread's part of the block's share of the loss (1/n) sum BCE + (l2/2) |w|^2: the
    // second term in block 0, its points' BCE (lanes of q = 0) in order
    double bacc = 0.0, lacc = (double)half_l2 * tn_fit_stage<DIM, NT, L>(S, P, H,
                                                              loss_part && blockIdx.x == 0);
    __syncthreads();
    f32x4_tn acc[L > 1 ? L - 1 : 1][NT];      // dW_l, rows 16 wv .., tile columns
    f32x4_tn gb[L > 1 ? L - 1 : 1][NT];       // db_l of the lane's units, l >= 1
    f32x4_tn g0[DIM + 1][NT], gv[NT];         // dW_0 by input and db_0; dv
    float gr = 0.0f;                          // db_o
    const f32x4_tn zero = {};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        gv[t] = zero;
#pragma unroll
        for (int k = 0; k <= DIM; ++k) g0[k][t] = zero;
#pragma unroll
        for (int l = 1; l < L; ++l) acc[l - 1][t] = gb[l - 1][t] = zero;
    }
    const int64_t groups = (n + 63) / 64;
    for (int64_t g = blockIdx.x; g < groups; g += blocks) {
        const bool ok = g * 64 + wv * kTnPts + c16 < n;
        // opaque per group: keeps the weights' LDS reads inside the loop
        int cr = c16, ur = u4;
        asm volatile("" : "+v"(cr), "+v"(ur));
        float xv[DIM];
#pragma unroll
        for (int k = 0; k < DIM; ++k) xv[k] = xn[k];
        const bool yes = yn;
        request(g + blocks);
        f32x4_tn a[L][NT], d[L][NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int u0 = 16 * t + ur;
            const float4 bb = tn_ld4(&S.bias[0][u0]);
            float z[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
            for (int k = 0; k < DIM; ++k) {
                const float4 w = tn_ld4(&S.w0t[k][u0]);
                z[0] = fmaf(w.x, xv[k], z[0]);
                z[1] = fmaf(w.y, xv[k], z[1]);
                z[2] = fmaf(w.z, xv[k], z[2]);
                z[3] = fmaf(w.w, xv[k], z[3]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float av, dv;
                tanh_slope(z[v], av, dv);
                a[0][t][v] = av;
                d[0][t][v] = dv;
            }
        }
#pragma unroll
        for (int l = 1; l < L; ++l) {
            f32x4_tn z[NT];
#pragma unroll
            for (int to = 0; to < NT; ++to) {
                const float4 bb = tn_ld4(&S.bias[l][16 * to + ur]);
                z[to][0] = bb.x;
                z[to][1] = bb.y;
                z[to][2] = bb.z;
                z[to][3] = bb.w;
            }
            const float *W = S.w[l - 1] + cr * WS + ur;
#pragma unroll
            for (int ti = 0; ti < NT; ++ti) {
                float4 w[NT];
#pragma unroll
                for (int to = 0; to < NT; ++to) w[to] = tn_ld4(W + 16 * to * WS + 16 * ti);
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int to = 0; to < NT; ++to)
                        z[to] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            v == 0 ? w[to].x : (v == 1 ? w[to].y : (v == 2 ? w[to].z : w[to].w)),
                            a[l - 1][ti][v], z[to], 0, 0, 0);
            }
#pragma unroll
            for (int to = 0; to < NT; ++to)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float av, dv;
                    tanh_slope(z[to][v], av, dv);
                    a[l][to][v] = av;
                    d[l][to][v] = dv;
                }
        }
        float p = 0.0f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float4 vv = tn_ld4(&S.vo[16 * t + ur]);
            p = fmaf(vv.x, a[L - 1][t][0], p);
            p = fmaf(vv.y, a[L - 1][t][1], p);
            p = fmaf(vv.z, a[L - 1][t][2], p);
            p = fmaf(vv.w, a[L - 1][t][3], p);
        }
        const float s = tn_sum4(p) + S.bo;
        const float yv = yes ? 1.0f : 0.0f;
        // dBCE/ds = sigma(s) - y as sigma(s) (y = 0) or -sigma(-s) (y = 1): full relative
        // accuracy also where sigma(s) rounds to y; e1 = exp(-|s|)
        const float e1 = exp2_fast(-fabsf(s) * kLog2e);
        const float inv = 1.0f / (1.0f + e1);
        const float sig_pos = s >= 0.0f ? inv : e1 * inv, sig_neg = s >= 0.0f ? e1 * inv : inv;
        const float r = ok ? (yes ? -sig_neg : sig_pos) * inv_n : 0.0f;
        if (ok && q == 0 && loss_part) bacc += (double)(fmaxf(s, 0.0f) - yv * s + log1pf(e1));
        gr += q == 0 ? r : 0.0f;
        f32x4_tn e[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float4 vv = tn_ld4(&S.vo[16 * t + ur]);
            e[t][0] = r * vv.x * d[L - 1][t][0];
            e[t][1] = r * vv.y * d[L - 1][t][1];
            e[t][2] = r * vv.z * d[L - 1][t][2];
            e[t][3] = r * vv.w * d[L - 1][t][3];
#pragma unroll
            for (int v = 0; v < 4; ++v) gv[t][v] = fmaf(r, a[L - 1][t][v], gv[t][v]);
        }
#pragma unroll
        for (int l = L - 1; l >= 1; --l) {
            // e = e_{l+1}: its part of dW_l and db_l, then e_l
            __syncthreads();  // every wave is done with the previous layer's points
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int at = (16 * t + u4 + v) * kTnPtRow + wv * kTnPts + c16;
                    S.xs[at] = e[t][v];
                    S.ys[at] = a[l - 1][t][v];
                    gb[l - 1][t][v] += e[t][v];
                }
            __syncthreads();
            f32x4_tn G[NT];
            const float *W = S.w[l - 1] + ur * WS + cr;
#pragma unroll
            for (int to = 0; to < NT; ++to)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int ti = 0; ti < NT; ++ti)
                        G[ti] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            W[(16 * to + v) * WS + 16 * ti], e[to][v],
                            (to == 0 && v == 0) ? zero : G[ti], 0, 0, 0);
            if (wv < NT) {
                const float *X = S.xs + (16 * wv + c16) * kTnPtRow + 16 * q;
                const float *Y = S.ys + c16 * kTnPtRow + 16 * q;
#pragma unroll
                for (int m = 0; m < 16; ++m)
#pragma unroll
                    for (int co = 0; co < NT; ++co)
                        acc[l - 1][co] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            X[m], Y[16 * co * kTnPtRow + m], acc[l - 1][co], 0, 0, 0);
            }
#pragma unroll
            for (int ti = 0; ti < NT; ++ti)
#pragma unroll
                for (int v = 0; v < 4; ++v) e[ti][v] = G[ti][v] * d[l - 1][ti][v];
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int k = 0; k < DIM; ++k) g0[k][t][v] = fmaf(e[t][v], xv[k], g0[k][t][v]);
                g0[DIM][t][v] += e[t][v];
            }
    }

    float *out = part + (size_t)blockIdx.x * np;
    // dW_l: entry v of lane (c16, q) in a tile is (row 4q + v, column c16)
#pragma unroll
    for (int l = 1; l < L; ++l)
#pragma unroll
        for (int co = 0; co < NT; ++co)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int o = 16 * wv + u4 + v, c = 16 * co + c16;
                if (wv < NT && o < H && c < H) out[tn_w_off(l, DIM, H) + o * H + c] = acc[l - 1][co][v];
            }
    // the per-lane sums: over the 16 points of a wave, then the waves in order
    float *cr = S.cross[wv];
    auto put = [&](int set, const f32x4_tn(&val)[NT]) {
        constexpr int PER = 4 / NT;  // lanes that hold one sum
        float w[4 * NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) w[4 * t + v] = val[t][v];
        const float f = tn_scatter16<4 * NT>(w, c16);
        const int k = c16 / PER;
        if (c16 % PER == 0) cr[set * HP + 16 * (k >> 2) + u4 + (k & 3)] = f;
    };
#pragma unroll
    for (int k = 0; k <= DIM; ++k) put(k, g0[k]);
#pragma unroll
    for (int l = 1; l < L; ++l) put(DIM + l, gb[l - 1]);
    put(DIM + L, gv);
    gr = tn_sum16(gr);  // lanes of q = 0
    if (lane == 0) cr[(DIM + 1 + L) * HP] = gr;
    if (loss_part) {
        lacc += bacc / (double)n;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) lacc += __shfl_xor(lacc, off, 64);
        if (lane == 0) S.rb[wv] = lacc;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < (DIM + 1 + L) * HP + 1; e += kTnBlock) {
        const float t = ((S.cross[0][e] + S.cross[1][e]) + S.cross[2][e]) + S.cross[3][e];
        const int set = e / HP, u = e % HP;
        if (e == (DIM + 1 + L) * HP) out[tn_w_off(L, DIM, H) + H] = t;  // b_o
        else if (u >= H) continue;
        else if (set < DIM) out[u * DIM + set] = t;                      // W_0
        else if (set < DIM + L) {                                        // b_l, l = set - DIM
            const int l = set - DIM;
            out[tn_w_off(l, DIM, H) + (int64_t)H * (l == 0 ? DIM : H) + u] = t;
        } else out[tn_w_off(L, DIM, H) + u] = t;                         // v
    }
    if (loss_part && threadIdx.x == 0)
        loss_part[blockIdx.x] = ((S.rb[0] + S.rb[1]) + S.rb[2]) + S.rb[3];
}

static size_t al256t(size_t b) { return (b + 255) & ~(size_t)255; }

// Blocks of k_tanh_fit (and partial rows) for n points: 64 points each, at most one block per
// CU, which then takes several groups.
static int tn_fit_blocks(int64_t n) {
    const int64_t g = (n + 63) / 64;
    return (int)(g < 256 ? g : 256);
}

static int64_t tn_nparams(const pdmp_tanh_net &net) {
    const int64_t H = net.hidden, L = net.n_hidden;
    return H * net.dim + H + (L - 1) * (H * H + H) + H + 1;
}

size_t tanh_fit_ws_bytes(const pdmp_tanh_net &net, int64_t n) {
    const int64_t np = tn_nparams(net);
    return al256t((size_t)tn_fit_blocks(n) * np * 4) + al256t((size_t)np * 4) + al256t(256 * 8);
}

template <int DIM, int NT, int L>
static void tn_fit_launch(const pdmp_tanh_net &net, const float *x, const uint8_t *y, int64_t n,
                          float l2, float *part, double *loss, hipStream_t st) {
    hipLaunchKernelGGL((k_tanh_fit<DIM, NT, L>), dim3((unsigned)tn_fit_blocks(n)), dim3(kTnBlock), 0,
                       st, net.params, net.hidden, x, y, n, (float)(1.0 / (double)n),
                       tn_nparams(net), 0.5f * l2, part, loss);
}

template <int DIM, int NT>
static void tn_fit_depth(const pdmp_tanh_net &net, const float *x, const uint8_t *y, int64_t n,
                         float l2, float *part, double *loss, hipStream_t st) {
    switch (net.n_hidden) {
        case 1: tn_fit_launch<DIM, NT, 1>(net, x, y, n, l2, part, loss, st); break;
        case 2: tn_fit_launch<DIM, NT, 2>(net, x, y, n, l2, part, loss, st); break;
        case 3: tn_fit_launch<DIM, NT, 3>(net, x, y, n, l2, part, loss, st); break;
        default: tn_fit_launch<DIM, NT, 4>(net, x, y, n, l2, part, loss, st); break;
    }
}

// One Adam step's state and coefficients (bc1 = 1/(1 - beta1^t), bc2 = 1/(1 - beta2^t));
// m == nullptr: no update.
struct TnAdam {
    float *m, *v;
    float lr, b1, b2, eps, bc1, bc2;
};

// grad[j] = sum_{r < rows} part[r np + j] (sixteen phases summing the rows r = ph mod 16 in
// increasing order, four loads at a time, the phases added in order) + l2 w on the weight
// entries, then the Adam step of parameter j on it (the update of k_adam).  With loss, one
// block past those of the parameters adds the blocks' shares of it (from k_tanh_fit).
constexpr int kTnSumPh = 16;
__global__ void __launch_bounds__(64 * kTnSumPh)
k_tanh_sum(const float *__restrict__ part, int rows, int64_t np, int dim, int H, int L, float l2,
           float *__restrict__ grad, float *__restrict__ P, TnAdam ad,
           const double *__restrict__ loss_part, float *__restrict__ loss) {
    __shared__ double sh[kTnSumPh][64];
    const int cl = threadIdx.x & 63, ph = threadIdx.x >> 6;
    const int64_t j = (int64_t)blockIdx.x * 64 + cl;
    if ((int64_t)blockIdx.x * 64 >= np) {  // the loss block
        if (ph != 0) return;
        double t = 0.0;
        for (int i = cl; i < rows; i += 64) t += loss_part[i];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
        if (cl == 0) *loss = (float)t;
        return;
    }
    double acc = 0.0;
    if (j < np) {
        int r = ph;
        for (; r + 3 * kTnSumPh < rows; r += 4 * kTnSumPh) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = part[(size_t)(r + u * kTnSumPh) * np + j];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc += v[u];
        }
        for (; r < rows; r += kTnSumPh) acc += part[(size_t)r * np + j];
    }
    sh[ph][cl] = acc;
    __syncthreads();
    if (ph != 0 || j >= np) return;
    double t = sh[0][cl];
#pragma unroll
    for (int q = 1; q < kTnSumPh; ++q) t += sh[q][cl];
    const float w = P[j];
    float gk = (float)t;
    if (tn_is_weight(j, dim, H, L)) gk = fmaf(l2, w, gk);
    grad[j] = gk;
    if (!ad.m) return;
    const float mk = ad.b1 * ad.m[j] + (1.0f - ad.b1) * gk;
    const float vk = ad.b2 * ad.v[j] + (1.0f - ad.b2) * gk * gk;
    ad.m[j] = mk;
    ad.v[j] = vk;
    const float mh = mk * ad.bc1, vh = vk * ad.bc2;
    P[j] = w - ad.lr * mh / (sqrtf(vh) + ad.eps);
}

// Loss (nullable, device [1]) and gradient (device [np]) of the fit objective at the
// current parameters, and with ad.m the Adam step on that gradient in the same pass
// over it.  `ws` holds tanh_fit_ws_bytes(net, n) bytes.
static int32_t tanh_loss_grad_step(const pdmp_tanh_net &net, const float *x, const uint8_t *y,
                                   int64_t n, float l2, float *loss, float *grad, void *ws,
                                   const TnAdam &ad, hipStream_t st) {
    const int dim = net.dim, H = net.hidden, L = net.n_hidden, rows = tn_fit_blocks(n);
    const int64_t np = tn_nparams(net);
    char *p = (char *)ws;
    float *part = (float *)p;
    p += al256t((size_t)rows * np * 4) + al256t((size_t)np * 4);
    double *loss_part = loss ? (double *)p : nullptr;  // per k_tanh_fit block

#define PDMP_TNFIT(D)                                                        \
    if (H <= 16) tn_fit_depth<D, 1>(net, x, y, n, l2, part, loss_part, st);       \
    else if (H <= 32) tn_fit_depth<D, 2>(net, x, y, n, l2, part, loss_part, st);  \
    else tn_fit_depth<D, 4>(net, x, y, n, l2, part, loss_part, st)
    if (dim == 2) {
        PDMP_TNFIT(2);
    } else {
        PDMP_TNFIT(3);
    }
#undef PDMP_TNFIT
    if (int32_t e = check_launch("k_tanh_fit")) return e;
    hipLaunchKernelGGL(k_tanh_sum, dim3((unsigned)((np + 63) / 64 + (loss ? 1 : 0))),
                       dim3(64 * kTnSumPh), 0, st, part, rows, np, dim, H, L, l2, grad,
                       const_cast<float *>(net.params), ad, loss_part, loss);
    return check_launch("k_tanh_sum");
}

int32_t launch_tanh_loss_grad(const pdmp_tanh_net &net, const float *x, const uint8_t *y,
                              int64_t n, float l2, float *loss, float *grad, void *ws,
                              hipStream_t st) {
    return tanh_loss_grad_step(net, x, y, n, l2, loss, grad, ws, TnAdam{}, st);
}

// `steps` full-batch Adam steps on the fit objective; the parameters (net.params)
// are updated in place, m and v are the Adam state, the step counter continues from t0.
int32_t launch_tanh_fit(const pdmp_tanh_net &net, const float *x, const uint8_t *y, int64_t n,
                        int steps, float lr, float l2, float b1, float b2, float eps, float *m,
                        float *v, int t0, float *loss_out, void *ws, hipStream_t st) {
    float *grad = (float *)((char *)ws + al256t((size_t)tn_fit_blocks(n) * tn_nparams(net) * 4));
    for (int t = 0; t < steps; ++t) {
        const int tt1 = t0 + t + 1;
        TnAdam ad;
        ad.m = m;
        ad.v = v;
        ad.lr = lr;
        ad.b1 = b1;
        ad.b2 = b2;
        ad.eps = eps;
        ad.bc1 = (float)(1.0 / (1.0 - std::pow((double)b1, (double)tt1)));
        ad.bc2 = (float)(1.0 / (1.0 - std::pow((double)b2, (double)tt1)));
        if (int32_t e = tanh_loss_grad_step(net, x, y, n, l2, loss_out ? loss_out + t : nullptr,
                                            grad, ws, ad, st))
            return e;
    }
    return PDMP_OK;
}
}  // namespace pdmp
