// grid3d.hip -- occupancy, joint-space morph and body-point check for hinges on a
// regular 3-D grid of up to 16 points per axis, as dense contractions on the matrix
// cores (FP16 or BF16 MFMA at FP32 accuracy, mfma_split.h).
//
// With hinges h_{a + G0 (b + G1 c)} = (X_a, Y_b, Z_c), carried padded to G0 = G1 = 16, the feature factorises,
// phi = ex_a ey_b ez_c, so with rows r = b + 16 c of W[r][a] = w_{a + G0 (b + G1 c)}
//   U_r = sum_a W[r][a] ex_a,   V_r = sum_a W[r][a] ex_a (x - X_a)        (MFMA)
//   s        = sum_c ez_c sum_b ey_b U_r + beta
//   ds/dx    = -(1/l^2) sum_c ez_c sum_b ey_b V_r
//   ds/dy    = -(1/l^2) sum_c ez_c sum_b ey_b (y - Y_b) U_r
//   ds/dz    = -(1/l^2) sum_c ez_c (z - Z_c) sum_b ey_b U_r
// the same s and grad s as the pairwise sum (rounding aside) for G0 + 16 + G2
// exponentials and two (16 G2) x G0 matrix-vector products per point.  32 points
// per wave go through the 32x32x16 MFMAs (A = W rows, B = [ex | ex dx] of the lane's
// own point, k = a, G0 = 16 in one k-step; two-part FP16 splits of both and three
// products per contraction, or three-way bf16 splits and six products when the
// operands' range needs FP32's exponent range; on grids below 16^3 with weights that no
// split carries, the pairwise sum in the same kernels); each 32-row tile holds two z-planes
// (c = 2t, 2t+1), so in the accumulator layout lane l owns the fixed y indices
// b = (8(v/4) + 4(l/32) + v%4) mod 16 and the y/z contractions need only per-lane
// tables of ey and ez.  The U terms are summed over z first (per y slot, the plane sums
// with ez and with ez (z - Z_c), then one y contraction after the tiles: 2 instead of 3
// multiply-adds per accumulator value and none per plane), the V term over y first.
// The two lanes of a point are summed by one xor-32 exchange (bit-identical).
//
// Arm mapping: a wave carries 4 configurations x 8 body points of one link at a
// time (lane = 8*config + point, mirrored in the upper 32 lanes), walks the links
// from the tip down, and keeps only the running suffix sums of the Eq. 3 pull-back.
#include <type_traits>

#include "mfma_split.h"
#include "pdmp_common.h"

namespace pdmp {

constexpr int kG3Block = 256;

// The x contraction runs on one of two split schemes (mfma_split.h): two-part FP16
// splits with three products where the operands' range allows, three-part BF16
// splits with six products otherwise.  The workspace morph and both arm kernels
// (morph and body-point check, each block running 7 links per configuration) test
// the range; a single workspace evaluation, whose blocks mostly stage W, skips the
// test and keeps the BF16 scheme.
static_assert(kG3Block == 64 * kSplitWaves, "the scheme test's block");

// Axis sizes of the launch's grid, each at most 16.  FULL: all three are 16 (compile-time
// sizes, every tile loop unrolled).  Otherwise the grid is carried padded to 16 x 16 x
// 2 ceil(G2 / 2): the padding's weights are zero and its axis coordinates repeat the last
// hinge's, so every padded operand is finite wherever the real ones are and adds exact
// zeros; only the ceil(G2 / 2) tiles that hold a real plane are walked.
//
// A padded grid has the choice between the contraction and the pairwise FP32 sum, so the
// contraction keeps to that sum's accuracy and range (errors below: root mean square over
// the absolute sums against 64 bits, a ratio to the pairwise kernel's):
//   * ex = exp2(-dx^2) is rounded as there and scaled by 2^c afterwards (ldexp).  The FULL
//     kernels add c to the exponent's argument, one instruction fewer per value; that sum's
//     rounding, 2^-21 of ex at c = 15, makes a gradient's error 1.06 to 1.6 times the
//     pairwise one (15^3 to 6^3 hinges), the separate scaling 0.83 to 1.12.
//   * Grids of at most kG3Fine per axis have too few terms for the two-part splits' rounding
//     to average out (1.12 at 6^3, 1.05 at 7^3, 0.98 at 8^3 and above): the FP16 scheme
//     takes three parts and six products there (0.97 and below).
//   * Up to kG3Tiny per axis the logit is off by up to 1.08 on any split, three
//     exponentials to one: single evaluations and the body-point check stay pairwise (the
//     gradient, 1.00 and below, does not).
//   * The BF16 scheme scales ex by 2^kG3Bf16Scale, so that the third part of the smallest
//     normal feature (2^-126) keeps all its bits.
//   * Weights that are not finite, or on the BF16 scheme outside [2^-100, 2^80), take the
//     pairwise sum in the kernel (kG3Direct).
enum G3Scheme { kG3Bf16 = 0, kG3Fp16 = 1, kG3Direct = 2, kG3Fp16Fine = 3 };  // SplitScheme::fp16
constexpr int kG3Fine = 7, kG3Tiny = 5;
constexpr int kG3Bf16Scale = 24;
constexpr uint32_t kG3Bf16Bottom = (127u - 100) << 23, kG3Bf16Top = (127u + 80) << 23;
struct G3Dims {
    int g0, g1, g2;
};
__host__ __device__ inline bool g3_within(const G3Dims &g, int most) {
    return g.g0 <= most && g.g1 <= most && g.g2 <= most;
}
// The grid as the evaluations see it: its axis sizes and its weights in memory.
struct G3Grid : G3Dims {
    const float *weights;
};

constexpr int kG3Tiles = 8;                    // 32-row tiles: 16 planes of 16 rows
constexpr int kG3Frag = 3 * kG3Tiles * 64;     // 16-byte fragments: up to 3 parts x tiles
constexpr int kG3Max = 16;

template <bool FULL>
__device__ __forceinline__ int g3_tiles(const G3Dims &g) {
    return FULL ? kG3Tiles : (g.g2 + 1) / 2;
}

// Weight W[r][a], r = b + 16 c, of the padded grid (0 in the padding).  The load itself is
// unconditional (entry 0 in the padding), so a thread's loads go out together.
template <bool FULL>
__device__ __forceinline__ float g3_weight(const float *__restrict__ weights, const G3Dims &g,
                                           int r, int a) {
    if (FULL) return weights[a + 16 * r];
    const int b = r & 15, c = r >> 4;
    const bool in = a < g.g0 && b < g.g1 && c < g.g2;
    const float w = weights[in ? a + g.g0 * (b + g.g1 * c) : 0];
    return in ? w : 0.0f;
}

template <bool FULL>
__device__ __forceinline__ void g3_axes(float *ax, float *ay, float *az,
                                        const float *__restrict__ hinges, const G3Dims &g,
                                        float kappa) {
    const int g0 = FULL ? 16 : g.g0, g1 = FULL ? 16 : g.g1, g2 = FULL ? 16 : g.g2;
    const int M = g0 * g1 * g2;
    if (threadIdx.x >= kG3Max) return;
    const int i = threadIdx.x;
    ax[i] = kappa * hinges[min(i, g0 - 1)];
    ay[i] = kappa * hinges[M + g0 * min(i, g1 - 1)];
    az[i] = kappa * hinges[2 * M + g0 * g1 * min(i, g2 - 1)];
}

// The third FP16 part of v from its first two (split2h).
__device__ __forceinline__ f16x8_t third_h(const float (&v)[8], const f16x8_t &p1,
                                           const f16x8_t &p2) {
    f16x8_t p3;
#pragma unroll
    for (int j = 0; j < 8; ++j) p3[j] = (_Float16)((v[j] - (float)p1[j]) - (float)p2[j]);
    return p3;
}

// acc += (a1 + a2 + a3)(b1 + b2 + b3) less the terms past the third order.
__device__ __forceinline__ f32x16_t mfma_h6(const f16x8_t &a1, const f16x8_t &a2, const f16x8_t &a3,
                                            const f16x8_t &b1, const f16x8_t &b2, const f16x8_t &b3,
                                            f32x16_t acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a3, b1, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, b2, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b3, acc, 0, 0, 0);
    return mfma_h3(a1, a2, b1, b2, acc);
}

// Stage W fragments (frag[(p*8 + t)*64 + lane] = part p of W[32t + lane%32][8(lane/32)
// + j], j < 8: three bf16 parts, or two FP16 parts of 2^sw W) and the prescaled axes
// into LDS, choosing the scheme when allow16 (else the BF16 parts, without the check when
// FULL).  All threads of the block of NW waves call it; the caller synchronises before
// reading the fragments.
template <bool FULL, int NW>
__device__ __forceinline__ SplitScheme g3_stage(uint4 *fraw, float *ax, float *ay, float *az,
                                             SplitRangeN<NW> &rg, const float *__restrict__ hinges,
                                             const float *__restrict__ weights, const G3Dims &g,
                                             float kappa, bool allow16) {
    constexpr int BT = 64 * NW;
    const int nf = 64 * g3_tiles<FULL>(g);
    if (!allow16) {
        // BF16 parts straight from global memory; a padded grid's weights are tested on the way
        bf16x8_t *frag = reinterpret_cast<bf16x8_t *>(fraw);
        bool out = false;
        for (int idx = threadIdx.x; idx < nf; idx += BT) {
            const int ln = idx & 63, t = idx >> 6;
            const int r = 32 * t + (ln & 31);
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = g3_weight<FULL>(weights, g, r, 8 * (ln >> 5) + j);
            bf16x8_t p1, p2, p3;
            split3(v, p1, p2, p3);
            frag[(0 * kG3Tiles + t) * 64 + ln] = p1;
            frag[(1 * kG3Tiles + t) * 64 + ln] = p2;
            frag[(2 * kG3Tiles + t) * 64 + ln] = p3;
            if (!FULL) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t u = __float_as_uint(v[j]) & 0x7fffffffu;
                    out = out || u >= kG3Bf16Top || (u != 0 && u < kG3Bf16Bottom);
                }
            }
        }
        g3_axes<FULL>(ax, ay, az, hinges, g, kappa);
        return SplitScheme{!FULL && __syncthreads_or(out) ? kG3Direct : kG3Bf16, 0, 0.0f, 0.0f};
    }
    constexpr int NI = (kG3Tiles * 64 + BT - 1) / BT;
    const float axis = split_axis(hinges, FULL ? 16 : g.g0, kappa);
    float w8[NI][8];
    uint32_t mx = 0, mn = 0xffffffffu;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int idx = threadIdx.x + it * BT;
        const int ln = idx & 63, r = 32 * (idx >> 6) + (ln & 31);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float w = idx < kG3Tiles * 64 ? g3_weight<FULL>(weights, g, r, 8 * (ln >> 5) + j)
                                                : 0.0f;
            w8[it][j] = w;
            const uint32_t u = __float_as_uint(w) & 0x7fffffffu;
            mx = max(mx, u);
            if (u != 0) mn = min(mn, u);
        }
    }
    g3_axes<FULL>(ax, ay, az, hinges, g, kappa);
    SplitScheme sc = split_decide(mx, mn, axis, FULL ? 16 : g.g0, rg);
    if (!FULL) {
        if (sc.fp16 && g3_within(g, kG3Fine)) sc.fp16 = kG3Fp16Fine;
        if (sc.fp16 == kG3Bf16) {
            bool ok = true;
#pragma unroll
            for (int w = 0; w < NW; ++w)
                ok = ok && rg.wmax[w] < kG3Bf16Top && rg.wmin[w] >= kG3Bf16Bottom;
            sc.fp16 = __builtin_amdgcn_readfirstlane(ok ? kG3Bf16 : kG3Direct);
            sc.sw = 0;
        }
    }
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int idx = threadIdx.x + it * BT;
        if (idx >= nf || sc.fp16 == kG3Direct) break;
        const int ln = idx & 63, t = idx >> 6;
        if (sc.fp16) {
            f16x8_t *frag = reinterpret_cast<f16x8_t *>(fraw);
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = ldexpf(w8[it][j], sc.sw);
            f16x8_t p1, p2;
            split2h(v, p1, p2);
            frag[(0 * kG3Tiles + t) * 64 + ln] = p1;
            frag[(1 * kG3Tiles + t) * 64 + ln] = p2;
            if (!FULL && sc.fp16 == kG3Fp16Fine) frag[(2 * kG3Tiles + t) * 64 + ln] = third_h(v, p1, p2);
        } else {
            bf16x8_t *frag = reinterpret_cast<bf16x8_t *>(fraw);
            bf16x8_t p1, p2, p3;
            split3(w8[it], p1, p2, p3);
            frag[(0 * kG3Tiles + t) * 64 + ln] = p1;
            frag[(1 * kG3Tiles + t) * 64 + ln] = p2;
            frag[(2 * kG3Tiles + t) * 64 + ln] = p3;
        }
    }
    return sc;
}

// The pairwise sums, over the hinges themselves (the lane and its xor-32 partner take every
// other one of a row along x).
template <bool GRAD>
__device__ __forceinline__ void g3_direct(const G3Grid &gr, int pair, const float *ax,
                                          const float *ay, const float *az, float xs, float ys,
                                          float zs, float &s, float &sx, float &sy, float &sz) {
    s = sx = sy = sz = 0.0f;
    for (int r = 0; r < gr.g1 * gr.g2; ++r) {
        const float dy = ys - ay[r % gr.g1], dz = zs - az[r / gr.g1];
        for (int a = (threadIdx.x & 63) >> 5; a < gr.g0; a += 2) {
            const float dx = xs - ax[a];
            const float e = exp2_fast(-fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
            const float wp = gr.weights[a + gr.g0 * r] * e;
            s += wp;
            if (GRAD) {
                sx = fmaf(wp, dx, sx);
                sy = fmaf(wp, dy, sy);
                sz = fmaf(wp, dz, sz);
            }
        }
    }
    s = pair_sum(s, pair);
    if (GRAD) {
        sx = pair_sum(sx, pair);
        sy = pair_sum(sy, pair);
        sz = pair_sum(sz, pair);
    }
}

// s (without beta) and, with GRAD, the unscaled logit-gradient sums (sx, sy, sz) at the
// prescaled point (xs, ys, zs) this lane shares with its xor-32 partner, on the
// block's scheme (SCH = sc.fp16), over the grid's tiles (8 when FULL).
template <bool FULL, bool GRAD, int SCH>
__device__ __forceinline__ void g3_point(const uint4 *fraw, const SplitScheme &sc, const G3Grid &gr,
                                         int pair, const float *ax, const float *ay,
                                         const float *az, float xs, float ys, float zs, float &s,
                                         float &sx, float &sy, float &sz) {
    static_assert(!FULL || SCH == kG3Bf16 || SCH == kG3Fp16, "padded grids only");
    if constexpr (SCH == kG3Direct) {
        g3_direct<GRAD>(gr, pair, ax, ay, az, xs, ys, zs, s, sx, sy, sz);
        return;
    }
    constexpr bool FINE = SCH == kG3Fp16Fine, F16 = SCH == kG3Fp16 || FINE;
    const int nt = g3_tiles<FULL>(gr);
    const int lane0 = threadIdx.x & 63, h = lane0 >> 5;
    // The weight fragments are the same at every call; an opaque copy of the lane
    // index keeps the compiler from hoisting their LDS reads out of the callers'
    // loops into registers.
    int lane = lane0;
    asm volatile("" : "+v"(lane));
    bf16x8_t e1, e2, e3, d1, d2, d3;
    f16x8_t h1, h2, h3, k1, k2, k3;
    int c = 0;  // this point's operand scale 2^c (FP16 scheme, padded grids)
    {
        float cf = 0.0f;
        if (F16) {
            c = split_scale_exp(xs, sc.gmin, sc.gmax);
            cf = (float)c;
        } else if (!FULL) {
            c = kG3Bf16Scale;
        }
        float e[8], de[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float d = xs - ax[8 * h + j];
            if (FULL) e[j] = exp2_fast(F16 ? fmaf(-d, d, cf) : -d * d);
            else e[j] = ldexpf(exp2_fast(-d * d), c);
            de[j] = e[j] * d;
        }
        if (F16) {
            split2h(e, h1, h2);
            if (GRAD) split2h(de, k1, k2);
            if (FINE) h3 = third_h(e, h1, h2);
            if (FINE && GRAD) k3 = third_h(de, k1, k2);
        } else {
            split3(e, e1, e2, e3);
            if (GRAD) split3(de, d1, d2, d3);
        }
    }
    // ey of the lane's 8 distinct y indices; the U terms z first (per y slot u the
    // plane sums q_u = sum_c ez_c U_(u,c) and qz_u with dez_c, contracted with ey and
    // ey dy after the tiles), the V term y first per plane
    float ey[8], q[8], qz[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int b = 8 * (u >> 2) + 4 * h + (u & 3);
        const float d = ys - ay[b];
        ey[u] = exp2_fast(-d * d);
        q[u] = qz[u] = 0.0f;
    }
    sx = 0.0f;
    constexpr int UN = FULL ? kG3Tiles : 1;
#pragma unroll UN
    for (int t = 0; t < (FULL ? kG3Tiles : nt); ++t) {
        // the two z-planes of this tile
        float ez[2], dez[2];
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
            const float d = zs - az[2 * t + cc];
            ez[cc] = exp2_fast(-d * d);
            dez[cc] = ez[cc] * d;
        }
        // one k-step (the padded x axis) from the zero accumulator
        const f32x16_t zero = {};
        f32x16_t U, V;
        if (F16) {
            const f16x8_t *frag = reinterpret_cast<const f16x8_t *>(fraw);
            const f16x8_t a1 = frag[(0 * kG3Tiles + t) * 64 + lane];
            const f16x8_t a2 = frag[(1 * kG3Tiles + t) * 64 + lane];
            if (FINE) {
                const f16x8_t a3 = frag[(2 * kG3Tiles + t) * 64 + lane];
                U = mfma_h6(a1, a2, a3, h1, h2, h3, zero);
                if (GRAD) V = mfma_h6(a1, a2, a3, k1, k2, k3, zero);
            } else {
                U = mfma_h3(a1, a2, h1, h2, zero);
                if (GRAD) V = mfma_h3(a1, a2, k1, k2, zero);
            }
        } else {
            const bf16x8_t *frag = reinterpret_cast<const bf16x8_t *>(fraw);
            const bf16x8_t a1 = frag[(0 * kG3Tiles + t) * 64 + lane];
            const bf16x8_t a2 = frag[(1 * kG3Tiles + t) * 64 + lane];
            const bf16x8_t a3 = frag[(2 * kG3Tiles + t) * 64 + lane];
            U = mfma_x6(a1, a2, a3, e1, e2, e3, zero);
            if (GRAD) V = mfma_x6(a1, a2, a3, d1, d2, d3, zero);
        }
        // row i = 8(v/4) + 4h + v%4 of tile t: b = i mod 16 (y slot v%8), c = 2t + v/8,
        // so U[u] and U[u + 8] share slot u on the tile's two planes
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            q[u] = fmaf(ez[1], U[u + 8], fmaf(ez[0], U[u], q[u]));
            if (GRAD) qz[u] = fmaf(dez[1], U[u + 8], fmaf(dez[0], U[u], qz[u]));
        }
        if (GRAD) {
#pragma unroll
            for (int cz = 0; cz < 2; ++cz) {
                float pyx = 0.0f;
#pragma unroll
                for (int u = 0; u < 8; ++u) pyx = fmaf(ey[u], V[8 * cz + u], pyx);
                sx = fmaf(ez[cz], pyx, sx);
            }
        }
    }
    s = sy = sz = 0.0f;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        s = fmaf(ey[u], q[u], s);
        if (GRAD) {
            const int b = 8 * (u >> 2) + 4 * h + (u & 3);
            sy = fmaf(ey[u] * (ys - ay[b]), q[u], sy);
            sz = fmaf(ey[u], qz[u], sz);
        }
    }
    s = pair_sum(s, pair);
    if (GRAD) {
        sx = pair_sum(sx, pair);
        sy = pair_sum(sy, pair);
        sz = pair_sum(sz, pair);
    }
    if (F16 || !FULL) {
        const int un = -(sc.sw + c);
        s = ldexpf(s, un);
        if (GRAD) {
            sx = ldexpf(sx, un);
            sy = ldexpf(sy, un);
            sz = ldexpf(sz, un);
        }
    }
}

// f with the block's scheme as a compile-time constant.
template <bool FULL, bool ALLOW16, class F>
__device__ __forceinline__ void g3_by_scheme(int scheme, F &&f) {
    if (ALLOW16 && scheme == kG3Fp16) {
        f(std::integral_constant<int, kG3Fp16>{});
    } else if (FULL || scheme == kG3Bf16) {
        f(std::integral_constant<int, kG3Bf16>{});
    } else if constexpr (!FULL) {
        if (ALLOW16 && scheme == kG3Fp16Fine) f(std::integral_constant<int, kG3Fp16Fine>{});
        else f(std::integral_constant<int, kG3Direct>{});
    }
}

// ---- workspace points [3][n]: eval / grad / morph, 32 points per wave ----
template <bool FULL, int MODE, int SCH>
__device__ __forceinline__ void g3_ws_body(const uint4 *fraw, const SplitScheme &sc, const G3Grid &gr, const float *ax,
                                           const float *ay, const float *az, float beta,
                                           float kappa, float gscale, const float *x_in,
                                           int64_t n, int T, float eta, float *c_out,
                                           float *s_out, float *g_out, float *x_out,
                                           const Traj &tr, int nb) {
    const int lane = threadIdx.x & 63, pair = pair_address();
    const int64_t stride = (int64_t)nb * 128;
    int64_t i = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32 + (lane & 31);
    const int64_t base = i - (lane & 31);  // the wave's first point
    auto load = [&](int64_t at, float &px, float &py, float &pz) {
        const int64_t ic = at < n ? at : n - 1;
        px = x_in[ic], py = x_in[(size_t)n + ic], pz = x_in[2 * (size_t)n + ic];
    };
    float x, y, z;
    load(i, x, y, z);
    if (MODE != kMorph) {
        // a block walks its points 128 x nb at a time, the next ones requested ahead
        for (int64_t b = base; b < n; b += stride, i += stride) {
            float nx, ny, nz;
            load(i + stride, nx, ny, nz);
            float s, sx, sy, sz, c, sp;
            g3_point<FULL, MODE != kEval, SCH>(fraw, sc, gr, pair, ax, ay, az, kappa * x, kappa * y,
                                               kappa * z, s, sx, sy, sz);
            x = nx, y = ny, z = nz;
            if ((lane >> 5) != 0 || i >= n) continue;
            sigmoid_and_slope(s + beta, c, sp);
            if (c_out) c_out[i] = c;
            if (MODE == kEval) {
                if (s_out) s_out[i] = s + beta;
            } else {
                const float f = -sp * gscale;
                g_out[i] = f * sx;
                g_out[(size_t)n + i] = f * sy;
                g_out[2 * (size_t)n + i] = f * sz;
            }
        }
        return;
    }
    float s, sx, sy, sz;
    int64_t tc;
    const bool rec = (lane >> 5) == 0 && traj_col(tr, i, n, tc);
    for (int st = 0; st < T; ++st) {
        if (rec) traj_put<3>(tr, st, tc, {x, y, z});
        g3_point<FULL, true, SCH>(fraw, sc, gr, pair, ax, ay, az, kappa * x, kappa * y, kappa * z, s, sx,
                                  sy, sz);
        float c, sp;
        sigmoid_and_slope(s + beta, c, sp);
        const float step = eta * sp * gscale;
        x = fmaf(step, sx, x);
        y = fmaf(step, sy, y);
        z = fmaf(step, sz, z);
    }
    if (rec) traj_put<3>(tr, T, tc, {x, y, z});
    if ((lane >> 5) != 0 || i >= n) return;
    x_out[i] = x;
    x_out[(size_t)n + i] = y;
    x_out[2 * (size_t)n + i] = z;
}

template <bool FULL, int MODE>
__global__ void __launch_bounds__(kG3Block)
__attribute__((amdgpu_waves_per_eu(MODE == kMorph ? 3 : 1)))
k_grid3d_ws(const float *__restrict__ hinges, const float *__restrict__ weights, G3Dims g,
            float kappa, float gscale, const float *x_in, int64_t n, int T, float eta, float *c_out,
            float *s_out, float *g_out, float *x_out, Traj tr, GridCheck gc) {
    __shared__ uint4 fraw[kG3Frag];
    __shared__ float ax[kG3Max], ay[kG3Max], az[kG3Max];
    __shared__ SplitRange rg;
    if ((int)blockIdx.x >= gc.nb) {
        grid_check_part(hinges, 3, g.g0 * g.g1 * g.g2, g.g0, g.g1, gc.word, blockIdx.x - gc.nb,
                        gridDim.x - gc.nb);
        return;
    }
    // the range check pays off over a morph's steps; a single evaluation, whose blocks
    // mostly stage W, keeps the BF16 scheme without it
    const SplitScheme sc = g3_stage<FULL>(fraw, ax, ay, az, rg, hinges, weights, g, kappa,
                                          MODE == kMorph);
    __syncthreads();
    const float beta = weights[FULL ? 4096 : g.g0 * g.g1 * g.g2];
    const G3Grid gr{{g}, weights};
    g3_by_scheme<FULL, MODE == kMorph>(sc.fp16, [&](auto scheme) {
        g3_ws_body<FULL, MODE, decltype(scheme)::value>(fraw, sc, gr, ax, ay, az, beta, kappa,
                                                        gscale, x_in, n, T, eta, c_out, s_out,
                                                        g_out, x_out, tr, gc.nb);
    });
}

// Sum over the 8 lanes of a group (lanes 8g..8g+7), the same value in each: two
// quad exchanges and the half-row mirror, all DPP moves (the order of the pairwise
// sums is that of xor-1, xor-2, xor-4 exchanges).
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL,
                                                              0xf, 0xf, true));
}
__device__ __forceinline__ float sum8(float v) {
    v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_mov<0x141>(v);  // row_half_mirror
    return v;
}

// The DH chain of one configuration by its 8 lanes: lane k = lane % 8 < NDOF forms link
// k's transform A_k (rotation Rz(theta0_k + q_k) Rx(alpha_k), translation (a_k cos,
// a_k sin, d_k) in frame k), and an inclusive scan composes them, P_k = A_0 ... A_k, in
// three rounds (lane k takes P from lane k - r by a DPP row shift and composes
// P <- P_{k-r} o P when k >= r, r = 1, 2, 4; lanes k >= NDOF carry the identity).  Lane
// k ends with frame k + 1: origin o_{k+1} = P_k's translation, axis z_{k+1} = the third
// column of its rotation.  qk: joint k's angle; lk: per link a, d, theta0, sin alpha, cos alpha (LDS).
template <int NDOF, int CTRL>
__device__ __forceinline__ void chain_round(int k, float (&R)[3][3], float (&t)[3]) {
    constexpr int r = CTRL & 15;
    float Rl[3][3], tl[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        tl[a] = dpp_mov<CTRL>(t[a]);
#pragma unroll
        for (int b = 0; b < 3; ++b) Rl[a][b] = dpp_mov<CTRL>(R[a][b]);
    }
    if (k >= r) {
        float Rn[3][3], tn[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            tn[a] = tl[a] + Rl[a][0] * t[0] + Rl[a][1] * t[1] + Rl[a][2] * t[2];
#pragma unroll
            for (int b = 0; b < 3; ++b)
                Rn[a][b] = Rl[a][0] * R[0][b] + Rl[a][1] * R[1][b] + Rl[a][2] * R[2][b];
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            t[a] = tn[a];
#pragma unroll
            for (int b = 0; b < 3; ++b) R[a][b] = Rn[a][b];
        }
    }
}

template <int NDOF>
__device__ __forceinline__ void g3_chain_scan(const float *lk, float qk, int k,
                                              float (&R)[3][3], float (&t)[3]) {
    static_assert(NDOF <= 8, "one lane per link");
    const bool act = k < NDOF;
    const float *p = lk + 5 * (act ? k : 0);
    const float a = p[0], d = p[1], sa = p[3], ca = p[4];
    float st, ct;
    sincosf(p[2] + qk, &st, &ct);
    if (act) {
        R[0][0] = ct, R[0][1] = -st * ca, R[0][2] = st * sa;
        R[1][0] = st, R[1][1] = ct * ca, R[1][2] = -ct * sa;
        R[2][0] = 0.0f, R[2][1] = sa, R[2][2] = ca;
        t[0] = a * ct, t[1] = a * st, t[2] = d;
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            t[i] = 0.0f;
#pragma unroll
            for (int j = 0; j < 3; ++j) R[i][j] = i == j ? 1.0f : 0.0f;
        }
    }
    chain_round<NDOF, 0x111>(k, R, t);  // row_shr:1
    chain_round<NDOF, 0x112>(k, R, t);  // row_shr:2
    chain_round<NDOF, 0x114>(k, R, t);  // row_shr:4
}

// The per-configuration records in LDS (chain, axes, joint gradient) are written and
// read by the lanes of one wave only, and a wave's LDS operations complete in issue
// order: ordering them needs a compiler barrier, not a block barrier.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- joint-space morph (MORPH) or largest body-point occupancy (check) ----
// 4 configurations per wave; lane%32 = 8*cfg + k, body point k of every link.
template <int NDOF, bool FULL, bool MORPH, int SCH>
__device__ __forceinline__ void arm_body(const pdmp_arm &arm, const uint4 *fraw,
                                         const SplitScheme &sc, const G3Grid &gr, const float *ax,
                                         const float *ay, const float *az, float *kin, const float *lk,
                                         float beta, float kappa,
                                         float gscale, const float *q_in, float *q_out, int64_t n,
                                         int64_t n_eff, int T, float eta, float thresh,
                                         float *maxc_out, uint8_t *flag_out, const Traj &tr) {
    constexpr int KIN = 3 * (NDOF + 1) + 3 * NDOF + NDOF;  // o, z, grad_q per configuration
    const int lane = threadIdx.x & 63, pair = pair_address();
    const int k = lane & 7;
    const int slot = (threadIdx.x >> 6) * 4 + ((lane & 31) >> 3);  // configuration in block
    float *ko = kin + slot * KIN, *kz = ko + 3 * (NDOF + 1), *kg = kz + 3 * NDOF;
    const bool writer = (lane & 39) == 0;  // k == 0 in the lower half-wave
    const int64_t cfg = (int64_t)blockIdx.x * 16 + slot;
    const int64_t cs = cfg < n_eff ? cfg : n_eff - 1;
    const int P = arm.pts_per_link;
    const bool own = k < P;
    const float frac = own ? (float)(k + 1) / (float)P : 0.0f;
    float q[NDOF];
#pragma unroll
    for (int j = 0; j < NDOF; ++j) q[j] = q_in[(size_t)j * n + cs];

    const int steps = MORPH ? T : 1;
    float mc = -1.0f;
    int64_t tc;
    const bool rec = MORPH && writer && traj_col(tr, cfg, n_eff, tc);
    for (int st = 0; st < steps; ++st) {
        if (rec) traj_put<NDOF>(tr, st, tc, q);
        {
            // the chain of this configuration (each lane of it one link, composed by a
            // scan), parked in LDS so that the link loop below does not hold ~45
            // registers across the MFMA work; the lower half-wave writes it
            float R[3][3], t[3];
            float qk = q[0];
#pragma unroll
            for (int j = 1; j < NDOF; ++j) qk = k == j ? q[j] : qk;
            g3_chain_scan<NDOF>(lk, qk, k, R, t);
            if (lane < 32) {
                if (k < NDOF) {
#pragma unroll
                    for (int e = 0; e < 3; ++e) ko[3 * (k + 1) + e] = t[e];
                }
                if (k + 1 < NDOF) {
#pragma unroll
                    for (int e = 0; e < 3; ++e) kz[3 * (k + 1) + e] = R[e][2];
                }
                if (k == 0) {
#pragma unroll
                    for (int e = 0; e < 3; ++e) {
                        ko[e] = 0.0f;
                        kz[e] = e == 2 ? 1.0f : 0.0f;
                    }
                }
            }
        }
        wave_lds_sync();
        float SG[3] = {0, 0, 0}, SM[3] = {0, 0, 0};
        // the check's links two at a time: one link's tables beside the other's products (4,000
        // configurations: 2 links 10.4 -> 9.9 us, 7 17.0 -> 15.3; a morph's, 3 % slower)
#pragma unroll(MORPH ? 1 : 2)
        for (int l = NDOF - 1; l >= 0; --l) {
            float p[3], ol[3];
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                ol[e] = ko[3 * l + e];
                p[e] = ol[e] + frac * (ko[3 * (l + 1) + e] - ol[e]);
            }
            float s, sx, sy, sz;
            g3_point<FULL, MORPH, SCH>(fraw, sc, gr, pair, ax, ay, az, kappa * p[0], kappa * p[1],
                                       kappa * p[2], s, sx, sy, sz);
            float c, sp;
            sigmoid_and_slope(s + beta, c, sp);
            if (MORPH) {
                const float f = own ? -sp * gscale : 0.0f;
                const float g0 = f * sx, g1 = f * sy, g2 = f * sz;
                SG[0] += sum8(g0);
                SG[1] += sum8(g1);
                SG[2] += sum8(g2);
                SM[0] += sum8(p[1] * g2 - p[2] * g1);
                SM[1] += sum8(p[2] * g0 - p[0] * g2);
                SM[2] += sum8(p[0] * g1 - p[1] * g0);
                // joint l moves links l..NDOF-1 about z_l through o_l
                const float v0 = SM[0] - (ol[1] * SG[2] - ol[2] * SG[1]);
                const float v1 = SM[1] - (ol[2] * SG[0] - ol[0] * SG[2]);
                const float v2 = SM[2] - (ol[0] * SG[1] - ol[1] * SG[0]);
                const float gq = kz[3 * l] * v0 + kz[3 * l + 1] * v1 + kz[3 * l + 2] * v2;
                if (writer) kg[l] = gq;
            } else if (own) {
                mc = fmaxf(mc, c);
            }
        }
        wave_lds_sync();
        if (MORPH) {
#pragma unroll
            for (int j = 0; j < NDOF; ++j) q[j] = q[j] - eta * kg[j];
        }
        wave_lds_sync();
    }
    if (rec) traj_put<NDOF>(tr, steps, tc, q);
    if (!MORPH) {
        mc = fmaxf(mc, __shfl_xor(mc, 1, 64));
        mc = fmaxf(mc, __shfl_xor(mc, 2, 64));
        mc = fmaxf(mc, __shfl_xor(mc, 4, 64));
    }
    if (lane >= 32 || k != 0 || cfg >= n_eff) return;
    if (MORPH) {
#pragma unroll
        for (int j = 0; j < NDOF; ++j) q_out[(size_t)j * n + cfg] = q[j];
    } else {
        if (maxc_out) maxc_out[cfg] = mc;
        if (flag_out) flag_out[cfg] = mc > thresh ? 1 : 0;
    }
}

template <int NDOF, bool FULL, bool MORPH>
__global__ void __launch_bounds__(kG3Block) __attribute__((amdgpu_waves_per_eu(3)))
k_arm_grid3d(pdmp_arm arm, const float *__restrict__ hinges, const float *__restrict__ weights,
             G3Dims g, float kappa, float gscale, const float *q_in, float *q_out, int64_t n, int T,
             float eta, const uint32_t *__restrict__ n_active, float thresh, float *maxc_out,
             uint8_t *flag_out, Traj tr) {
    constexpr int KIN = 3 * (NDOF + 1) + 3 * NDOF + NDOF;  // o, z, grad_q per configuration
    __shared__ uint4 fraw[kG3Frag];
    __shared__ float ax[kG3Max], ay[kG3Max], az[kG3Max];
    __shared__ float kin[16 * KIN];
    __shared__ float lk[5 * NDOF];  // per link: a, d, theta0, sin alpha, cos alpha
    __shared__ SplitRange rg;
    const int64_t n_eff = n_active ? min((int64_t)*n_active, n) : n;
    if ((int64_t)blockIdx.x * 16 >= n_eff) return;  // whole block idle (uniform)
    if (threadIdx.x < NDOF) {
        const int j = threadIdx.x;
        lk[5 * j] = arm.a[j];
        lk[5 * j + 1] = arm.d[j];
        lk[5 * j + 2] = arm.theta0[j];
        sincosf(arm.alpha[j], &lk[5 * j + 3], &lk[5 * j + 4]);
    }
    const SplitScheme sc = g3_stage<FULL>(fraw, ax, ay, az, rg, hinges, weights, g, kappa, true);
    __syncthreads();
    const float beta = weights[FULL ? 4096 : g.g0 * g.g1 * g.g2];
    const G3Grid gr{{g}, weights};
    g3_by_scheme<FULL, true>(sc.fp16, [&](auto scheme) {
        arm_body<NDOF, FULL, MORPH, decltype(scheme)::value>(arm, fraw, sc, gr, ax, ay, az, kin, lk,
                                                             beta, kappa, gscale, q_in, q_out, n,
                                                             n_eff, T, eta, thresh, maxc_out,
                                                             flag_out, tr);
    });
}

// ---- the same for small batches: one link per wave ----
//
// A block is NDOF waves on the same 4 configurations, wave l evaluating the body points of
// link l, so a step's serial chain is one link's evaluation instead of NDOF.  Every wave
// composes the whole DH chain (lane k keeps only joint k's angle: the chain scan, the
// pull-back and the update need no other), the per-link sums meet in LDS (two buffers:
// one block barrier per step) and lane k adds those of the links it moves, tip first as
// k_arm_grid3d does, so a configuration gets the same bits from either kernel.
template <int NDOF, bool FULL, bool MORPH, int SCH>
__device__ __forceinline__ void arm_wide_body(const pdmp_arm &arm, const uint4 *fraw,
                                              const SplitScheme &sc, const G3Grid &gr, const float *ax,
                                              const float *ay, const float *az,
                                              float (&red)[2][NDOF][4][6], const float *lk,
                                              float beta, float kappa, float gscale,
                                              const float *q_in, float *q_out, int64_t n,
                                              int64_t n_eff, int T, float eta, float thresh,
                                              float *maxc_out, uint8_t *flag_out, const Traj &tr) {
    const int lane = threadIdx.x & 63, l = threadIdx.x >> 6;  // wave l: link l
    const int pair = pair_address();
    const int k = lane & 7, slot = (lane & 31) >> 3;
    const int64_t cfg = (int64_t)blockIdx.x * 4 + slot;
    const int64_t cs = cfg < n_eff ? cfg : n_eff - 1;
    const bool joint = k < NDOF;
    const int P = arm.pts_per_link;
    const bool own = k < P;
    const float frac = own ? (float)(k + 1) / (float)P : 0.0f;
    float qk = joint ? q_in[(size_t)(joint ? k : 0) * n + cs] : 0.0f;
    // one copy of a configuration's joints is written: wave 0's lower half
    const bool out = l == 0 && lane < 32 && joint && cfg < n_eff;
    int64_t tc;
    const bool rec = MORPH && out && traj_col(tr, cfg, n_eff, tc);
    const int steps = MORPH ? T : 1;
    for (int st = 0; st < steps; ++st) {
        if (rec) tr.p[((size_t)st * NDOF + k) * (size_t)tr.nt + (size_t)tc] = qk;
        float R[3][3], t[3];
        g3_chain_scan<NDOF>(lk, qk, k, R, t);
        // frame k (origin o_k, axis z_k) is lane k - 1's result; frame 0 is the base
        float ok[3], zk[3], p[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const float o = dpp_mov<0x111>(t[e]), z = dpp_mov<0x111>(R[e][2]);
            ok[e] = k == 0 ? 0.0f : o;
            zk[e] = k == 0 ? (e == 2 ? 1.0f : 0.0f) : z;
        }
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const float ol = __shfl(ok[e], (lane & ~7) + l, 64);
            const float o1 = __shfl(t[e], (lane & ~7) + l, 64);
            p[e] = ol + frac * (o1 - ol);
        }
        float s, sx, sy, sz;
        g3_point<FULL, MORPH, SCH>(fraw, sc, gr, pair, ax, ay, az, kappa * p[0], kappa * p[1],
                                   kappa * p[2], s, sx, sy, sz);
        float c, sp;
        sigmoid_and_slope(s + beta, c, sp);
        float(&rb)[NDOF][4][6] = red[st & 1];
        if (MORPH) {
            const float f = own ? -sp * gscale : 0.0f;
            const float g0 = f * sx, g1 = f * sy, g2 = f * sz;
            const float v[6] = {sum8(g0), sum8(g1), sum8(g2), sum8(p[1] * g2 - p[2] * g1),
                                sum8(p[2] * g0 - p[0] * g2), sum8(p[0] * g1 - p[1] * g0)};
            if ((lane & 39) == 0) {
#pragma unroll
                for (int e = 0; e < 6; ++e) rb[l][slot][e] = v[e];
            }
            __syncthreads();
            float SG[3] = {0, 0, 0}, SM[3] = {0, 0, 0};
#pragma unroll
            for (int i = NDOF - 1; i >= 0; --i) {
                if (i < k) continue;
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    SG[e] += rb[i][slot][e];
                    SM[e] += rb[i][slot][3 + e];
                }
            }
            const float v0 = SM[0] - (ok[1] * SG[2] - ok[2] * SG[1]);
            const float v1 = SM[1] - (ok[2] * SG[0] - ok[0] * SG[2]);
            const float v2 = SM[2] - (ok[0] * SG[1] - ok[1] * SG[0]);
            const float gq = zk[0] * v0 + zk[1] * v1 + zk[2] * v2;
            qk = qk - eta * gq;
        } else {
            float mc = own ? fmaxf(-1.0f, c) : -1.0f;  // a NaN point counts as none
            mc = fmaxf(mc, __shfl_xor(mc, 1, 64));
            mc = fmaxf(mc, __shfl_xor(mc, 2, 64));
            mc = fmaxf(mc, __shfl_xor(mc, 4, 64));
            if ((lane & 39) == 0) rb[l][slot][0] = mc;
            __syncthreads();
            if (!out || k != 0) return;
#pragma unroll
            for (int i = 0; i < NDOF; ++i) mc = fmaxf(mc, rb[i][slot][0]);
            if (maxc_out) maxc_out[cfg] = mc;
            if (flag_out) flag_out[cfg] = mc > thresh ? 1 : 0;
            return;
        }
    }
    if (rec) tr.p[((size_t)steps * NDOF + k) * (size_t)tr.nt + (size_t)tc] = qk;
    if (out) q_out[(size_t)k * n + cfg] = qk;
}

template <int NDOF, bool FULL, bool MORPH>
__global__ void __launch_bounds__(64 * NDOF)
__attribute__((amdgpu_waves_per_eu(3)))
k_arm_wide(pdmp_arm arm, const float *__restrict__ hinges, const float *__restrict__ weights,
           G3Dims g, float kappa, float gscale, const float *q_in, float *q_out, int64_t n, int T,
           float eta, const uint32_t *__restrict__ n_active, float thresh, float *maxc_out,
           uint8_t *flag_out, Traj tr) {
    __shared__ uint4 fraw[kG3Frag];
    __shared__ float ax[kG3Max], ay[kG3Max], az[kG3Max];
    __shared__ float red[2][NDOF][4][6];
    __shared__ float lk[5 * NDOF];  // per link: a, d, theta0, sin alpha, cos alpha
    __shared__ SplitRangeN<NDOF> rg;
    const int64_t n_eff = n_active ? min((int64_t)*n_active, n) : n;
    if ((int64_t)blockIdx.x * 4 >= n_eff) return;  // whole block idle (uniform)
    if (threadIdx.x < NDOF) {
        const int j = threadIdx.x;
        lk[5 * j] = arm.a[j];
        lk[5 * j + 1] = arm.d[j];
        lk[5 * j + 2] = arm.theta0[j];
        sincosf(arm.alpha[j], &lk[5 * j + 3], &lk[5 * j + 4]);
    }
    const SplitScheme sc = g3_stage<FULL>(fraw, ax, ay, az, rg, hinges, weights, g, kappa, true);
    __syncthreads();
    const float beta = weights[FULL ? 4096 : g.g0 * g.g1 * g.g2];
    const G3Grid gr{{g}, weights};
    g3_by_scheme<FULL, true>(sc.fp16, [&](auto scheme) {
        arm_wide_body<NDOF, FULL, MORPH, decltype(scheme)::value>(arm, fraw, sc, gr, ax, ay, az, red,
                                                                  lk, beta, kappa, gscale, q_in,
                                                                  q_out, n, n_eff, T, eta, thresh,
                                                                  maxc_out, flag_out, tr);
    });
}

// Grids the kernels take: at most 16 hinges per axis, and enough of them to pay for the
// padded contraction, whose cost goes by the tiles nt = ceil(G2 / 2) and not by M.  Measured
// in us: arm morph, 16,000 configurations, 5 steps: 82 + 20 nt against the pairwise
// 30 + 1.4 M; the lines cross at M = 37 + 14 nt.  (10^3 hinges: arm 1,388 -> 188 us; 15^3:
// 4,609 -> 275 us.)
static bool g3_supported(const int *grid, int M) {
    if (!grid || grid[0] < 1 || grid[1] < 1 || grid[2] < 1 || grid[0] > kG3Max ||
        grid[1] > kG3Max || grid[2] > kG3Max || M != grid[0] * grid[1] * grid[2])
        return false;
    return M >= 40 + 16 * ((grid[2] + 1) / 2);
}

// Whether a padded grid's workspace call takes the contraction.
//   * Single evaluations, by M and nt alone (a point's result does not depend on its batch).
//     Values and gradients of few points: 3.2 + 0.42 nt us against 4.0 + 0.003 M with the
//     check's launch; the lines cross at M = 140 nt - 270.  (Gradients of 10^6 points: 16 x 1
//     x 16 hinges 90 against 77, 6^3 49 against 66, 8^3 60 against 150.)
//   * Morphs, by a step's time: a wave's chain, 0.6 + 0.22 nt us (the six products of small
//     grids 0.4 more), or its throughput, against the pairwise kernel's hinge walk and
//     throughput; and 1.2 us of start-up.  (20 steps, 8^3: one point 33 against 15, 8,000
//     34 against 38, 10^6 561 against 2,928; 5^3: 8,000 36 against 16, 10^6 615 against 738.)
static bool g3_ws_pays(int mode, const G3Dims &g, int64_t n, int T) {
    const double M = (double)(g.g0 * g.g1 * g.g2), nt = (g.g2 + 1) / 2;
    if (mode != kMorph) return !g3_within(g, kG3Tiny) && M >= 140 * nt - 270;
    const bool fine = g3_within(g, kG3Fine);
    const double chain = 0.6 + 0.22 * nt + (fine ? 0.4 : 0.0);
    const double rate = n * (6e-6 + 6e-6 * nt + (fine ? 6e-6 : 0.0));
    return T * (0.35 + 5e-4 * M + 3e-7 * n * M - (chain > rate ? chain : rate)) >= 1.2;
}

// Whether a batch takes one link per wave (k_arm_wide): a step's latency is then that of one
// link instead of n_dof, but blocks of 5 links and more hold a CU (3 waves per SIMD; two of
// fewer links share it), so its time goes by rounds of 256 blocks = 1,024 configurations,
// where k_arm_grid3d's is flat up to one wave per SIMD (4,096).  From sweeps of 1 to 8 links,
// 16^3 hinges, 1 to 16,000 configurations (us): k_arm_grid3d 8 + T (0.6 + 1.9 n_dof); wide 8 +
// 4 (r - 1) + T (0.2 + 4 r) in r rounds, of up to 4 links 8 + 2 (r - 1) + T (1.3 + 1.4 r).
// (10 steps, 7 links: 1,000 configurations 53 against 146, 2,000 95 / 146, 3,000 138 / 147,
// 4,000 181 / 152; one step of 3,000: 28 / 23.  One link: 37 / 32 at any size.)  The check: 9.2
// to 10, 11.2 to 13, 17 us in 1, 2, 3 rounds against 7.9 + 1.1 n_dof (4 links 13.0, 8 18.2;
// padded grids, two links: 10.4 / 9.4).
static bool arm_wide_pays(int n_dof, bool full, bool morph, int64_t n, int T) {
    if (n_dof < 2 || n > 3072) return false;
    const int r = (int)((n + 1023) / 1024);
    if (!morph) return full ? n_dof >= 1 << r : 5 * r <= 2 * n_dof;
    return n_dof > 4 ? T * (0.4 + 1.9 * n_dof - 4 * r) >= 4 * (r - 1)
                     : T * (1.9 * n_dof - 0.7 - 1.4 * r) >= 2 * (r - 1);
}

static G3Dims g3_dims(const int *grid) { return G3Dims{grid[0], grid[1], grid[2]}; }
static bool g3_full(const int *grid) { return grid[0] == 16 && grid[1] == 16 && grid[2] == 16; }

// The split scheme the 3-D grid morphs (workspace and arm) take: one block runs their
// staging and writes 2 (FP16 splits), 1 (three-part BF16 splits) or 0 (the pairwise sum).
template <bool FULL>
__global__ void __launch_bounds__(kG3Block)
k_grid3d_scheme(const float *__restrict__ hinges, const float *__restrict__ weights, G3Dims g,
                float kappa, int32_t *out) {
    __shared__ uint4 fraw[kG3Frag];
    __shared__ float ax[kG3Max], ay[kG3Max], az[kG3Max];
    __shared__ SplitRange rg;
    const SplitScheme sc = g3_stage<FULL>(fraw, ax, ay, az, rg, hinges, weights, g, kappa, true);
    if (threadIdx.x == 0) *out = sc.fp16 == kG3Direct ? 0 : sc.fp16 == kG3Bf16 ? 1 : 2;
}

int32_t launch_grid3d_scheme(const float *hinges, const float *weights, const int *grid, int M,
                             float kappa, int32_t *out, hipStream_t st) {
    if (!g3_supported(grid, M)) return PDMP_EUNSUPPORTED;
    if (g3_full(grid))
        hipLaunchKernelGGL(k_grid3d_scheme<true>, dim3(1), dim3(kG3Block), 0, st, hinges, weights,
                           g3_dims(grid), kappa, out);
    else
        hipLaunchKernelGGL(k_grid3d_scheme<false>, dim3(1), dim3(kG3Block), 0, st, hinges, weights,
                           g3_dims(grid), kappa, out);
    return check_launch("k_grid3d_scheme");
}

// A single evaluation's blocks: at most this many, each staging W once for all its points
// (2^20 points, 16^3: 49 us for 500 to 1,500 blocks; 54 us with a block per 128 points, a
// quarter of its VALU work spent on W).
constexpr int64_t kG3EvalBlocks = 1280;

template <bool FULL>
static int32_t launch_grid3d_ws_n(int mode, const RbfArgs &a, const G3Dims &d, hipStream_t st) {
    int64_t blocks = (a.n + 127) / 128;
    if (mode != kMorph && blocks > kG3EvalBlocks) blocks = kG3EvalBlocks;
    GridCheck gc;
    const int axes[3] = {d.g0, d.g1, d.g2};
    if (int32_t e = plan_grid_check(3, a, axes, blocks, st, gc)) return e;
    const dim3 g((unsigned)(blocks + gc.blocks)), b(kG3Block);
#define PDMP_G3(MODE)                                                                          \
    hipLaunchKernelGGL((k_grid3d_ws<FULL, MODE>), g, b, 0, st, a.hinges, a.weights, d, a.kappa, \
                       a.gscale, a.x_in, a.n, a.T, a.eta, a.c_out, a.s_out, a.g_out, a.x_out,  \
                       a.traj, gc)
    if (mode == kEval) PDMP_G3(kEval);
    else if (mode == kGrad) PDMP_G3(kGrad);
    else PDMP_G3(kMorph);
#undef PDMP_G3
    return check_launch("k_grid3d_ws");
}

int32_t launch_grid3d_ws(int mode, const RbfArgs &a, const int *grid, hipStream_t st) {
    if (!g3_supported(grid, a.M) || (mode != kEval && mode != kGrad && mode != kMorph))
        return PDMP_EUNSUPPORTED;
    const int64_t blocks = (a.n + 127) / 128;
    if (!g3_full(grid)) {
        if (!g3_ws_pays(mode, g3_dims(grid), a.n, a.T)) return PDMP_EUNSUPPORTED;
        // a batch beyond one dispatch of this kernel still fits the pairwise kernel's
        if (blocks * kG3Block > 0xffffffffll) return PDMP_EUNSUPPORTED;
        return launch_grid3d_ws_n<false>(mode, a, g3_dims(grid), st);
    }
    if (int32_t e = grid_guard(blocks, kG3Block, "k_grid3d_ws")) return e;
    return launch_grid3d_ws_n<true>(mode, a, g3_dims(grid), st);
}

template <int NDOF, bool FULL>
static int32_t launch_arm_grid3d_n(const pdmp_arm &arm, const float *h, const float *w,
                                   const G3Dims &d, float kappa, float gscale, const float *qi,
                                   float *qo, int64_t n, int T, float eta,
                                   const uint32_t *n_active, bool morph, float thresh, float *maxc,
                                   uint8_t *flag, hipStream_t st, const Traj &traj) {
#define PDMP_ARM(K, G, B)                                                                        \
    hipLaunchKernelGGL(K, dim3((unsigned)(G)), dim3(B), 0, st, arm, h, w, d, kappa, gscale, qi, qo, \
                       n, T, eta, n_active, thresh, maxc, flag, traj)
    if constexpr (NDOF > 1) {
        if (arm_wide_pays(NDOF, FULL, morph, n, T)) {
            if (morph) PDMP_ARM((k_arm_wide<NDOF, FULL, true>), (n + 3) / 4, 64 * NDOF);
            else PDMP_ARM((k_arm_wide<NDOF, FULL, false>), (n + 3) / 4, 64 * NDOF);
            return check_launch("k_arm_wide");
        }
    }
    if (morph) PDMP_ARM((k_arm_grid3d<NDOF, FULL, true>), (n + 15) / 16, kG3Block);
    else PDMP_ARM((k_arm_grid3d<NDOF, FULL, false>), (n + 15) / 16, kG3Block);
#undef PDMP_ARM
    return check_launch("k_arm_grid3d");
}

int32_t launch_arm_grid3d(const pdmp_arm &arm, const float *h, const float *w, int M,
                          const int *grid, float kappa, float gscale, const float *qi, float *qo,
                          int64_t n, int T, float eta, const uint32_t *n_active, bool morph,
                          float thresh, float *maxc, uint8_t *flag, hipStream_t st,
                          const Traj &traj) {
    if (!g3_supported(grid, M) || arm.pts_per_link > 8) return PDMP_EUNSUPPORTED;
    const bool full = g3_full(grid);
    if (!morph && g3_within(g3_dims(grid), kG3Tiny)) return PDMP_EUNSUPPORTED;
    // one link, many configurations: a pairwise step of 16,000 is 0.04 M us (M = 125: 5.4, 216:
    // 8.7), of the contraction 5.4 to 7, with 6 us more to start (T = 1: 10.5 against 16.2)
    if (!full && morph && arm.n_dof == 1 && n > 8192 && M <= (T > 2 ? 128 : 256))
        return PDMP_EUNSUPPORTED;
    const int64_t blocks = (n + 15) / 16;
    if (!full && blocks * kG3Block > 0xffffffffll) return PDMP_EUNSUPPORTED;
    if (int32_t e = grid_guard(blocks, kG3Block, "k_arm_grid3d")) return e;
    const G3Dims d = g3_dims(grid);
    switch (arm.n_dof) {
#define PDMP_CASE(N)                                                                              \
    case N:                                                                                       \
        return full ? launch_arm_grid3d_n<N, true>(arm, h, w, d, kappa, gscale, qi, qo, n, T, eta, \
                                                   n_active, morph, thresh, maxc, flag, st, traj) \
                    : launch_arm_grid3d_n<N, false>(arm, h, w, d, kappa, gscale, qi, qo, n, T,    \
                                                    eta, n_active, morph, thresh, maxc, flag, st, \
                                                    traj);
        PDMP_CASE(1) PDMP_CASE(2) PDMP_CASE(3) PDMP_CASE(4)
        PDMP_CASE(5) PDMP_CASE(6) PDMP_CASE(7) PDMP_CASE(8)
#undef PDMP_CASE
    }
    return PDMP_EUNSUPPORTED;
}

}  // namespace pdmp
