// occupancy.hip -- RBF logistic occupancy (value, input gradient) and the fused
// T-step explicit-Euler workspace morph, for gfx950.
//
// Occupancy (Sec. 3.1, Hilbert-map form): s(x) = sum_j w_j exp(-|x-h_j|^2/(2 l^2)) + beta,
// c = sigma(s), grad c = sigma'(s) grad s, grad s = -(1/l^2) sum_j w_j phi_j (x - h_j).
// Morph (Sec. 3.2, Eq. 1 by Euler's method): x <- x - eta * grad c(x), T times.
//
// Mapping.  The work is FP32 VALU + v_exp_f32 bound (one exp and 3*DIM+2 VALU per
// sample-hinge pair), not HBM bound: samples stream in once and out once.
//   * Hinges live in LDS for the whole launch when they fit (64 KiB: 4096 3-D or
//     5504 2-D hinges), staged as chunks of four: DIM float4 rows of prescaled
//     coordinates kappa*h and one float4 row of weights, so one ds_read_b128 per row
//     feeds four hinges.  Larger hinge sets are streamed
//     through LDS tile by tile inside each step.
//   * Coordinates are prescaled by kappa = sqrt(log2(e)/(2 l^2)) so that
//     phi = exp2(-|kappa x - kappa h|^2) needs no multiply before v_exp_f32.
//   * G lanes share SPL samples (the launcher's rule below); each lane sums a strided
//     subset of hinge chunks and the G partial sums are combined by exchanges that leave
//     bit-identical totals in all G lanes, so their redundant copies of the state stay
//     equal.
//   * The T-step loop runs in registers; the state touches HBM only at the ends.
#include "pdmp_common.h"
#include "rbf_split.h"

namespace pdmp {

// LDS place (in float4) of row k of chunk c, rows being DIM coordinates and the weights of a
// chunk of four hinges: a row of IW chunks after the other, IW the lanes (up to 16) that
// read neighbouring chunks, so their 16-byte reads are contiguous and the rows of a chunk
// lie at fixed distances.
template <int G>
constexpr int chunk_iw() { return G < 16 ? G : 16; }

template <int DIM, int IW>
__device__ __forceinline__ int chunk_at(int c, int k) {
    return ((c / IW) * (DIM + 1) + k) * IW + c % IW;
}

// Copy hinge chunks [c0, c0 + nc) into LDS, prescaled, zero-padded past M.
template <int DIM, int IW>
__device__ __forceinline__ void stage_chunks(float4 *lds, const float *__restrict__ hinges,
                                             const float *__restrict__ weights, int M,
                                             float kappa, int c0, int nc) {
    float *f = reinterpret_cast<float *>(lds);
    for (int idx = threadIdx.x; idx < nc * 4; idx += blockDim.x) {
        const int j = c0 * 4 + idx, u = idx & 3;
        const bool ok = j < M;
#pragma unroll
        for (int k = 0; k < DIM; ++k)
            f[chunk_at<DIM, IW>(idx >> 2, k) * 4 + u] = ok ? kappa * hinges[(size_t)k * M + j] : 0.0f;
        f[chunk_at<DIM, IW>(idx >> 2, DIM) * 4 + u] = ok ? weights[j] : 0.0f;
    }
}

// Accumulate the chunk at ch into SPL samples' sums (GRAD: the gradient's too).
template <int DIM, int SPL, int IW, bool GRAD>
__device__ __forceinline__ void chunk_accumulate(const float4 *__restrict__ ch,
                                                 const float (&xs)[SPL][DIM], float (&as)[SPL],
                                                 float (&ag)[SPL][DIM]) {
    float4 hc[DIM];
#pragma unroll
    for (int k = 0; k < DIM; ++k) hc[k] = ch[k * IW];
    const float4 wv = ch[DIM * IW];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
            float d[DIM];
            d[0] = xs[s][0] - f4c(hc[0], u);
            float r2 = d[0] * d[0];
#pragma unroll
            for (int k = 1; k < DIM; ++k) {
                d[k] = xs[s][k] - f4c(hc[k], u);
                r2 = fmaf(d[k], d[k], r2);
            }
            const float wp = f4c(wv, u) * exp2_fast(-r2);
            as[s] += wp;
            if (!GRAD) continue;
#pragma unroll
            for (int k = 0; k < DIM; ++k) ag[s][k] = fmaf(wp, d[k], ag[s][k]);
        }
    }
}

// Sum over the G lanes of a group, the same value in each: exchanges within a row of 16 by
// DPP moves, across rows by lane swaps.
template <int CTRL>
__device__ __forceinline__ float dpp_get(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL,
                                                              0xf, 0xf, true));
}
template <int G>
__device__ __forceinline__ float group_sum(float v) {
    if (G >= 2) v += dpp_get<0xB1>(v);    // quad_perm [1,0,3,2]
    if (G >= 4) v += dpp_get<0x4E>(v);    // quad_perm [2,3,0,1]
    if (G >= 8) v += dpp_get<0x141>(v);   // row_half_mirror
    if (G >= 16) v += dpp_get<0x140>(v);  // row_mirror
    if (G >= 32) {
        const uint32_t u = __float_as_uint(v);
        const auto x = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        v = __uint_as_float(x[0]) + __uint_as_float(x[1]);
    }
    if (G >= 64) {
        const uint32_t u = __float_as_uint(v);
        const auto x = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        v = __uint_as_float(x[0]) + __uint_as_float(x[1]);
    }
    return v;
}

// MODE kEval   : c_out[n] (nullable), s_out[n] (nullable).  With gridDim.y > 1 the
//                hinge chunks are split into ranges of `cps` chunks, block row y sums
//                range y only and writes s_out[y*n + i] (partial sums, no bias).
// MODE kGrad   : c_out[n] (nullable), g_out[DIM][n] = sigma'(s) grad s
// MODE kGradBwd: g_out[DIM][n] = g_in[i] * (chain ? sigma'(s) : 1) * grad s
// MODE kMorph  : x_out[DIM][n] after T steps (x_out may equal x_in)
// The bias is *bias_ptr (nullable: no bias).
template <int DIM, int SPL, int G, int BLOCK, int MODE>
__global__ void __launch_bounds__(BLOCK)
k_rbf(const float *__restrict__ hinges, const float *__restrict__ weights, int M,
      const float *__restrict__ bias_ptr, float kappa, float gscale, const float *x_in, int64_t n,
      int T, float eta, float *c_out, float *s_out, float *g_out, float *x_out,
      const float *__restrict__ g_in, int chain, int cps, Traj tr) {
    constexpr int IW = chunk_iw<G>();
    constexpr int TILE = rbf_tile_chunks<DIM>();
    // values of one sample are few instructions per LDS read: two chunks at a time hide its latency
    // (26,000 samples, 2,600 hinges: 19.3 -> 18.4 us; weight gradient, 2^20 points, 700
    // hinges: 244 -> 212)
    constexpr int UN = MODE == kEval && SPL == 1 ? 2 : 1;
    extern __shared__ float4 lds[];

    const int nchunks_all = chunks_for(M);
    const int cbeg = (int)blockIdx.y * cps;                  // this block row's hinge chunks
    const int nchunks = min(cps, nchunks_all - cbeg);
    const int ntiles = (nchunks + TILE - 1) / TILE;
    const int lg = threadIdx.x % G;
    constexpr int GPB = BLOCK / G;  // sample groups per block
    const int64_t base = (int64_t)blockIdx.x * GPB * SPL + threadIdx.x / G;

    int64_t idx[SPL];
    float x[SPL][DIM];
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
        idx[s] = base + (int64_t)s * GPB;
        const int64_t i = idx[s] < n ? idx[s] : n - 1;  // tail lanes shadow a valid sample
#pragma unroll
        for (int k = 0; k < DIM; ++k) x[s][k] = x_in[(size_t)k * n + i];
    }
    const float beta = bias_ptr ? *bias_ptr : 0.0f;

    if (ntiles == 1) {
        stage_chunks<DIM, IW>(lds, hinges, weights, M, kappa, cbeg, nchunks);
        __syncthreads();
    }

    const int steps = (MODE == kMorph) ? T : 1;
    int64_t tc[SPL];
    bool rec[SPL];
#pragma unroll
    for (int s = 0; s < SPL; ++s) rec[s] = MODE == kMorph && lg == 0 && traj_col(tr, idx[s], n, tc[s]);
    float as[SPL], ag[SPL][DIM];
    for (int t = 0; t < steps; ++t) {
#pragma unroll
        for (int s = 0; s < SPL; ++s)
            if (rec[s]) traj_put<DIM>(tr, t, tc[s], x[s]);
        float xs[SPL][DIM];
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
            as[s] = 0.0f;
#pragma unroll
            for (int k = 0; k < DIM; ++k) {
                xs[s][k] = kappa * x[s][k];
                ag[s][k] = 0.0f;
            }
        }
        for (int tile = 0; tile < ntiles; ++tile) {
            const int c0 = tile * TILE;
            const int nc = min(TILE, nchunks - c0);
            if (ntiles > 1) {
                __syncthreads();
                stage_chunks<DIM, IW>(lds, hinges, weights, M, kappa, cbeg + c0, nc);
                __syncthreads();
            }
            const float4 *ch = lds + chunk_at<DIM, IW>(lg, 0);
#pragma unroll UN
            for (int c = lg; c < nc; c += G, ch += G * (DIM + 1))
                chunk_accumulate<DIM, SPL, IW, MODE != kEval>(ch, xs, as, ag);
        }
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
            if (G > 1) {
                as[s] = group_sum<G>(as[s]);
#pragma unroll
                for (int k = 0; k < DIM && MODE != kEval; ++k) ag[s][k] = group_sum<G>(ag[s][k]);
            }
            if (MODE == kMorph) {
                float c, sp;
                sigmoid_and_slope(as[s] + beta, c, sp);
                // x - eta * sigma' * grad s,  grad s = -gscale * ag
                const float step = eta * sp * gscale;
#pragma unroll
                for (int k = 0; k < DIM; ++k) x[s][k] = fmaf(step, ag[s][k], x[s][k]);
            }
        }
    }

#pragma unroll
    for (int s = 0; s < SPL; ++s)
        if (rec[s]) traj_put<DIM>(tr, steps, tc[s], x[s]);
    if (lg != 0) return;
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
        if (idx[s] >= n) continue;
        const size_t i = (size_t)idx[s];
        if (MODE == kMorph) {
#pragma unroll
            for (int k = 0; k < DIM; ++k) x_out[(size_t)k * n + i] = x[s][k];
        } else if (MODE == kEval) {
            const float sv = as[s] + beta;
            if (c_out) {
                float c, sp;
                sigmoid_and_slope(sv, c, sp);
                c_out[i] = c;
            }
            if (s_out) s_out[(size_t)blockIdx.y * n + i] = sv;
        } else {
            const float sv = as[s] + beta;
            float c, sp;
            sigmoid_and_slope(sv, c, sp);
            float f;
            if (MODE == kGrad) {
                if (c_out) c_out[i] = c;
                f = -sp * gscale;
            } else {
                f = -g_in[i] * (chain ? sp : 1.0f) * gscale;
            }
#pragma unroll
            for (int k = 0; k < DIM; ++k) g_out[(size_t)k * n + i] = f * ag[s][k];
        }
    }
}

// ---------------------------------------------------------------- launcher ---

template <int DIM, int SPL, int G, int BLOCK, int MODE>
static int32_t launch_rbf_v(const RbfArgs &a, hipStream_t st) {
    constexpr int TILE = rbf_tile_chunks<DIM>(), IW = chunk_iw<G>();
    const int nchunks = chunks_for(a.M);
    const int splits = a.splits > 1 ? a.splits : 1;
    const int cps = (nchunks + splits - 1) / splits;
    const int used = ((cps < TILE ? cps : TILE) + IW - 1) / IW * IW;
    const size_t lds = (size_t)used * ChunkLayout<DIM>::kBytes;
    const int64_t per_block = (int64_t)(BLOCK / G) * SPL;
    const int64_t blocks = (a.n + per_block - 1) / per_block;
    if (int32_t e = grid_guard(blocks, BLOCK, "k_rbf")) return e;
    hipLaunchKernelGGL((k_rbf<DIM, SPL, G, BLOCK, MODE>), dim3((unsigned)blocks, (unsigned)splits),
                       dim3(BLOCK), lds, st, a.hinges, a.weights, a.M, a.bias, a.kappa, a.gscale,
                       a.x_in, a.n, a.T, a.eta, a.c_out, a.s_out, a.g_out, a.x_out, a.g_in,
                       a.chain, cps, a.traj);
    return check_launch("k_rbf");
}

// Lanes per sample (G), samples per lane (SPL) and block size, by what binds the launch; us.
//   * Few samples: the length of a lane's hinge walk.  G = 64 up to 1,000 + 8 M samples, at
//     most 5,000 (morph step, 1,000 samples and 4,000 hinges: 2.4 against 7.8 with G = 16;
//     4,096: 5.1 against 7.8; the lines cross between 5,000 and 8,000 there, with 200 hinges
//     between 3,000 and 5,000, with 100 between 1,500 and 3,000; up to 64 hinges the lanes
//     past the last chunk idle and the exchanges remain: 8 steps, 30 hinges, 5,000 samples: 8.8
//     against 4.8).  512 threads for single evaluations, which stage the hinges for as little
//     work as one step, and for 53 KiB and more of hinges (below; 6,000 hinges, 5,000 samples,
//     4 steps: 119 -> 62).
//   * More: the LDS reads of hinges and the waves in flight.  16 lanes that read 16
//     consecutive chunks leave both clear (10 steps, 40,001 samples, 2-D: 4,000 hinges 368, four
//     lanes per sample 512; 1,000 hinges 99 against 131; 600,000 samples, 4,000 hinges:
//     5,125, one lane per sample and two samples per lane 9,060).  512 threads stage the
//     hinges half as often and keep many of them from holding the CU to few waves, but 256 CUs
//     of such blocks may end on a round of 32 samples per CU that 256 threads would not need.
//     512 where they do not (14,000 samples, 2,000 hinges, one evaluation: 0.92 of the time;
//     10,000: 1.01 to 1.05, over 8 steps 1.16); always where two blocks' hinges at most fit a
//     CU (53 KiB; 10,000 samples, 5,000 hinges: 0.72), which includes hinges past one tile
//     (26,000 samples, 6,000 hinges, 4 steps: 281 -> 200), from 65,536 samples on above 40 KiB
//     (evaluations of 100,003 samples, 4,096 hinges: 80 against 108), and for single
//     evaluations of 20,000 and more above 32 KiB (26,000, 3,000 hinges: 0.93).  64 lanes again
//     between 8,192 and 11,000 samples, where a second round of 16 lanes would be half
//     empty (10,000 samples, 4,000 hinges, 8 steps: 0.77 of the time; 1,400: 0.91; 600: 1.11).
//   * Few hinges: the exchanges of a step's end, so as few lanes as fill the chip (two waves
//     per SIMD).  Below 600 hinges 8 from 12,000 samples (16,000, 200 hinges, 8 steps: 14.5
//     against 18.3 with 16), below 64 always (16 lanes walk half a chunk); from 30,000 four
//     below 300 hinges and 8 above (30,000, 100 hinges, 8 steps: 14.7 against 18.2 with 8); one
//     where the blocks of 256 samples fill nine tenths of their rounds (131,072, 30 hinges, 8
//     steps: 13.5 against 19.1 with 8; 200,000, 200 hinges, three blocks and a bit per CU: 100
//     against four lanes' 94); one always for 8 hinges and fewer, and from 120,000 below 64.  8 below 1,200 hinges from
//     60,000 on (65,536 samples, 1,044 hinges: 130 against 138; 300,000, 850: 458 against 480).
//   * Batches that fill whole rounds of 512 blocks of 2,048 samples: one lane per sample, two
//     samples per lane, no exchanges (2^20 samples, 5 steps: 900 hinges 1,024 against
//     1,127, 3-D 4,096 hinges 5,884 against 6,143); a poorly filled last round costs more than
//     that (600,000 samples above; single evaluations lose less, 1,500,000 samples on 2,000 3-D
//     hinges, seven tenths filled: 600 against 687).  Also from 2^27 samples, where 16 threads per sample
//     would pass one dispatch.
template <int DIM, int MODE>
static int32_t launch_rbf_dim(const RbfArgs &a, hipStream_t st) {
    const bool single = MODE != kMorph || a.T <= 1;
    const int lds = chunks_for(a.M) * ChunkLayout<DIM>::kBytes;
    const bool two = lds > 53 * 1024;  // two blocks at most share a CU
    // samples in blocks of `per` fill at least tenths/10 of their rounds of `slots` blocks
    auto fills = [&](int64_t per, int64_t slots, int tenths) {
        const int64_t b = (a.n + per - 1) / per;
        return 10 * b >= tenths * ((b + slots - 1) / slots * slots);
    };
    const bool wide = a.n >= (1 << 19) && (a.M <= 8 || fills(2048, 512, MODE != kMorph ? 7 : 9));
    if (!(wide && (a.M <= 8 || a.M >= 600)) && a.n < (1 << 27) &&
        (a.M <= 8 || (a.n >= 120000 && (a.M < 64 || (a.M < 600 && fills(256, 256, 9))))))
        return launch_rbf_v<DIM, 1, 1, 256, MODE>(a, st);
    if (wide || a.n >= (1 << 27)) return launch_rbf_v<DIM, 2, 1, 1024, MODE>(a, st);
    if (a.M >= 64 && a.n <= 5000 && a.n <= 1000 + 8 * (int64_t)a.M)
        return single || two ? launch_rbf_v<DIM, 1, 64, 512, MODE>(a, st)
                             : launch_rbf_v<DIM, 1, 64, 256, MODE>(a, st);
    if (a.M < 300 && a.n >= 30000) return launch_rbf_v<DIM, 1, 4, 256, MODE>(a, st);
    if (a.M < 64 || (a.M < 600 && a.n >= 12000) || (a.M < 1200 && a.n >= 60000))
        return launch_rbf_v<DIM, 1, 8, 256, MODE>(a, st);
    if (a.M >= 1400 && a.n > 8192 && a.n <= 11000) return launch_rbf_v<DIM, 1, 64, 512, MODE>(a, st);
    auto round_up = [&](int64_t per) { return (a.n + 256 * per - 1) / (256 * per) * per; };
    if (two || round_up(32) <= round_up(16) ||
        (lds > 40 * 1024 && a.n >= 65536) || (lds > 32 * 1024 && single && a.n >= 20000))
        return launch_rbf_v<DIM, 1, 16, 512, MODE>(a, st);
    return launch_rbf_v<DIM, 1, 16, 256, MODE>(a, st);
}

template <int DIM>
static int32_t launch_rbf_mode(int mode, const RbfArgs &a, hipStream_t st) {
    switch (mode) {
        case kEval: return launch_rbf_dim<DIM, kEval>(a, st);
        case kGrad: return launch_rbf_dim<DIM, kGrad>(a, st);
        case kGradBwd: return launch_rbf_dim<DIM, kGradBwd>(a, st);
        default: return launch_rbf_dim<DIM, kMorph>(a, st);
    }
}

int32_t launch_rbf(int dim, int mode, const RbfArgs &a, hipStream_t st) {
    return dim == 2 ? launch_rbf_mode<2>(mode, a, st) : launch_rbf_mode<3>(mode, a, st);
}

// A weight gradient: lanes are hinges (rbf_split.h) and every lane reads the same points.
int32_t launch_rbf_wgrad(int dim, const RbfArgs &a, int hinges_per_block, hipStream_t st) {
    if (hinges_per_block == 512)
        return dim == 2 ? launch_rbf_v<2, 2, 1, 256, kEval>(a, st)
                        : launch_rbf_v<3, 2, 1, 256, kEval>(a, st);
    return dim == 2 ? launch_rbf_v<2, 1, 1, 256, kEval>(a, st)
                    : launch_rbf_v<3, 1, 1, 256, kEval>(a, st);
}

int32_t launch_occ_any(int dim, int mode, const RbfArgs &a, const int *grid, hipStream_t st) {
    if (grid && grid[0] > 0 && a.splits <= 1) {
        const int32_t r = dim == 2 ? launch_grid2d(mode, a, grid[0], grid[1], st)
                                   : launch_grid3d_ws(mode, a, grid, st);
        if (r != PDMP_EUNSUPPORTED) return r;  // other grids take the pairwise sum
    }
    if (a.check_grid)
        if (int32_t e = launch_grid_check(dim, a.hinges, a.M, grid, st)) return e;
    return launch_rbf(dim, mode, a, st);
}

}  // namespace pdmp
