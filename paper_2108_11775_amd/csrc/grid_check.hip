// grid_check.hip -- device-side check of the tensor-grid statement of an occupancy.
//
// An occupancy whose `grid` field is set is evaluated through the per-axis
// factorisation, which reads only the axis entries of the hinge array (X0[i] = h[i],
// X1[i] = h[M + g0 i], X2[i] = h[2M + g0 g1 i]).  With such a launch the entry
// points enqueue this check on the same stream, before it or inside it: every hinge j = i0 + g0 (i1 + g1 i2)
// must equal (X0[i0], X1[i1], X2[i2]) (by value; a NaN coordinate fails).  A mismatch
// sets a sticky per-device word that pdmp_sync reports as PDMP_EINVAL and clears;
// the launch itself runs to completion (its results are then undefined).
//
// Small evaluations and morphs on a grid take the check into their own launch, as blocks
// past their own (plan_grid_check): a launch is 3 us of the host's time and 3 us of the
// stream's, beside 3 to 15 us for the whole work of such a call.
#include <atomic>

#include "pdmp_common.h"

namespace pdmp {

__device__ uint32_t g_grid_mismatch = 0;

__global__ void __launch_bounds__(256)
k_grid_check(const float *__restrict__ h, int dim, int M, int g0, int g1) {
    grid_check_part(h, dim, M, g0, g1, &g_grid_mismatch, blockIdx.x, gridDim.x);
}

int32_t launch_grid_check(int dim, const float *hinges, int M, const int *grid, hipStream_t st) {
    const int blocks = (M + 255) / 256 < 64 ? (M + 255) / 256 : 64;
    hipLaunchKernelGGL(k_grid_check, dim3(blocks), dim3(256), 0, st, hinges, dim, M, grid[0],
                       grid[1]);
    return check_launch("k_grid_check");
}

// The mismatch word's address on each device: a kernel of another file cannot name it.  (A
// launch of the check's own takes the word of the device that it runs on.)
static std::atomic<uint32_t *> g_word[64];

static uint32_t *mismatch_word(hipStream_t st) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    // a stream of another device: its kernels must not write to this one's word
    hipDevice_t on = dev;
    if (st && hipStreamGetDevice(st, &on) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    if (on != dev) return nullptr;
    uint32_t *p = g_word[dev].load(std::memory_order_acquire);
    if (p) return p;
    // first call on the device; left for a later one while the stream is captured
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone)
        return nullptr;
    void *v = nullptr;
    if (hipGetSymbolAddress(&v, HIP_SYMBOL(g_grid_mismatch)) != hipSuccess) return nullptr;
    g_word[dev].store((uint32_t *)v, std::memory_order_release);
    return (uint32_t *)v;
}

// Beyond this many blocks the launch is a few percent of the call, and the kernel's own
// blocks come first.
constexpr int64_t kFusedCheckBlocks = 4096;

int32_t plan_grid_check(int dim, const RbfArgs &a, const int *grid, int64_t blocks, hipStream_t st,
                        GridCheck &gc) {
    gc = GridCheck();
    gc.nb = (int)blocks;
    if (!a.check_grid) return PDMP_OK;
    if (blocks <= kFusedCheckBlocks) gc.word = mismatch_word(st);
    if (!gc.word) return launch_grid_check(dim, a.hinges, a.M, grid, st);
    gc.blocks = (a.M + 1023) / 1024;  // four hinges per thread
    return PDMP_OK;
}

// Reads and clears the current device's mismatch word (host-synchronous).
int32_t take_grid_mismatch(bool &mismatch) {
    uint32_t v = 0;
    hipError_t e = hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_grid_mismatch), sizeof(v), 0,
                                       hipMemcpyDeviceToHost);
    if (e == hipSuccess && v != 0) {
        const uint32_t zero = 0;
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_grid_mismatch), &zero, sizeof(zero), 0,
                              hipMemcpyHostToDevice);
    }
    if (e != hipSuccess) {
        set_error("grid check word: %s", hipGetErrorString(e));
        return PDMP_EDEVICE;
    }
    mismatch = v != 0;
    return PDMP_OK;
}

}  // namespace pdmp
