// Base GEMV as a kernel of its own (k = 0, or when the compensation runs in
// separate kernels).  The device code is in gemv_body.h.
#include <hip/hip_runtime.h>

#include "gemv_body.h"

namespace decdec {
namespace {

// Eight wavefronts a SIMD (kernels.h), so that two workgroups of 16 fit a compute unit: with the cap taken off, one does, and
// gate + up of the Llama-3-8B shape runs in two rounds (32 layers 921 us instead of 846).  Four where four tiles in flight
// need up to 104 vector registers.
template <int KIND, int WPB, int NBUF>
__global__ __launch_bounds__(WPB * 64) __attribute__((amdgpu_waves_per_eu(NBUF == 2 ? 8 : 4))) void gemv_kernel(const CallArgs a) {
    touch_args(a);
    gemv_block<KIND, WPB, NBUF>(a, (int)blockIdx.x);
}

template <int KIND, int WPB>
hipError_t launch_depth(const CallArgs& a, hipStream_t stream, const KernelTimer* tm) {
    const dim3 grid((unsigned)(a.tiles * a.gslices)), block(WPB * 64);
    if (a.gpw > 2) return launch_kernel(tm, gemv_kernel<KIND, WPB, 4>, grid, block, 0, stream, a);  // tiles a wave keeps in flight
    return launch_kernel(tm, gemv_kernel<KIND, WPB, 2>, grid, block, 0, stream, a);
}

template <int KIND>
hipError_t launch_waves(const CallArgs& a, int wpb, hipStream_t stream, const KernelTimer* tm) {
    switch (wpb) {
        case 4: return launch_depth<KIND, 4>(a, stream, tm);
        case 8: return launch_depth<KIND, 8>(a, stream, tm);
        case 16: return launch_depth<KIND, 16>(a, stream, tm);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

GemvPlan gemv_plan(long tiles, int G, int gpw_request, int wpb_request) {
    // One group per wavefront, so that a wavefront requests all its weights at once, as long as the chip
    // holds the wavefronts that makes at one time; two groups beyond that.  A K-slice more costs one atomic
    // per column (finalize.h), so the slices are not kept few: small matrices take small workgroups, which
    // start sooner and spread over more compute units; in between, the largest workgroups (a workgroup that
    // walks all of K alone writes y itself); the largest matrices run in several rounds of workgroups,
    // which medium workgroups fill more evenly.  Read from a sweep over the shapes of Llama-3 8B and 70B.
    GemvPlan p;
    const long units = tiles * G;  // (tile, group) pairs = wavefront iterations
    p.wpb = wpb_request > 0 ? wpb_request : units <= 4096 ? 4 : units <= 16384 ? 16 : 8;
    p.gpw = gpw_request > 0 ? gpw_request : units <= 12288 ? 1 : 2;
    int per_block = p.gpw * p.wpb;
    p.slices = (G + per_block - 1) / per_block;
    while (p.slices > kMaxGemvSlices) {
        ++p.gpw;
        per_block = p.gpw * p.wpb;
        p.slices = (G + per_block - 1) / per_block;
    }
    return p;
}

hipError_t launch_gemv(int kind, const CallArgs& a, int wpb, hipStream_t stream, const KernelTimer* tm) {
    switch (kind) {
        case PACK_U4: return launch_waves<PACK_U4>(a, wpb, stream, tm);
        case PACK_U3: return launch_waves<PACK_U3>(a, wpb, stream, tm);
        case PACK_LUT3: return launch_waves<PACK_LUT3>(a, wpb, stream, tm);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace decdec
