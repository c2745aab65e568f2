// One launch for a whole compensated GEMV (DecDEC Section 4.1): the first
// `nfetch` workgroups of the grid do steps 1-3 (selection for themselves, then
// zero-copy fetch of the selected residual rows and the residual GEMV), all
// other workgroups do the base GEMV.
//
// Why one grid instead of the paper's two streams (Section 4.1, 4.3): measured
// on MI355X, handing work from one hardware queue to another costs about 10 us
// per join, more than the base GEMV itself for Llama-3-8B shapes, and a GEMV
// kernel that runs beside the fetch kernel from another queue starts late and
// runs 5-7x slower.  Inside one grid the fetch workgroups are dispatched first
// (lowest workgroup ids), the GEMV workgroups fill the rest of the chip and
// finish while the fetch workgroups are still waiting for the host link, and
// every workgroup adds its part sums into the per-column accumulators, the
// last arrival writing y (finalize.h), so nothing has to be joined and nothing
// else has to be launched.  How many workgroups fetch (the paper's n_tb,
// Section 4.4) follows from the number of wavefronts that share the rows of a
// column segment (decdec_ws_set_fetch_split).
#include <hip/hip_runtime.h>

#include "fetch_body.h"
#include "gemv_body.h"

namespace decdec {
namespace {

// Eight wavefronts a SIMD (kernels.h), so that the base-GEMV workgroups keep the memory busy: with the cap taken off the
// Llama-3-8B layers with rows in GPU memory take 145.7 us a step instead of 141.5, four layers without compensation 111.2
// instead of 103.6.  Six where the vector registers allow no more: eight chunks of keys per thread, or 2-bit rows (16 column
// sums and 16 row pieces a lane), need up to 80.  Up to 24 scalar values wait in the lanes of a vector register where they
// are not used; that costs nothing that could be measured, whereas 32-43 of them with 4-bit rows, many out of the row loop,
// cost 2-5 % of a small step.
template <int KIND, int RBITS, int SELECT_NCH>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(SELECT_NCH == 8 || RBITS == 2 ? 6 : 8)))
void compensated_gemv_kernel(const CallArgs a) {
    touch_args(a);
    const int bid = (int)blockIdx.x;
    if (bid < a.nfetch) {
        fetch_block<RBITS, SELECT_NCH>(a, bid);
    } else {
        gemv_block<KIND, kWavesPerBlock, 2>(a, bid - a.nfetch);
    }
}

template <int KIND, int RBITS>
hipError_t launch_nch(const CallArgs& a, int nch, hipStream_t stream, const KernelTimer* tm) {
    const dim3 grid((unsigned)(a.nfetch + a.tiles * a.gslices)), block(kBlockThreads);
    const unsigned lds = selection_lds_bytes(nch, a.k);
    switch (nch) {
        case 0: return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 0>, grid, block, lds, stream, a);
        case 1: return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 1>, grid, block, lds, stream, a);
        case 2: return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 2>, grid, block, lds, stream, a);
        case 4: return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 4>, grid, block, lds, stream, a);
        case 8: return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 8>, grid, block, lds, stream, a);
        default: return hipErrorInvalidValue;
    }
}

template <int KIND>
hipError_t launch_rfmt(int rfmt, const CallArgs& a, int nch, hipStream_t stream, const KernelTimer* tm) {
    switch (rfmt) {
        case 0: return launch_nch<KIND, 16>(a, nch, stream, tm);
        case 1: return launch_nch<KIND, 4>(a, nch, stream, tm);
        case 2: return launch_nch<KIND, 2>(a, nch, stream, tm);
        case 3: return launch_nch<KIND, 8>(a, nch, stream, tm);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_compensated_gemv(int kind, int rfmt, const CallArgs& a, int select_chunks, hipStream_t stream,
                                   const KernelTimer* tm) {
    switch (kind) {
        case PACK_U4: return launch_rfmt<PACK_U4>(rfmt, a, select_chunks, stream, tm);
        case PACK_U3: return launch_rfmt<PACK_U3>(rfmt, a, select_chunks, stream, tm);
        case PACK_LUT3: return launch_rfmt<PACK_LUT3>(rfmt, a, select_chunks, stream, tm);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace decdec
