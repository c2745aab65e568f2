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

#include <algorithm>

#include "fetch_body.h"
#include "gemv_body.h"

namespace decdec {
namespace {

// Eight wavefronts a SIMD (kernels.h), so that the base-GEMV workgroups keep the memory busy.  They take 64 columns a
// wavefront: with blocks of 16 columns Llama-3-8B layers with rows in GPU memory take 141 us a step instead of 134.  Six
// where the vector registers allow no more: eight chunks of keys per thread, or 2-bit rows (16 column sums and 16 row pieces
// a lane), need up to 80.
//
// DEPTH 2: the base GEMV takes more than one turn per wavefront, two at a time (28672 x 8192 in 4 bits, one at a time 23.4 us,
// two 21.6).  A kernel of its own, because one that does either takes up to 4 % longer where there is one turn.
template <int KIND, int RBITS, int SELECT_NCH, int DEPTH>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(SELECT_NCH == 8 || RBITS == 2 ? 6 : 8)))
void compensated_gemv_kernel(const CallArgs a) {
    touch_args(a);
    const int bid = (int)blockIdx.x;
    if (bid < a.nfetch) {
        fetch_block<RBITS, SELECT_NCH>(a, bid);
    } else {
        gemv_block<KIND, kOneGridCols, kWavesPerBlock, DEPTH>(a, bid - a.nfetch, kWavesPerBlock);
    }
}

template <int KIND, int RBITS, int DEPTH>
hipError_t launch_nch(const CallArgs& a, int nch, bool over_link, hipStream_t stream, const KernelTimer* tm) {
    const dim3 grid((unsigned)(a.nfetch + a.tiles * (kTileCols / kOneGridCols) * a.gslices)), block(kBlockThreads);
    const unsigned lds = std::max(one_grid_lds(KIND, RBITS, nch, a.k, (long)a.tiles * a.gslices, over_link),
                                  fetch_lds_bytes<RBITS>(a, nch));
    switch (nch) {
        case 0: return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 0, DEPTH>, grid, block, lds, stream, a);
        case 1: return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 1, DEPTH>, grid, block, lds, stream, a);
        case 2: return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 2, DEPTH>, grid, block, lds, stream, a);
        case 4: return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 4, DEPTH>, grid, block, lds, stream, a);
        default: break;
    }
    // eight chunks: more than 128 groups, which 16 K-slices of eight wavefronts do not cover in one turn
    if (nch != 8 || DEPTH != 2) return hipErrorInvalidValue;
    return launch_kernel(tm, compensated_gemv_kernel<KIND, RBITS, 8, 2>, grid, block, lds, stream, a);
}

template <int KIND, int RBITS>
hipError_t launch_turns(const CallArgs& a, int nch, bool over_link, hipStream_t stream, const KernelTimer* tm) {
    return a.gpw > 1 ? launch_nch<KIND, RBITS, 2>(a, nch, over_link, stream, tm) : launch_nch<KIND, RBITS, 0>(a, nch, over_link, stream, tm);
}

template <int KIND>
hipError_t launch_rfmt(int rfmt, const CallArgs& a, int nch, bool over_link, hipStream_t stream, const KernelTimer* tm) {
    switch (rfmt) {
        case 0: return launch_turns<KIND, 16>(a, nch, over_link, stream, tm);
        case 1: return launch_turns<KIND, 4>(a, nch, over_link, stream, tm);
        case 2: return launch_turns<KIND, 2>(a, nch, over_link, stream, tm);
        case 3: return launch_turns<KIND, 8>(a, nch, over_link, stream, tm);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Dynamic LDS: the selection, and where fewer workgroups on a compute unit are better, what keeps another one out.
//
// With rows behind the link and more than 4096 channels a small call lasts as long as its selection and its rows, and the base
// GEMV of the same compute unit slows the selection down.  That pays while the base GEMV is about one round of workgroups:
// four per compute unit, two more in 3 bits, whose tiles are worked off faster, one more beside fp16 rows, which take longer
// on the link (not in the codebook format).  Where it lasts longer, a fourth of the wavefronts that keep the memory busy is
// missing.  us with four and with three, 3-bit / 4-bit / codebook:
//   14336 x 4096 (896 workgroups), 28 4-bit rows 8.7 / 9.2 / 8.8 and 8.5 / 8.8 / 8.5;  8192 x 8192 (1024), 8 fp16 rows 8.9 / 9.1
//   / 9.9 and 8.9 / 9.0 / 9.2;  8192 x 10240 (1280), 8 fp16 rows 9.9 / 10.5 / 10.9 and 9.5 / 10.1 / 11.2, 16 4-bit rows 9.3 /
//   10.1 / 10.1 and 9.1 / 10.4 / 10.6;  14336 x 8192 (1792), 14 fp16 rows 12.3 / 12.4 / 13.3 and 11.6 / 12.6 / 13.6, 28 4-bit
//   rows 11.1 / 12.0 / 12.9 and 11.2 / 12.6 / 13.4;  8192 x 57344, 8 fp16 rows 43.6 / 47.5 / 50.4 and 46.7 / 51.8 / 53.7.
// Up to 4096 channels, where the selection is short, no difference; with rows in GPU memory, where the base GEMV is what lasts,
// 7.3 and 7.8 (14336 x 4096, 286 fp16 rows).
// Kernels with eight chunks of keys per thread have registers for three workgroups only, and so have those with 2-bit rows:
// two of these instead, up to 2.5 workgroups of the base GEMV per compute unit (a codebook loses 9 % at three).  us with three
// and with two:  7680 x 4992 (624), 2 rows 7.3 / 7.5 / 7.2 and 7.1 / 7.1 / 7.1;  8192 x 6144 (768), 2 rows 7.4 / 7.9 / 7.5 and
// 7.4 / 7.9 / 8.2;  8192 x 8192 (1024), 2 rows 7.8 / 8.6 / 8.9 and 8.8 / 9.5 / 9.7.
unsigned one_grid_lds(int kind, int rbits, int nch, int k, long base_workgroups, bool over_link) {
    constexpr unsigned kCuLds = 160 * 1024, kLdsOfThree = 42 * 1024, kLdsOfTwo = 55 * 1024;
    static_assert(3 * kLdsOfThree <= kCuLds && 4 * kLdsOfThree > kCuLds, "three workgroups");
    static_assert(2 * kLdsOfTwo <= kCuLds && 3 * kLdsOfTwo > kCuLds, "two workgroups");
    constexpr unsigned kGemvLds = sizeof(float) * kWavesPerBlock * kOneGridCols;
    constexpr unsigned kStatic = sizeof(FetchLds<16, 2>) + kGemvLds, kStatic2 = sizeof(FetchLds<2, 2>) + kGemvLds;
    static_assert(sizeof(FetchLds<16, 2>) == sizeof(FetchLds<8, 2>) && sizeof(FetchLds<16, 2>) == sizeof(FetchLds<4, 2>) &&
                  sizeof(FetchLds<16, 2>) == sizeof(FetchLds<16, 4>) && sizeof(FetchLds<2, 2>) == sizeof(FetchLds<2, 4>), "one size");
    const unsigned lds = selection_lds_bytes(nch, k);
    if (!over_link || (nch != 2 && nch != 4)) return lds;
    if (rbits == 2) return 2 * base_workgroups <= 5 * kCus ? std::max(lds, kLdsOfTwo - kStatic2) : lds;
    const int rounds = 4 + (kind == PACK_U3 ? 2 : 0) + (rbits == 16 && kind != PACK_LUT3 ? 1 : 0);
    return base_workgroups <= rounds * kCus ? std::max(lds, kLdsOfThree - kStatic) : lds;
}

hipError_t launch_compensated_gemv(int kind, int rfmt, const CallArgs& a, int select_chunks, bool over_link, hipStream_t stream,
                                   const KernelTimer* tm) {
    switch (kind) {
        case PACK_U4: return launch_rfmt<PACK_U4>(rfmt, a, select_chunks, over_link, stream, tm);
        case PACK_U3: return launch_rfmt<PACK_U3>(rfmt, a, select_chunks, over_link, stream, tm);
        case PACK_LUT3: return launch_rfmt<PACK_LUT3>(rfmt, a, select_chunks, over_link, stream, tm);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace decdec
