// Step 1 of dynamic error compensation (DecDEC Section 4.1): sc_indices, the k
// input channels with the largest |x|, and x[sc_indices], as a kernel of its
// own.  The paper's kernel uses an approximate, chunked bucket Top-K (Section
// 4.3); this is the exact Top-K it uses as its quality reference (Section 5.2).
// The algorithm is in select_block.h; one workgroup does the whole selection
// (one chunk of 8 channels per thread up to 4096 channels, two to eight above).
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "select_block.h"

namespace decdec {
namespace {

template <int THREADS, int NCH, bool RADIX = false>
__global__ __launch_bounds__(THREADS) void select_topk_kernel(const uint16_t* __restrict__ x, int K, int k,
                                                             int32_t* __restrict__ idx_out,
                                                             uint16_t* __restrict__ xsel_out) {
    __shared__ SelectShared<THREADS, NCH> sh;
    uint4 ch[NCH];
    const auto select = [&](const auto& run) {
        load_keys(x, run, ch);
        block_select_topk<THREADS, NCH, RADIX>(ch, run, K, k, sh, idx_out, xsel_out);
    };
    if constexpr (RADIX || NCH == 1) {
        select(FullRuns<THREADS, NCH>(K / 8));
    } else {
        select(ChosenRuns<THREADS, NCH>(K / 8, k));
    }
}

}  // namespace

hipError_t launch_select_topk(const void* x, int K, int k, int32_t* idx_out, void* xsel_out, hipStream_t stream,
                              const KernelTimer* tm) {
    const uint16_t* xp = static_cast<const uint16_t*>(x);
    uint16_t* xs = static_cast<uint16_t*>(xsel_out);
    const dim3 one(1);
    // one chunk of 8 channels per thread as long as that gives enough threads: no list of chunks is needed then
    if (K <= 2048) return launch_kernel(tm, select_topk_kernel<256, 1>, one, dim3(256), 0, stream, xp, K, k, idx_out, xs);
    if (K <= 4096) return launch_kernel(tm, select_topk_kernel<512, 1>, one, dim3(512), 0, stream, xp, K, k, idx_out, xs);
    // Above, by chunks with eight wavefronts (select_block.h); a k too large for the chunk form has 1024 threads and kernels without
    // that form, with the marked keys' words chosen by comparisons.  us, the kernel with both forms -> without: K = 14336, k =
    // 1433: 7.24 -> 7.14; 28672, 2867: 11.53 -> 11.40; 32768, 3276: 12.14 -> 11.98.
    const bool radix = !select_tries_chunks(K / 8, k);
    if (!radix && K <= 8192) return launch_kernel(tm, select_topk_kernel<512, 2>, one, dim3(512), 0, stream, xp, K, k, idx_out, xs);
    if (!radix && K <= 16384) return launch_kernel(tm, select_topk_kernel<512, 4>, one, dim3(512), 0, stream, xp, K, k, idx_out, xs);
    if (!radix && K <= 32768) return launch_kernel(tm, select_topk_kernel<512, 8>, one, dim3(512), 0, stream, xp, K, k, idx_out, xs);
    if (K <= 8192) return launch_kernel(tm, select_topk_kernel<1024, 1, true>, one, dim3(1024), 0, stream, xp, K, k, idx_out, xs);
    if (K <= 16384) return launch_kernel(tm, select_topk_kernel<1024, 2, true>, one, dim3(1024), 0, stream, xp, K, k, idx_out, xs);
    if (K <= 32768) return launch_kernel(tm, select_topk_kernel<1024, 4, true>, one, dim3(1024), 0, stream, xp, K, k, idx_out, xs);
    return launch_kernel(tm, radix ? select_topk_kernel<1024, 8, true> : select_topk_kernel<1024, 8>, one, dim3(1024), 0, stream,
                         xp, K, k, idx_out, xs);
}

}  // namespace decdec
