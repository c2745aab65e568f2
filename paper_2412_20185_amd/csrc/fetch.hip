// Residual fetch + residual GEMV as a kernel of its own.  The device code is
// in fetch_body.h.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fetch_body.h"

namespace decdec {
namespace {

template <int BITS, int SELECT_NCH>
__global__ __launch_bounds__(kBlockThreads) void fetch_kernel(const CallArgs a) {
    touch_args(a);
    fetch_block<BITS, SELECT_NCH>(a, (int)blockIdx.x);
}

}  // namespace

FetchPlan fetch_plan(int rfmt, const MultiShape& sh, int k, int row_split, bool in_hbm, bool selects) {
    FetchPlan p;
    p.segments = 0;
    for (int m = 0; m < sh.n; ++m) p.segments += (sh.N[m] + kFetchSegmentCols - 1) / kFetchSegmentCols;
    // Host link: about 128 wavefronts x 4 KiB of row loads each = 512 KiB of requests in flight saturate it.
    // Rows in device memory: latency bound, so eight times as many wavefronts.
    const int waves = in_hbm ? 1024 : 128;
    // wavefronts that share the rows of one segment
    int per_segment = row_split > 0 ? row_split : (waves + p.segments - 1) / p.segments;
    // fp16 rows: one workgroup per segment is enough once there are eight segments (64 wavefronts already
    // fill the link, and every column has one part sum fewer to add); measured 0.6 % on the Llama-3-8B layer
    if (row_split <= 0 && !in_hbm && rfmt == 0 && p.segments >= 8 && per_segment > kWavesPerBlock)
        per_segment = kWavesPerBlock;
    // Rows in device memory: every workgroup more makes the selection once more beside the base GEMV and adds one more part sum
    // per column, so no more of them than have four rows per wavefront.  us, one grid: 4096 x 14336 (codebook), 60 4-bit rows
    // 8.3 -> 7.7; 8192 x 8192, 80 fp16 rows 7.4 -> 7.0.  With eight rows or more 4096 x 6144, 60 4-bit rows takes 6.6, not 6.3.
    if (row_split <= 0 && in_hbm) {
        constexpr int rows = 4 * kWavesPerBlock;
        per_segment = std::min(per_segment, (k + rows - 1) / rows * kWavesPerBlock);
    }
    if (per_segment > kMaxFetchSlices * kWavesPerBlock) per_segment = kMaxFetchSlices * kWavesPerBlock;
    if (per_segment > k) per_segment = k;
    if (per_segment < 1) per_segment = 1;

    // Rows asked for while the selection goes on (fetch_body.h).  They take about 0.35 us of the selection and use the link for
    // up to 1.2 (4096 channels) to 2 (14336) before it is over: not with few bytes to fetch, nor where so many workgroups share
    // a segment's rows that a good part is asked for by the wrong one, nor with so many segments that one row per wavefront
    // is more than the link takes in that time.  us without and with, fp16 / 8-bit / 4-bit rows: 4096 x 4096, k = 60 14.9 -> 13.9 /
    // 10.5 -> 9.2 / 8.1 -> 7.1; 14336 x 4096, k = 210 38.2 -> 36.9 / 22.4 -> 21.4 / 15.4 -> 14.7; but 4096 x 28672, k = 81
    // 87.2 -> 88.7 (fp16).  Between 54 and 64 KiB, 90 sizes (1024, 4096 and 14336 channels by 512 to 4096 columns, all three
    // formats), the time is 6 % less to 5 % more with it (1024 x 1024, 32 fp16 rows 6.58 -> 6.83, 4096 x 4096, 8 of them
    // 6.63 -> 6.22); at 24 KiB 2 % less to 9 % more.  A requested split is kept as it is, without.
    constexpr int row_bits[] = {16, 4, 2, 8};
    const int segment_bytes = kFetchSegmentCols / 8 * row_bits[rfmt];
    const size_t bytes = (size_t)p.segments * segment_bytes * k;
    const int one_each = p.segments * kWavesPerBlock * segment_bytes;  // a row per wavefront
    constexpr int kLinkBytes = 256 * 1024;
    // Above 16384 channels the kernels have no such code (kAsksEarly), and eight wavefronts of each workgroup delay the base GEMV:
    // us with three to seven and with eight, 60 4-bit rows, 17408 x 28672 (4-bit weights) 43.5 and 46.3, 28672 x 22016 42.1 and
    // 44.3; 200 rows of 28672 x 16384 39.6 and 39.3.
    constexpr int kEarlyMaxK = 4 * 8 * kBlockThreads;
    static_assert(kAsksEarly<16, 4> && !kAsksEarly<16, 8>, "four chunks of eight keys per thread");
    p.early = 0;
    if (sh.K <= kEarlyMaxK && row_split <= 0 && !in_hbm && rfmt != 2 && bytes > 64 * 1024 && per_segment <= 4 * kWavesPerBlock &&
        one_each <= kLinkBytes && select_tries_chunks(sh.K / 8, k)) {
        if (selects) p.early = std::min((kLinkBytes + one_each - 1) / one_each, 2048 / segment_bytes);
        // All wavefronts take rows then, where that is no slower with a supplied selection either: who selects must not show in
        // how the rows are split, because y has the bits of that split.  us with three to seven wavefronts of each workgroup ->
        // with eight: 60 4-bit rows, selecting 5120 x 13824 13.9 -> 12.7, 4096 x 28672 21.5 -> 20.8, supplied 4096 x 12288 12.8 ->
        // 11.7, 4096 x 28672 21.1 -> 20.5; beyond 28672 columns, 20 to 90 rows, 4 % more to 8 % less.  8-bit rows above 32
        // segments, if eight wavefronts have more than a batch (8) each, selecting / supplied: 4096 x 20480, k = 100 42.8 -> 42.0 /
        // 42.3 -> 40.8; but k = 60 27.8 -> 27.1 / 25.9 -> 27.1, and up to 32 segments 4096 x 12288, k = 60 19.3 -> 18.3 / 17.3 ->
        // 18.7, 8192 x 12288, k = 330 78.2 -> 80.2 / 78.0 -> 77.4.  fp16 rows stay as they are: 14336 x 16384, k = 33 26.3 ->
        // 28.8 / 25.2 -> 26.7.
        const bool all = rfmt == 1 || (rfmt == 3 && p.segments > 32 && k > 8 * kWavesPerBlock);
        if (all && p.segments * kWavesPerBlock <= 448) per_segment = std::min(std::max(per_segment, kWavesPerBlock), k);
    }
    p.slices = (per_segment + kWavesPerBlock - 1) / kWavesPerBlock;
    p.row_waves = (per_segment + p.slices - 1) / p.slices;
    // With the rows of a segment in one workgroup, a look at the accumulators behind the requests of a batch: who sees the base
    // GEMV's part sums there writes y without the trip of an atomic.  It is a trip to memory itself, which the rows behind it wait
    // for, and a long one while the base GEMV adds its sums: only with fp16 rows (fewer bits 1 to 6 % slower) that take more than
    // 16 us of the link, or a base GEMV of 8 Mi weights at most.  us without and with: 4096 x 6144, k = 96 25.7 and 25.4, 14336 x
    // 6144, k = 122 32.5 and 31.9, 8192 x 8192, k = 61 23.4 and 22.8, 2048 x 4096, k = 32 9.4 and 9.2; but 14336 x 6144, k = 24
    // 10.7 and 11.6, 8192 x 4096, k = 65 15.1 and 15.5, 14336 x 8192, k = 20 11.6 and 14.1; above 16 segments 8192 x 16384, k =
    // 163 100.4 and 101.3.
    constexpr size_t kLookBytes = 920000;
    const bool rows_last = bytes > kLookBytes || (size_t)sh.K * sh.col0[sh.n] <= (size_t)1 << 23;
    p.look = p.early > 0 && rfmt == 0 && p.slices == 1 && p.segments <= 16 && rows_last;
    return p;
}

int fetch_select_chunks(int K, int k) {
    // In-kernel selection: the keys of a workgroup stay in registers (at most 8 chunks of 8 per thread)
    // and the selection must fit in LDS.
    constexpr int per_chunk_round = 8 * kBlockThreads;  // channels covered by one chunk per thread
    if (k < 1 || k > 4096 || K > 8 * per_chunk_round) return 0;
    return K <= per_chunk_round ? 1 : K <= 2 * per_chunk_round ? 2 : K <= 4 * per_chunk_round ? 4 : 8;
}

template <int BITS, int NCH>
static hipError_t launch_fetch_kernel(const CallArgs& a, hipStream_t stream, const KernelTimer* tm) {
    return launch_kernel(tm, fetch_kernel<BITS, NCH>, dim3((unsigned)(a.segments * a.cslices)), dim3(kBlockThreads),
                         fetch_lds_bytes<BITS>(a, NCH), stream, a);
}

template <int NCH>
static hipError_t launch_fetch_nch(int rfmt, const CallArgs& a, hipStream_t stream, const KernelTimer* tm) {
    switch (rfmt) {
        case 0: return launch_fetch_kernel<16, NCH>(a, stream, tm);
        case 1: return launch_fetch_kernel<4, NCH>(a, stream, tm);
        case 2: return launch_fetch_kernel<2, NCH>(a, stream, tm);
        default: return launch_fetch_kernel<8, NCH>(a, stream, tm);
    }
}

hipError_t launch_fetch(int rfmt, const CallArgs& a, int select_chunks, hipStream_t stream, const KernelTimer* tm) {
    switch (select_chunks) {
        case 0: return launch_fetch_nch<0>(rfmt, a, stream, tm);
        case 1: return launch_fetch_nch<1>(rfmt, a, stream, tm);
        case 2: return launch_fetch_nch<2>(rfmt, a, stream, tm);
        case 4: return launch_fetch_nch<4>(rfmt, a, stream, tm);
        case 8: return launch_fetch_nch<8>(rfmt, a, stream, tm);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace decdec
