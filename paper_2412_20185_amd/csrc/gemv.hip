// Base GEMV as a kernel of its own (k = 0, or when the compensation runs in
// separate kernels).  The device code is in gemv_body.h.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gemv_body.h"

namespace decdec {
namespace {

// Eight wavefronts a SIMD (kernels.h): a wavefront holds one tile or two, and the others of its compute unit cover its trip to
// memory.  Four where it holds kDeepTiles.
template <int KIND, int COLS, int WAVES, int DEPTH>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(DEPTH <= 2 ? 8 : 4))) void gemv_kernel(const CallArgs a) {
    touch_args(a);
    asm volatile("" ::"s"(a.tiles), "s"(a.waves));
    gemv_block<KIND, COLS, WAVES, DEPTH>(a, (int)blockIdx.x, a.waves);
}

template <int KIND, int COLS, int DEPTH = 1>
hipError_t launch_waves(const CallArgs& a, hipStream_t stream, const KernelTimer* tm) {
    const dim3 grid((unsigned)(a.tiles * (kTileCols / COLS) * a.gslices)), block(workgroup_waves(a.waves) * 64);
    switch (workgroup_waves(a.waves)) {
        case 4: return launch_kernel(tm, gemv_kernel<KIND, COLS, 4, DEPTH>, grid, block, 0, stream, a);
        case 8: return launch_kernel(tm, gemv_kernel<KIND, COLS, 8, DEPTH>, grid, block, 0, stream, a);
        default: return launch_kernel(tm, gemv_kernel<KIND, COLS, 16, DEPTH>, grid, block, 0, stream, a);
    }
}

template <int KIND>
hipError_t launch_cols(const CallArgs& a, const GemvPlan& plan, hipStream_t stream, const KernelTimer* tm) {
    switch (plan.cols) {
        case 16: return launch_waves<KIND, 16>(a, stream, tm);
        case 32: return launch_waves<KIND, 32>(a, stream, tm);
        case 64: break;
        default: return hipErrorInvalidValue;
    }
    if (plan.depth == kDeepTiles) return launch_waves<KIND, 64, kDeepTiles>(a, stream, tm);
    if (plan.depth != 2) return launch_waves<KIND, 64>(a, stream, tm);
    const dim3 grid((unsigned)(a.tiles * a.gslices)), block(workgroup_waves(a.waves) * 64);
    switch (workgroup_waves(a.waves)) {  // gemv_plan has two tiles with these only
        case 8: return launch_kernel(tm, gemv_kernel<KIND, 64, 8, 2>, grid, block, 0, stream, a);
        case 16: return launch_kernel(tm, gemv_kernel<KIND, 64, 16, 2>, grid, block, 0, stream, a);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

namespace {

constexpr int kSimds = 4 * kCus;
int ceil_div(long a, long b) { return (int)((a + b - 1) / b); }

// `waves` wavefronts of `cols` columns, `gpw` turns each; as many slices as that takes, at most kMaxGemvSlices.
GemvPlan sliced(int G, int cols, int waves, int gpw) {
    const int turns = ceil_div(G, kTileCols / cols);  // of one wavefront over all of K
    gpw = std::max(gpw, ceil_div(turns, (long)waves * kMaxGemvSlices));
    return GemvPlan{cols, waves, gpw, ceil_div(turns, (long)waves * gpw)};
}

// What a caller asks for, in wavefronts of 64 columns; 0 is left to the library.
GemvPlan requested(int kind, long tiles, int G, int gpw, int waves) {
    // Two turns where they let one workgroup cover all of K, of matrices wide enough for that: 4096 x 28672 by 16 wavefronts
    // 11.5 -> 9.9 us.
    if (gpw == 0) gpw = tiles >= kCus && waves < G && G <= 2 * waves ? 2 : 1;
    // Four wavefronts start sooner where the chip holds all of them at one time (2048 x 2048, one turn: eight take 3.8 us, four
    // 3.5; 4096 x 4096, codebook, four turns: 7.6 and 5.8), 16 where those cover all of K of a wide matrix (4096 x 28672, two
    // turns, 4 bit: eight 12.8, 16 11.5; 8192 x 28672, four turns, 3 bit: 18.5 and 17.6), eight otherwise (14336 x 4096, four
    // turns: eight 7.8, 16 10.4).
    if (waves == 0) waves = G > 8 && tiles * G <= 4096 ? 4 : tiles >= kCus && G > 8 * gpw && G <= 16 * gpw ? 16 : 8;
    GemvPlan p = sliced(G, 64, waves, gpw);
    // Several tiles on their way where the chain of turns is long for the number of wavefronts (those with work) that hide one
    // another's trips: eight turns per wavefront of a SIMD, three in the codebook format, whose turns take longer.  us with one
    // tile and with kDeepTiles, 3-bit / 4-bit / codebook:
    //   28672 x 8192, 4 wavefronts x 56 turns: 48.8 / 48.8 / 55.4 and 31.1 / 31.8 / 37.6;  14336 x 4096, 4 x 28: 25.2 / 25.1 /
    //   28.7 and 16.5 / 16.6 / 19.8;  4096 x 28672, 8 x 14: 16.9 / 17.2 / 20.6 and 14.6 / 15.5 / 17.3;  8192 x 8192, 8 x 8
    //   (8 per SIMD): 11.0 / 11.0 / 13.2 and 10.1 / 10.9 / 11.5;  28672 x 8192, 8 x 14 (7 per SIMD): 19.1 / 20.7 / 22.3 and
    //   18.5 / 22.1 / 20.1.
    const long working = tiles * ceil_div(G, p.gpw);
    if (p.gpw > 1 && tiles * p.slices * waves <= 4 * kSimds &&
        (long)std::min(p.gpw, G) * kSimds >= (kind == PACK_LUT3 ? 3 : 8) * working)
        p.depth = kDeepTiles;
    return p;
}

GemvPlan plan_of(int kind, long tiles, int G, int gpw_request, int waves_request, bool one_grid, bool over_link) {
    if (one_grid) {
        // A K-slice fewer is an atomic per column fewer, and in the codebook format the codebook once less; a turn more lets a
        // workgroup last longer, which is what fills the chip less evenly.  Two turns from three rounds of wavefronts at eight a
        // SIMD on; in 3 bits only with rows behind the link, in 4 bits not.  us with one turn and with two, 3-bit / 4-bit /
        // codebook:  8192 x 57344, 8 fp16 rows 43.0 / 47.8 / 49.6 and 39.8 / 49.1 / 44.0;  14336 x 14336, 14 fp16 rows 17.3 /
        // 19.8 / 20.1 and 16.7 / 20.1 / 19.5;  8192 x 20480, 16 4-bit rows 13.7 / 15.9 / 16.8 and 14.4 / 16.6 / 17.6;
        // 4096 x 57344, 80 fp16 rows in GPU memory 19.2 / 23.4 / 21.9 and 20.1 / 24.0 / 21.2.
        const bool two = tiles * G >= 3 * 8 * kSimds && (kind == PACK_LUT3 || (kind == PACK_U3 && over_link));
        return sliced(G, kOneGridCols, kWavesPerBlock, gpw_request > 0 ? gpw_request : two ? 2 : 1);
    }
    if (gpw_request > 0 || waves_request > 0) return requested(kind, tiles, G, gpw_request, waves_request);

    // One tile per wavefront, but for the widest matrices.  us per call in graph replays on rotating weights, 3-bit / 4-bit /
    // codebook; first a plan of 64 columns only, cut in K-slices, with two groups per wavefront from 12288 tiles on -> this one.
    //
    // One workgroup over all of K, which writes y itself, where that still gives the chip enough to do.
    //   4096 x 4096: 4.10 / 4.44 / 4.38 -> 3.59 / 3.82 / 3.68;  4096 x 28672, codebook: 12.4 -> 10.9;
    //   1024 x 1024: 3.2 / 3.3 / 3.3 -> 2.7 / 2.6 / 2.7;  8192 x 4096: 5.17 / 5.70 / 5.49 -> 4.66 / 5.38 / 4.84
    //
    // In blocks of 64 columns a load is 1 KiB in one piece, and x and the sum over wavefronts are there once per 64 columns: so
    // where the columns are many enough to keep the compute units evenly busy with them, to `share` of the last round.  us for
    // blocks of 16 or 32 columns and of 64:
    const auto even = [&](double share) { return tiles >= share * kCus * ceil_div(tiles, kCus); };
    int turns = 0;  // per wavefront, of 64 columns; 0: narrower blocks
    if (G <= 8) {
        // Few groups are few wavefronts a workgroup, so that small workgroups start all over the chip; but just above one round
        // half as wide blocks are more even.  256 x 1024 2.40 / 2.23 / 2.55 and 2.30 / 2.14 / 2.48;  256 x 43008 4.6 / 4.6 / 5.0
        // and 3.1 / 3.3 / 3.5;  1024 x 14336 3.35 / 3.51 / 3.73 and 3.29 / 3.45 / 3.61;  1024 x 24576 4.07 / 4.55 / 4.60 and
        // 4.07 / 4.32 / 4.56;  1024 x 22528 3.85 / 4.20 / 4.29 and 4.03 / 4.38 / 4.50;  below 128 tiles 768 x 4096 8 % slower.
        turns = G <= 2 ? tiles >= 16 : tiles >= kCus / 2 && (G <= 4 || tiles <= kCus || tiles > 2 * kCus || even(0.75));
    } else if (G <= 16) {
        // One group per wavefront, while the chip holds the workgroups of 16 at one time (two per compute unit):
        // 2048 x 14336 4.28 / 4.74 / 4.87 and 4.17 / 4.56 / 4.70;  2048 x 28672 6.18 / 7.14 / 6.61 and 5.81 / 6.71 / 6.67;
        // 2048 x 24576 (0.75) 5.64 / 6.47 / 6.06 and 5.59 / 6.34 / 6.63;  2048 x 36864 7.2 / 8.5 / 8.2 and 8.0 / 8.9 / 9.1.
        // Beyond that two by half as many wavefronts, both asked for at once:
        // 1152 x 49152 (1) 6.9 / 7.1 / 7.9 and 5.8 / 6.6 / 6.5;  2048 x 45056 (0.92) 8.3 / 9.8 / 9.0 and 7.8 / 9.2 / 8.8;
        // 2048 x 57152 (0.87) 9.4 / 11.0 / 11.6 and 9.4 / 11.3 / 11.1;  2048 x 40960 (0.83) 7.7 / 9.1 / 8.4 and 7.7 / 9.0 / 8.8.
        turns = tiles <= 2 * kCus ? even(0.875) : even(0.9) ? 2 : 0;
    } else if (G <= 32 && tiles > kCus && even(0.85)) {
        // Two groups per wavefront likewise: 4096 x 28672 (0.875) 9.8 / 11.7 / 11.1 and 9.4 / 11.2 / 10.9;
        // 3584 x 28672 9.0 / 10.6 / 10.4 and 9.2 / 10.7 / 10.6;  2176 x 57152 (0.872) 12.6 / 14.0 / 14.4 and 11.1 / 12.4 / 12.2;
        // 4096 x 49152 (1) 15.2 / 18.2 / 17.5 and 14.2 / 17.1 / 16.4;  3072 x 40960 (0.83) 10.5 / 12.3 / 12.3 and 10.7 / 12.4 /
        // 11.8;  4096 x 36864 (0.75) 11.9 / 14.3 / 13.7 and 12.5 / 15.3 / 14.6.  One after the other 4096 x 28672 takes 9.7 /
        // 11.3 / 11.1.
        turns = 2;
    }
    if (turns > 0) return GemvPlan{64, ceil_div(G, turns), turns, 1, turns};
    const int turns16 = ceil_div(G, 4), turns32 = ceil_div(G, 2);
    const long blocks16 = 4 * tiles, blocks32 = 2 * tiles;
    const int rounds16 = ceil_div(blocks16, kCus), rounds32 = ceil_div(blocks32, kCus);
    if (turns16 <= 8) {
        // Blocks of 32 columns where those of 16 would leave compute units idle in their last round and twice as wide ones
        // do not take longer for it: N = 5120, 6144 and 14336 with K = 4096 4.42 -> 4.29, 4.52 -> 4.37, 6.83 -> 6.43.
        if (turns32 <= 16 && blocks16 % kCus != 0 && rounds16 == 2 * rounds32) return GemvPlan{32, turns32, 1, 1};
        return GemvPlan{16, turns16, 1, 1};
    }
    // Up to K = 8192 the same with up to 16 wavefronts and one workgroup per compute unit, or half as many as there are; up to
    // 6144 also with two.  us for that and for slices: 8192 x 4096 4.6 and 5.1, 5120 x 8192 5.5 and 5.9; but 8192 x 1024 3.9
    // and 3.5, 8192 x 5120 6.3 and 5.7, 8192 x 8192 in 4 bits 8.9 and 8.6.
    if (turns16 <= 16 && blocks16 >= kCus / 2 && (blocks16 <= kCus || (blocks16 == 2 * kCus && turns16 <= 12)))
        return GemvPlan{16, turns16, 1, 1};
    // K-slices, one atomic per column each (finalize.h): workgroups of four wavefronts while the chip holds all of them at one
    // time, which start sooner; else of eight at most, in the widest blocks whose slices are few enough.
    //   8192 x 10240: 9.6 / 11.1 / 10.1 -> 8.5 / 10.0 / 9.9;  28672 x 8192: 18.5 / 22.6 / 21.5 -> 17.2 / 21.1 / 20.9;
    //   13824 x 5120: 8.7 / 10.0 / 9.7 -> 7.7 / 8.9 / 8.9;  8192 x 5120 by four and by eight: 5.7 and 5.9
    if (G <= 4 * kMaxGemvSlices && tiles * G <= 8192) return sliced(G, 64, 4, 1);
    // With codebooks, and in 3 bits above 16384 channels, half as many slices of two tiles on their way once there are several
    // rounds of workgroups.  us so and by the slices below, one tile a wavefront:
    //   8192 x 30400 17.9 / 22.4 / 21.1 and 17.6 / 21.8 / 22.2;  14336 x 30400 28.7 / 37.5 / 33.4 and 27.9 / 35.9 / 36.5;
    //   16512 x 8192 11.8 / 14.4 / 13.3 and 11.5 / 13.2 / 14.7;  20480 x 14336 20.9 / 25.3 / 23.9 and 20.3 / 24.4 / 26.0;
    //   26752 x 30400 51.5 / 64.8 / 60.5 and 54.9 / 64.2 / 67.8;  16512 x 4096 8.0 / 9.3 / 9.1 and 7.5 / 8.3 / 8.9.
    const long units = tiles * G;
    const bool many_groups = G > 8 * kMaxGemvSlices;
    if (kind == PACK_LUT3 ? units >= (many_groups ? 12 : 28) * kSimds : kind == PACK_U3 && many_groups && units >= 48 * kSimds) {
        GemvPlan p = sliced(G, 64, 8, 2);
        if (p.gpw == 2) p.depth = 2;
        return p;
    }
    if (G <= 8 * kMaxGemvSlices) {
        // More slices of fewer wavefronts, if all workgroups still start at one time (four per compute unit): 14336 x 4096 in
        // 14 and 16 slices 7.24 / 8.27 / 7.67 and 7.10 / 7.91 / 7.41 (8704 x 4096 in 9 and 14: 5.96 -> 5.74); in 16 slices of
        // 13824 x 4608, which do not, 7.6 instead of 7.3.
        const int slices = std::max(ceil_div(G, 8), (int)std::min<long>(4 * kCus / tiles, kMaxGemvSlices));
        return sliced(G, 64, ceil_div(G, slices), 1);
    }
    return sliced(G, G <= 16 * kMaxGemvSlices ? 32 : 16, 8, 1);
}

}  // namespace

GemvPlan gemv_plan(int kind, long tiles, int G, int gpw_request, int waves_request, bool one_grid, bool over_link) {
    const GemvPlan p = plan_of(kind, tiles, G, gpw_request, waves_request, one_grid, over_link);
    // A grid has fewer than 2^32 threads (inside the one-grid kernel half of them at most): one workgroup of eight per tile where
    // the plan would take more, from 2^20 tiles on.
    const long threads = tiles * (kTileCols / p.cols) * p.slices * workgroup_waves(p.waves) * 64;
    return threads < (one_grid ? 1L << 31 : 1L << 32) ? p : GemvPlan{64, 8, ceil_div(G, 8), 1, 1};
}

hipError_t launch_gemv(int kind, const CallArgs& a, const GemvPlan& plan, hipStream_t stream, const KernelTimer* tm) {
    switch (kind) {
        case PACK_U4: return launch_cols<PACK_U4>(a, plan, stream, tm);
        case PACK_U3: return launch_cols<PACK_U3>(a, plan, stream, tm);
        case PACK_LUT3: return launch_cols<PACK_LUT3>(a, plan, stream, tm);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace decdec
