// Internal launch interface between the C-ABI layer (api.hip) and the kernel
// translation units.  Every launcher validates nothing: api.hip has already
// checked shapes against what the kernels and their grids assume.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>

namespace decdec {

// Workgroup size of the base-GEMV, residual and fused kernels (one wavefront = one unit of work in all of them).
constexpr int kBlockThreads = 512;
constexpr int kWavesPerBlock = kBlockThreads / 64;

// Eight wavefronts a SIMD take at most 64 vector and 80 scalar registers each.  The compiler's occupancy remark promises
// eight up to 100 scalar registers, but the chip takes some for itself: of 512 workgroups of 1024 threads all start at once
// at 80 registers, and 256 have to wait at 82.

constexpr int kCus = 256;               // compute units of the card
constexpr int kFetchSegmentCols = 512;  // output columns of one column segment = threads of a fetch workgroup
constexpr int kMaxGemvSlices = 16;   // part sums per column the base GEMV may contribute (K-slices)
constexpr int kMaxFetchSlices = 16;  // part sums per column the residual kernel may contribute (row slices)
constexpr int kSelectMaxK = 65536;

// Optional pair of events that receive the begin and end timestamps of one
// kernel dispatch (what a kernel trace reports as its duration).
struct KernelTimer {
    hipEvent_t start, stop;
};

// Launches `kernel`; with a timer the dispatch's own timestamps go to its events.
template <typename F, typename... Args>
inline hipError_t launch_kernel(const KernelTimer* tm, F kernel, dim3 grid, dim3 block, unsigned lds,
                                hipStream_t stream, Args... args) {
    if (tm != nullptr) {
        hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, tm->start, tm->stop, 0, args...);
    } else {
        kernel<<<grid, block, lds, stream>>>(args...);
    }
    return hipGetLastError();
}

// One call handles up to kMaxMulti weight matrices that share the activation
// vector x (q/k/v, gate/up): their columns are treated as one concatenated
// output of Ntot = sum N_m columns; matrix m owns columns [col0[m], col0[m]+N[m]).
constexpr int kMaxMulti = 4;

struct MultiShape {
    int n;                    // matrices in this call
    int K;                    // shared input channels
    int N[kMaxMulti];         // output columns per matrix
    int col0[kMaxMulti + 1];  // first concatenated column of matrix m; col0[n] = Ntot
};

// Kernel arguments of the base-GEMV, residual and one-grid kernels.  They arrive cold: every 64-byte line of them is
// a trip to memory for the first wavefront of a compute unit that reads it, and a kernel here runs for only a few such
// trips.  So one matrix is one line, everything else is two, and touch_args asks for all of them at once, before
// anything waits for a value: what is read by index afterwards, the matrix a workgroup falls into, is then at hand.
struct alignas(64) MatArgs {
    const uint4* Wq;
    const uint16_t* scales;
    const uint16_t* zeros_or_lut;
    const uint4* R;       // residual rows
    const uint16_t* Rs;   // fp16 [N] column scales (integer residuals) or null
    _Float16* y;
    int N;
    int col0;      // first concatenated column
    int tile_end;  // 64-column tiles of the matrices up to and including this one
    int seg_end;   // 512-column segments likewise
};
static_assert(sizeof(MatArgs) == 64, "one line");

struct CallArgs {
    MatArgs mat[kMaxMulti];
    const uint16_t* x;
    unsigned long long* acc;  // one word per concatenated column, zero between calls; null: the producers leave fp32
                              // partial rows and a separate kernel adds them
    int n;                    // matrices
    int G;                    // groups of 128 input channels
    int gslices, gpw, waves;  // base GEMV: K-slices, turns per wavefront, wavefronts per workgroup
    unsigned gdiv;            // reciprocal_of(gslices)
    int producers;            // part sums per column: gslices + cslices
    int direct;               // 1: the base GEMV is the only producer and has one slice: it writes y itself
    int Ntot;
    float* gpart;             // fp32 [gslices][Ntot]   (acc == null only)
    int k;
    int cslices, row_waves;   // workgroups per column segment, wavefronts of each that share its rows
    int rows_per;             // rows of each of these wavefronts, rounded up
    unsigned cdiv;            // reciprocal_of(cslices)
    int early;                // rows a wavefront may ask for before the selection is complete
    int look;                 // 1: a workgroup looks at the accumulators before it adds to them
    int nfetch;               // workgroups of the residual part of the one-grid kernel
    int32_t* idx;             // the selection: written by the kernel that selects, read by the others
    uint16_t* xsel;
    float* cpart;             // fp32 [cslices][Ntot]   (acc == null only)
    int tiles, segments;      // over all matrices
};

// i / d as the high word of i * reciprocal_of(d), for d <= 16 and i < 2^28 (a grid of more would need more weights
// than the card holds): one scalar multiplication where a division takes forty instructions ahead of the first load.
inline unsigned reciprocal_of(int d) { return d > 1 ? (unsigned)((0x100000000ull + d - 1) / d) : 0u; }
__device__ __forceinline__ int divide_by(int i, unsigned reciprocal) {
    return reciprocal ? (int)__umulhi((unsigned)i, reciprocal) : i;
}

__device__ __forceinline__ void touch_args(const CallArgs& a) {
    asm volatile("" ::"s"(a.mat[0].N), "s"(a.mat[1].N), "s"(a.mat[2].N), "s"(a.mat[3].N), "s"(a.x), "s"(a.xsel), "s"(a.n),
                 "s"(a.mat[0].tile_end), "s"(a.mat[1].tile_end), "s"(a.mat[2].tile_end), "s"(a.gslices), "s"(a.gdiv),
                 "s"(a.gpw), "s"(a.G), "s"(a.nfetch));
}

// Has a value in a register by here.  What an asm statement returns is a pointer of unknown address space,
// and accesses through it are flat ones, which count as LDS accesses too and are waited for together with all of them:
// pointers are held as pointers to global memory.
__device__ __forceinline__ void hold_scalar(int& a, int& b, int& c) { asm volatile("" : "+s"(a), "+s"(b), "+s"(c)); }
__device__ __forceinline__ void hold_vector(uint32_t& v) { asm volatile("" : "+v"(v)); }
template <typename T>
__device__ __forceinline__ void hold_scalar(T*& p) {
    auto global = (__attribute__((address_space(1))) T*)p;
    asm volatile("" : "+s"(global));
    p = (T*)global;
}

// What the lanes of a wavefront have written to LDS is there for its other lanes.
__device__ __forceinline__ void wave_writes_seen() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// gemv.hip ---------------------------------------------------------------
// How the work is cut: a wavefront takes `cols` columns (16, 32 or 64) of 64 / cols groups of 128 input channels at a time,
// `gpw` times, the tiles of `depth` turns on their way at one time (1, 2 or kDeepTiles; more than 1 with 64 columns only);
// workgroups with `waves` such wavefronts (at most 16; they have workgroup_waves of them), `slices` workgroups (and part sums
// per column) per block of `cols` columns.  Requests of 0 leave the choice to the library; others are for 64 columns.
// one_grid: inside the one-grid kernel, where cols is kOneGridCols, waves kWavesPerBlock and depth 1 (several
// turns are worked off two at a time); over_link: with residual rows in host memory.
constexpr int kDeepTiles = 4;
struct GemvPlan {
    int cols, waves, gpw, slices, depth = 1;
};
inline int workgroup_waves(int waves) { return waves <= 4 ? 4 : waves <= 8 ? 8 : 16; }
constexpr int kOneGridCols = 64;
GemvPlan gemv_plan(int kind, long tiles, int G, int gpw_request, int waves_request, bool one_grid, bool over_link);
hipError_t launch_gemv(int kind, const CallArgs& a, const GemvPlan& plan, hipStream_t stream, const KernelTimer* tm = nullptr);

// select.hip -------------------------------------------------------------
hipError_t launch_select_topk(const void* x, int K, int k, int32_t* idx_out, void* xsel_out, hipStream_t stream,
                              const KernelTimer* tm = nullptr);

// select_bucket.hip ------------------------------------------------------
// The paper's approximate Top-K: k_chunk channels per 1024-channel chunk (K a multiple of 1024).
hipError_t launch_select_bucket(const void* x, int K, int k_chunk, float b0, float b15, int32_t* idx_out,
                                void* xsel_out, hipStream_t stream, const KernelTimer* tm = nullptr);

// fetch.hip --------------------------------------------------------------
// How the residual kernel is laid out: `segments` column segments (one 16-byte piece per lane and row; all
// matrices of the call together) x `slices` workgroups per segment; `row_waves` wavefronts of each workgroup
// share its rows; `early`: rows that a wavefront may ask for before the selection is complete; `look`: whether a workgroup that
// has asked for rows early looks at the accumulators before it adds to them.
struct FetchPlan {
    int segments, slices, row_waves, early, look;
};
// row_split: requested workgroups per segment (0 = automatic); in_hbm: the residual rows are in device
// memory, not behind the host link.
// selects: the kernel makes the selection itself.
FetchPlan fetch_plan(int rfmt, const MultiShape& sh, int k, int row_split, bool in_hbm, bool selects);
// select_chunks (from fetch_select_chunks) > 0: the kernel runs the exact top-k on x itself and writes
// the selection to a.idx / a.xsel; 0: they hold the selection already (x is not read).
int fetch_select_chunks(int K, int k);
hipError_t launch_fetch(int rfmt, const CallArgs& a, int select_chunks, hipStream_t stream,
                        const KernelTimer* tm = nullptr);

// fused.hip -------------------------------------------------------------
// Base GEMV and residual kernel in one grid (the fetch workgroups come first).  over_link: residual rows in host memory.
hipError_t launch_compensated_gemv(int kind, int rfmt, const CallArgs& a, int select_chunks, bool over_link, hipStream_t stream,
                                   const KernelTimer* tm = nullptr);

// Bytes of dynamic LDS per workgroup of it.
unsigned one_grid_lds(int kind, int rbits, int nch, int k, long base_workgroups, bool over_link);

// accumulate.hip ---------------------------------------------------------
// y_m[n] = fp16( sum_s gpart[s][col0[m]+n] + sum_r cpart[r][col0[m]+n] ), the terms added in the fixed point of finalize.h
hipError_t launch_accumulate(const MultiShape& sh, void* const* y, const float* gpart, int gslices,
                             const float* cpart, int cslices, hipStream_t stream, const KernelTimer* tm = nullptr);

// A fill kernel (not hipMemsetAsync, so that callers may capture the call in a graph).
hipError_t launch_clear_u32(unsigned* p, int n, hipStream_t stream);

// quantize.hip -----------------------------------------------------------
hipError_t launch_quantize_uniform(int bits, const float* W, void* Wq, void* scales, void* zeros, void* R, int K,
                                   int N, hipStream_t stream);
hipError_t launch_residual_f32(int kind, const float* W, const void* Wq, const void* scales, const void* zeros_or_lut,
                               float* R, int K, int N, hipStream_t stream);
// Which of the two searches for the column scales a matrix gets; they give the same bits.
bool residual_scale_by_bounds(int bits, int K, int N);
hipError_t launch_quantize_residual(int bits, const float* R, void* codes_out, void* scales_out, int K, int N,
                                    hipStream_t stream);

}  // namespace decdec
