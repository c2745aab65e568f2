// Offline preparation of the residuals on the device (DecDEC Section 4.2).
//
//   residual_f32_kernel     R = W - W_hat for weights already quantised and
//                           packed (any base quantiser: the paper applies
//                           DecDEC on top of third-party quantisers, Section
//                           5.2), one fp32 subtraction per element.
//   residual_scale_kernel   per output column the scale S of the b-bit
//                           symmetric quantiser  Q(r) = clip(rint(r / S),
//                           -qmax, qmax),  qmax = 2^(b-1) - 1, found by grid
//                           search for the least squared error over
//                           S = fp16(alpha * max|r| / qmax), alpha = 0.30,
//                           0.31, ..., 1.00 (a tie keeps the larger alpha).
//   residual_encode_kernel  the codes, packed row by row for the fetch kernel.
//
// Scales and codes have the bits that one IEEE fp64 operation per step gives,
// the error of a column summed over its rows in ascending order, so that a CPU
// can reproduce them; the search takes fewer, fused steps with the same results
// (residual_scale_kernel says why they are the same).  The conversion of a scale
// to fp16 is one round-to-nearest-even done with integer arithmetic.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "layout.h"

namespace decdec {
namespace {

#pragma clang fp contract(off)

template <int KIND>
__global__ __launch_bounds__(256) void residual_f32_kernel(const float* __restrict__ W,
                                                          const uint32_t* __restrict__ Wq,
                                                          const _Float16* __restrict__ scales,
                                                          const _Float16* __restrict__ zeros_or_lut,
                                                          float* __restrict__ R, int N, int G, int tiles) {
    const int lane = threadIdx.x & 63;
    const int tile_id = blockIdx.x * 4 + (threadIdx.x >> 6);  // = nt * G + g
    if (tile_id >= tiles) return;
    const int nt = tile_id / G, g = tile_id - nt * G;
    const int n = nt * kTileCols + lane;

    uint32_t words[words_per_lane(KIND)];
    const uint4* tile = reinterpret_cast<const uint4*>(Wq + (size_t)tile_id * (tile_bytes(KIND) / 4));
#pragma unroll
    for (int p = 0; p < words_per_lane(KIND) / 4; ++p) {
        const uint4 v = tile[p * kTileCols + lane];
        words[4 * p] = v.x;
        words[4 * p + 1] = v.y;
        words[4 * p + 2] = v.z;
        words[4 * p + 3] = v.w;
    }
    float s = 0.f, z = 0.f, lut[8];
    if constexpr (KIND == PACK_LUT3) {
#pragma unroll
        for (int c = 0; c < 8; ++c) lut[c] = (float)zeros_or_lut[(size_t)n * 8 + c];
    } else {
        s = (float)scales[(size_t)g * N + n];
        z = (float)zeros_or_lut[(size_t)g * N + n];
    }
#pragma unroll
    for (int i = 0; i < kGroup; ++i) {
        constexpr int kind = KIND;
        const CodeSlot slot = code_slot(kind, i);
        uint32_t q = 0;
#pragma unroll
        for (int r = 0; r < slot.nruns; ++r) {
            const BitRun br = slot.run[r];
            q |= ((words[br.word] >> br.bit) & ((1u << br.nbits) - 1u)) << br.code_bit;
        }
        float w_hat;
        if constexpr (KIND == PACK_LUT3) {
            w_hat = lut[0];
#pragma unroll
            for (int c = 1; c < 8; ++c) w_hat = q == (uint32_t)c ? lut[c] : w_hat;
        } else {
            w_hat = s * ((float)q - z);  // exact: an 11-bit scale times an integer below 16
        }
        const size_t at = ((size_t)g * kGroup + i) * N + n;
        R[at] = W[at] - w_hat;
    }
}

// fp16 bits of v >= 0 (finite), rounded to nearest even: what a correctly
// rounded conversion of the fp64 value gives.
__device__ __forceinline__ uint16_t half_bits_rne(double v) {
    if (!(v > 0.0)) return 0;
    if (v >= 65520.0) return 0x7C00;                       // rounds to infinity
    if (v < 6.103515625e-05) return (uint16_t)rint(v * 16777216.0);  // below 2^-14: multiples of 2^-24
    const int e = (int)((__double_as_longlong(v) >> 52) & 0x7FF) - 1023;  // 2^e <= v < 2^(e+1), -14 <= e <= 15
    const double scaled = v * __longlong_as_double((long long)(1023 + 10 - e) << 52);  // in [1024, 2048), exact
    const int r = (int)rint(scaled);                        // 1024 .. 2048
    return (uint16_t)(((e + 15) << 10) + (r - 1024));       // r = 2048 carries into the exponent
}

__device__ __forceinline__ double half_bits_to_double(uint16_t h) {
    return (double)(float)__builtin_bit_cast(_Float16, h);
}

constexpr int kAlphas = 71;       // 0.30 ... 1.00
constexpr int kScaleRows = 128;   // rows of a column block staged in LDS at a time
constexpr int kMaxSlots = 80;     // threads that share a column's candidates x candidates per thread, at most

// One workgroup = COLS columns; SLOTS = 64 * WAVES / COLS threads share a column's 71 candidate scales, APT of them
// each, so that K x 71 dependent sums per column become 71 independent chains of K, spread over the chip (one thread
// per column left three quarters of the compute units without work and walked the column six times).  The workgroup
// reads its columns twice: for max|r|, and then tile by tile through LDS, as |r| in fp64, the next tile being loaded
// while the candidates walk the current one.
//
// Bound by fp64 issue: five instructions per (element, candidate).  They give the bits of the plain form
//     q = clip(rint(r / S), -qmax, qmax),   d = r - S q,   err = err + d d        (one rounding each)
// because
//   * |r| gives the same d d as r (every step is odd in r), and needs one clip instead of two;
//   * |r| fl(1/S) is off from r / S by less than 2^-43 (|r| / S < 1000: S is at least half of 0.3 max|r| / qmax, and
//     where it is replaced by 1, |r| < 2^-15), while a quotient that is not a half-integer is at least 2^-25 away from
//     one (S is a multiple of 2^(e-10) and |r| >= S / 2 one of 2^(e-24), S < 2^(e+1)): the same integer; and where it is
//     one, both neighbours give |d| = S / 2;
//   * adding 1.5 * 2^52 in the same fused step rounds to that integer (the products lie far below 2^51);
//   * d has at most 24 significant bits and S q at most 18, so r - S q and d d are exact, fused or not.
// That is for finite values.  An infinity or a NaN in the column makes err a NaN for every candidate, and a NaN is never
// the least error: the column gets S = 1.  Rows beyond K count as zeros: they leave err as it is.
// A 4096 x 4096 layer prepared with 4-bit residual codes: 18.8 -> 0.47 ms, of which the search is now 0.26 (0.15 at
// the issue rate) and the way of the codes to pinned host memory 0.15.
template <int COLS, int WAVES, int APT>
__global__ __launch_bounds__(64 * WAVES) void residual_scale_kernel(const float* __restrict__ R, int K, int N,
                                                                   double qmax, _Float16* __restrict__ scales_out) {
    constexpr int THREADS = 64 * WAVES, SLOTS = THREADS / COLS;
    constexpr int PER_TILE = (kScaleRows * COLS + THREADS - 1) / THREADS;  // elements of a tile per thread
    static_assert(SLOTS * COLS == THREADS && SLOTS * APT >= kAlphas && SLOTS * APT <= kMaxSlots, "scale search shape");
    __shared__ double tile[kScaleRows * COLS];
    __shared__ double s_err[kMaxSlots][COLS];
    __shared__ uint16_t s_bits[kMaxSlots][COLS];
    __shared__ float s_max[SLOTS][COLS];

    const int tid = threadIdx.x;
    const int col = tid % COLS, slot = tid / COLS;
    // Workgroups go to the eight XCDs in turn: give each XCD's L2 adjacent columns, so that it reads a line once.
    const int blocks = (int)gridDim.x, xcd = (int)blockIdx.x % 8;
    const int block = xcd * (blocks / 8) + min(xcd, blocks % 8) + (int)blockIdx.x / 8;
    const float* src = R + (size_t)block * COLS + col;

    float mx = 0.f;
    int k = slot;
    for (; k + 7 * SLOTS < K; k += 8 * SLOTS) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = src[(size_t)(k + i * SLOTS) * N];
#pragma unroll
        for (int i = 0; i < 8; ++i) mx = fmaxf(mx, fabsf(v[i]));
    }
    for (; k < K; k += SLOTS) mx = fmaxf(mx, fabsf(src[(size_t)k * N]));
    s_max[slot][col] = mx;
    __syncthreads();
    for (int s = 0; s < SLOTS; ++s) mx = fmaxf(mx, s_max[s][col]);
    const double m = (double)mx;

    double S[APT], inv[APT], err[APT];
#pragma unroll
    for (int a = 0; a < APT; ++a) {
        const int c = slot * APT + a;
        const double alpha = (double)(30 + min(c, kAlphas - 1)) / 100.0;
        uint16_t h = half_bits_rne(alpha * m / qmax);
        if (h == 0) h = 0x3C00;  // an all-zero (or vanishing) column gets S = 1
        s_bits[c][col] = h;
        S[a] = half_bits_to_double(h);
        inv[a] = 1.0 / S[a];
        err[a] = 0.0;
    }

    constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52
    float next[PER_TILE];
    const auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < PER_TILE; ++i) {
            const int r = slot + i * SLOTS;
            next[i] = r < kScaleRows && k0 + r < K ? src[(size_t)(k0 + r) * N] : 0.f;
        }
    };
    load(0);
    for (int k0 = 0; k0 < K; k0 += kScaleRows) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER_TILE; ++i) {
            const int r = slot + i * SLOTS;
            if (r < kScaleRows) tile[r * COLS + col] = fabs((double)next[i]);
        }
        __syncthreads();
        load(k0 + kScaleRows);
#pragma unroll 8
        for (int r = 0; r < kScaleRows; ++r) {
            const double v = tile[r * COLS + col];
#pragma unroll
            for (int a = 0; a < APT; ++a) {
                const double q = fmin(__builtin_fma(v, inv[a], kMagic) - kMagic, qmax);
                const double d = __builtin_fma(-S[a], q, v);
                err[a] = __builtin_fma(d, d, err[a]);
            }
        }
    }
#pragma unroll
    for (int a = 0; a < APT; ++a) s_err[slot * APT + a][col] = err[a];
    __syncthreads();
    if (tid < COLS) {
        double best_err = __longlong_as_double(0x7FF0000000000000LL);  // +inf
        uint16_t best = 0x3C00;                                        // 1.0
        for (int a = 0; a < kAlphas; ++a) {
            if (s_err[a][tid] <= best_err) {
                best_err = s_err[a][tid];
                best = s_bits[a][tid];
            }
        }
        scales_out[(size_t)block * COLS + tid] = __builtin_bit_cast(_Float16, best);
    }
}

// One thread per 32-bit word of the packed rows: 32 / BITS columns of one row.
template <int BITS>
__global__ __launch_bounds__(256) void residual_encode_kernel(const float* __restrict__ R,
                                                             const _Float16* __restrict__ scales,
                                                             uint32_t* __restrict__ out, int K, int N) {
    constexpr int CPW = 32 / BITS;
    const double qmax = (double)((1 << (BITS - 1)) - 1);
    const int words_per_row = N / CPW;
    const size_t id = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= (size_t)K * words_per_row) return;
    const int k = (int)(id / words_per_row), w = (int)(id - (size_t)k * words_per_row);
    uint32_t word = 0;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int n = w * CPW + i;
        const double S = (double)(float)scales[n];
        const int q = (int)fmin(fmax(rint((double)R[(size_t)k * N + n] / S), -qmax), qmax);
        word |= ((uint32_t)q & ((1u << BITS) - 1u)) << (BITS * i);
    }
    out[id] = word;
}

}  // namespace

hipError_t launch_residual_f32(int kind, const float* W, const void* Wq, const void* scales, const void* zeros_or_lut,
                               float* R, int K, int N, hipStream_t stream) {
    const int G = K / kGroup, tiles = (N / kTileCols) * G;
    const dim3 grid((unsigned)((tiles + 3) / 4)), block(256);
    const uint32_t* q = static_cast<const uint32_t*>(Wq);
    const _Float16* s = static_cast<const _Float16*>(scales);
    const _Float16* z = static_cast<const _Float16*>(zeros_or_lut);
    switch (kind) {
        case PACK_U4: residual_f32_kernel<PACK_U4><<<grid, block, 0, stream>>>(W, q, s, z, R, N, G, tiles); break;
        case PACK_U3: residual_f32_kernel<PACK_U3><<<grid, block, 0, stream>>>(W, q, s, z, R, N, G, tiles); break;
        case PACK_LUT3: residual_f32_kernel<PACK_LUT3><<<grid, block, 0, stream>>>(W, q, s, z, R, N, G, tiles); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_quantize_residual(int bits, const float* R, void* codes_out, void* scales_out, int K, int N,
                                    hipStream_t stream) {
    if (bits != 2 && bits != 4 && bits != 8) return hipErrorInvalidValue;
    const double qmax = (double)((1 << (bits - 1)) - 1);
    _Float16* S = static_cast<_Float16*>(scales_out);
    // N is a multiple of 16.  Few columns: narrow blocks with one candidate per thread, so that every compute unit has
    // work; many: wide blocks, which read whole 64-byte pieces of a row and convert and load it for more candidates at
    // once.  The line at 6144 columns: three workgroups of nine wavefronts fit a compute unit, so that up to there all
    // run at once.  With 4096 rows, search and encoding into GPU memory, blocks of 4 / 8 / 16 columns, us: N = 256
    // 110 / 146 / 340; 1024 119 / 152 / 346; 2048 186 / 165 / 353; 4096 304 / 267 / 358; 6144 434 / 383 / 510; 8192
    // 549 / 616 / 520; 14336 961 / 984 / 921.
    if (N <= 1024) {
        residual_scale_kernel<4, 5, 1><<<dim3((unsigned)(N / 4)), dim3(320), 0, stream>>>(R, K, N, qmax, S);
    } else if (N <= 6144) {
        residual_scale_kernel<8, 9, 1><<<dim3((unsigned)(N / 8)), dim3(576), 0, stream>>>(R, K, N, qmax, S);
    } else {
        residual_scale_kernel<16, 4, 5><<<dim3((unsigned)(N / 16)), dim3(256), 0, stream>>>(R, K, N, qmax, S);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t words = (size_t)K * (size_t)(N / (32 / bits));
    const dim3 grid((unsigned)((words + 255) / 256)), block(256);
    uint32_t* out = static_cast<uint32_t*>(codes_out);
    if (bits == 2) residual_encode_kernel<2><<<grid, block, 0, stream>>>(R, S, out, K, N);
    if (bits == 4) residual_encode_kernel<4><<<grid, block, 0, stream>>>(R, S, out, K, N);
    if (bits == 8) residual_encode_kernel<8><<<grid, block, 0, stream>>>(R, S, out, K, N);
    return hipGetLastError();
}

}  // namespace decdec
