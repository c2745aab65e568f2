// Offline preparation of the residuals on the device (DecDEC Section 4.2).
//
//   residual_f32_kernel     R = W - W_hat for weights already quantised and
//                           packed (any base quantiser: the paper applies
//                           DecDEC on top of third-party quantisers, Section
//                           5.2), one fp32 subtraction per element.
//   residual_scale_kernel, residual_scale_bounds_kernel
//                           per output column the scale S of the b-bit
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
// (add_error says why they are the same) and, where there are rows enough, sums
// only the candidates that may be the least.  The conversion of a scale to fp16
// is one round-to-nearest-even done with integer arithmetic.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"
#include "layout.h"

namespace decdec {
namespace {

#pragma clang fp contract(off)

// One workgroup per tile, each of its four wavefronts 32 of the 128 channels (quantize.hip): 1024 x 1024 8.6 us -> 5.7.
constexpr int kParts = 4, kPartRows = kGroup / kParts;

// Bit p: a code of the channels of part PART has a bit in 16-byte piece p of a lane.
constexpr unsigned pieces_of_part(int kind, int part) {
    unsigned used = 0;
    for (int i = 0; i < kPartRows; ++i) {
        const CodeSlot slot = code_slot(kind, part * kPartRows + i);
        for (int r = 0; r < slot.nruns; ++r) used |= 1u << (slot.run[r].word / 4);
    }
    return used;
}

template <int KIND, int PART>
__device__ __forceinline__ void residual_part(const float* __restrict__ W, const uint4* __restrict__ tile,
                                              const _Float16* __restrict__ scales, const _Float16* __restrict__ zeros_or_lut,
                                              float* __restrict__ R, int N, int g, int n, int lane) {
    constexpr unsigned used = pieces_of_part(KIND, PART);
    uint32_t words[words_per_lane(KIND)];
#pragma unroll
    for (int p = 0; p < words_per_lane(KIND) / 4; ++p) {
        const uint4 v = (used >> p & 1u) ? tile[p * kTileCols + lane] : make_uint4(0, 0, 0, 0);
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
    const size_t at = ((size_t)g * kGroup + PART * kPartRows) * N + n;
    float w[kPartRows];
#pragma unroll
    for (int i = 0; i < kPartRows; ++i) w[i] = W[at + (size_t)i * N];
#pragma unroll
    for (int i = 0; i < kPartRows; ++i) {
        constexpr int kind = KIND, first = PART * kPartRows;
        const CodeSlot slot = code_slot(kind, first + i);
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
        R[at + (size_t)i * N] = w[i] - w_hat;
    }
}

template <int KIND>
__global__ __launch_bounds__(kParts * 64) void residual_f32_kernel(const float* __restrict__ W, const uint32_t* __restrict__ Wq,
                                                                  const _Float16* __restrict__ scales,
                                                                  const _Float16* __restrict__ zeros_or_lut,
                                                                  float* __restrict__ R, int N, int G) {
    const int lane = threadIdx.x & 63;
    const int tile_id = blockIdx.x;  // = nt * G + g
    const int nt = tile_id / G, g = tile_id - nt * G;
    const int n = nt * kTileCols + lane;
    const uint4* tile = reinterpret_cast<const uint4*>(Wq + (size_t)tile_id * (tile_bytes(KIND) / 4));
    switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
        case 0: residual_part<KIND, 0>(W, tile, scales, zeros_or_lut, R, N, g, n, lane); break;
        case 1: residual_part<KIND, 1>(W, tile, scales, zeros_or_lut, R, N, g, n, lane); break;
        case 2: residual_part<KIND, 2>(W, tile, scales, zeros_or_lut, R, N, g, n, lane); break;
        default: residual_part<KIND, 3>(W, tile, scales, zeros_or_lut, R, N, g, n, lane); break;
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

constexpr int kAlphas = 71;      // 0.30 ... 1.00
constexpr int kBins = 1024;      // of |r| / max|r|
constexpr int kPosBits = 26;     // |r| / max|r| as a whole number
constexpr int kSumBits = 44;     // field of the sum of positions in a bin's word, the count above it
constexpr int kMaxHistRows = 1 << (kSumBits - kPosBits);
constexpr int kSlots = 64;       // threads that share a column's rows
constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52
constexpr double kInf = __builtin_huge_val();

__device__ __forceinline__ uint16_t candidate_bits(int c, double m, double qmax) {
    const uint16_t h = half_bits_rne((double)(30 + c) / 100.0 * m / qmax);
    return h == 0 ? 0x3C00 : h;  // a vanishing column gets S = 1
}

// Squared error of one value v = |r| under scale S, added to err.  Five instructions that give the bits of the plain form
//     q = clip(rint(r / S), -qmax, qmax),   d = r - S q,   err = err + d d        (one rounding each)
// because
//   * |r| gives the same d d as r (every step is odd in r), and needs one clip instead of two;
//   * |r| fl(1/S) is off from r / S by less than 2^-43 (|r| / S < 1000: S is at least half of 0.3 max|r| / qmax, and
//     where it is replaced by 1, |r| < 2^-15), while a quotient that is not a half-integer is at least 2^-25 away from
//     one (S is a multiple of 2^(e-10) and |r| >= S / 2 one of 2^(e-24), S < 2^(e+1)): the same integer; and where it is
//     one, both neighbours give |d| = S / 2;
//   * adding 1.5 * 2^52 in the same fused step rounds to that integer (the products lie far below 2^51);
//   * d has at most 24 significant bits and S q at most 18, so r - S q and d d are exact, fused or not.
__device__ __forceinline__ double add_error(double v, double S, double inv, double qmax, double err) {
    const double q = fmin(__builtin_fma(v, inv, kMagic) - kMagic, qmax);
    const double d = __builtin_fma(-S, q, v);
    return __builtin_fma(d, d, err);
}

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int d = 1; d < 64; d *= 2) v = fmin(v, __shfl_xor(v, d, 64));
    return v;
}

constexpr int kScaleRows = 128;   // rows of a column block staged in LDS at a time
constexpr int kMaxSlots = 80;     // threads that share a column's candidates x candidates per thread, at most

// One workgroup = COLS columns; SLOTS = 64 * WAVES / COLS threads share a column's 71 candidate scales, APT of them
// each, so that K x 71 dependent sums per column become 71 independent chains of K, spread over the chip (one thread
// per column left three quarters of the compute units without work and walked the column six times).  The workgroup
// reads its columns twice: for max|r|, and then tile by tile through LDS, as |r| in fp64, the next tile being loaded
// while the candidates walk the current one.
//
// Bound by fp64 issue: add_error for every (element, candidate).  That is for finite values.  An infinity or a NaN in the
// column makes err a NaN for every candidate, and a NaN is never the least error: the column gets S = 1.  Rows beyond K
// count as zeros: they leave err as it is.
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
        const uint16_t h = candidate_bits(min(c, kAlphas - 1), m, qmax);
        s_bits[c][col] = h;
        S[a] = half_bits_to_double(h);
        inv[a] = 1.0 / S[a];
        err[a] = 0.0;
    }

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
                err[a] = add_error(v, S[a], inv[a], qmax, err[a]);
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

// The same scales.  One workgroup = COLS columns, kSlots threads each.  Nearly all candidates are ruled out by bounds first, so
// that what bounds the kernel is reading the columns three times (in 8 bits the bounds themselves, 127 steps a candidate):
//
//   1. max|r| of every column.
//   2. A histogram of |r|: per bin the number of values and the sum of their positions (26-bit whole numbers), one 64-bit
//      LDS atomic per value; then its sums from every bin up.
//   3. With q = sum_j [v > t_j], t_j = (j + 1/2) S, the error less sum v^2, which all candidates share, is
//          -2 S sum_j A_j + S^2 sum_j (2j + 1) C_j,     A_j, C_j = sum and number of the values above t_j.
//      The bins above the one that holds t_j belong to A_j and C_j whole.  A value v inside that bin, if counted above,
//      changes the error by -2 S (v - t_j), and the true error takes the better of both for every value; so with n values of
//      mean mu in a bin [lo, hi] the gain lies between 2 S n max(0, mu - t_j) and 2 S n (mu - lo)(hi - t_j) / (hi - lo).
//      That bounds a candidate's error to about 3e-4 of it (4 bits), rounding of the positions included.  Candidates whose
//      lower bound exceeds the least upper bound are out; one is left, or two or three.
//   4. Where more than one is left: their errors, the rows spread over the column's threads.
//   5. The result is to be the least of sums taken in ascending row order.  Sums of K terms that are not negative are off by
//      at most K 2^-53 of themselves in that order, and by (K / 64 + 80) 2^-53 here; only if two candidates are closer than
//      twice both are they summed again, in that order.
//
// Columns with an infinity or a NaN: err is a NaN for every candidate in the plain form, and a NaN is never the least error:
// S = 1.  A candidate that overflows fp16 likewise.
template <int COLS, int LEVELS, int PER_PASS>
__global__ __launch_bounds__(kSlots * COLS) void residual_scale_bounds_kernel(const float* __restrict__ R, int K, int N,
                                                                             _Float16* __restrict__ scales_out) {
    constexpr int kStride = kBins + 1;  // sums from bin b up; none from kBins up
    __shared__ unsigned long long hist[COLS * kStride];
    __shared__ unsigned s_max[COLS];
    __shared__ uint16_t s_bits[COLS][kAlphas + 1];  // fp16 scale of every candidate; one more that equals none
    __shared__ unsigned char s_left[COLS][kAlphas + 1];  // candidates that are left
    __shared__ int s_count[COLS], s_most;
    // after the bounds the histogram's place holds the errors of the candidates that are left
    double* s_err = reinterpret_cast<double*>(hist);         // [COLS][kAlphas]
    double* s_part = s_err + COLS * kAlphas;                 // [COLS wavefronts][PER_PASS][COLS]
    static_assert(COLS * kAlphas + COLS * PER_PASS * COLS <= COLS * kStride, "errors fit in the histogram's place");

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = tid % COLS, slot = tid / COLS;
    constexpr double qmax = (double)LEVELS;
    // Workgroups go to the eight XCDs in turn: give each XCD's L2 adjacent columns, so that it reads a line once.
    const int blocks = (int)gridDim.x, xcd = (int)blockIdx.x % 8;
    const int block = xcd * (blocks / 8) + min(xcd, blocks % 8) + (int)blockIdx.x / 8;
    const float* src = R + (size_t)block * COLS + col;
    const auto each_row = [&](auto&& f) {
        int k = slot;
        for (; k + 7 * kSlots < K; k += 8 * kSlots) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = src[(size_t)(k + i * kSlots) * N];
#pragma unroll
            for (int i = 0; i < 8; ++i) f(fabsf(v[i]));
        }
        for (; k < K; k += kSlots) f(fabsf(src[(size_t)k * N]));
    };

    for (int i = tid; i < COLS * kStride; i += kSlots * COLS) hist[i] = 0;
    if (tid < COLS) s_max[tid] = 0;
    if (tid == 0) s_most = 0;
    __syncthreads();
    unsigned mx = 0;  // as bits, which puts infinity and NaN above every number
    each_row([&](float v) { mx = max(mx, __builtin_bit_cast(unsigned, v)); });
#pragma unroll
    for (int d = COLS; d < 64; d *= 2) mx = max(mx, (unsigned)__shfl_xor((int)mx, d, 64));
    if (lane < COLS) atomicMax(&s_max[col], mx);
    __syncthreads();

    {
        // v * to_pos < 2^26 for v <= max|r|.  Columns whose scales all vanish, or that hold no numbers, have no use for it.
        const unsigned bits = s_max[col];
        const double m = (double)__builtin_bit_cast(float, bits);
        const bool usable = bits < 0x7F800000u && m > 1e-30;
        const float to_pos = usable ? (float)(67108800.0 / m) : 0.f;
        if (usable) {
            each_row([&](float v) {
                const unsigned p = (unsigned)(v * to_pos);
                atomicAdd(&hist[col * kStride + (p >> (kPosBits - 10))], (1ull << kSumBits) | p);
            });
        }
        __syncthreads();
        // Wavefront w turns column w's bins into sums from bin b up.
        unsigned long long* h = hist + wave * kStride;
        unsigned long long s[kBins / 64], above = 0;
#pragma unroll
        for (int i = 0; i < kBins / 64; ++i) s[i] = h[i * 64 + 63 - lane];
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
#pragma unroll
            for (int i = 0; i < kBins / 64; ++i) {
                const unsigned long long o = __shfl_up(s[i], d, 64);
                s[i] += lane >= d ? o : 0ull;
            }
        }
#pragma unroll
        for (int i = kBins / 64 - 1; i >= 0; --i) {
            const unsigned long long total = __shfl(s[i], 63, 64);
            h[i * 64 + 63 - lane] = s[i] + above;
            above += total;
        }
    }
    __syncthreads();

    // Wavefront w decides for column w, a lane per candidate.
    const int n = block * COLS + wave;
    const unsigned mbits = s_max[wave];
    const double m = (double)__builtin_bit_cast(float, mbits);
    const bool finite = mbits < 0x7F800000u;
    const bool bounded = finite && m > 1e-30;
    {
        double lower[2], upper[2], least = kInf;
        uint16_t bits[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int c = r * 64 + lane;
            lower[r] = upper[r] = kInf;
            bits[r] = 0x7C00;
            if (c >= kAlphas) continue;
            bits[r] = finite ? candidate_bits(c, m, qmax) : 0x7C00;
            s_bits[wave][c] = bits[r];
            if (bits[r] == 0x7C00) continue;
            lower[r] = -kInf;
            if (!bounded) continue;
            // in units of positions
            const double to_pos = (double)(float)(67108800.0 / m), S = half_bits_to_double(bits[r]) * to_pos;
            const unsigned long long* h = hist + wave * kStride;
            constexpr double kSlack = 5.0;  // a position: truncated, of a product rounded to 24 bits of 26
            constexpr unsigned long long kSumMask = (1ull << kSumBits) - 1;
            double sum_a = 0.0, sum_c = 0.0, gain_hi = 0.0, gain_lo = 0.0, sum_q = 0.0;
#pragma unroll
            for (int j = 0; j < LEVELS; ++j) {
                const double t = ((double)j + 0.5) * S;
                const int b = (int)fmin(t * (1.0 / (1 << (kPosBits - 10))), (double)kBins);  // kBins: above every value
                const unsigned long long up = h[min(b + 1, kBins)], own = h[b] - up;
                const double a_n = (double)(up >> kSumBits), o_n = (double)(own >> kSumBits);
                sum_a += (double)(up & kSumMask) + 0.5 * a_n;
                sum_c += (2.0 * j + 1.0) * a_n;
                const double before_n = (double)((h[max(b - 1, 0)] - h[b]) >> kSumBits);  // may be above t by rounding
                sum_q += a_n + o_n + before_n;
                const double lo = (double)b * (1 << (kPosBits - 10)) - kSlack, hi = lo + (1 << (kPosBits - 10)) + 2.0 * kSlack;
                const double o_sum = (double)(own & kSumMask) + 0.5 * o_n;  // n mu
                gain_lo += fmax(0.0, o_sum - o_n * t);
                gain_hi += fmax(0.0, o_sum - o_n * lo) * (hi - t) * (1.0 / ((1 << (kPosBits - 10)) + 2.0 * kSlack));
            }
            const double f = S * (S * sum_c - 2.0 * sum_a), slack = S * (2.0 * kSlack * sum_q + 1e-9 * (sum_a + S * sum_c));
            upper[r] = f - 2.0 * S * gain_lo + slack;
            lower[r] = f - 2.0 * S * gain_hi - slack;
            least = fmin(least, upper[r]);
        }
        least = wave_min(least);
        if (lane == 0) s_bits[wave][kAlphas] = 0;
        wave_writes_seen();
        int count = 0;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int c = r * 64 + lane;
            // of equal scales the one with the larger alpha
            const bool left = c < kAlphas && bits[r] != 0x7C00 && lower[r] <= least && s_bits[wave][c + 1] != bits[r];
            const unsigned long long mask = __ballot(left);
            if (left) s_left[wave][count + __builtin_popcountll(mask & ((1ull << lane) - 1))] = (unsigned char)c;
            count += __builtin_popcountll(mask);
        }
        wave_writes_seen();
        if (lane == 0) {
            if (count <= 1) scales_out[n] = __builtin_bit_cast(_Float16, count == 1 ? s_bits[wave][s_left[wave][0]] : (uint16_t)0x3C00);
            s_count[wave] = count <= 1 ? 0 : count;
            if (count > 1) atomicMax(&s_most, count);
        }
    }
    __syncthreads();

    const int rounds = (s_most + PER_PASS - 1) / PER_PASS, mine = s_count[col];
    for (int r = 0; r < rounds; ++r) {
        double S[PER_PASS], inv[PER_PASS], err[PER_PASS];
#pragma unroll
        for (int a = 0; a < PER_PASS; ++a) {
            const int i = min(r * PER_PASS + a, max(mine - 1, 0));
            S[a] = mine > 0 ? half_bits_to_double(s_bits[col][s_left[col][i]]) : 1.0;
            inv[a] = 1.0 / S[a];
            err[a] = 0.0;
        }
        // For all columns of the workgroup as many as the one with the most has left, which is two as a rule: four each, 4096 x
        // 4096 took 63 us for 4 bits and 74 for 2 instead of 59 and 48.
        const auto sum_errors = [&](auto count) {
            each_row([&](float f) {
                const double v = (double)f;
#pragma unroll
                for (int a = 0; a < decltype(count)::value; ++a) err[a] = add_error(v, S[a], inv[a], qmax, err[a]);
            });
        };
        if (s_most - r * PER_PASS <= 2) {
            sum_errors(std::integral_constant<int, 2>());
        } else {
            sum_errors(std::integral_constant<int, PER_PASS>());
        }
#pragma unroll
        for (int a = 0; a < PER_PASS; ++a) {
#pragma unroll
            for (int d = COLS; d < 64; d *= 2) err[a] += __shfl_xor(err[a], d, 64);
            if (lane < COLS) s_part[(wave * PER_PASS + a) * COLS + lane] = err[a];
        }
        __syncthreads();
        if (tid < PER_PASS * COLS) {
            const int a = tid / COLS, c = tid % COLS, i = r * PER_PASS + a;
            double sum = 0.0;
            for (int w = 0; w < COLS; ++w) sum += s_part[(w * PER_PASS + a) * COLS + c];
            if (i < s_count[c]) s_err[c * kAlphas + i] = sum;
        }
        __syncthreads();
    }

    const int count = s_count[wave];
    if (count == 0) return;
    const double tolerance = 2.0 * ((double)K * (1.0 + 1.0 / kSlots) + 80.0) * 1.2e-16;
    double err[2], best = kInf;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int i = r * 64 + lane;
        err[r] = i < count ? s_err[wave * kAlphas + i] : kInf;
        best = fmin(best, err[r]);
    }
    best = wave_min(best);
    bool close[2];
    int n_close = 0;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        close[r] = r * 64 + lane < count && err[r] <= best * (1.0 + tolerance);
        n_close += __builtin_popcountll(__ballot(close[r]));
    }
    if (n_close > 1 && best > 0.0) {
        // too close to tell: the sums in ascending row order
        const float* column = R + n;
        double S[2], inv[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            S[r] = close[r] ? half_bits_to_double(s_bits[wave][s_left[wave][r * 64 + lane]]) : 1.0;
            inv[r] = 1.0 / S[r];
            err[r] = 0.0;
        }
        int k = 0;
        for (; k + 8 <= K; k += 8) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = column[(size_t)(k + i) * N];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
#pragma unroll
                for (int r = 0; r < 2; ++r) err[r] = add_error((double)fabsf(v[i]), S[r], inv[r], qmax, err[r]);
            }
        }
        for (; k < K; ++k) {
#pragma unroll
            for (int r = 0; r < 2; ++r) err[r] = add_error((double)fabsf(column[(size_t)k * N]), S[r], inv[r], qmax, err[r]);
        }
        best = kInf;
#pragma unroll
        for (int r = 0; r < 2; ++r) best = fmin(best, close[r] ? err[r] : kInf);
        best = wave_min(best);
    }
    // the last one, that is the one with the largest alpha, of those with the least error
    int at = -1;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const unsigned long long mask = __ballot(close[r] && err[r] == best);
        if (mask) at = r * 64 + 63 - __builtin_clzll(mask);
    }
    if (lane == 0) scales_out[n] = __builtin_bit_cast(_Float16, at < 0 ? (uint16_t)0x3C00 : s_bits[wave][s_left[wave][at]]);
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

// N is a multiple of 16.
void launch_scale_direct(const float* R, int K, int N, double qmax, _Float16* S, hipStream_t stream) {
    // Few columns: narrow blocks with one candidate per thread, so that every compute unit has
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
}

template <int LEVELS>
void launch_scale_bounds(const float* R, int K, int N, _Float16* S, hipStream_t stream) {
    // as many columns per workgroup (their histograms fill the LDS) as leave about a workgroup for every compute unit
    if (N <= 1024) {
        residual_scale_bounds_kernel<4, LEVELS, 4><<<dim3((unsigned)(N / 4)), dim3(4 * kSlots), 0, stream>>>(R, K, N, S);
    } else if (N <= 2048) {
        residual_scale_bounds_kernel<8, LEVELS, 4><<<dim3((unsigned)(N / 8)), dim3(8 * kSlots), 0, stream>>>(R, K, N, S);
    } else {
        residual_scale_bounds_kernel<16, LEVELS, 4><<<dim3((unsigned)(N / 16)), dim3(16 * kSlots), 0, stream>>>(R, K, N, S);
    }
}

}  // namespace

hipError_t launch_residual_f32(int kind, const float* W, const void* Wq, const void* scales, const void* zeros_or_lut,
                               float* R, int K, int N, hipStream_t stream) {
    const int G = K / kGroup, tiles = (N / kTileCols) * G;
    const dim3 grid((unsigned)tiles), block(kParts * 64);
    const uint32_t* q = static_cast<const uint32_t*>(Wq);
    const _Float16* s = static_cast<const _Float16*>(scales);
    const _Float16* z = static_cast<const _Float16*>(zeros_or_lut);
    switch (kind) {
        case PACK_U4: residual_f32_kernel<PACK_U4><<<grid, block, 0, stream>>>(W, q, s, z, R, N, G); break;
        case PACK_U3: residual_f32_kernel<PACK_U3><<<grid, block, 0, stream>>>(W, q, s, z, R, N, G); break;
        case PACK_LUT3: residual_f32_kernel<PACK_LUT3><<<grid, block, 0, stream>>>(W, q, s, z, R, N, G); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Bounds first, where they pay: not for few rows, which for 8 bits, with 127 steps per candidate, are more; nor from
// kMaxHistRows on, where the fields of a bin's word are too small, nor where a grid would have 2^32 threads.  us, search and
// encoding into GPU memory, all candidates in fp64 / bounds first, 4 bits: 256 x 4096 25 / 29; 256 x 1024 16 / 16; 512 x 4096
// 44 / 33; 1024 x 1024 35 / 17; 4096 x 256 106 / 23; 4096 x 4096 264 / 80; 14336 x 4096 901 / 220; 4096 x 14336 908 / 255.
// 8 bits, residuals of the 3-bit quantiser: 1024 x 1024 36 / 74; 2048 x 4096 153 / 184; 3072 x 4096 212 / 199; 4096 x 1024
// 113 / 87; 4096 x 4096 275 / 209; 14336 x 4096 915 / 451; 4096 x 14336 921 / 747.
bool residual_scale_by_bounds(int bits, int K, int N) {
    return K >= (bits == 8 ? 4096 : 384) && K < kMaxHistRows && (long)N * kSlots < 1L << 32;
}

hipError_t launch_quantize_residual(int bits, const float* R, void* codes_out, void* scales_out, int K, int N,
                                    hipStream_t stream) {
    if (bits != 2 && bits != 4 && bits != 8) return hipErrorInvalidValue;
    _Float16* S = static_cast<_Float16*>(scales_out);
    if (!residual_scale_by_bounds(bits, K, N)) {
        launch_scale_direct(R, K, N, (double)((1 << (bits - 1)) - 1), S, stream);
    } else if (bits == 8) {
        launch_scale_bounds<127>(R, K, N, S, stream);
    } else if (bits == 4) {
        launch_scale_bounds<7>(R, K, N, S, stream);
    } else {
        launch_scale_bounds<1>(R, K, N, S, stream);
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
