// Offline preparation on the device: uniform min/max group-128 quantiser that
// writes the packed codes (layout.h), the fp16 scales and zero points, and the
// fp16 residual R = W - W_hat that DecDEC keeps in CPU memory (Section 3.1).
// The paper takes its base quantisers from third-party work (Section 5.2) and
// prints no formula; the formula is stated in decdec.h.  Every decision is one
// IEEE fp32 operation (correctly rounded divide, no fusion that changes a
// result), so the codes are reproducible bit for bit on a CPU.
//
// One workgroup handles one tile (128 input channels x 64 columns), each of its four wavefronts 32 of the channels, one lane
// per column: a row of W is one 256-byte load, the lane's 32 values stay in registers, and the column's range is taken over
// the wavefronts through LDS.  With a whole tile per wavefront (128 loads, divisions and codes in a row, 128 wavefronts
// for a 1024 x 1024 matrix) that took 9.8 us instead of 5.7, 4096 x 4096 20 instead of 16.5.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "layout.h"

namespace decdec {
namespace {

constexpr int kParts = 4, kPartRows = kGroup / kParts;  // wavefronts of a tile, channels of each

// The codes of the 32 channels of part PART, as their bits of the lane's words of the tile, and the fp16 residual.
template <int KIND, int PART>
__device__ __forceinline__ void encode_part(const float (&w)[kPartRows], float s, float z, float qmax,
                                            uint32_t (&words)[words_per_lane(KIND)], _Float16* R, int N) {
#pragma unroll
    for (int i = 0; i < kPartRows; ++i) {
        const float qf = fminf(fmaxf(rintf(w[i] / s) + z, 0.f), qmax);
        const uint32_t q = (uint32_t)qf;
        constexpr int kind = KIND, first = PART * kPartRows;
        const CodeSlot slot = code_slot(kind, first + i);
#pragma unroll
        for (int r = 0; r < slot.nruns; ++r) {
            const BitRun br = slot.run[r];
            words[br.word] |= ((q >> br.code_bit) & ((1u << br.nbits) - 1u)) << br.bit;
        }
        if (R != nullptr) R[(size_t)i * N] = (_Float16)(w[i] - s * (qf - z));
    }
}

template <int KIND, int BITS>
__global__ __launch_bounds__(kParts * 64) void quantize_uniform_kernel(const float* __restrict__ W, uint32_t* __restrict__ Wq,
                                                              _Float16* __restrict__ scales,
                                                              _Float16* __restrict__ zeros, _Float16* __restrict__ R,
                                                              int N, int G) {
    constexpr int kWords = words_per_lane(KIND);
    __shared__ float s_lo[kParts][kTileCols], s_hi[kParts][kTileCols];
    __shared__ uint32_t s_words[kWords][kTileCols];
    const int lane = threadIdx.x & 63;
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile_id = blockIdx.x;  // = nt * G + g
    const int nt = tile_id / G, g = tile_id - nt * G;
    const int n = nt * kTileCols + lane;
    const size_t at = ((size_t)g * kGroup + part * kPartRows) * N + n;

    float w[kPartRows];
#pragma unroll
    for (int i = 0; i < kPartRows; ++i) w[i] = W[at + (size_t)i * N];
#pragma unroll
    for (int i = part; i < kWords; i += kParts) s_words[i][lane] = 0u;
    float lo = w[0], hi = w[0];
#pragma unroll
    for (int i = 1; i < kPartRows; ++i) {
        lo = fminf(lo, w[i]);
        hi = fmaxf(hi, w[i]);
    }
    s_lo[part][lane] = lo;
    s_hi[part][lane] = hi;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
        lo = fminf(lo, s_lo[p][lane]);
        hi = fmaxf(hi, s_hi[p][lane]);
    }
    constexpr float qmax = (float)((1 << BITS) - 1);
    _Float16 s16 = (_Float16)((hi - lo) / qmax);
    if (s16 == (_Float16)0.f) s16 = (_Float16)1.f;
    const float s = (float)s16;
    const float z = fminf(fmaxf(rintf(-lo / s), 0.f), qmax) + 0.f;  // + 0: a zero point is never -0

    uint32_t words[kWords];
#pragma unroll
    for (int i = 0; i < kWords; ++i) words[i] = 0u;
    _Float16* r = R != nullptr ? R + at : nullptr;
    switch (part) {
        case 0: encode_part<KIND, 0>(w, s, z, qmax, words, r, N); break;
        case 1: encode_part<KIND, 1>(w, s, z, qmax, words, r, N); break;
        case 2: encode_part<KIND, 2>(w, s, z, qmax, words, r, N); break;
        default: encode_part<KIND, 3>(w, s, z, qmax, words, r, N); break;
    }
    // words that hold codes of more than one part meet in LDS
#pragma unroll
    for (int i = 0; i < kWords; ++i)
        if (words[i] != 0u) atomicOr(&s_words[i][lane], words[i]);
    __syncthreads();
    if (part < kWords / 4) {
        const uint4 v = make_uint4(s_words[4 * part][lane], s_words[4 * part + 1][lane], s_words[4 * part + 2][lane],
                                   s_words[4 * part + 3][lane]);
        reinterpret_cast<uint4*>(Wq + (size_t)tile_id * (tile_bytes(KIND) / 4))[part * kTileCols + lane] = v;
    }
    if (part == 0) scales[(size_t)g * N + n] = s16;
    if (part == 1) zeros[(size_t)g * N + n] = (_Float16)z;
}

}  // namespace

hipError_t launch_quantize_uniform(int bits, const float* W, void* Wq, void* scales, void* zeros, void* R, int K,
                                   int N, hipStream_t stream) {
    const int G = K / kGroup, tiles = (N / kTileCols) * G;
    const dim3 grid((unsigned)tiles), block(kParts * 64);
    if (bits == 4) {
        quantize_uniform_kernel<PACK_U4, 4><<<grid, block, 0, stream>>>(
            W, static_cast<uint32_t*>(Wq), static_cast<_Float16*>(scales), static_cast<_Float16*>(zeros),
            static_cast<_Float16*>(R), N, G);
    } else if (bits == 3) {
        quantize_uniform_kernel<PACK_U3, 3><<<grid, block, 0, stream>>>(
            W, static_cast<uint32_t*>(Wq), static_cast<_Float16*>(scales), static_cast<_Float16*>(zeros),
            static_cast<_Float16*>(R), N, G);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace decdec
