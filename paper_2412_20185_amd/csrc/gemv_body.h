// Device code of the base GEMV (included by gemv.hip and fused.hip).
//
// Base GEMV  o_b = W_hat x  for 3/4-bit weights at batch 1 (DecDEC Section 4.1:
// the base GEMV the compensation runs beside; Section 2.2: weights are
// de-quantised on the fly and multiplied with fp16 activations).
//
// gfx950 design.  The work is a stream over the packed weights (HBM bound), so
// there is no MFMA here; what has to be kept small is the number of vector
// instructions per weight, and what stands in front of and behind the stream:
//   * a lane owns one output column of one 128-channel quantisation group (=
//     one tile of 64 columns, see layout.h) at a time.  A wavefront takes 64
//     columns of one group, 32 of two or 16 of four: with narrow blocks of
//     columns a small matrix still has a workgroup for every compute unit when
//     one workgroup covers all of K, and nothing has to be added across
//     workgroups.  A 128-bit load of a wavefront is four contiguous pieces of
//     256 bytes or fewer, longer ones;
//   * a lane never converts a code: a masked code field inside the fp16
//     mantissa is the subnormal  code * 2^(p-24), which v_dot2_f32_f16
//     multiplies with an (x[2j], x[2j+1]) pair and accumulates in fp32; fields
//     are used at two bit positions p (4 and 7), each with its own
//     accumulators, combined once per group;
//   * every row of 16 lanes holds the 64 activation pairs of its group, four a
//     lane, loaded beside the weights; the dot reads the pair it needs from
//     another lane of the row as it goes (dot2_x);
//   * the zero point is factored out of the inner loop:
//     sum_k s (q_k - z) x_k = s (sum_k q_k x_k - z sum_k x_k), with the
//     group's sum of x formed once per row by a DPP reduction;
//   * a wavefront asks for one tile and works it off; what hides the trip to
//     memory is the other wavefronts of the compute unit (gemv_plan says how
//     many workgroups of how many wavefronts).  Only where a caller asks for
//     long chains of few wavefronts are several tiles on their way;
//   * a workgroup adds the sums of its wavefronts through LDS and either writes
//     y itself (it covers all of K and there is no residual term) or adds them
//     into the per-column accumulators with one atomic per column (finalize.h).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "finalize.h"
#include "kernels.h"
#include "layout.h"

namespace decdec {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float acc) {
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, a), __builtin_bit_cast(half2_t, b), acc, false);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xF, false));
}

// Sum over the 16 lanes of a row, in every lane of it.
__device__ __forceinline__ float row_sum(float v) {
    v += dpp_move<0xB1, 0xF>(v);   // quad_perm [1,0,3,2]
    v += dpp_move<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
    v += dpp_move<0x141, 0xF>(v);  // row_half_mirror
    v += dpp_move<0x140, 0xF>(v);  // row_mirror
    return v;
}

// Sum over the lanes that are a multiple of COLS apart, in every one of them.
template <int COLS>
__device__ __forceinline__ float sum_over_groups(float v) {
    if constexpr (COLS <= 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
        v = __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
    }
    if constexpr (COLS <= 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
        v = __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
    }
    return v;
}

// A field at bits p..p+b-1 of an fp16 pattern with nothing else set is the
// subnormal code * 2^(p-24).  The dot unit keeps full fp32 accuracy for such
// operands only when the field's top bit is mantissa bit 6 or above, so every
// field is moved to p = 4 or p = 7 first; accumulators are rescaled by 2^-p
// and by 2^24 once per group.
constexpr float kTwoPow24 = 16777216.f;

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// acc += code pair . activation pair J of the group.  Every row of 16 lanes holds the group's 64 pairs, lane l the pairs
// 4 l .. 4 l + 3, and the dot reads the pair from its lane of the row (row_newbcast): an activation costs no instruction, no
// LDS access and no scalar register, and the rows of a wavefront may work on different groups.  With eight wavefronts a SIMD
// it takes the time of a dot with a scalar operand, 4.2 cycles (an AND or a shift 2.3), with one alone 5.7 instead of 5.1.
// The compiler neither forms this instruction nor knows what is
// inside an asm statement: the two waits that it would insert itself are in dot_operands_ready and dot_results_ready.
template <int J>
__device__ __forceinline__ float dot2_x(uint32_t code, const uint4& x, float acc) {
    const uint32_t v = (J & 3) == 0 ? x.x : (J & 3) == 1 ? x.y : (J & 3) == 2 ? x.z : x.w;
    asm("v_dot2c_f32_f16_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(v), "v"(code), "n"(J >> 2));
    return acc;
}
// A register that a DPP operand names must not have been written by either of the two vector instructions in front.
__device__ __forceinline__ void dot_operands_ready(uint4& x) {
    asm volatile("s_nop 1" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w));
}
// Three wait states between a dot and another kind of instruction that reads its result.
__device__ __forceinline__ void dot_results_ready(float& a, float& b) { asm("s_nop 2" : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void dot_results_ready(float& a, float& b, float& c, float& d) {
    asm("s_nop 2" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}

// f(0) ... f(TO - 1), the argument a compile-time constant.
template <int TO, int FROM = 0, typename F>
__device__ __forceinline__ void unroll(F&& f) {
    if constexpr (FROM < TO) {
        f(std::integral_constant<int, FROM>{});
        unroll<TO, FROM + 1>(f);
    }
}

// Partial sums of one group for one lane.
template <int KIND>
struct GroupAcc;

// 4-bit layout: word w, nibble i of each half -> pair 4w + i.
template <>
struct GroupAcc<PACK_U4> {
    float a = 0.f, b = 0.f, c = 0.f, d = 0.f;
    __device__ __forceinline__ void add(const uint32_t* wd, const uint4& x) {
        unroll<16>([&](auto W) {
            constexpr int w = decltype(W)::value;
            const uint32_t t = wd[w];
            a = dot2_x<4 * w + 0>((t << 4) & 0x00F000F0u, x, a);
            b = dot2_x<4 * w + 1>(t & 0x00F000F0u, x, b);
            c = dot2_x<4 * w + 2>((t >> 4) & 0x00F000F0u, x, c);
            d = dot2_x<4 * w + 3>((t >> 8) & 0x00F000F0u, x, d);
        });
        dot_results_ready(a, b, c, d);
    }
    __device__ __forceinline__ float sum() const { return ((a + b) + (c + d)) * (kTwoPow24 / 16.f); }
};

// 3-bit layout: fields at bits 0-2, 4-6, 7-9, 10-12, 13-15 of each half and a spare bit 3 that carries one bit of
// pair 60 + w / 3.
template <>
struct GroupAcc<PACK_U3> {
    float a4 = 0.f, b4 = 0.f, c4 = 0.f, a7 = 0.f, b7 = 0.f;
    float e[3] = {0.f, 0.f, 0.f};
    __device__ __forceinline__ void add(const uint32_t* wd, const uint4& x) {
        unroll<12>([&](auto W) {
            constexpr int w = decltype(W)::value;
            const uint32_t t = wd[w], lo = t << 4, hi = t >> 6;
            a4 = dot2_x<5 * w + 0>(lo & 0x00700070u, x, a4);        // bits 0-2
            b4 = dot2_x<5 * w + 1>(t & 0x00700070u, x, b4);         // bits 4-6
            a7 = dot2_x<5 * w + 2>(t & 0x03800380u, x, a7);         // bits 7-9
            c4 = dot2_x<5 * w + 3>(hi & 0x00700070u, x, c4);        // bits 10-12
            b7 = dot2_x<5 * w + 4>(hi & 0x03800380u, x, b7);        // bits 13-15
            e[w % 3] = dot2_x<60 + w / 3>(lo & 0x00800080u, x, e[w % 3]);  // spare bit 3
        });
        dot_results_ready(a4, b4, c4, a7);
        dot_results_ready(b7, e[0], e[1], e[2]);
    }
    __device__ __forceinline__ float sum() const {
        const float at7 = (a7 + b7) + ((e[0] + 2.f * e[1]) + 4.f * e[2]);
        return (((a4 + b4) + c4) * 0.0625f + at7 * 0.0078125f) * kTwoPow24;
    }
};

// Per-lane codebook as byte tables for v_perm_b32 lookups.
struct LutTables {
    uint32_t lo03, lo47, hi03, hi47;
};

__device__ __forceinline__ LutTables make_lut_tables(uint4 l) {
    // l.x = (e0,e1)  l.y = (e2,e3)  l.z = (e4,e5)  l.w = (e6,e7) as fp16 pairs
    LutTables t;
    t.lo03 = __builtin_amdgcn_perm(l.y, l.x, 0x06040200u);
    t.hi03 = __builtin_amdgcn_perm(l.y, l.x, 0x07050301u);
    t.lo47 = __builtin_amdgcn_perm(l.w, l.z, 0x06040200u);
    t.hi47 = __builtin_amdgcn_perm(l.w, l.z, 0x07050301u);
    return t;
}

// LUT layout: the byte selectors of three words, looked up in the column's codebook.
template <>
struct GroupAcc<PACK_LUT3> {
    LutTables T;
    float acc0 = 0.f, acc1 = 0.f;
    __device__ __forceinline__ void add(const uint32_t* wd, const uint4& x) {
        unroll<4>([&](auto B) {
            constexpr int b = decltype(B)::value;
            const uint32_t w0 = wd[3 * b], w1 = wd[3 * b + 1], w2 = wd[3 * b + 2];
            uint32_t sel[8];
            sel[0] = w0 & 0x07070707u;
            sel[1] = (w0 >> 3) & 0x07070707u;
            sel[2] = w1 & 0x07070707u;
            sel[3] = (w1 >> 3) & 0x07070707u;
            sel[4] = w2 & 0x07070707u;
            sel[5] = (w2 >> 3) & 0x07070707u;
            sel[6] = ((w0 >> 6) & 0x03030303u) | ((w2 >> 4) & 0x04040404u);
            sel[7] = ((w1 >> 6) & 0x03030303u) | ((w2 >> 5) & 0x04040404u);
            unroll<8>([&](auto S) {
                constexpr int s = decltype(S)::value;
                const uint32_t lo = __builtin_amdgcn_perm(T.lo47, T.lo03, sel[s]);
                const uint32_t hi = __builtin_amdgcn_perm(T.hi47, T.hi03, sel[s]);
                const uint32_t p01 = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
                const uint32_t p23 = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
                acc0 = dot2_x<16 * b + 2 * s>(p01, x, acc0);
                acc1 = dot2_x<16 * b + 2 * s + 1>(p23, x, acc1);
            });
        });
        dot_results_ready(acc0, acc1);
    }
    __device__ __forceinline__ float sum() const { return acc0 + acc1; }
};

// 128-bit load of data that is read exactly once (the weight stream).
__device__ __forceinline__ uint4 load_streaming(const uint4* p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// What one lane holds of one tile while it is in flight.
template <int KIND>
struct TileRegs {
    uint4 x;         // this lane's four activation pairs of the group
    uint4 q[words_per_lane(KIND) / 4];
    uint16_t s, z;   // fp16 scale and zero point of (group, column)   (uniform formats)
};

// tile: the lane's first piece.
template <int KIND>
__device__ __forceinline__ void load_tile(TileRegs<KIND>& r, const uint4* __restrict__ tile,
                                          const uint16_t* __restrict__ scales,
                                          const uint16_t* __restrict__ zeros, const uint4* __restrict__ x128,
                                          int g, int N, int n, int lane) {
    constexpr int P = words_per_lane(KIND) / 4;
    r.x = x128[g * 16 + (lane & 15)];
#pragma unroll
    for (int p = 0; p < P; ++p) r.q[p] = load_streaming(tile + p * kTileCols);
    if constexpr (KIND != PACK_LUT3) {
        r.s = scales[(size_t)g * N + n];
        r.z = zeros[(size_t)g * N + n];
    }
}

template <int KIND>
__device__ __forceinline__ float tile_dot(TileRegs<KIND>& r, const LutTables& T) {
    constexpr int P = words_per_lane(KIND) / 4;
    dot_operands_ready(r.x);
    uint32_t wd[4 * P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        wd[4 * p] = r.q[p].x;
        wd[4 * p + 1] = r.q[p].y;
        wd[4 * p + 2] = r.q[p].z;
        wd[4 * p + 3] = r.q[p].w;
    }
    GroupAcc<KIND> acc;
    if constexpr (KIND == PACK_LUT3) acc.T = T;
    acc.add(wd, r.x);
    if constexpr (KIND == PACK_LUT3) {
        return acc.sum();
    } else {
        constexpr uint32_t kOnes = 0x3C003C00u;  // (1, 1)
        const float xs = dot2(r.x.w, kOnes, dot2(r.x.z, kOnes, dot2(r.x.y, kOnes, dot2(r.x.x, kOnes, 0.f))));
        const float gs = row_sum(xs);  // sum of the group's 128 activations
        const float s = (float)__builtin_bit_cast(_Float16, r.s);
        const float z = (float)__builtin_bit_cast(_Float16, r.z);
        return s * (acc.sum() - z * gs);
    }
}

// Work of workgroup `bid`: COLS columns of one tile of one of the matrices, K-slice ks of a.gslices.  The first
// `waves` of its WAVES wavefronts take 64 / COLS groups at a time, one per COLS lanes, a.gpw times each, with the tiles of
// DEPTH turns on their way (0: a.gpw is 1).
//
// Adjacent blocks of fewer than 64 columns share the 128-byte lines of the scales and zero points (and lie in one tile):
// they go to one XCD, whose L2 then reads a line once (workgroups go to the eight XCDs in turn).
template <int KIND, int COLS, int WAVES, int DEPTH>
__device__ __forceinline__ void gemv_block(const CallArgs& a, int bid, int waves) {
    constexpr int P = words_per_lane(KIND) / 4;  // 16-byte pieces per lane per tile
    constexpr int kTileStride = P * kTileCols;   // uint4 per tile
    constexpr int GPI = kTileCols / COLS;        // groups of a wavefront at a time = column blocks of a tile
    __shared__ float red[WAVES * COLS];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int block = divide_by(bid, a.gdiv);  // of COLS columns, over all matrices
    const int ks = bid - block * a.gslices;
    if constexpr (GPI > 1) {
        const int t = block % (8 * GPI), base = block - t;
        if (base + 8 * GPI <= a.tiles * GPI) block = base + (t % 8) * GPI + t / 8;
    }
    const int gt = block / GPI, part = block % GPI;  // tile over all matrices, block of the tile
    int m = 0, tile0 = 0;
#pragma unroll
    for (int i = 0; i < kMaxMulti - 1; ++i) {
        if (i + 1 < a.n && gt >= a.mat[i].tile_end) {
            m = i + 1;
            tile0 = a.mat[i].tile_end;
        }
    }
    const MatArgs& mat = a.mat[m];
    const int nt = gt - tile0;
    const int N = mat.N, G = a.G, gpw = a.gpw;
    const int tcol = part * COLS + lane % COLS;
    const int n = nt * kTileCols + tcol;
    const uint16_t* scales = mat.scales;
    const uint16_t* zeros_or_lut = mat.zeros_or_lut;
    const uint4* x128 = reinterpret_cast<const uint4*>(a.x);
    // for the end: read now, so that the last step does not begin with a trip to memory
    int col0 = mat.col0, producers = a.producers, direct = a.direct;
    hold_scalar(col0, producers, direct);
    _Float16* y = mat.y;
    hold_scalar(y);
    unsigned long long* acc = a.acc;
    hold_scalar(acc);

    float total = 0.f;
    const uint4* column = mat.Wq + (size_t)nt * G * kTileStride + tcol;
    const int g_first = (ks * waves + wave) * gpw * GPI;  // wave-uniform
    const int g_end = wave < waves ? min(g_first + gpw * GPI, G) : 0;
    const auto load = [&](TileRegs<KIND>& r, int g) {
        load_tile<KIND>(r, column + (size_t)g * kTileStride, scales, zeros_or_lut, x128, g, N, n, lane);
    };
    const auto load_codebook = [&] {
        uint4 c{};
        if constexpr (KIND == PACK_LUT3) c = reinterpret_cast<const uint4*>(zeros_or_lut)[n];
        return c;
    };
    // One turn, from the loads on.  Lanes beyond the last group read it once more and add nothing.
    const auto turn = [&](int g0) {
        const int mine = g0 + (GPI > 1 ? lane / COLS : 0), g = GPI > 1 ? min(mine, G - 1) : mine;
        const uint4 codebook = load_codebook();
        TileRegs<KIND> r;
        load(r, g);
        const float v = tile_dot<KIND>(r, make_lut_tables(codebook));
        total += GPI == 1 || mine < G ? v : 0.f;
    };
    if constexpr (DEPTH > 2) {
        // Long chains of few wavefronts (gemv.hip): DEPTH tiles on their way.  The loop asks for one wherever it has used
        // one, without conditions: where it depends on the path how many requests are on their way, the compiler waits for all.
        TileRegs<KIND> r[DEPTH];
        int g = g_first;
        if (g + DEPTH <= g_end) {
            const uint4 codebook = load_codebook();
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) load(r[i], g + i);
            const LutTables T = make_lut_tables(codebook);
            for (; g + 2 * DEPTH <= g_end; g += DEPTH) {
#pragma unroll
                for (int i = 0; i < DEPTH; ++i) {
                    total += tile_dot<KIND>(r[i], T);
                    load(r[i], g + i + DEPTH);
                }
            }
            const int left = g_end - g - DEPTH;  // fewer than DEPTH, besides those on their way
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) {
                total += tile_dot<KIND>(r[i], T);
                if (i < left) load(r[i], g + i + DEPTH);
            }
#pragma unroll
            for (int i = 0; i < DEPTH - 1; ++i)
                if (i < left) total += tile_dot<KIND>(r[i], T);
        } else if (g < g_end) {
            const uint4 codebook = load_codebook();
#pragma unroll
            for (int i = 0; i < DEPTH - 1; ++i)
                if (g + i < g_end) load(r[i], g + i);
            const LutTables T = make_lut_tables(codebook);
#pragma unroll
            for (int i = 0; i < DEPTH - 1; ++i)
                if (g + i < g_end) total += tile_dot<KIND>(r[i], T);
        }
    } else if constexpr (DEPTH == 2) {
        // Both tiles of two turns asked for before the first is worked off.
        int g = g_first;
        for (; g + 1 < g_end; g += 2) {
            const uint4 codebook = load_codebook();
            TileRegs<KIND> r0, r1;
            load(r0, g);
            load(r1, g + 1);
            const LutTables T = make_lut_tables(codebook);
            total += tile_dot<KIND>(r0, T);
            total += tile_dot<KIND>(r1, T);
        }
        if (g < g_end) turn(g);
    } else if (DEPTH == 0 || gpw == 1) {
        // The usual single turn as straight code: in a loop the compiler waits for all of a tile before it starts on the first
        // word (4096 x 28672: 11.5 instead of 10.2 us).
        if (g_first < g_end) turn(g_first);
    } else {
        int g0 = g_first;
        asm volatile("" : "+s"(g0));  // nothing in common with the straight code, which the compiler would move in front of both
        for (; g0 < g_end; g0 += GPI) turn(g0);
    }

    total = sum_over_groups<COLS>(total);
    if (COLS == 64 || lane < COLS) red[wave * COLS + lane] = total;
    __syncthreads();
    if (wave == 0) {
        // 64 / COLS wavefronts' sums a load; a fixed tree over the loads, which are independent of one another
        constexpr int kLoads = WAVES / GPI;
        static_assert(kLoads * GPI == WAVES, "whole loads");
        float v[kLoads];
#pragma unroll
        for (int i = 0; i < kLoads; ++i) v[i] = red[i * 64 + lane];
#pragma unroll
        for (int span = 1; span < kLoads; span *= 2)
#pragma unroll
            for (int w = 0; w + span < kLoads; w += 2 * span) v[w] += v[w + span];
        const float sum = sum_over_groups<COLS>(v[0]);
        if (lane < COLS) {
            if (direct) {
                y[n] = (_Float16)sum;
            } else if (acc != nullptr) {
                arrive(acc + col0 + n, y + n, producers, sum);
            } else {
                a.gpart[(size_t)ks * a.Ntot + col0 + n] = sum;
            }
        }
    }
}

}  // namespace decdec
