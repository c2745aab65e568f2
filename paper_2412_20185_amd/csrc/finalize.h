// Step 4 of dynamic error compensation (DecDEC Section 4.1), o = o_b + o_dec,
// folded into the kernels that produce the two terms.
//
// The paper adds o_dec into o_b with atomics from its fused kernel (Section
// 4.3 "Kernel Fusion").  So does this: every producer of a column (the base
// GEMV once per K-slice, the residual kernel once per slice of the selected
// channels) adds its fp32 part sum into one 64-bit word per output column with
// a single returning atomic.  Floating-point atomics would make the result
// depend on who came first; the word therefore holds the sum in fixed point
// (integer addition is associative, so every arrival order gives the same
// bits) and, in its low six bits, the number of producers that have arrived:
//
//     word = (sum of rint(v * 2^30)) * 64  +  arrivals
//
// The producer whose atomic returns arrivals == producers - 1 holds the whole
// sum (returned value + own term), rounds it once to fp16, writes y and stores
// zero to the word for the next call.  A producer that has read the word earlier
// in the call and saw all others there does the same without adding
// (arrive_after_look).  One memory round trip per producer, no partial rows, no
// fences (each column is a location of its own), nobody waits, and no extra launch.
//
// Range and resolution: a part sum is clamped to +-2^21 before conversion
// (far outside fp16's +-65504, so a clamped term can only make y infinite, or
// meet a clamped term of the other sign: inputs are assumed finite and y
// representable); up to 32 producers then stay below 2^57 in the 58-bit signed
// sum field.  The step 2^-30 is finer than the last place of an fp32 part sum
// of magnitude 2^-7 or more, and 2^-6 of fp16's smallest subnormal: the fixed
// point sum is at least as accurate as an fp32 sum in any order.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace decdec {

constexpr float kFixedScale = 1073741824.f;       // 2^30
constexpr float kFixedInvScale = 1.f / 1073741824.f;
constexpr float kFixedLimit = 2097152.f;          // 2^21
constexpr int kArrivalBits = 6;                   // producers per column <= 32 < 2^6
static_assert(kMaxGemvSlices + kMaxFetchSlices <= 32, "32 clamped terms of 2^51 stay below 2^57");
static_assert(kMaxGemvSlices + kMaxFetchSlices < (1 << kArrivalBits), "the arrival count must fit its field");

// fp32 part sum -> fixed point (round to nearest even; NaN takes the lower clamp, so it leaves -inf in y).
__device__ __forceinline__ long long to_fixed(float v) {
    v = fminf(fmaxf(v, -kFixedLimit), kFixedLimit);
    return (long long)rintf(v * kFixedScale);
}

// Fixed-point sum -> the fp16 result (one rounding to fp32, exact scaling, one rounding to fp16).
__device__ __forceinline__ _Float16 from_fixed(long long s) { return (_Float16)((float)s * kFixedInvScale); }

// The producer that knows the others' sum writes the result and leaves zero for the next call.
__device__ __forceinline__ void finish(unsigned long long* word, _Float16* y, unsigned long long sum) {
    *y = from_fixed((long long)sum >> kArrivalBits);
    __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What the other producers have added so far.
__device__ __forceinline__ unsigned long long arrived_so_far(const unsigned long long* word) {
    return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long term_of(float v) {
    return ((unsigned long long)to_fixed(v) << kArrivalBits) + 1ull;
}
__device__ __forceinline__ bool others_arrived(unsigned long long word, int producers) {
    return (int)(word & ((1ull << kArrivalBits) - 1)) + 1 == producers;
}

// One thread per column: add part sum v into the column's accumulator.  Called once by every one of the `producers`
// of that column; the last one writes *y.
__device__ __forceinline__ void arrive(unsigned long long* word, _Float16* y, int producers, float v) {
    const unsigned long long term = term_of(v);
    const unsigned long long old = __hip_atomic_fetch_add(word, term, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (others_arrived(old, producers)) finish(word, y, old + term);
}

// The same, with what the word has shown earlier in this call: who has seen all others arrive is the last one and need not add.
__device__ __forceinline__ void arrive_after_look(unsigned long long* word, _Float16* y, int producers, float v,
                                                  unsigned long long seen) {
    if (others_arrived(seen, producers)) {
        finish(word, y, seen + term_of(v));
    } else {
        arrive(word, y, producers, v);
    }
}

}  // namespace decdec
