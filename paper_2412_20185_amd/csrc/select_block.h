// Workgroup-level exact top-k of |x| (DecDEC Section 4.1 step 1 with the exact
// Top-K of Section 5.2; a tie at the cut goes to the lower index).  Used by the
// stand-alone selection kernel and by kernels that select for themselves.
//
// x is read once and stays in registers, in chunks of 8 keys: a wavefront owns a
// run of consecutive chunks, of which lane l holds chunk l, l + 64, ...
// (one coalesced 128-bit load each), so inside a wavefront the channel order is
// (j, lane, position in the chunk) and wavefronts follow one another.  The order
// of |x| is the order of the 15-bit key (fp16 bits, sign cleared).  Output is in
// ascending index order.
//
// What bounds the selection is the instruction issue of the one compute unit it
// runs on, so few instructions may touch every key.  Two forms:
//
//   chunks (list_chunks, select_listed), when k is at most a third of the number
//   of chunks and at most 576 (beyond, the bound is too low to exclude much): k
//   chunks hold a key at least as large as the k-th largest chunk maximum, so that
//   is a lower bound of the k-th largest key.
//     1. chunk maxima by packed 16-bit maxima; a 256-bin LDS histogram of their
//        high 8 bits gives the bin that holds the k-th largest; its lower edge L
//        is the bound;
//     2. every wavefront lists its chunks with a maximum >= L, in order, in its
//        own part of an LDS list and takes them back one to three per lane (left
//        out when every thread has one chunk), so that no barrier and no sum over
//        wavefronts stands in front of the next step.  A wavefront with more of
//        them than its list holds then puts the others there and reads them when
//        they are needed.  Fewer than k chunks have a maximum in a bin above;
//        nearly always all of these maxima are selected, and a caller may act on
//        them while the rest is found out (`ask`);
//     3. a 256-bin LDS histogram of key - L over their keys gives T, the k-th
//        largest key itself, and how many keys equal to T are needed; only when
//        T >= L + 255 (large |x| crowded into few chunks) it is formed twice more,
//        over 128-key bins and inside the bin that holds T;
//     4. masks of the keys > T and == T and one prefix sum place every selected
//        element.
//   radix (select_by_radix), for larger k, or when the bound is zero (fewer than k
//   chunks with a key of 2^-17 or more) or a wavefront has more than two lists of
//   chunks (384 of up to 512): LDS histograms of all keys over their high 8 and
//   low 7 bits, then masks and prefix sums over every key.
// Every phase is a chain of dependent instructions of a few wavefronts, about 2 ns each, and of LDS trips (with all of its
// instructions in the cache it takes the same time): finding a bin and marking keys take as few as they can.
// Stand-alone kernel in graph replays, radix for every key -> chunks, us: K = 1024, k = 32: 3.4 -> 2.7; 4096, 60:
// 3.7 -> 3.0; 8192, 81: 5.4 -> 3.4; 14336, 286: 6.3 -> 3.9; 28672, 286: 9.8 -> 4.6.  One list for all wavefronts, which
// takes two barriers and a sum over them, took 0.5 more (K = 8192 up) of 1024 threads; the lists of sixteen wavefronts 0.6 more
// than those of eight, because each of them issues the steps 3 and 4 for a quarter of its lanes only.  With k = 400 of 4096
// the bound is so low that the chunks took 5.4 against 3.5 for radix.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "kernels.h"

namespace decdec {

constexpr int kSelectMaxChunks = 8;  // 8-key chunks per thread at most

constexpr int kMaxByChunks = 576;    // the bin of L alone can make the list 1.77 times as long as k (|x| normal, k 1 % of K)
// Chunks with a key that may be selected in a wavefront's list.  Of 1020 such chunks in all, each of eight wavefronts has 128 +- 10
// where the channels' magnitudes are alike; where they fall along the channels the first wavefronts have more.
template <int THREADS, int NCH>
constexpr int kListedPerWave = THREADS <= 512 && NCH == 8 ? 192 : 128;

__host__ __device__ inline bool select_tries_chunks(int nchunks, int k) { return 3 * k <= nchunks && k <= kMaxByChunks; }

// LDS of the selection; nothing in it is needed afterwards, so it may share its place with other data.
template <int THREADS, int NCH>
struct SelectShared {
    static constexpr int kListed = NCH <= 1 ? 1 : THREADS / 64 * kListedPerWave<THREADS, NCH>;
    uint4 list[kListed];
    uint16_t list_chunk[kListed];
    __attribute__((aligned(16))) unsigned hist1[256];
    __attribute__((aligned(16))) unsigned hist2[256];
    __attribute__((aligned(16))) unsigned wtot[16];  // per wave: (keys > T) | (keys == T) << 16
    int overflow;                                     // 1: a wavefront's list, filled twice, is too short
    uint16_t asked[THREADS / 64][8];                  // for the caller's `ask`
};

template <int CTRL, int ROW_MASK, bool BOUND_CTRL>
__device__ __forceinline__ unsigned dpp_u32(unsigned v) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, BOUND_CTRL);
}

// Inclusive prefix sum over the 64 lanes of a wavefront (DPP row shifts and row broadcasts).
__device__ __forceinline__ unsigned wave_incl_scan(unsigned v) {
    v += dpp_u32<0x111, 0xF, true>(v);   // row_shr:1, zero shifted in
    v += dpp_u32<0x112, 0xF, true>(v);   // row_shr:2
    v += dpp_u32<0x114, 0xF, true>(v);   // row_shr:4
    v += dpp_u32<0x118, 0xF, true>(v);   // row_shr:8 -> inclusive scan inside each row of 16
    v += dpp_u32<0x142, 0xA, false>(v);  // row_bcast15: rows 1 and 3 add the total of the row before
    v += dpp_u32<0x143, 0xC, false>(v);  // row_bcast31: rows 2 and 3 add the total of rows 0-1
    return v;
}

// Run by all 64 lanes of a wavefront.  hist (16-byte aligned) holds NB = 64 * PER bins in ascending key order whose
// sum has at least kk >= 1 entries.  Finds the bin with fewer than kk entries in the bins above it and at least kk
// in the bins from it up; returns it and kk - (entries above it) in every lane.
template <int PER>
__device__ __forceinline__ void wave_find_bin(const unsigned* hist, unsigned kk, unsigned& bin, unsigned& rem, int lane) {
    static_assert(PER == 4 || PER == 2, "bins per lane");
    unsigned c[PER];
    if constexpr (PER == 4) {
        const uint4 v = reinterpret_cast<const uint4*>(hist)[lane];
        c[0] = v.x;
        c[1] = v.y;
        c[2] = v.z;
        c[3] = v.w;
    } else {
        const uint2 v = reinterpret_cast<const uint2*>(hist)[lane];
        c[0] = v.x;
        c[1] = v.y;
    }
    unsigned from[PER];  // entries in the lane's bins from this one up
    from[PER - 1] = c[PER - 1];
#pragma unroll
    for (int j = PER - 2; j >= 0; --j) from[j] = from[j + 1] + c[j];
    const unsigned incl = wave_incl_scan(from[0]);
    const unsigned above = (unsigned)__builtin_amdgcn_readlane((int)incl, 63) - incl;  // entries above this lane's bins
    const unsigned want = kk - above;  // of the lane's own entries; 0 or "negative" where the bins above have enough
    const unsigned long long mask = __ballot(want - 1u < from[0]);  // one lane unless the histogram is short of kk entries
    unsigned b_l = (unsigned)(lane * PER + PER - 1), over = 0;  // over: entries of the lane above its bin
#pragma unroll
    for (int j = PER - 1; j >= 1; --j) {
        const bool below = from[j] < want;
        b_l -= below;
        over = below ? from[j] : over;
    }
    const int src = mask ? __builtin_ctzll(mask) : 0;
    bin = (unsigned)__builtin_amdgcn_readlane((int)b_l, src);
    rem = (unsigned)__builtin_amdgcn_readlane((int)(want - over), src);
}

// Word e / 2 of a chunk, by its bits or (MANY) by comparisons: the former is the quicker one where few keys of a chunk are
// marked, the latter where many are (select.hip).  The words come by value: chosen by reference they would be kept in
// scratch memory.
template <bool MANY>
__device__ __forceinline__ uint32_t word_of(uint32_t x, uint32_t y, uint32_t z, uint32_t w, int e) {
    if constexpr (MANY) {
        uint32_t r = e >= 2 ? y : x;
        r = e >= 4 ? z : r;
        return e >= 6 ? w : r;
    } else {
        const uint32_t lo = e & 2 ? y : x, hi = e & 2 ? w : z;
        return e & 4 ? hi : lo;
    }
}
__device__ __forceinline__ unsigned key_of(const uint4& c, int e) {
    const uint32_t w = word_of<false>(c.x, c.y, c.z, c.w, e);
    return ((e & 1) ? (w >> 16) : w) & 0x7FFFu;
}
template <bool MANY = false>
__device__ __forceinline__ uint16_t raw_of(const uint4& c, int e) {
    const uint32_t w = word_of<MANY>(c.x, c.y, c.z, c.w, e);
    return (uint16_t)((e & 1) ? (w >> 16) : (w & 0xFFFFu));
}

typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned pk_max_u16(unsigned a, unsigned b) {
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a),
                                                                  __builtin_bit_cast(ushort2_t, b)));
}

__device__ __forceinline__ unsigned chunk_max(const uint4& c) {
    const unsigned m = pk_max_u16(pk_max_u16(c.x & 0x7FFF7FFFu, c.y & 0x7FFF7FFFu),
                                  pk_max_u16(c.z & 0x7FFF7FFFu, c.w & 0x7FFF7FFFu));
    return max(m >> 16, m & 0xFFFFu);
}

// Number of set bits of a lane mask in front of this lane.
__device__ __forceinline__ unsigned lanes_before(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// Sum of the waves' totals in front of `wave`.
template <int WAVES>
__device__ __forceinline__ unsigned totals_before(const unsigned* wtot, int wave) {
    unsigned before = 0;
#pragma unroll
    for (int w = 0; w < WAVES; w += 4) {
        const uint4 t = *reinterpret_cast<const uint4*>(wtot + w);
        before += (w < wave ? t.x : 0u) + (w + 1 < wave ? t.y : 0u) + (w + 2 < wave ? t.z : 0u) + (w + 3 < wave ? t.w : 0u);
    }
    return before;
}

// Writes the marked keys of one chunk: all of `gt`, of `eq` those with fewer than `need` equal keys in front.  `tag`: 0, or a
// key's position in the chunk (low three bits) and what its index gets from bit 16 on.
template <bool MANY = false>
__device__ __forceinline__ void write_marked(const uint4& c, int channel0, unsigned gt, unsigned eq, unsigned pos_gt,
                                             unsigned seen_eq, unsigned need, unsigned k, int32_t* idx_out,
                                             uint16_t* xsel_out, unsigned tag = 0) {
    unsigned m = gt | eq;
    while (m) {
        const int e = __builtin_ctz(m);
        m &= m - 1;
        const bool is_gt = (gt >> e) & 1u;
        const unsigned pos = pos_gt + min(seen_eq, need);
        // pos < k always holds for a taken key; the bound keeps a logic error from writing outside
        if ((is_gt || seen_eq < need) && pos < k) {
            idx_out[pos] = (channel0 + e) | ((unsigned)e == (tag & 7u) ? (int)(tag >> 3 << 16) : 0);
            if (xsel_out) xsel_out[pos] = raw_of<MANY>(c, e);
        }
        pos_gt += is_gt;
        seen_eq += !is_gt;
    }
}

// Bit e: key e of the chunk is > below (below <= 0x7FFF), two keys at a time: with the sign bits set, no half borrows from the
// other, and a half's sign bit stays where its key is large enough.  (Packed saturating subtractions and minima become
// comparisons, selects and byte permutes in the compiler's hands, half as many instructions again.)
__device__ __forceinline__ unsigned mark_above(const uint4& c, unsigned below) {
    constexpr unsigned kSigns = 0x80008000u;
    const unsigned lim = (below + 1) * 0x10001u;
    const unsigned w[4] = {c.x, c.y, c.z, c.w};
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) m = (m >> 2) | (((w[i] | kSigns) - lim) & kSigns);
    return ((m >> 9) | (m >> 24)) & 0xFFu;  // bits 9 + 2 i and 25 + 2 i: the two keys of word i
}

// Bit e of gt / eq: key e of the chunk is > T / == T (T >= 1).
__device__ __forceinline__ void mark_chunk(const uint4& c, unsigned T, unsigned& gt, unsigned& eq) {
    gt = mark_above(c, T);
    eq = mark_above(c, T - 1) & ~gt;
}

// The chunks of a thread: chunk(j) for those j that has(j) is true for.  The runs of the wavefronts are 64 * NCH chunks, with which
// the fewest have any (each issues the steps 3 and 4, however few chunks it lists) ...
// (With two and four chunks per thread they are compared with what is left of the run: the lane masks that are kept when they are
// compared with nchunks are more than the residual kernels have scalar registers for.  With eight that takes 22016 x 2048 0.6 us
// longer.)
template <int THREADS, int NCH>
struct FullRuns {
    static constexpr bool kOfAll = NCH == 1 || NCH == 8 || THREADS > 512;
    int first, left;  // left: all chunks, or those of the run from `first` on
    __device__ __forceinline__ explicit FullRuns(int nchunks) {
        const int wave = kOfAll ? (int)threadIdx.x >> 6 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        const int lane = threadIdx.x & 63;
        first = wave * 64 * NCH + lane;
        left = kOfAll ? nchunks : min(64 * NCH, nchunks - wave * 64 * NCH) - lane;
    }
    __device__ __forceinline__ bool has(int j) const { return (kOfAll ? first : 0) + 64 * j < left; }
    __device__ __forceinline__ int chunk(int j) const { return first + 64 * j; }
};
// ... or, for a k with which full ones would make the lists long (the bin of L makes them up to 1.77 times k), all alike.  us, full
// runs and even ones: K = 22016, k = 220 4.3 and 4.5; 16512, 516, where five wavefronts would list 190 chunks each, 5.6 and 5.4.
// Not in residual kernels: what the choice costs in front of their first load is 1 % of 14336 x 4096, 6 % of 22016 x 2048.
template <int THREADS, int NCH>
struct ChosenRuns {
    int first, left;  // left: chunks of the run from `first` on
    __device__ __forceinline__ ChosenRuns(int nchunks, int k) {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
        const bool even = k > 40 * ((nchunks + 64 * NCH - 1) / (64 * NCH));
        const int each = even ? (nchunks + THREADS / 64 - 1) / (THREADS / 64) : 64 * NCH;
        first = wave * each + lane;
        left = min(each, nchunks - wave * each) - lane;
    }
    __device__ __forceinline__ bool has(int j) const { return 64 * j < left; }
    __device__ __forceinline__ int chunk(int j) const { return first + 64 * j; }
};

// A lane's chunks once those that cannot matter are gone: entries lane, lane + 64, ... of the wavefront's list.
template <int THREADS, int NCH>
struct Listed {
    static constexpr int kList = NCH == 1 ? 64 : kListedPerWave<THREADS, NCH>;
    static constexpr int kPer = kList / 64;
    static constexpr bool kMayBeMore = NCH * 64 > kList;  // more than the list holds: the others then take their place in LDS,
    static constexpr bool kMayOverflow = NCH * 64 > 2 * kList;  // and not even that is enough: sh.overflow
    uint4 keys[kPer];
    int chunk[kPer];
    int count = 0;   // chunks of this wavefront
    unsigned L = 0;  // the bound; 0: the chunks do not give one

    // f(keys, chunk) in all lanes for 64 at a time of those that are more (keys of 0 in lanes that have none).  Few wavefronts
    // have any, and they have a trip to LDS for them at every step; kept in registers they would cost every kernel 10 to 20.
    template <typename F>
    __device__ __forceinline__ void each_more(const SelectShared<THREADS, NCH>& sh, const F& f) const {
        if constexpr (kMayBeMore) {
            if (__builtin_expect(count > kList, 0)) {
                const int lane = threadIdx.x & 63, at = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) * kList;
#pragma unroll 1
                for (int i = 0; i < count - kList; i += 64) {
                    const bool have = i + lane < count - kList;
                    const int e = at + min(i + lane, count - kList - 1);
                    uint4 c = sh.list[e];
                    if (!have) c = make_uint4(0, 0, 0, 0);
                    f(c, (int)sh.list_chunk[e]);
                }
            }
        }
    }
};

// Steps 1 and 2.  Requires 1 <= k <= nchunks and sh.hist1 cleared (with a barrier behind).
template <int THREADS, int NCH, typename Runs>
__device__ __forceinline__ void list_chunks(const uint4 (&ch)[NCH], const Runs& run, int k, SelectShared<THREADS, NCH>& sh,
                                            Listed<THREADS, NCH>& out) {
    typedef Listed<THREADS, NCH> L_t;
    constexpr int LIST = L_t::kList;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    unsigned cm[NCH];  // absent chunks: 0
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        cm[j] = chunk_max(ch[j]);
        if (run.has(j)) atomicAdd(&sh.hist1[cm[j] >> 7], 1u);
    }
    __syncthreads();
    unsigned bin, need;
    wave_find_bin<4>(sh.hist1, (unsigned)k, bin, need, lane);
    const unsigned L = bin << 7;
    out.L = L;
    if (L == 0) return;
    if constexpr (NCH == 1) {
        out.keys[0] = ch[0];
        out.chunk[0] = run.chunk(0);
        out.count = 64;
    } else {
        uint4* list = sh.list + wave * LIST;
        uint16_t* list_chunk = sh.list_chunk + wave * LIST;
        // entries from `from` on to the list; returns how many there are in all
        const auto fill = [&](int from, const auto& top) {
            int count = 0;
#pragma unroll
            for (int j = 0; j < NCH; ++j) {
                const bool wanted = top(j) >= L;
                const unsigned long long b = __ballot(wanted);
                const int at = count + (int)lanes_before(b) - from;
                if (wanted && (!L_t::kMayBeMore || (unsigned)at < (unsigned)LIST)) {
                    list[at] = ch[j];
                    list_chunk[at] = (uint16_t)run.chunk(j);
                }
                count += (int)__builtin_popcountll(b);
            }
            wave_writes_seen();
            return count;
        };
        out.count = fill(0, [&](int j) { return cm[j]; });
#pragma unroll
        for (int p = 0; p < L_t::kPer; ++p) {
            const int i = 64 * p + lane;
            out.keys[p] = make_uint4(0, 0, 0, 0);  // keys below L: never taken
            out.chunk[p] = 0;
            if (i < out.count) {
                out.keys[p] = list[i];
                out.chunk[p] = list_chunk[i];
            }
        }
        if constexpr (L_t::kMayBeMore) {
            if (__builtin_expect(out.count > LIST, 0)) {
                wave_writes_seen();  // it has been read
                (void)fill(LIST, [&](int j) { return chunk_max(ch[j]); });
                if (L_t::kMayOverflow && out.count > 2 * LIST) {
                    if (lane == 0) sh.overflow = 1;
                    out.count = 0;  // all go to the radix form: many equal keys are not counted here too
                }
            }
        }
    }
}

// Steps 3 and 4.  Requires L != 0 and sh.hist2 cleared.  False, in all threads, when a list was too short: nothing has been
// written to the outputs then.
template <int THREADS, int NCH>
__device__ __forceinline__ bool select_listed(const Listed<THREADS, NCH>& l, int k, SelectShared<THREADS, NCH>& sh,
                                              int32_t* idx_out, uint16_t* xsel_out, unsigned tag) {
    typedef Listed<THREADS, NCH> L_t;
    constexpr int PER = L_t::kPer;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned T = l.L, bin, need;
    int shift = 0;  // bins of 2^shift keys from T on; the last one takes everything above
    const auto count_keys = [&](const uint4& c) {
        unsigned m = mark_above(c, T - 1);
        while (m) {
            atomicAdd(&sh.hist2[min((key_of(c, __builtin_ctz(m)) - T) >> shift, 255u)], 1u);
            m &= m - 1;
        }
    };
    while (true) {
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            if (64 * p >= l.count) break;  // wave-uniform
            count_keys(l.keys[p]);
        }
        l.each_more(sh, [&](const uint4& c, int) { count_keys(c); });
        __syncthreads();
        if (L_t::kMayOverflow && __builtin_amdgcn_readfirstlane(sh.overflow)) return false;
        wave_find_bin<4>(sh.hist2, (unsigned)k, bin, need, lane);  // need: keys equal to T to take (>= 1) in the end
        T += bin << shift;
        if (shift == 0 && bin < 255) break;
        shift = shift == 0 ? 7 : 0;  // 256 bins of 128 cover every key; then 128 keys at the most
        __syncthreads();
        for (int i = tid; i < 256; i += THREADS) sh.hist2[i] = 0;
        __syncthreads();
    }

    unsigned gt[PER], eq[PER], at[PER], total = 0;  // at: marked keys of this wavefront in front of the chunk's
    const auto mark_and_count = [&](const uint4& c, unsigned& g, unsigned& e, unsigned& a) {
        mark_chunk(c, T, g, e);
        const unsigned cnt = (unsigned)__builtin_popcount(g) | ((unsigned)__builtin_popcount(e) << 16);
        const unsigned incl = wave_incl_scan(cnt) + total;
        a = incl - cnt;
        total = PER == 1 ? incl : (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
    };
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        gt[p] = eq[p] = at[p] = 0;
        if (64 * p >= l.count) break;
        mark_and_count(l.keys[p], gt[p], eq[p], at[p]);
    }
    const unsigned listed = total;
    unsigned g, e, a;
    l.each_more(sh, [&](const uint4& c, int) { mark_and_count(c, g, e, a); });
    if (lane == 63) sh.wtot[wave] = total;
    __syncthreads();
    // fewer than k keys > T, and at most 65535 equal ones in front of any key: no carry between the halves
    const unsigned before = totals_before<THREADS / 64>(sh.wtot, wave);
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        if (64 * p >= l.count) break;
        write_marked(l.keys[p], l.chunk[p] * 8, gt[p], eq[p], (before + at[p]) & 0xFFFFu, (before + at[p]) >> 16, need, (unsigned)k,
                     idx_out, xsel_out, p == 0 ? tag : 0u);
    }
    total = listed;
    l.each_more(sh, [&](const uint4& c, int chunk) {
        mark_and_count(c, g, e, a);
        write_marked(c, chunk * 8, g, e, (before + a) & 0xFFFFu, (before + a) >> 16, need, (unsigned)k, idx_out, xsel_out);
    });
    return true;
}

// Any 1 <= k <= K.  Requires sh.hist1, sh.hist2 cleared (with a barrier behind).  MANY: many keys per chunk are marked.
template <int THREADS, int NCH, bool MANY = false, typename Runs>
__device__ __forceinline__ void select_by_radix(const uint4 (&ch)[NCH], const Runs& run, int k, SelectShared<THREADS, NCH>& sh,
                                                int32_t* idx_out, uint16_t* xsel_out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    // pass 1: high 8 bits of the key
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        if (run.has(j)) {
#pragma unroll
            for (int e = 0; e < 8; ++e) atomicAdd(&sh.hist1[key_of(ch[j], e) >> 7], 1u);
        }
    }
    __syncthreads();
    unsigned b1, rem1;
    wave_find_bin<4>(sh.hist1, (unsigned)k, b1, rem1, lane);

    // pass 2: low 7 bits of the keys inside bin b1
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        if (run.has(j)) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const unsigned key = key_of(ch[j], e);
                if ((key >> 7) == b1) atomicAdd(&sh.hist2[key & 127u], 1u);
            }
        }
    }
    __syncthreads();
    unsigned b2, need;  // need: keys equal to T to take (>= 1)
    wave_find_bin<2>(sh.hist2, rem1, b2, need, lane);
    const unsigned T = (b1 << 7) | b2;

    // compaction in index order; counts are packed as (> T) | (== T) << 16 (at most 4096 each per wavefront: no
    // carry between the halves)
    unsigned gtm[NCH], eqm[NCH], excl[NCH];  // excl: this wave's marked keys at lower indices (earlier rounds, lower lanes)
    unsigned wave_cnt = 0;                    // uniform: marked keys of the rounds so far
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        gtm[j] = eqm[j] = 0;
        if (run.has(j)) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const unsigned key = key_of(ch[j], e);
                gtm[j] |= (unsigned)(key > T) << e;
                eqm[j] |= (unsigned)(key == T) << e;
            }
        }
        const unsigned cnt = (unsigned)__builtin_popcount(gtm[j]) | ((unsigned)__builtin_popcount(eqm[j]) << 16);
        const unsigned incl = wave_incl_scan(cnt);
        excl[j] = wave_cnt + incl - cnt;
        wave_cnt += (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
    }
    if (lane == 0) sh.wtot[wave] = wave_cnt;
    __syncthreads();
    unsigned base_gt = 0, base_eq = 0;  // marked keys of the wavefronts before this one
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        const unsigned t = sh.wtot[w];
        base_gt += w < wave ? (t & 0xFFFFu) : 0u;
        base_eq += w < wave ? (t >> 16) : 0u;
    }
#pragma unroll
    for (int j = 0; j < NCH; ++j)
        write_marked<MANY>(ch[j], run.chunk(j) * 8, gtm[j], eqm[j], base_gt + (excl[j] & 0xFFFFu), base_eq + (excl[j] >> 16), need,
                     (unsigned)k, idx_out, xsel_out);
}

// The keys of a thread.  Requires K a multiple of 8, K <= 8 * THREADS * NCH and x 16-byte aligned.
template <int NCH, typename Runs>
__device__ __forceinline__ void load_keys(const uint16_t* __restrict__ x, const Runs& run, uint4 (&ch)[NCH]) {
    const uint4* x128 = reinterpret_cast<const uint4*>(x);
#pragma unroll
    for (int j = 0; j < NCH; ++j) ch[j] = run.has(j) ? x128[run.chunk(j)] : make_uint4(0, 0, 0, 0);
}

// The caller does not act on a part of the selection.
struct AskNothing {
    __device__ __forceinline__ unsigned operator()(const uint4&, int, unsigned, unsigned) const { return 0; }
};

// All THREADS threads of the workgroup call this, with their keys (load_keys) and their runs, and 1 <= k <= K.  idx_out / xsel_out
// may point to global memory or LDS; xsel_out may be null.  Ends with the outputs
// written but not yet synchronised (the caller adds the barrier it needs).  RADIX: the caller knows that
// select_tries_chunks(K / 8, k) is false.
//
// ask(a chunk's keys, the chunk, its maximum, edge): called once by every lane, on every path, with its first listed chunk (maximum
// 0: none).  Fewer than k chunks have a maximum >= edge.  Returns the lane's tag (write_marked), which only a selection by
// chunks writes.
template <int THREADS, int NCH, bool RADIX = false, typename Runs, typename Ask = AskNothing>
__device__ __forceinline__ void block_select_topk(const uint4 (&ch)[NCH], const Runs& run, int K, int k, SelectShared<THREADS, NCH>& sh,
                                                  int32_t* idx_out, uint16_t* xsel_out, const Ask& ask = Ask()) {
    static_assert(THREADS % 256 == 0 && THREADS / 64 <= 16 && NCH <= kSelectMaxChunks, "select shape");
    const int tid = threadIdx.x, nchunks = K / 8;
    const auto clear = [&] {
        for (int i = tid; i < 256; i += THREADS) sh.hist1[i] = sh.hist2[i] = 0;
        if (Listed<THREADS, NCH>::kMayOverflow && tid == 0) sh.overflow = 0;
        __syncthreads();
    };
    clear();
    if constexpr (!std::is_same_v<Ask, AskNothing>) {  // on every path, see `ask`
        const bool chunks = select_tries_chunks(nchunks, k);
        Listed<THREADS, NCH> l;
        if (chunks) list_chunks(ch, run, k, sh, l);
        const unsigned tag = ask(l.keys[0], l.chunk[0], l.L != 0 ? chunk_max(l.keys[0]) : 0u, l.L + 128);
        if (l.L != 0 && select_listed(l, k, sh, idx_out, xsel_out, tag)) return;
        if (chunks) {
            __syncthreads();
            clear();
        }
    } else if (!RADIX && select_tries_chunks(nchunks, k)) {
        Listed<THREADS, NCH> l;
        list_chunks(ch, run, k, sh, l);
        if (l.L != 0 && select_listed(l, k, sh, idx_out, xsel_out, 0)) return;
        __syncthreads();
        clear();
    }
    select_by_radix<THREADS, NCH, RADIX>(ch, run, k, sh, idx_out, xsel_out);
}

}  // namespace decdec
