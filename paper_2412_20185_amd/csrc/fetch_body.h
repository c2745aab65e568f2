// Device code of the residual kernel (included by fetch.hip and fused.hip).
//
// Steps 2 and 3 of dynamic error compensation (DecDEC Section 4.1): fetch the
// residual rows of the selected input channels from pinned CPU memory and
// multiply them with x[sc_indices]:  o_dec[n] = sum_j R_hat[s_j][n] * x[s_j].
//
// Zero-copy (Section 4.3): the kernel reads the rows in place over the host
// link with plain 128-bit loads; a wavefront covers 1 KiB of one row per load,
// so requests are cache-line sized and contiguous per row (Section 4.2: each
// input-channel row is contiguous in CPU memory).  As in the paper's kernel
// (Section 4.3 "Kernel Fusion") the unit of ownership is a column segment: a
// workgroup owns the 1 KiB-per-row segment `wc` of the rows it handles, so its
// sum over those rows never leaves the compute unit.  The selected rows of a
// segment are spread over the wavefronts of the workgroup (and over `slices`
// workgroups when one workgroup does not put enough requests in flight: the
// knob that plays the role of n_tb in Section 4.4); the wavefronts' sums meet
// in LDS and the workgroup contributes ONE fp32 part sum per column of the segment.
//
// Selection inside the kernel (SELECT_NCH > 0): every workgroup first runs the
// exact top-k of select_block.h on x for itself and keeps sc_indices and
// x[sc_indices] in LDS, so step 1 costs no launch of its own and no trip
// through global memory (the paper's fused kernel does step 1 inside the
// kernel too, Section 4.3, but needs a grid-wide barrier because its
// selection is spread over the thread blocks; an exact select that is cheap
// enough to repeat per workgroup needs none).  Workgroup 0 also writes the
// selection to global memory for the caller.
//
// The link stands idle until the first row is requested: 2.0 us of a call with
// 4096 channels, 3.4 with 14336 (stamps of the first workgroup).  But once the
// bound of the selection is known, after 0.8 / 1.2 us, most of the selected
// channels are: the maxima of the chunks in a bin above.  EARLY (below) requests
// their rows then; the selection marks those that it has (a tag beside the
// index), and they are worked off in their place among the others, so that the
// sum has the same bits.  A row that is not selected after all is dropped.
// 4096 x 4096, 60 4-bit rows 8.4 -> 7.1 us; 14336 x 4096, 56 8-bit rows 10.9 ->
// 9.8; 5120 x 13824, 60 4-bit rows 15.0 -> 12.7.  What it costs is the issue of
// the requests (a wavefront's request of 1 KiB occupies its compute unit for
// about 50 ns, and the wavefronts that wait for it also make the selection).
#pragma once
#include <hip/hip_runtime.h>

#include "finalize.h"
#include "kernels.h"
#include "layout.h"
#include "select_block.h"

namespace decdec {

__device__ __forceinline__ float h2f(uint32_t bits16) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}

// sc_indices / x[sc_indices] as the fetch loops see them: global memory, or LDS
// after an in-kernel selection.
struct Selection {
    const int32_t* idx;
    const uint16_t* xsel;
};

// `ask`: select_block.h.  What it adds to an index is above bit 15 (K <= 32768 here).
template <int SELECT_NCH, typename Ask>
__device__ __forceinline__ Selection obtain_selection(const uint4* keys, int K, int k, int32_t* idx_g, uint16_t* xsel_g,
                                                      SelectShared<kBlockThreads, SELECT_NCH>& sh, int bid, const Ask& ask) {
    if constexpr (SELECT_NCH > 0) {
        extern __shared__ uint4 s_sel_raw[];
        int32_t* idx_l = reinterpret_cast<int32_t*>(s_sel_raw);
        uint16_t* xs_l = reinterpret_cast<uint16_t*>(idx_l + k);
        uint4 ch[SELECT_NCH];
#pragma unroll
        for (int j = 0; j < SELECT_NCH; ++j) ch[j] = keys[j];
        block_select_topk<kBlockThreads, SELECT_NCH>(ch, FullRuns<kBlockThreads, SELECT_NCH>(K / 8), K, k, sh, idx_l, xs_l, ask);
        __syncthreads();
        if (bid == 0) {
            for (int i = threadIdx.x; i < k; i += kBlockThreads) {
                idx_g[i] = idx_l[i] & 0xFFFF;
                xsel_g[i] = xs_l[i];
            }
        }
        return Selection{idx_l, xs_l};
    } else {
        return Selection{idx_g, xsel_g};
    }
}

// Wave-uniform load of data that this kernel does not write, through the scalar cache.  The compiler does so by itself only
// while no asm statement stands in front.  A supplied selection's row numbers read by vector loads cost a trip of their own
// per batch of rows: 81 fp16 rows of 4096 columns by two wavefronts a segment 21.1 -> 28.6 us.
__device__ __forceinline__ int load_constant(const int32_t* p) {
    return *(const __attribute__((address_space(4))) int32_t*)(uintptr_t)p;
}

// What one lane loads of one row: 8 columns (16 of 2-bit codes), BITS bits each; never less than 4 bytes.
template <int BITS>
struct RowPiece;
template <>
struct RowPiece<16> {
    typedef uint4 type;
};
template <>
struct RowPiece<8> {
    typedef uint2 type;
};
template <>
struct RowPiece<4> {
    typedef uint32_t type;
};
template <>
struct RowPiece<2> {
    typedef uint32_t type;
};

// acc[i] += value of column i of the piece * xs.
template <int BITS, int CPL>
__device__ __forceinline__ void accumulate_piece(const typename RowPiece<BITS>::type& v, float xs, float (&acc)[CPL]) {
    if constexpr (BITS == 16) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            acc[2 * c] = fmaf(h2f(w[c] & 0xFFFFu), xs, acc[2 * c]);
            acc[2 * c + 1] = fmaf(h2f(w[c] >> 16), xs, acc[2 * c + 1]);
        }
    } else if constexpr (BITS == 8) {
        const uint32_t w[2] = {v.x, v.y};
#pragma unroll
        for (int i = 0; i < 8; ++i)
            acc[i] = fmaf((float)((int)(w[i >> 2] << (24 - 8 * (i & 3))) >> 24), xs, acc[i]);
    } else {
        const uint32_t w = v;  // CPL two's-complement fields of BITS bits
#pragma unroll
        for (int i = 0; i < CPL; ++i)
            acc[i] = fmaf((float)((int)(w << (32 - BITS * (i + 1))) >> (32 - BITS)), xs, acc[i]);
    }
}

template <int BITS>
constexpr int kLaneCols = BITS == 2 ? 16 : 8;                                  // columns per lane
template <int BITS>
constexpr int kLoadRows = 64 / (kFetchSegmentCols / kLaneCols<BITS>);  // rows a wavefront loads with one instruction

// Rows asked for while the selection goes on: 32 bytes a lane, in registers until the selection is complete.  Not with
// 2-bit rows, nor with eight chunks of keys per thread, where there are no registers for them.
template <int BITS, int SELECT_NCH>
constexpr bool kAsksEarly = SELECT_NCH > 0 && SELECT_NCH < 8 && BITS != 2;
template <int BITS>
constexpr int kLanesPerEarlyRow = kFetchSegmentCols * BITS / 128;  // 16 bytes each
template <int BITS>
constexpr int kEarlyRows = 2 * 64 / kLanesPerEarlyRow<BITS>;  // per wavefront
static_assert(kEarlyRows<4> <= 8, "SelectShared::asked");
// Rows that a wavefront has LDS for: both 16-byte pieces of its lanes, or the first ones where that is enough, as it is in wide
// matrices.  Their base GEMV outlasts few rows, and a workgroup starts earlier where the LDS holds one more than the wavefronts
// that fit, because those of another that have ended leave its LDS behind: 20 4-bit rows, 4-bit weights, 8192 x 16384 13.1 us
// with 31 KiB a workgroup, 13.5 with 32 (33 as allocated) or 39; 14336 x 16384 20.9 and 21.1.
template <int BITS>
__host__ __device__ constexpr int early_slots(int early) {
    return early <= kEarlyRows<BITS> / 2 ? kEarlyRows<BITS> / 2 : kEarlyRows<BITS>;
}

// The selection and the sum over the wavefronts follow one another and share their LDS.
template <int BITS, int SELECT_NCH>
union FetchLds {
    float red[kWavesPerBlock * kLoadRows<BITS>][kFetchSegmentCols];
    SelectShared<kBlockThreads, SELECT_NCH> sh;
    __device__ FetchLds() {}
};

// Dynamic LDS: int32 idx[k] and fp16 xsel[k] of a selection made here, then the rows asked for early.
__host__ __device__ inline unsigned selection_lds_bytes(int select_chunks, int k) {
    return select_chunks > 0 ? (unsigned)(((size_t)k * 6 + 15) / 16 * 16) : 0u;
}
// Host: of a kernel that selects for itself.
template <int BITS>
inline unsigned fetch_lds_bytes(const CallArgs& a, int select_chunks) {
    const unsigned early = a.early > 0 ? kWavesPerBlock * early_slots<BITS>(a.early) * (kFetchSegmentCols * BITS / 8) : 0u;
    return selection_lds_bytes(select_chunks, a.k) + early;
}

// One workgroup = one column segment of 512 columns x the rows of row slice rs.  A lane reads 8 columns of a
// row (16, 8 or 4 bytes for fp16, 8-bit and 4-bit rows: a wavefront 1 KiB down to 256 bytes of contiguous
// row) or 16 columns of a 2-bit row (4 bytes; the two halves of a wavefront then take different rows).
// Wavefront w < row_waves takes a contiguous share of the workgroup's rows and keeps 4 KiB of row loads in
// flight in every format.  BITS = 16: fp16 rows.  BITS = 2, 4, 8: integer residuals (Section 4.2: 4-bit
// symmetric with one scale per output column; 2- and 8-bit are the variants of the paper's bit-width study,
// Table 2),  o_dec[n] = S[n] * sum_j q[s_j][n] x[s_j].
//
// After the row loop the sums of the wavefronts (and half-wavefronts) are added through LDS in a fixed
// order: thread t of the workgroup ends up with the segment's sum for column t and adds it into the
// column's accumulator (finalize.h), or, when a separate kernel does the adding, writes it to row rs of cpart.
//
// Workgroup `bid` is slice rs = bid % a.cslices of segment bid / a.cslices, counted over all matrices.
//
// EARLY: rows are asked for while the selection goes on (a.early of them per wavefront at most); code of its own, because the
// few instructions that this takes on the way would cost calls without it up to 0.5 us.  fetch_plan says which calls.
template <int BITS, int SELECT_NCH, bool EARLY>
__device__ __forceinline__ void fetch_block(const CallArgs& a, int bid, FetchLds<BITS, SELECT_NCH>& lds) {
    typedef typename RowPiece<BITS>::type piece_t;
    constexpr int CPL = kLaneCols<BITS>, SUB = kLoadRows<BITS>;
    constexpr int LPR = kFetchSegmentCols / CPL;        // lanes that cover the segment's part of one row
    constexpr int UNROLL = (4096 / 64) / (int)sizeof(piece_t);  // loads in flight per lane: 4 KiB per wavefront
    static_assert(kBlockThreads == kFetchSegmentCols, "one thread per column of the segment");
    static_assert(!EARLY || kAsksEarly<BITS, SELECT_NCH>, "early rows");
    auto& red = lds.red;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k = a.k, K = a.G * kGroup;
    // the keys are asked for before anything else: the selection is the first link of this workgroup's chain of waits
    uint4 keys[SELECT_NCH > 0 ? SELECT_NCH : 1];
    if constexpr (SELECT_NCH > 0) load_keys(a.x, FullRuns<kBlockThreads, SELECT_NCH>(K / 8), keys);
    const int row_waves = a.row_waves, slices = a.cslices;
    const int seg = divide_by(bid, a.cdiv);
    const int rs = bid - seg * slices;
    int m = 0, seg0 = 0;
#pragma unroll
    for (int i = 0; i < kMaxMulti - 1; ++i) {
        if (i + 1 < a.n && seg >= a.mat[i].seg_end) {
            m = i + 1;
            seg0 = a.mat[i].seg_end;
        }
    }
    const int wc = seg - seg0;
    const MatArgs& mat = a.mat[m];
    int N = mat.N, col0 = mat.col0, producers = a.producers;
    const uint4* rows_base = mat.R;
    const uint16_t* Rs = mat.Rs;
    _Float16* y = mat.y;
    unsigned long long* acc_words = a.acc;
    hold_scalar(N, col0, producers);
    hold_scalar(rows_base);
    hold_scalar(Rs);
    hold_scalar(y);
    hold_scalar(acc_words);

    const int ocol = wc * kFetchSegmentCols + tid;  // the column this thread owns after the LDS round
    const bool owns = ocol < N;
    // The column scale is requested in front of the selection and first touched (hold_vector) behind the rows.  Converted where
    // it is loaded, as the compiler has it, it is waited for in front of the first row request: us, before -> now: 4096 x 28672,
    // 60 4-bit rows 22.8 -> 21.8; 14336 x 4096, 56 8-bit rows 11.4 -> 11.0; 210 8-bit rows in GPU memory 8.4 -> 7.9.  (With eight
    // chunks of keys per thread there is no register for it during the selection.)
    constexpr bool kScaleFirst = SELECT_NCH < 8;
    uint32_t sraw = 0;
    if constexpr (BITS != 16 && kScaleFirst) sraw = Rs[min(ocol, N - 1)];

    // This wavefront's part of the rows that are nearly certain is asked for before the selection is complete.  Where several
    // workgroups share a segment's rows, each takes those of the channels that are likely to be in its share.  The requests
    // are made on every path, if need be for the first bytes of x: loads that only some paths make are waited for where the
    // paths meet.
    uint4 early0, early1;
    const auto ask = [&](const uint4& chunk_keys, int chunk, unsigned top, unsigned edge) -> unsigned {
        unsigned tag = 0;
        if constexpr (EARLY) {
            constexpr int LPE = kLanesPerEarlyRow<BITS>;
            const int most = wave * slices / kWavesPerBlock == rs ? a.early : 0;
            const bool wanted = top >= edge;
            const unsigned long long b = __ballot(wanted);
            const int rank = (int)lanes_before(b), n = min((int)__builtin_popcountll(b), most);
            uint16_t* asked = lds.sh.asked[wave];
            if (wanted && rank < n) {
                const int e = __builtin_ctz(mark_above(chunk_keys, top - 1));
                asked[rank] = (uint16_t)(chunk * 8 + e);
                tag = (unsigned)e | (unsigned)(wave * early_slots<BITS>(a.early) + rank + 1) << 3;
            }
            wave_writes_seen();
            const unsigned pieces = (unsigned)N * BITS / 128;
            const unsigned at = wc * LPE + lane % LPE;
            const int i0 = lane / LPE, i1 = 64 / LPE + lane / LPE;
            const uint4* none = reinterpret_cast<const uint4*>(a.x);
            const uint4 *p0 = rows_base + (size_t)asked[i0] * pieces + at, *p1 = rows_base + (size_t)asked[i1] * pieces + at;
            p0 = i0 < n && at < pieces ? p0 : none;
            p1 = i1 < n && at < pieces ? p1 : none;
            early0 = *p0;
            early1 = *p1;
        }
        return tag;
    };
    const Selection sel = [&] {
        if constexpr (EARLY) {
            return obtain_selection<SELECT_NCH>(keys, K, k, a.idx, a.xsel, lds.sh, bid, ask);
        } else {
            return obtain_selection<SELECT_NCH>(keys, K, k, a.idx, a.xsel, lds.sh, bid, AskNothing());
        }
    }();
    if constexpr (BITS != 16 && !kScaleFirst) {
        sraw = Rs[min(ocol, N - 1)];
        __builtin_amdgcn_sched_barrier(0);  // not among the row requests
    }
    const int32_t* idx = sel.idx;
    const uint16_t* xsel = sel.xsel;
    const piece_t* __restrict__ R = reinterpret_cast<const piece_t*>(rows_base);
    const int sub = lane / LPR;                       // which of the SUB rows of a load instruction
    const int piece = wc * LPR + (lane % LPR);      // this lane's CPL columns of a row
    const bool active = piece * CPL < N;
    const size_t row_pieces = (size_t)(N / CPL);
    // rows of this wavefront: slice (rs, wave) out of slices * row_waves equal shares of the k selected rows
    const int rows_per = a.rows_per;
    const int j0 = min((rs * row_waves + wave) * rows_per, k);
    const int j1 = wave < row_waves ? min(j0 + rows_per, k) : j0;


    // Behind the requests of a batch a look at the column's accumulator (fetch_plan says when): a workgroup that sees the base
    // GEMV's part sums there writes y without the trip of an atomic.  Decided at run time: compiled without it, the loop takes 1 to
    // 7 % longer with 61 to 122 rows of 4096 x 4096.
    const bool looks = EARLY && BITS == 16 && a.look != 0 && acc_words != nullptr;
    unsigned long long seen = 0;

    float acc[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) acc[i] = 0.f;
    // A batch of up to UNROLL rows in sets of up to 8.  In a set every request is made, those without a row of their own for the
    // first bytes of x.  So what was asked for early can be waited for alone; and sixteen conditions cost more than the requests
    // that they save (4-bit rows, 4096 x 4096, 60 of them in GPU memory 6.06 us with conditions and 5.46 without, over the link
    // 8.37 and 8.06), eight or four less (210 8-bit rows of 14336 x 4096 in GPU memory 7.8 and 8.1, 81 fp16 rows 5.33 and 5.53).
    constexpr bool kAllRequests = EARLY || (BITS == 4 && SELECT_NCH > 0);
    if constexpr (kAllRequests) {
        constexpr int SET = UNROLL < 8 ? UNROLL : 8;
        const char* lane_row = reinterpret_cast<const char*>(rows_base) + min(piece, (int)row_pieces - 1) * (int)sizeof(piece_t);
        const char* none = reinterpret_cast<const char*>(a.x);
        const unsigned row_bytes = (unsigned)row_pieces * (unsigned)sizeof(piece_t);
        extern __shared__ uint4 s_sel_raw[];
        uint4* early_lds = s_sel_raw + selection_lds_bytes(SELECT_NCH, k) / 16;
        bool asked = EARLY;
        int j = j0;
        do {
            piece_t v[UNROLL];
#pragma unroll
            for (int u0 = 0; u0 < UNROLL; u0 += SET) {
                if (u0 > 0 && j + u0 >= j1) break;
                unsigned entry[SET];
#pragma unroll
                for (int u = 0; u < SET; ++u) entry[u] = (unsigned)idx[min(j + u0 + u, k - 1)];
#pragma unroll
                for (int u = 0; u < SET; ++u) {
                    const unsigned limit = j + u0 + u < j1 ? (unsigned)K : 0u;
                    const char* row = lane_row + (unsigned long long)entry[u] * row_bytes;
                    row = entry[u] < limit ? row : none;  // a tag: it has been asked for
                    v[u0 + u] = *reinterpret_cast<const piece_t*>(row);
                }
            }
            if (looks) seen = arrived_so_far(acc_words + col0 + min(ocol, N - 1));
            if constexpr (EARLY) {
                if (asked) {
                    asked = false;
                    const bool both = early_slots<BITS>(a.early) == kEarlyRows<BITS>;
                    uint4* to = early_lds + (both ? wave * 128 : wave * 64) + lane;
                    to[0] = early0;
                    // on every path, if need be to a place that nobody reads: with a condition 14336 x 4096 takes 0.15 us more
                    to = both ? to + 64 : reinterpret_cast<uint4*>(red) + lane;
                    to[0] = early1;
                    __syncthreads();
                }
            }
#pragma unroll
            for (int u0 = 0; u0 < UNROLL; u0 += SET) {
                if (j + u0 >= j1) break;
                uint32_t xraw[SET];
#pragma unroll
                for (int u = 0; u < SET; ++u) xraw[u] = xsel[min(j + u0 + u, j1 - 1)];
                if constexpr (EARLY) {
                    const char* early_piece = reinterpret_cast<const char*>(early_lds) + lane * sizeof(piece_t);
                    piece_t w[SET];
                    unsigned slot[SET];  // 0: not asked for early
#pragma unroll
                    for (int u = 0; u < SET; ++u) slot[u] = (unsigned)__builtin_amdgcn_readfirstlane(idx[min(j + u0 + u, j1 - 1)]) >> 16;
#pragma unroll
                    for (int u = 0; u < SET; ++u)
                        w[u] = *reinterpret_cast<const piece_t*>(early_piece + (max(slot[u], 1u) - 1) * (kFetchSegmentCols * BITS / 8));
#pragma unroll
                    for (int u = 0; u < SET; ++u)
                        if (j + u0 + u < j1) accumulate_piece<BITS, CPL>(slot[u] ? w[u] : v[u0 + u], h2f(xraw[u]), acc);
                } else {
#pragma unroll
                    for (int u = 0; u < SET; ++u)
                        if (j + u0 + u < j1) accumulate_piece<BITS, CPL>(v[u0 + u], h2f(xraw[u]), acc);
                }
            }
            j += UNROLL;
        } while (j < j1);
    }
    for (int j = kAllRequests ? j1 : j0; j < j1; j += UNROLL * SUB) {
        piece_t v[UNROLL];
        float xs[UNROLL];
        int row[UNROLL];
        uint32_t xraw[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {  // indices and activations first, so that no row load waits for them
            const int jj = min(j + u * SUB + sub, j1 - 1);
            if constexpr (SELECT_NCH == 0 && SUB == 1) {
                row[u] = load_constant(idx + jj);
            } else {
                row[u] = idx[jj];
            }
            xraw[u] = xsel[jj];
        }
        if constexpr (BITS == 4) {
            // The activation of a row that does not count is cleared where the row is requested, so that the row's lane mask
            // ends there: sixteen masks, kept until the activations are used, do not fit beside the rest into the 80 scalar
            // registers that leave room for eight wavefronts a SIMD.  All activations have to be there before the first
            // request: the requests are conditional, so that a wait for one activation between them waits for rows too
            // (1194 4-bit rows of 4096 columns, selection supplied: 53 instead of 49 us).
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) hold_vector(xraw[u]);
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const bool valid = j + u < j1 && (unsigned)row[u] < (unsigned)K;
                v[u] = piece_t{};
                if (valid && active) v[u] = R[(size_t)row[u] * row_pieces + piece];
                xraw[u] = valid ? xraw[u] : 0;
                hold_vector(xraw[u]);
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) xs[u] = h2f(xraw[u]);
        } else {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                v[u] = piece_t{};
                if (j + u * SUB + sub < j1 && active && (unsigned)row[u] < (unsigned)K)
                    v[u] = R[(size_t)row[u] * row_pieces + piece];
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                xs[u] = (j + u * SUB + sub < j1 && (unsigned)row[u] < (unsigned)K) ? h2f(xraw[u]) : 0.f;
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            if (j + u * SUB < j1) accumulate_piece<BITS, CPL>(v[u], xs[u], acc);  // wave-uniform: rows it does not have cost nothing
    }

    // Sum over the wavefronts (and their halves) of the workgroup.
    if (wave < row_waves) {
        float4* dst = reinterpret_cast<float4*>(&red[wave * SUB + sub][(lane % LPR) * CPL]);
#pragma unroll
        for (int i = 0; i < CPL / 4; ++i) dst[i] = make_float4(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]);
    }
    __syncthreads();
    float val = red[0][tid];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock * SUB; ++w)
        if (w < row_waves * SUB) val += red[w][tid];  // wave-uniform
    if constexpr (BITS != 16) {
        hold_vector(sraw);
        val *= h2f(sraw);
    }

    if (owns) {
        if (acc_words != nullptr) {
            if (looks) {
                arrive_after_look(acc_words + col0 + ocol, y + ocol, producers, val, seen);
            } else {
                arrive(acc_words + col0 + ocol, y + ocol, producers, val);
            }
        } else {
            a.cpart[(size_t)rs * a.Ntot + col0 + ocol] = val;
        }
    }
}

template <int BITS, int SELECT_NCH>
__device__ __forceinline__ void fetch_block(const CallArgs& a, int bid) {
    __shared__ FetchLds<BITS, SELECT_NCH> lds;
    if constexpr (kAsksEarly<BITS, SELECT_NCH>) {
        if (a.early > 0) {
            fetch_block<BITS, SELECT_NCH, true>(a, bid, lds);
            return;
        }
    }
    fetch_block<BITS, SELECT_NCH, false>(a, bid, lds);
}

}  // namespace decdec
