// Stage 2 (Sec. 3.2.2): one level of hierarchical pruning.
//
//   row_stats_kernel     MFMA pass 1 over all keys: per (head, text query) sum of the causal softmax, relative to a
//                        number of its own, in the log2 domain, per workgroup; leaves the queries in MFMA fragment order
//   merge_stats_kernel   merges the per-workgroup partial sums into one normaliser per row (pass 2 does it for itself where
//                        they are few)
//   col_sums_kernel      MFMA pass 2 over the visual keys: recomputes the logits and adds up the
//                        probabilities of every visual key over the rows of a workgroup
//   narrow_row_stats_kernel, narrow_col_sums_kernel   the two passes for at most 64 query rows per kv head
//   score_select_kernel  score_j = w_e(j) * mean probability per tile; the workgroup that arrives last selects per class
//                        (radix select) and writes the ascending index list
//   prepare_kernel, select_kernel, write_index_kernel   the same steps where that one workgroup is no match for them (see
//                        one_launch_selection): scores; one workgroup per class walks all keys; one workgroup per 1024-token tile
//                        applies the keep rule and writes the index list and the carried metadata
//   gather_rows_kernel   compaction of the hidden states (hidden_index_kernel + the row mover of stage 3 when
//                        the output is the input buffer) and, after score_select_kernel, of the carried metadata
//
// A batch of videos of one shape runs as one launch of every kernel: blockIdx.z is the video, every pointer
// advances by that video's stride, and the per-video workspaces lie one after the other.
//
// Both MFMA passes are query-stationary: a wave keeps the fragments of its own 32-row blocks of queries in
// registers and the workgroup streams its range of keys through LDS.  The contraction index may be
// permuted freely as long as both operands agree; here lane half h = lane/32 owns the contiguous half h
// of the head dimension, so every fragment is a contiguous 16-byte chunk of a row.
#include <algorithm>
#include <mutex>

#include "common.h"
#include "score_plan.h"

namespace metok {

constexpr float kNegBig = -1.0e30f;
constexpr float kPosBig = 1.0e30f;

// v_exp_f32 without the denormal-range fix-up of exp2f(): a result below 2^-126 may flush to zero (it is a softmax term that
// small).
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <typename T> struct Mma;
template <> struct Mma<bf16_t> {
    static constexpr int kChunkElems = 8;          // one 16-byte chunk feeds one 32x32x16 MFMA
    static constexpr int kMfmaPerChunk = 1;
    static __device__ __forceinline__ f32x16_t mma(const uint4& a, const uint4& b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    }
};
template <> struct Mma<float> {
    static constexpr int kChunkElems = 4;          // one chunk feeds four 32x32x2 MFMAs
    static constexpr int kMfmaPerChunk = 4;
    static __device__ __forceinline__ f32x16_t mma(const uint4& a, const uint4& b, f32x16_t c) {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
        return c;
    }
};

// fp32 rows multiplied as bf16.  An element is the sum of three bf16 numbers, each the nearest to what the ones before leave, without a
// rounding (the last has at most eight bits left); of the nine products of two such numbers six are taken, each with 16 times the rate of
// an fp32 MFMA: 192 cycles of the matrix pipe per 32 x 32 x 16 products instead of 512.  The other three, middle by last and last by
// last, are together below 2^-24 of the whole (0.9 at most) and of either sign.  (Parts that are cut off all have the sign of their
// element: the three reach 7.8 x 2^-24 and shrink every product.)
// Root mean square error of a sum against 64 bits, in units of its size, fp32 MFMA / parts, normal elements of which n of a row are not
// 0: n = 1 2.54e-8 / 2.61e-8, 2 3.1e-8 / 2.6e-8, 4 4.0e-8 / 2.7e-8, 8 5.3e-8 / 2.9e-8, all 64 14.3e-8 / 4.9e-8, all 128 20.2e-8 / 6.5e-8;
// parts cut off 6.9e-8 up to n = 8, then 7.5e-8 and 8.5e-8.
// Whole calls by graph replay, fp32 MFMA / parts: 28 heads on 4 x 64 queries of 128 elements, 8 x 4000 tokens 352 / 242 us, 24000 tokens
// 287 / 204; see split_products for where they are taken.
struct split_t { float value; };
template <> struct Mma<split_t> : Mma<float> {};

// 16-byte operand registers of a lane for a row block or a subtile: its NCH pieces of memory, or three numbers for each of their elements
template <typename T, int NCH> constexpr int kOperands = std::is_same<T, split_t>::value ? NCH / 2 * 3 : NCH;

__device__ __forceinline__ bool is_finite_bits(uint32_t x) { return (x & 0x7f800000u) != 0x7f800000u; }

// Four elements -> their leading, middle and last parts.  For elements beyond kPartsBelow the caller takes exact_parts instead.
__device__ __forceinline__ void split_piece(const uint4& x, uint2 (&part)[3]) {
    float e[4] = {__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w)};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        part[p] = make_uint2(pack_bf16x2(e[0], e[1]), pack_bf16x2(e[2], e[3]));
        if (p < 2) { e[0] -= bf16_lo(part[p].x); e[1] -= bf16_hi(part[p].x); e[2] -= bf16_lo(part[p].y); e[3] -= bf16_hi(part[p].y); }
    }
}
// Elements below this are multiplied in parts: no sum of 128 of their products leaves the range of float, whatever the order, and parts
// too small for a bf16 number of full precision (below 2^-126) are less than 2^-58 of a logit together.
// One comparison of the largest magnitude, above which infinities and NaNs are: with four of floats the 5000 tokens at split_products took
// 36.5 us.
constexpr uint32_t kPartsBelow = 0x5d000000u;                      // 2^59
__device__ __forceinline__ bool all_fit(const uint4& x) {
    auto magnitude = [](uint32_t e) { return e & 0x7fffffffu; };
    return max(max(magnitude(x.x), magnitude(x.y)), max(magnitude(x.z), magnitude(x.w))) < kPartsBelow;
}
// The same for elements of which some do not fit: parts that joined_piece puts together again (short of less than 2^-133).  The leading
// part of the largest must not round to infinity, so they are cut off; what is not finite is its leading part alone, a NaN stays one.
__device__ __forceinline__ uint32_t quiet(uint32_t x) { return (x & 0x7fffffffu) > 0x7f800000u ? x | 0x00400000u : x; }
__device__ __forceinline__ uint32_t below_leading(uint32_t x) { return __float_as_uint(__uint_as_float(x) - __uint_as_float(x & 0xffff0000u)); }
__device__ __forceinline__ uint32_t upper_halves(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }
__device__ __forceinline__ void exact_parts(const uint4& x, uint2 (&part)[3]) {
    const uint32_t e[4] = {quiet(x.x), quiet(x.y), quiet(x.z), quiet(x.w)};
    uint32_t lead[4], mid[4], last[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool f = is_finite_bits(e[i]);
        lead[i] = e[i];
        mid[i] = f ? below_leading(e[i]) : 0u;
        last[i] = f ? below_leading(mid[i]) : 0u;
    }
    part[0] = make_uint2(upper_halves(lead[0], lead[1]), upper_halves(lead[2], lead[3]));
    part[1] = make_uint2(upper_halves(mid[0], mid[1]), upper_halves(mid[2], mid[3]));
    part[2] = make_uint2(upper_halves(last[0], last[1]), upper_halves(last[2], last[3]));
}
// Piece c of the 2 n pieces that the operands f[3 n] were made of
__device__ __forceinline__ uint4 joined_piece(const uint4* f, int c) {
    const uint4* a = f + c / 2 * 3;
    uint32_t w[3][2];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        w[p][0] = c & 1 ? a[p].z : a[p].x; w[p][1] = c & 1 ? a[p].w : a[p].y;
        asm volatile("" : "+v"(w[p][0]), "+v"(w[p][1]));            // made where it is used, not kept from one subtile to the next
    }
    auto element = [&](int i) {
        auto part = [&](int p) { return i & 1 ? bf16_hi(w[p][i >> 1]) : bf16_lo(w[p][i >> 1]); };
        return __float_as_uint(part(0) + part(1) + part(2));
    };
    return make_uint4(element(0), element(1), element(2), element(3));
}
// Operands of a row block from its pieces; true: every element of the lane fits.
template <typename T, int NCH>
__device__ __forceinline__ bool make_operands(const uint4 (&raw)[NCH], uint4 (&op)[kOperands<T, NCH>]) {
    bool fit = true;
    if constexpr (std::is_same<T, split_t>::value) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) fit = fit && all_fit(raw[c]);
#pragma unroll
        for (int c = 0; c < NCH; c += 2) {
            uint2 a[3], b[3];
            if (fit) { split_piece(raw[c], a); split_piece(raw[c + 1], b); } else { exact_parts(raw[c], a); exact_parts(raw[c + 1], b); }
#pragma unroll
            for (int p = 0; p < 3; ++p) op[c / 2 * 3 + p] = make_uint4(a[p].x, a[p].y, b[p].x, b[p].y);
        }
    } else {
#pragma unroll
        for (int c = 0; c < NCH; ++c) op[c] = raw[c];
    }
    return fit;
}

// Kept visual tokens of every video of a batch (the quotas of a video added up), passed by value.
struct BatchKeep { int32_t n[METOK_MAX_BATCH]; };

// ---------------------------------------------------------------------------------------------
// Both MFMA passes are query-stationary: wave w of a workgroup keeps the fragments of its own row
// blocks (local blocks w, w + 8, ...) in registers for the whole kernel, and the workgroup streams its
// contiguous range of keys through LDS, one stage of SUBS 32-key subtiles at a time (kStageBuffers
// stages in LDS, one barrier per stage).  A stage is stored in fragment order,
//     kbuf[(sub * NCH + c) * 64 + lane],   lane = key % 32 + 32 * half,
// so a wave reads the NCH fragments of a subtile with conflict-free 16-byte LDS reads and uses them
// against every row block it owns.
// ---------------------------------------------------------------------------------------------
template <typename T, int NCH, int SUBS>
struct KeyStage {
    static constexpr int kKeys = SUBS * 32;
    static constexpr int kPieces = SUBS * NCH * 64;                // 16-byte pieces of memory per stage
    static constexpr int kSlots = SUBS * kOperands<T, NCH> * 64;   // of LDS
    static constexpr int kPerThread = (kPieces + kScoreThreads - 1) / kScoreThreads;

    // piece id -> (key in stage, half, chunk); the key runs fastest so that the LDS writes of a wave are contiguous
    static __device__ __forceinline__ void load(u32x4_t (&v)[kPerThread], const T* __restrict__ k_head, int64_t j0, int64_t S, int dh) {
        constexpr int CE = Mma<T>::kChunkElems;
#pragma unroll
        for (int u = 0; u < kPerThread; ++u) {
            int id = threadIdx.x + u * kScoreThreads;
            id = id < kPieces ? id : 0;                             // surplus threads repeat piece 0 and do not store it
            const int jl = id % kKeys, p = id / kKeys;
            int64_t j = j0 + jl;
            j = j < S ? j : S - 1;                                  // stages may overhang the sequence; masked later
            // S < 2^31: one 32 x 32 -> 64 bit multiply instead of a 64-bit one in every stage
            const size_t row = static_cast<size_t>(static_cast<uint32_t>(j)) * static_cast<uint32_t>(dh);
            v[u] = *reinterpret_cast<const u32x4_t*>(k_head + row + (p / NCH) * (dh / 2) + (p % NCH) * CE);
        }
    }
    // UNCHECKED_ROUNDS: rounds in which every thread of the workgroup owns a piece skip the bounds check,
    // which keeps a branch out of the caller's loop body.
    template <bool UNCHECKED_ROUNDS = false>
    static __device__ __forceinline__ void store(const u32x4_t (&v)[kPerThread], uint4* __restrict__ kbuf) {
#pragma unroll
        for (int u = 0; u < kPerThread; ++u) {
            const int id = threadIdx.x + u * kScoreThreads;
            const int jl = id % kKeys, p = id / kKeys;
            if ((UNCHECKED_ROUNDS && (u + 1) * kScoreThreads <= kPieces) || id < kPieces)
                reinterpret_cast<u32x4_t*>(kbuf)[((jl >> 5) * NCH + (p % NCH)) * 64 + (jl & 31) + 32 * (p / NCH)] = v[u];
        }
    }
    // Three parts of every element; false: an element of this thread does not fit.
    static __device__ __forceinline__ bool store_split(const u32x4_t (&v)[kPerThread], uint4* __restrict__ kbuf) {
        bool fit = true;
#pragma unroll
        for (int u = 0; u < kPerThread; ++u) {
            const int id = threadIdx.x + u * kScoreThreads;
            const int jl = id % kKeys, p = id / kKeys, c = p % NCH;
            const uint4 x = make_uint4(v[u].x, v[u].y, v[u].z, v[u].w);
            uint2 part[3];
            if (__builtin_expect(all_fit(x), 1)) split_piece(x, part);
            else { fit = false; exact_parts(x, part); }
            uint2* dst = reinterpret_cast<uint2*>(kbuf) + 2 * (((jl >> 5) * (NCH / 2 * 3) + c / 2 * 3) * 64 + (jl & 31) + 32 * (p / NCH)) + (c & 1);
            if ((u + 1) * kScoreThreads <= kPieces || id < kPieces) {
#pragma unroll
                for (int q = 0; q < 3; ++q) dst[2 * 64 * q] = part[q];
            }
        }
        return fit;
    }
};

// Query fragments in MFMA operand order, written once per call (by the first workgroups of pass 1) for pass 2:
//     qfrag[((kvh * rb_total + rb) * NCH + c) * 64 + lane],  row = 32 rb + lane % 32, half = lane / 32,
// 16 bytes each (elements half * dh/2 + c * CE ... of the row); rows past the last query are zero.
// A wave then fetches a fragment with one fully coalesced 1 KB load instead of 64 strided 16-byte pieces.
//
// Pass 1 takes its fragments from the rows themselves.  The rows of a block lie one after the other (row r of kv head v is
// row v * R + r of q_text), so a wave loads them in memory order, 1 KB a time, and turns them into fragments through a
// part of LDS of its own: kRows rows a round, piece p of a row at p ^ (row mod pieces), which spreads both the writes
// (pieces of a row) and the reads (one piece of 32 rows) over the banks.  A packing kernel in front
// took 3.2 us a call; this costs pass 1 about 1 us, with eight videos per launch 3 of the kernel's 5 us (one level of 2243
// tokens, 28 / 4 heads x 64 queries: 35.5 -> 33.4 us, of 5000 in fp32: 39.2 -> 37.0 us, eight videos of 36864 tokens: within
// the noise).
//
// Row blocks of the waves.  Block w belongs to wave w.  Of the x = nrb - 8 blocks beyond, block 8 + w is the second one of wave
// w; waves w and w + 4 sit on one SIMD, so with x = 1, 2, 5 or 6 one or two SIMDs have a block more than the others and every
// stage waits for them.  There the last x % 4 second blocks are shared with the waves two further on, which have one block
// only: the first wave takes subtile 0 of a stage, the other one subtile 1.  28 heads on 4 x 64 queries are 14 blocks (4, 4, 3,
// 3 a SIMD unshared, 3.5 shared): eight videos of 36864 tokens, pass 1 152 -> 144 us (1.05 PFLOP/s), pass 2 157 -> 151 us.  It
// costs two waves a load more before the first stage, so short ranges go unshared (where their rows are not split, see plan_score): 18432 tokens (5 stages) 17.7 -> 17.1 us in
// pass 1 but 13.8 -> 14.3 in pass 2, 2243 tokens (1 stage) 9.0 -> 9.4 and 6.2 -> 6.5.  Ranges below kMinPipelined stages do
// not take pass 1's software pipeline either (2243 tokens 9.4 -> 9.2 us).  Levels of 9 to 17 blocks, 300 to 24000 tokens, bf16 with 32
// to 128 elements and fp32 with 32 and 64, are none slower than before these lines were drawn.
constexpr int kMinPipelined = 4, kMinSharedRows = 4, kMinSharedCols = 8;         // stages of a workgroup
enum class SecondBlock { kNone, kBoth, kSubtile0, kSubtile1 };
template <int RBW>
__device__ __forceinline__ SecondBlock second_block(int nrb, int wave, bool share) {
    const int x = RBW == 2 ? nrb - kScoreWaves : 0, shared_from = share && ((x & 3) == 1 || (x & 3) == 2) ? x & ~3 : x;
    if (wave < x) return wave < shared_from ? SecondBlock::kBoth : SecondBlock::kSubtile0;
    return x > 0 && wave - 2 >= shared_from && wave - 2 < x ? SecondBlock::kSubtile1 : SecondBlock::kNone;
}
// Row block i of a wave among the workgroup's nrb, -1: it has none.
template <int RBW>
__device__ __forceinline__ int wave_block(int nrb, int wave, SecondBlock second, int i) {
    if (i == 0) return wave < nrb ? wave : -1;
    return second == SecondBlock::kNone ? -1 : kScoreWaves + wave - (second == SecondBlock::kSubtile1 ? 2 : 0);
}

template <typename T, int NCH, int RBW>
struct QueryRows {
    static constexpr int kPieces = 2 * NCH;                                    // 16-byte pieces of a row, a power of two
    static constexpr int kRows = kPieces > 16 ? 512 / kPieces : 32;            // rows per round: at most 8 KB per wave
    static constexpr int kRounds = 32 / kRows;
    static constexpr int kLoads = kRows * kPieces / 64;                        // per round
    static constexpr size_t kLdsBytes = static_cast<size_t>(kScoreWaves) * kRows * kPieces * sizeof(uint4);
    u32x4_t v[RBW][kRounds][kLoads];

    __device__ __forceinline__ void load(const T* __restrict__ q_text, const ScoreGeom& g, int kvh, int rb0, int nrb, int wave, SecondBlock second, int lane) {
        const u32x4_t* rows = reinterpret_cast<const u32x4_t*>(q_text) + static_cast<size_t>(kvh) * g.R * kPieces;
#pragma unroll
        for (int i = 0; i < RBW; ++i) {
            const int r0 = (rb0 + max(wave_block<RBW>(nrb, wave, second, i), 0)) * 32;
#pragma unroll
            for (int k = 0; k < kRounds; ++k)
#pragma unroll
                for (int u = 0; u < kLoads; ++u) {
                    const int id = u * 64 + lane;
                    const int r = min(r0 + k * kRows + id / kPieces, g.R - 1);     // rows past the last are cleared below
                    v[i][k][u] = rows[r * kPieces + id % kPieces];
                }
        }
    }
    // Only the wave itself uses its part of LDS, and a wave's LDS accesses complete in order.
    __device__ __forceinline__ void to_fragments(uint4 (&q)[RBW][NCH], uint4* lds, const ScoreGeom& g, int rb0, int nrb, int wave, SecondBlock second, int lane) {
        u32x4_t* own = reinterpret_cast<u32x4_t*>(lds) + wave * kRows * kPieces;
        const int row = lane & 31, half = lane >> 5;
#pragma unroll
        for (int i = 0; i < RBW; ++i) {
            const int rbl = wave_block<RBW>(nrb, wave, second, i);
            const bool ok = rbl >= 0 && (rb0 + rbl) * 32 + row < g.R;
#pragma unroll
            for (int k = 0; k < kRounds; ++k) {
#pragma unroll
                for (int u = 0; u < kLoads; ++u) {
                    const int id = u * 64 + lane, r = id / kPieces, p = id % kPieces;
                    own[r * kPieces + (p ^ (r & (kPieces - 1)))] = v[i][k][u];
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const int r = row % kRows;
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    const u32x4_t f = own[r * kPieces + ((half * NCH + c) ^ (r & (kPieces - 1)))];
                    if (k == 0 || row / kRows == k) q[i][c] = make_uint4(f.x, f.y, f.z, f.w);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
#pragma unroll
            for (int c = 0; c < NCH; ++c) if (!ok) q[i][c] = make_uint4(0, 0, 0, 0);
        }
    }
};

// q[i][c] belongs to row block i of the wave.
template <int NCH, int RBW>
__device__ __forceinline__ void load_qfrag(uint4 (&q)[RBW][NCH], const uint4* __restrict__ qfrag, const ScoreGeom& g, int kvh,
                                           int rb0, int nrb, int wave, SecondBlock second, int lane) {
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
        const int rbl = wave_block<RBW>(nrb, wave, second, i);
        const bool ok = rbl >= 0;
        const uint4* src = qfrag + (static_cast<size_t>(kvh) * g.rb_total + rb0 + (ok ? rbl : 0)) * NCH * 64 + lane;
#pragma unroll
        for (int c = 0; c < NCH; ++c) q[i][c] = ok ? src[c * 64] : make_uint4(0, 0, 0, 0);
    }
}

template <typename T, int NCH>
__device__ __forceinline__ f32x16_t mma_chain(const uint4 (&a)[NCH], const uint4 (&b)[NCH]) {
    f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NCH; ++c) acc = Mma<T>::mma(a[c], b[c], acc);
    return acc;
}

// The product of a subtile of split keys, operand c of the lane at keys[64 c], with a split row block; KEYS_FIRST: keys x queries.
// !FIT: some element may not (infinity times a part that is zero would be NaN): fp32 products.
template <int NCH, bool FIT, bool KEYS_FIRST>
__device__ __forceinline__ f32x16_t split_chain(const uint4* keys, const uint4 (&q)[NCH / 2 * 3]) {
    // The products of the leading parts have a sum of their own: a bf16 MFMA does not round to nearest what it adds to a sum.  Where they
    // went on from the sum of the others, rows of one element were 3.5e-8 off instead of 2.6e-8.  They run ahead of the others with 128
    // elements (one level of 24000 tokens, 28 heads on 4 x 64: 199 us, alternating 203) and alternate with them otherwise (4 x 9000
    // tokens, 16 heads x 100 queries of 64 elements: 203 us, alternating 188; with one sum 176).
    constexpr bool kAhead = NCH == 16;
    f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, small = acc;
    auto mma = [&](auto tag, f32x16_t& sum, const uint4& key, const uint4& row) {
        sum = KEYS_FIRST ? Mma<decltype(tag)>::mma(key, row, sum) : Mma<decltype(tag)>::mma(row, key, sum);
    };
    if constexpr (FIT && kAhead) {
#pragma unroll
        for (int c = 0; c < NCH / 2; ++c) mma(bf16_t(), acc, keys[3 * c * 64], q[3 * c]);
    }
#pragma unroll
    for (int c = 0; c < NCH / 2; ++c) {
        const uint4 k[3] = {keys[(3 * c) * 64], keys[(3 * c + 1) * 64], keys[(3 * c + 2) * 64]};
        const uint4* x = q + 3 * c;
        if constexpr (FIT) {
            mma(bf16_t(), small, k[2], x[0]);
            mma(bf16_t(), small, k[0], x[2]);
            mma(bf16_t(), small, k[1], x[1]);
            mma(bf16_t(), small, k[1], x[0]);
            mma(bf16_t(), small, k[0], x[1]);
            if constexpr (!kAhead) mma(bf16_t(), acc, k[0], x[0]);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                mma(float(), acc, joined_piece(k, i), joined_piece(x, i));
                __builtin_amdgcn_sched_barrier(0);                  // one piece at a time: no registers for what is hardly ever run
            }
        }
    }
    if constexpr (FIT) {
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] += small[e];
    }
    return acc;
}

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

__device__ __forceinline__ float max16(const f32x16_t& acc) {
    const float t0 = max3(acc[0], acc[1], acc[2]), t1 = max3(acc[3], acc[4], acc[5]), t2 = max3(acc[6], acc[7], acc[8]),
                t3 = max3(acc[9], acc[10], acc[11]), t4 = max3(acc[12], acc[13], acc[14]);
    return max3(max3(t0, t1, t2), max3(t3, t4, acc[15]), acc[15]);
}

// Softmax steps of one lane over its 16 accumulators (log2 domain).  m, what the terms are relative to, is a whole number not
// below the largest logit it was taken from, so that scaling a sum to another m is exact.
__device__ __forceinline__ float reference_above(float logit_max) { return fmaxf(kNegBig, ceilf(logit_max)); }

// l = mantissa in [0.5, 1): a sum far from 1 must not lose others, or be lost, when they meet at another m
__device__ __forceinline__ void normalise_softmax(float& m, float& l) {
    if (l > 0.f) { const int e = __builtin_amdgcn_frexp_expf(l); l = ldexpf(l, -e); m += static_cast<float>(e); }
}

// Every key is visible and m stays: the new sum.
__device__ __forceinline__ float softmax_sum(const f32x16_t& acc, float scale_log2, float m, float l) {
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) sum += fast_exp2(fmaf(acc[e], scale_log2, -m));
    return l + sum;
}

// Every key is visible and m follows the maximum.
__device__ __forceinline__ void softmax_step_full(const f32x16_t& acc, float scale_log2, float& m, float& l) {
    const float m_new = fmaxf(m, reference_above(max16(acc) * scale_log2));        // the scale is positive: max commutes with it
    l = softmax_sum(acc, scale_log2, m_new, l * fast_exp2(m - m_new));
    m = m_new;
}

// l becomes the sum that softmax_sum returned, unless it left the range of float in a lane: then the step is done once more with
// a larger m.
__device__ __forceinline__ void softmax_take(const f32x16_t& acc, float scale_log2, float& m, float& l, float sum) {
    if (__builtin_expect(__any(sum == INFINITY), 0)) {
        normalise_softmax(m, l);
        softmax_step_full(acc, scale_log2, m, l);
    } else {
        l = sum;
    }
}

// Keeps the MFMA chain that produces `acc` inside the scheduling region in which it was written: the value counts as
// used (and changed) here, so the chain cannot sink towards its first real use in a later region.
__device__ __forceinline__ void pin_accumulators(f32x16_t& acc) { asm volatile("" : "+v"(acc)); }

// Asks the scheduler to place `valu` vector instructions after each of the next `mfmas` MFMAs of the
// region, so that the softmax arithmetic of one block runs while the matrix pipe works on the next block.
template <int MFMAS, int VALU>
__device__ __forceinline__ void interleave_mfma_valu() {
#pragma unroll
    for (int z = 0; z < MFMAS; ++z) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
    }
}

// Online softmax step of one lane over its 16 accumulators with the causal / range mask applied:
// accumulator e is key j0 + 8 (e / 4) + 4 h + e % 4 and is visible iff that offset is <= lim.
__device__ __forceinline__ void softmax_step_masked(const f32x16_t& acc, float scale_log2, int h, int lim, float& m, float& l) {
    bool vis[16];
    float tmax = kNegBig;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        vis[e] = 8 * (e >> 2) + 4 * h + (e & 3) <= lim;
        if (vis[e]) tmax = fmaxf(tmax, acc[e] * scale_log2);
    }
    const float m_new = fmaxf(m, reference_above(tmax));
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) sum += vis[e] ? fast_exp2(fmaf(acc[e], scale_log2, -m_new)) : 0.f;
    l = l * fast_exp2(m - m_new) + sum;
    m = m_new;
}

// (m, l) stands for the sum l 2^m.
__device__ __forceinline__ void merge_softmax(float& m, float& l, float m2, float l2) {
    const float mm = fmaxf(m, m2);
    l = l * fast_exp2(m - mm) + l2 * fast_exp2(m2 - mm);
    m = mm;
}

// What pass 1 leaves of a workgroup's rows: their m, then their l (the sum of 2^logit over the workgroup's keys is l 2^m; one
// number, m + log2 l, would be half of it, but the sum of 40 rounded logarithms is measurably further from the row's).
__device__ __forceinline__ void store_partial(float* pstat, int rows, int r, float m, float l) {
    float* dst = pstat + (static_cast<size_t>(blockIdx.y) * gridDim.x + blockIdx.x) * rows * 2 + r;
    dst[0] = m;
    dst[rows] = l;
}
constexpr int kStageBuffers = 3;       // LDS stages: one in use, one ready (its first fragments are read early), one being filled

// ---------------------------------------------------------------------------------------------
// pass 1: blockIdx.x owns sub_per_wg consecutive 32-key subtiles of [key_begin, key_end),
// blockIdx.y = kvh * rs + split.  The product is taken as keys x queries, so a lane's 16 accumulators
// are 16 keys of ONE query row (row = lane % 32) and the online softmax state is one (max, sum) pair
// per lane and row block, in the log2 domain.
// pstat[((y * gridDim.x + x) * 2 + {0, 1}) * rbw * 32 + local_row]: see store_partial
//
// Key stages are fetched two ahead (global -> registers at the top of a stage, registers -> LDS at its
// end, one barrier per stage).  Where a workgroup has a row block for every wave, the stages in which every key is
// visible to every query run as one software pipeline over a wave's blocks (subtile, row block): the MFMA chain
// of block b + 1 is interleaved with the softmax arithmetic of block b, also across the barrier, and the
// fragments of the next stage's first subtile are read from LDS as soon as their registers are free.
// Stages that need the mask, and workgroups with fewer row blocks than waves, take the plain path.
//
// m is taken from a lane's keys of the first subtile and stays while whole subtiles are visible: terms relative to it keep
// their precision as long as none exceeds it by 2^127, and following the maximum is 14 of the 64 vector instructions of a
// block (eight videos of 36864 tokens: 160 -> 152 us).  A block whose sums left the range of float is added once more under a
// larger m, while its products are still there.  The question costs the same level 0.7 % (312.5 -> 314.5 us without its row
// gather); to let the whole workgroup start over instead made logits that jump by more than 2^127, or one key that is
// not finite, pass 1 twice as long (354 and 343 us with the running maximum, 490 and 454 so, 352 and 325 now).
// ---------------------------------------------------------------------------------------------
template <typename T, int NCH, int RBW, int SUBS>
__global__ __launch_bounds__(kScoreThreads) void row_stats_kernel(const T* __restrict__ q_text, const T* __restrict__ k_all,
                                                                  const ScoreGeom g, int sub_per_wg, float* __restrict__ pstat,
                                                                  uint4* __restrict__ qfrag, uint32_t* __restrict__ clear, int n_clear) {
    using Stage = KeyStage<T, NCH, SUBS>;
    extern __shared__ uint4 lds[];                      // the waves' query rows, then kStageBuffers stages
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = lane >> 5;
    const int kvh = blockIdx.y / g.rs, split = blockIdx.y % g.rs;
    const int rb0 = split * g.rbw;
    const int nrb = min(g.rbw, g.rb_total - rb0);
    __shared__ float2 shared_rows[2][64];
    constexpr int N = kOperands<T, NCH>;
    constexpr bool kSplit = std::is_same<T, split_t>::value;
    __shared__ int unfit[kSplit ? kStageBuffers : 1];          // the last stage of the buffer that held an element that does not fit
    q_text = of_video_elems(q_text, g.q_video);
    qfrag = of_video(qfrag, g.ws_video); pstat = of_video(pstat, g.ws_video); clear = of_video(clear, g.ws_video);
    const T* k_head = of_video_elems(k_all, g.k_video) + static_cast<size_t>(kvh) * g.S * g.dh;
    // as the first kernel of a call it clears the counters of the later ones
    if (blockIdx.x == 0 && blockIdx.y == 0 && static_cast<int>(threadIdx.x) < n_clear) clear[threadIdx.x] = 0u;

    const int64_t kb = g.key_begin + static_cast<int64_t>(blockIdx.x) * sub_per_wg * 32;
    const int64_t ke = min(g.key_end, kb + static_cast<int64_t>(sub_per_wg) * 32);
    const int n_stage = static_cast<int>((ke - kb + Stage::kKeys - 1) / Stage::kKeys);
    const int64_t text_start = g.S - g.Tq;
    const int64_t full_end = text_start < ke ? text_start : ke;
    const SecondBlock second = second_block<RBW>(nrb, wave, n_stage >= kMinSharedRows);
    // row blocks of this wave on the plain path, which shares none
    const int nrb_w = wave < nrb ? (second == SecondBlock::kBoth || second == SecondBlock::kSubtile0 ? 2 : 1) : 0;

    // the first two key stages and the queries are requested together: one memory round trip
    u32x4_t kv[Stage::kPerThread], kv1[Stage::kPerThread];
    Stage::load(kv, k_head, kb, g.S, g.dh);
    Stage::load(kv1, k_head, kb + (n_stage > 1 ? Stage::kKeys : 0), g.S, g.dh);
    uint4 q[RBW][N];
    bool fit_rows = true;
    if (kSplit && threadIdx.x < kStageBuffers) unfit[threadIdx.x] = -1;
    {
        QueryRows<T, NCH, RBW> rows;
        uint4 raw[RBW][NCH];
        rows.load(q_text, g, kvh, rb0, nrb, wave, second, lane);
        rows.to_fragments(raw, lds, g, rb0, nrb, wave, second, lane);
#pragma unroll
        for (int i = 0; i < RBW; ++i) fit_rows = make_operands<T, NCH>(raw[i], q[i]) && fit_rows;
        fit_rows = !__any(!fit_rows);
        __syncthreads();                                // the stages take over the waves' parts of LDS
    }
    auto store_stage = [&](const u32x4_t (&v)[Stage::kPerThread], int s) {
        uint4* kbuf = lds + (s % kStageBuffers) * Stage::kSlots;
        if constexpr (kSplit) { if (!Stage::store_split(v, kbuf)) unfit[s % kStageBuffers] = s; }
        else Stage::store(v, kbuf);
    };
    float m[RBW], l[RBW];
    store_stage(kv, 0);
    if (n_stage > 1) store_stage(kv1, 1);
    // Every load issued so far has to land before the loop: with query loads still pending at its head the
    // first use of a fragment inside would wait for ALL outstanding loads, the prefetch of later stages included.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    auto stage_buf = [&](int s) { return lds + (s % kStageBuffers) * Stage::kSlots; };
    auto prefetch = [&](int s) {          // global -> registers for stage s + 2
        if (s + 2 < n_stage) Stage::load(kv, k_head, kb + static_cast<int64_t>(s + 2) * Stage::kKeys, g.S, g.dh);
    };
    auto publish = [&](int s) {           // registers -> LDS; that buffer was last read before the previous barrier
        if (s + 2 < n_stage) store_stage(kv, s + 2);
        __syncthreads();
    };

    // stages s, s + 1, ... on the plain path; `online`: m follows the maximum
    auto plain_stages = [&](int s) {
        for (; s < n_stage; ++s) {
            const uint4* kbuf = stage_buf(s);
            const int64_t js = kb + static_cast<int64_t>(s) * Stage::kKeys;
            prefetch(s);
#pragma unroll
            for (int sub = 0; sub < SUBS; ++sub) {
                const int64_t j0 = js + sub * 32;
                if (j0 < ke && nrb_w > 0) {
                    const uint4* keys = kbuf + sub * N * 64 + lane;
                    uint4 kf[kSplit ? 1 : N];
                    bool fit = true;
                    if constexpr (kSplit) fit = fit_rows && unfit[s % kStageBuffers] != s;
                    else {
#pragma unroll
                        for (int c = 0; c < N; ++c) kf[c] = keys[c * 64];
                    }
                    const bool full = j0 + 32 <= full_end;      // every key of the subtile is visible to every query
#pragma unroll
                    for (int i = 0; i < RBW; ++i) {
                        if (i < nrb_w) {
                            f32x16_t acc;
                            if constexpr (!kSplit) acc = mma_chain<T, NCH>(kf, q[i]);
                            else if (fit) acc = split_chain<NCH, true, true>(keys, q[i]);
                            else acc = split_chain<NCH, false, true>(keys, q[i]);
                            if (full && j0 > kb) {
                                softmax_take(acc, g.scale_log2, m[i], l[i], softmax_sum(acc, g.scale_log2, m[i], l[i]));
                            } else if (full) {
                                softmax_step_full(acc, g.scale_log2, m[i], l[i]);
                            } else {
                                const int r = (rb0 + wave + kScoreWaves * i) * 32 + (lane & 31);
                                int64_t last = text_start + (r % g.Tq);            // causal: keys 0..last, and below ke
                                last = last < ke - 1 ? last : ke - 1;
                                const int64_t d = last - j0;
                                const int lim = d < 0 ? -1 : (d > 31 ? 31 : static_cast<int>(d));
                                softmax_step_masked(acc, g.scale_log2, h, lim, m[i], l[i]);
                            }
                        }
                    }
                }
            }
            publish(s);
        }
    };

#pragma unroll
    for (int i = 0; i < RBW; ++i) { m[i] = kNegBig; l[i] = 0.f; }
    int s = 0;
    if constexpr (RBW == 2 && SUBS == 2) {
        // Leading stages whose 64 keys are all visible to every query.  The choice is the same for every wave of the workgroup,
        // and whatever its row blocks are a wave meets the others at one barrier per stage.
        int n_fast = 0;
        if (nrb >= kScoreWaves) {
            const int64_t f = (full_end - kb) / Stage::kKeys;
            n_fast = f < kMinPipelined ? 0 : (f > n_stage ? n_stage : static_cast<int>(f));
        }
        if (n_fast > 0) {
            constexpr int kMfmas = NCH * Mma<T>::kMfmaPerChunk;
            constexpr int kValu = (49 + kMfmas - 1) / kMfmas;
            const int first = second == SecondBlock::kSubtile1 ? NCH * 64 : 0, later = NCH * 64 - first;
            uint4 kf0[NCH], kf1[NCH];
#pragma unroll
            for (int c = 0; c < NCH; ++c) kf0[c] = lds[c * 64 + lane + first];
            f32x16_t A, B = mma_chain<T, NCH>(kf0, q[1]);
            m[1] = reference_above(max16(B) * g.scale_log2);
            A = mma_chain<T, NCH>(kf0, q[0]);
            m[0] = reference_above(max16(A) * g.scale_log2);
            // the product of one block beside the softmax arithmetic of the block before
            auto phase = [&](f32x16_t& next, const uint4 (&kf)[NCH], const uint4 (&qf)[NCH], const f32x16_t& acc, int i) {
                next = mma_chain<T, NCH>(kf, qf);
                const float sum = softmax_sum(acc, g.scale_log2, m[i], l[i]);
                interleave_mfma_valu<kMfmas, kValu>();
                pin_accumulators(next);
                __builtin_amdgcn_sched_barrier(0);
                softmax_take(acc, g.scale_log2, m[i], l[i], sum);
            };
            // Which subtile of a stage comes first is a wave's own choice: one that shares a block takes its subtile of it
            // first, so that both waves of a pair do the same, block 0, block 1, block 0 of the other subtile.  The loads and
            // stores are free of branches, on clamped addresses (a stage is fetched twice, a free buffer is overwritten,
            // the product started for a stage that is not fast is dropped).
            for (; s < n_fast; ++s) {
                const uint4* kbuf = stage_buf(s);
                const int s2 = s + 2 < n_stage ? s + 2 : n_stage - 1;
                Stage::load(kv, k_head, kb + static_cast<int64_t>(s2) * Stage::kKeys, g.S, g.dh);
#pragma unroll
                for (int c = 0; c < NCH; ++c) kf1[c] = kbuf[c * 64 + lane + later];
                __builtin_amdgcn_sched_barrier(0);
                phase(B, kf0, q[1], A, 0);
                {   // first subtile of the next stage: published before the previous barrier
                    const uint4* knext = stage_buf(s + 1);
#pragma unroll
                    for (int c = 0; c < NCH; ++c) kf0[c] = knext[c * 64 + lane + first];
                }
                __builtin_amdgcn_sched_barrier(0);
                phase(A, kf1, q[0], B, 1);
                if (second == SecondBlock::kBoth) {
                    phase(B, kf1, q[1], A, 0);
                    Stage::template store<true>(kv, stage_buf(s + 2));
                    __syncthreads();
                    __builtin_amdgcn_sched_barrier(0);
                    phase(A, kf0, q[0], B, 1);
                } else {
                    Stage::template store<true>(kv, stage_buf(s + 2));
                    __syncthreads();
                    __builtin_amdgcn_sched_barrier(0);
                    phase(B, kf0, q[0], A, 0);
                    A = B;
                }
            }
        }
    }
    plain_stages(s);
    // the sums of a shared block's second subtiles, for the wave that owns it
    if constexpr (RBW == 2) if (second == SecondBlock::kSubtile1) shared_rows[wave & 1][lane] = make_float2(m[1], l[1]);
    lds_barrier();
    // Pass 2 reads the fragments that the first workgroup of each kv head and split leaves (here, behind the key stages,
    // whose loads would wait for the stores).
    if (blockIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < RBW; ++i) {
            const int rbl = wave_block<RBW>(nrb, wave, second, i);
            if (rbl >= 0 && rbl % kScoreWaves == wave) {
                uint4* dst = qfrag + (static_cast<size_t>(kvh) * g.rb_total + rb0 + rbl) * NCH * 64 + lane;
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    if constexpr (kSplit) dst[c * 64] = joined_piece(q[i], c);
                    else dst[c * 64] = q[i][c];
                }
            }
        }
    }
    // the two lane halves hold different keys of the same row
    const int rows_per_y = g.rbw * 32;
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
        const int rbl = wave + kScoreWaves * i;
        if (rbl < g.rbw) {
            normalise_softmax(m[i], l[i]);
            if (i == 1 && second == SecondBlock::kSubtile0) {
                float2 o = shared_rows[wave & 1][lane];
                normalise_softmax(o.x, o.y);
                merge_softmax(m[i], l[i], o.x, o.y);
            }
            merge_softmax(m[i], l[i], __shfl_xor(m[i], 32, 64), __shfl_xor(l[i], 32, 64));
            if (h == 0) store_partial(pstat, rows_per_y, rbl * 32 + lane, m[i], l[i]);
        }
    }
}

// (m, l) takes in N partials; those from `in` on are repetitions and do not count.
template <int N>
__device__ __forceinline__ void merge_partials(float& m, float& l, const float (&pm)[N], const float (&pl)[N], int in) {
    float mx = m;
#pragma unroll
    for (int u = 0; u < N; ++u) mx = fmaxf(mx, pm[u]);
    float sum = 0.f;
#pragma unroll
    for (int u = 0; u < N; ++u) sum += u < in ? pl[u] * fast_exp2(pm[u] - mx) : 0.f;
    l = l * fast_exp2(m - mx) + sum;
    m = mx;
}
__device__ __forceinline__ float row_norm(float m, float l, bool is_row) { return is_row && l > 0.f ? m + log2f(l) : kPosBig; }

// Normalisers of the rows of one workgroup row from the partials that the nx workgroups of pass 1 left, by
// every workgroup of pass 2 for itself: norm[r] = log2 of the row's whole sum, +big for padding rows.  Four neighbouring rows
// per 16-byte load, the threads of a row spread over the workgroups, and a thread's loads (2 kBatch in a round) on their way
// together, in the shadow of those for the keys and queries.  Called by the whole workgroup; ends with a barrier.
struct MergeShared { float4 m[kScoreThreads], l[kScoreThreads]; };
template <int kBatch>
__device__ __forceinline__ void merge_rows(const float* __restrict__ part, int nx, int rows, int first_row, int R, MergeShared& sh, float* norm) {
    const int lg = 32 - __clz(rows / 4 - 1);                        // rows / 4 <= 2^lg <= kScoreThreads / 4; rows is a multiple of 32
    const int quad = threadIdx.x & ((1 << lg) - 1), g = threadIdx.x >> lg, groups = kScoreThreads >> lg;
    const float4* src = reinterpret_cast<const float4*>(part) + min(quad, rows / 4 - 1);
    float m[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { m[i] = kNegBig; l[i] = 0.f; }
    for (int x0 = g; x0 < nx; x0 += groups * kBatch) {
        float4 vm[kBatch], vl[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const float4* p = src + static_cast<size_t>(min(x0 + u * groups, nx - 1)) * (rows / 2);      // past the end: the last one again
            vm[u] = p[0]; vl[u] = p[rows / 4];
        }
        const int in = (nx - x0 + groups - 1) / groups;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float pm[kBatch], pl[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                pm[u] = i == 0 ? vm[u].x : i == 1 ? vm[u].y : i == 2 ? vm[u].z : vm[u].w;
                pl[u] = i == 0 ? vl[u].x : i == 1 ? vl[u].y : i == 2 ? vl[u].z : vl[u].w;
            }
            merge_partials(m[i], l[i], pm, pl, in);
        }
    }
    sh.m[threadIdx.x] = make_float4(m[0], m[1], m[2], m[3]);
    sh.l[threadIdx.x] = make_float4(l[0], l[1], l[2], l[3]);
    lds_barrier();
    const int r = threadIdx.x;
    if (r < rows) {
        // the groups that had a partial, eight at a time: a row's threads are up to 64, and one after the other through all of them
        // was a chain of 1 us (300 tokens, 8 heads x 16 queries, kernels alone: 21.0 -> 18.8 us)
        const float* gm = reinterpret_cast<const float*>(sh.m) + r;
        const float* gl = reinterpret_cast<const float*>(sh.l) + r;
        const int used = min(groups, nx);
        float mm = kNegBig, ll = 0.f;
        for (int k = 0; k < used; k += 8) {
            float pm[8], pl[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int at = (min(k + u, used - 1) << lg) * 4;
                pm[u] = gm[at]; pl[u] = gl[at];
            }
            merge_partials(mm, ll, pm, pl, used - k);
        }
        norm[r] = row_norm(mm, ll, first_row + r < R);
    }
    lds_barrier();
}

// norm[y * rbw * 32 + local_row] = log2-domain normaliser max + log2(sum) of the row (+big for padding rows).
// Sixteen lanes share a row: each merges every 16th partial, then the lanes are merged pairwise.
__global__ __launch_bounds__(256) void merge_stats_kernel(const float* __restrict__ pstat, const ScoreGeom g, int nx,
                                                          float* __restrict__ norm) {
    const int rows_per_y = g.rbw * 32;
    const int total = g.Hkv * g.rs * rows_per_y;
    pstat = of_video(pstat, g.ws_video); norm = of_video(norm, g.ws_video);
    const int i = blockIdx.x * 16 + (threadIdx.x >> 4);
    const int p = threadIdx.x & 15;
    float mm = kNegBig, ll = 0.f;
    int y = 0, lr = 0;
    if (i < total) {
        y = i / rows_per_y; lr = i % rows_per_y;
        for (int x = p; x < nx; x += 16) {
            const float* src = pstat + (static_cast<size_t>(y) * nx + x) * rows_per_y * 2 + lr;
            merge_softmax(mm, ll, src[0], src[rows_per_y]);
        }
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
        merge_softmax(mm, ll, __shfl_xor(mm, off, 16), __shfl_xor(ll, off, 16));
    }
    if (i < total && p == 0) {
        const int r = (y % g.rs) * rows_per_y + lr;
        norm[i] = row_norm(mm, ll, r < g.R);
    }
}

// ---------------------------------------------------------------------------------------------
// pass 2: queries x keys, a lane's 16 accumulators are 16 rows of ONE key (key = lane % 32), and the
// normalisers of those rows stay in registers.  blockIdx.x owns sub_per_wg consecutive subtiles of the
// visual keys.  The eight per-wave partial column sums of a stage are added in wave order through LDS.
// colpart[y * n_vis + j] = sum over the rows of workgroup-row y of the probability of visual key j.
// ---------------------------------------------------------------------------------------------
// Grids of more workgroups than CUs run two (or three) to a CU where 128 (80) registers suffice, which the merge must not exceed:
// with eight partials a round in every kernel, 20 x 3000 tokens of 40 heads x 100 queries took 438 us for 389 with the merging kernel,
// in bf16 with 256 elements 934 for 810, and now, with four (two) a round, 381 and 793.
template <typename T, int NCH, int RBW> constexpr int kColWaves = (RBW == 2 && NCH > 4) || kOperands<T, NCH> > 16 ? 2 : 4;      // per SIMD
template <typename T, int NCH, int RBW, int SUBS>
__global__ __launch_bounds__(kScoreThreads, (kColWaves<T, NCH, RBW>)) void col_sums_kernel(const uint4* __restrict__ qfrag, const T* __restrict__ k_all,
                                                                 const ScoreGeom g, int sub_per_wg, const float* __restrict__ norm,
                                                                 const float* __restrict__ pstat, int nx1, float* __restrict__ colpart) {
    using Stage = KeyStage<T, NCH, SUBS>;
    extern __shared__ uint4 lds[];                      // two stages, then the column partials [2][waves][stage keys]
    float* cs = reinterpret_cast<float*>(lds + 2 * Stage::kSlots);
    __shared__ MergeShared red;
    constexpr int N = kOperands<T, NCH>;
    constexpr bool kSplit = std::is_same<T, split_t>::value;
    __shared__ int unfit[2];                       // see pass 1
    if (kSplit && threadIdx.x < 2) unfit[threadIdx.x] = -1;
    __shared__ __align__(16) float own_norm[kScoreThreads];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = lane >> 5;
    const int kvh = blockIdx.y / g.rs, split = blockIdx.y % g.rs;
    const int rb0 = split * g.rbw;
    const int nrb = min(g.rbw, g.rb_total - rb0);
    qfrag = of_video(qfrag, g.ws_video); norm = of_video(norm, g.ws_video); pstat = of_video(pstat, g.ws_video); colpart = of_video(colpart, g.ws_video);
    const T* k_head = of_video_elems(k_all, g.k_video) + static_cast<size_t>(kvh) * g.S * g.dh;

    const int vb = blockIdx.x * sub_per_wg * 32;                       // visual keys [vb, ve) of this workgroup
    const int ve = min(g.n_vis, vb + sub_per_wg * 32);
    const int n_stage = (ve - vb + Stage::kKeys - 1) / Stage::kKeys;
    // Subtiles of a stage that the wave takes of its second row block, bit by bit, and whether it has a first one: in vector
    // registers, because behind scalar branches the compiler spreads a subtile's LDS reads between its products (eight videos
    // of 36864 tokens: 166 us, now 151)
    const SecondBlock second = second_block<RBW>(nrb, wave, n_stage >= kMinSharedCols);
    int second_subtiles = second == SecondBlock::kBoth ? 3 : second == SecondBlock::kSubtile0 ? 1 : second == SecondBlock::kSubtile1 ? 2 : 0;
    int has_rows = wave < nrb ? 1 : 0;
    asm volatile("" : "+v"(second_subtiles), "+v"(has_rows));
    u32x4_t kv[Stage::kPerThread];
    Stage::load(kv, k_head, static_cast<int64_t>(g.vis_start) + vb, g.S, g.dh);

    uint4 raw[RBW][NCH];
    load_qfrag<NCH, RBW>(raw, qfrag, g, kvh, rb0, nrb, wave, second, lane);
    const float* rows_norm = norm + static_cast<size_t>(blockIdx.y) * g.rbw * 32;
    if (pstat) {                                                        // no kernel has merged the partials
        merge_rows<(RBW == 2 || NCH == 8 ? 4 : 2)>(pstat + static_cast<size_t>(blockIdx.y) * nx1 * g.rbw * 64, nx1, g.rbw * 32, rb0 * 32, g.R, red, own_norm);
        rows_norm = own_norm;
    }
    // accumulator e <-> query row 32 rbl + 8 (e / 4) + 4 h + e % 4
    float cr[RBW][16];
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
        const float* src = rows_norm + max(wave_block<RBW>(nrb, wave, second, i), 0) * 32 + 4 * h;
#pragma unroll
        for (int b4 = 0; b4 < 4; ++b4) {
            const float4 c4 = *reinterpret_cast<const float4*>(src + 8 * b4);
            cr[i][4 * b4 + 0] = c4.x; cr[i][4 * b4 + 1] = c4.y; cr[i][4 * b4 + 2] = c4.z; cr[i][4 * b4 + 3] = c4.w;
        }
    }
    uint4 q[RBW][N];
    bool fit_rows = true;
#pragma unroll
    for (int i = 0; i < RBW; ++i) fit_rows = make_operands<T, NCH>(raw[i], q[i]) && fit_rows;
    fit_rows = !__any(!fit_rows);
    auto store_stage = [&](int s) {
        uint4* kbuf = lds + (s & 1) * Stage::kSlots;
        if constexpr (kSplit) { if (!Stage::store_split(kv, kbuf)) unfit[s & 1] = s; }
        else Stage::store(kv, kbuf);
    };
    if (kSplit && !pstat) lds_barrier();        // unfit is ready
    store_stage(0);
    __builtin_amdgcn_s_waitcnt(0);      // queries and normalisers have landed: see row_stats_kernel
    __syncthreads();
    for (int s = 0; s < n_stage; ++s) {
        const uint4* kbuf = lds + (s & 1) * Stage::kSlots;
        float* csb = cs + (s & 1) * (kScoreWaves * Stage::kKeys);
        const int vs = vb + s * Stage::kKeys;
        if (s + 1 < n_stage) Stage::load(kv, k_head, static_cast<int64_t>(g.vis_start) + vs + Stage::kKeys, g.S, g.dh);
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub) {
            if (vs + sub * 32 < ve) {
                float colsum = 0.f;
                if (has_rows) {
                    const uint4* keys = kbuf + sub * N * 64 + lane;
                    uint4 kf[kSplit ? 1 : N];
                    bool fit = true;
                    if constexpr (kSplit) fit = fit_rows && unfit[s & 1] != s;
                    else {
#pragma unroll
                        for (int c = 0; c < N; ++c) kf[c] = keys[c * 64];
                    }
#pragma unroll
                    for (int i = 0; i < RBW; ++i) {
                        if (i == 0 || (second_subtiles >> sub & 1)) {
                            f32x16_t acc;
                            if constexpr (!kSplit) acc = mma_chain<T, NCH>(q[i], kf);
                            else if (fit) acc = split_chain<NCH, true, false>(keys, q[i]);
                            else acc = split_chain<NCH, false, false>(keys, q[i]);
#pragma unroll
                            for (int e = 0; e < 16; ++e) colsum += fast_exp2(fmaf(acc[e], g.scale_log2, -cr[i][e]));
                        }
                    }
                    colsum += __shfl_xor(colsum, 32, 64);
                }
                if (h == 0) csb[wave * Stage::kKeys + sub * 32 + lane] = colsum;
            }
        }
        if (s + 1 < n_stage) store_stage(s + 1);
        __syncthreads();
        if (threadIdx.x < Stage::kKeys) {
            const int j = vs + threadIdx.x;
            if (j < ve) {
                float a = 0.f;
#pragma unroll
                for (int w = 0; w < kScoreWaves; ++w) a += csb[w * Stage::kKeys + threadIdx.x];
                colpart[static_cast<size_t>(blockIdx.y) * g.n_vis + j] = a;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Narrow scores: at most 64 query rows per kv head (one query head per kv head with up to 64 text queries, or the last
// token's queries alone).  One or two 32-row blocks would leave six or seven of the eight waves above without work and
// every stage waiting for memory behind a barrier; what bounds this shape is the stream of keys.  Here every wave keeps all
// query rows (NB blocks of 16) in registers and walks its own 16-key subtiles of the workgroup's range, every eighth one,
// straight from memory into registers in MFMA fragment order and several subtiles ahead; no wave waits for another.
// 40 heads x 64 queries, 4571 keys of 128 bf16 (47 MB): row statistics 17.7 -> 15.6 us, column sums 15.9 -> 13.6 us (the
// shared stages took packed queries then, a launch of 3.2 us more; turning them itself costs their pass 1 about 1 us); the
// launch and the first loads are 5 us of each.  16 heads, 30064 keys of 64: 27.4 + 28.8 ->
// 15.1 + 14.8 us; the last token of 28 heads on 4, 18496 keys: 10.5 + 8.6 -> 8.0 + 6.1 us.  With more rows the loads cost
// more than they save: a wave's 1 KB load in fragment order takes 64 bytes of 16 rows (four times the address work of a
// contiguous one), and 28 blocks over four waves that each load their own fragments took 160 us where the shared stages
// above take 154.
// ---------------------------------------------------------------------------------------------
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
template <typename T> struct NarrowMma;
template <> struct NarrowMma<bf16_t> {             // one 16-byte chunk feeds one 16x16x32 MFMA
    static __device__ __forceinline__ f32x4_t mma(const u32x4_t& a, const u32x4_t& b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    }
};
template <> struct NarrowMma<float> {              // one chunk feeds four 16x16x4 MFMAs
    static __device__ __forceinline__ f32x4_t mma(const u32x4_t& a, const u32x4_t& b, f32x4_t c) {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
        return c;
    }
};
constexpr int kSubKeys = 16;
// Subtiles in registers: the one in work and those on their way.
constexpr int subtile_depth(int nch, int nb) { return nch * nb >= 32 ? 2 : (nch * nb >= 8 ? 4 : 6); }

// Rows j0 + lane % 16 (at most `last`, which stands in for the rows behind it) of [*, dh]: pieces 4 c + lane / 16.
template <typename T, int NCH>
__device__ __forceinline__ void load_fragments(u32x4_t (&f)[NCH], const T* __restrict__ base, int64_t j0, int64_t last, int dh) {
    constexpr int CE = Mma<T>::kChunkElems;
    const int lane = threadIdx.x & 63;
    int64_t j = j0 + (lane & 15);
    j = j < last ? j : last;
    // fewer than 2^31 rows: one 32 x 32 -> 64 bit multiply
    const T* row = base + static_cast<size_t>(static_cast<uint32_t>(j)) * static_cast<uint32_t>(dh) + (lane >> 4) * CE;
#pragma unroll
    for (int c = 0; c < NCH; ++c) f[c] = *reinterpret_cast<const u32x4_t*>(row + c * 4 * CE);
}

// The query rows of a kv head lie one after the other in q_text ([Hq, Tq, dh], group consecutive heads): no packing needed.
template <typename T, int NCH, int NB>
__device__ __forceinline__ void load_queries(u32x4_t (&q)[NB][NCH], const T* __restrict__ q_text, const ScoreGeom& g, int kvh) {
#pragma unroll
    for (int b = 0; b < NB; ++b) load_fragments<T, NCH>(q[b], q_text + static_cast<size_t>(kvh) * g.R * g.dh, b * 16, g.R - 1, g.dh);
}

// From eight fragments on the workgroup loads them once, into LDS, from where every wave takes them all.  A load in fragment order is 64
// bytes of 16 rows, and eight waves with 16 of them each ahead of their keys took 2.7 us of pass 1 and 2 of pass 2 for the addresses
// alone.  One level by graph replay, us: 4507 tokens, 40 heads x 64 queries of 128 elements 49.7 -> 46.5, 839 tokens 30.5 -> 25.9, 2924
// in fp32 79.8 -> 71.8; 7274, 16 heads x 64 of 64 30.1 -> 28.8.  With fewer fragments, or one row block, the barrier costs more than it
// saves: 439 tokens, 16 x 16 of 64 17.7 / 18.1, 12587 in fp32, 32 heads on 8 x 1 of 128 77.3 / 79.8.
template <int NCH, int NB> constexpr bool kShareQueries = NB >= 2 && NB * NCH >= 8;
template <typename T, int NCH, int NB>
struct SharedQueries {
    static constexpr int kFragments = NB * NCH, kRounds = (kFragments * 64 + kScoreThreads - 1) / kScoreThreads;
    u32x4_t v[kRounds];

    // piece id of the fragments: (block b, chunk c, lane) = (id / 64 / NCH, id / 64 % NCH, id % 64)
    __device__ __forceinline__ void load(const T* __restrict__ q_text, const ScoreGeom& g, int kvh) {
        const T* rows = q_text + static_cast<size_t>(kvh) * g.R * g.dh;
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int id = min(static_cast<int>(threadIdx.x) + u * kScoreThreads, kFragments * 64 - 1), f = id >> 6, lane = id & 63;
            const int row = min(f / NCH * 16 + (lane & 15), g.R - 1);
            v[u] = *reinterpret_cast<const u32x4_t*>(rows + static_cast<size_t>(row) * g.dh + (f % NCH * 4 + (lane >> 4)) * Mma<T>::kChunkElems);
        }
    }
    __device__ __forceinline__ void store(u32x4_t* lds) {
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int id = threadIdx.x + u * kScoreThreads;
            if ((u + 1) * kScoreThreads <= kFragments * 64 || id < kFragments * 64) lds[id] = v[u];
        }
    }
    // behind a barrier
    static __device__ __forceinline__ void take(u32x4_t (&q)[NB][NCH], const u32x4_t* lds) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int c = 0; c < NCH; ++c) q[b][c] = lds[(b * NCH + c) * 64 + lane];
    }
};

template <typename T, int NCH>
__device__ __forceinline__ f32x4_t narrow_chain(const u32x4_t (&a)[NCH], const u32x4_t (&b)[NCH]) {
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NCH; ++c) acc = NarrowMma<T>::mma(a[c], b[c], acc);
    return acc;
}

// Subtiles t = 0 .. n-1 of a wave: k[0 .. DEPTH-2] await the first ones, load(dst, t) requests subtile t, work(fragments, t).
template <int NCH, int DEPTH, typename LOAD, typename WORK>
__device__ __forceinline__ void walk_subtiles(u32x4_t (&k)[DEPTH][NCH], int n, LOAD&& load, WORK&& work) {
    for (int t0 = 0; t0 < n; t0 += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int t = t0 + d;
            if (t < n) {
                load(k[(d + DEPTH - 1) % DEPTH], t + DEPTH - 1);      // past the end: the last key again
                work(k[d], t);
            }
        }
    }
}

// pass 1 (see row_stats_kernel): keys x queries, a lane's 4 accumulators are 4 keys (4 (lane / 16) + e) of query row lane % 16.
template <typename T, int NCH, int NB>
__global__ __launch_bounds__(kScoreThreads) void narrow_row_stats_kernel(const T* __restrict__ q_text, const T* __restrict__ k_all,
                                                                         const ScoreGeom g, int sub_per_wg, float* __restrict__ pstat,
                                                                         uint32_t* __restrict__ clear, int n_clear) {
    constexpr int DEPTH = subtile_depth(NCH, NB);
    __shared__ float2 red[kScoreWaves][NB * 16];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = lane >> 4;
    const int kvh = blockIdx.y;
    q_text = of_video_elems(q_text, g.q_video); pstat = of_video(pstat, g.ws_video); clear = of_video(clear, g.ws_video);
    const T* k_head = of_video_elems(k_all, g.k_video) + static_cast<size_t>(kvh) * g.S * g.dh;
    // as the first kernel of a call it clears the counters of the later ones
    if (blockIdx.x == 0 && blockIdx.y == 0 && static_cast<int>(threadIdx.x) < n_clear) clear[threadIdx.x] = 0u;

    const int64_t kb = g.key_begin + static_cast<int64_t>(blockIdx.x) * sub_per_wg * 32;
    const int64_t ke = min(g.key_end, kb + static_cast<int64_t>(sub_per_wg) * 32);
    const int64_t text_start = g.S - g.Tq;
    const int64_t full_end = text_start < ke ? text_start : ke;      // keys below are visible to every query
    const int subs = static_cast<int>((ke - kb + kSubKeys - 1) / kSubKeys);
    const int n = subs > wave ? (subs - wave + kScoreWaves - 1) / kScoreWaves : 0;
    auto first_key = [&](int t) { return kb + static_cast<int64_t>(wave + t * kScoreWaves) * kSubKeys; };
    auto load = [&](u32x4_t (&dst)[NCH], int t) { load_fragments<T, NCH>(dst, k_head, first_key(t), ke - 1, g.dh); };
    // the first subtiles and the queries are requested together: one memory round trip
    u32x4_t k[DEPTH][NCH], q[NB][NCH];
    constexpr bool kShare = kShareQueries<NCH, NB>;
    __shared__ u32x4_t query_lds[kShare ? NB * NCH * 64 : 1];
    SharedQueries<T, NCH, NB> queries;
    if constexpr (kShare) queries.load(q_text, g, kvh);
    else load_queries<T, NCH, NB>(q, q_text, g, kvh);
#pragma unroll
    for (int d = 0; d < DEPTH - 1; ++d) load(k[d], d);
    if constexpr (kShare) {
        queries.store(query_lds);
        lds_barrier();
        queries.take(q, query_lds);
    }

    // m is the largest logit among the lane's keys of the first subtile and stays while whole subtiles are visible: terms
    // relative to it keep their precision as long as none exceeds it by 2^127, and the running maximum with its masks is
    // three quarters of the vector instructions.  A wave whose sums left the range of float starts over with the maximum.
    float m[NB], l[NB];
    for (bool online = false;; online = true) {
#pragma unroll
        for (int b = 0; b < NB; ++b) { m[b] = kNegBig; l[b] = 0.f; }
        walk_subtiles<NCH, DEPTH>(k, n, load, [&](const u32x4_t (&kf)[NCH], int t) {
            const int64_t j0 = first_key(t);
            f32x4_t x[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) x[b] = narrow_chain<T, NCH>(kf, q[b]);
            if (t > 0 && !online && j0 + kSubKeys <= full_end) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    float p[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) p[e] = fast_exp2(fmaf(x[b][e], g.scale_log2, -m[b]));
                    l[b] += (p[0] + p[1]) + (p[2] + p[3]);
                }
            } else {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    // causal: row r sees keys 0 .. text_start + r % Tq, and below ke
                    int64_t last = text_start + (b * 16 + (lane & 15)) % g.Tq;
                    last = (last < ke - 1 ? last : ke - 1) - j0;
                    const int lim = last < 0 ? -1 : (last < kSubKeys - 1 ? static_cast<int>(last) : kSubKeys - 1);
                    float mx = m[b];
#pragma unroll
                    for (int e = 0; e < 4; ++e) mx = 4 * h + e <= lim ? fmaxf(mx, x[b][e] * g.scale_log2) : mx;
                    float sum = 0.f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum += 4 * h + e <= lim ? fast_exp2(fmaf(x[b][e], g.scale_log2, -mx)) : 0.f;
                    l[b] = l[b] * fast_exp2(m[b] - mx) + sum;
                    m[b] = mx;
                }
            }
        });
        bool bad = false;
#pragma unroll
        for (int b = 0; b < NB; ++b) bad = bad || !(l[b] <= 3.0e38f);
        if (online || !__any(bad ? 1 : 0)) break;
#pragma unroll
        for (int d = 0; d < DEPTH - 1; ++d) load(k[d], d);
    }
    // the four lanes of a row hold different keys, and so do the waves
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        // l = mantissa in [0.5, 1): a sum far from 1 must not lose the others when they are scaled to its m
        if (l[b] > 0.f) { const int e = __builtin_amdgcn_frexp_expf(l[b]); l[b] = ldexpf(l[b], -e); m[b] += static_cast<float>(e); }
        merge_softmax(m[b], l[b], __shfl_xor(m[b], 16, 64), __shfl_xor(l[b], 16, 64));
        merge_softmax(m[b], l[b], __shfl_xor(m[b], 32, 64), __shfl_xor(l[b], 32, 64));
        if (lane < 16) red[wave][b * 16 + lane] = make_float2(m[b], l[b]);
    }
    __syncthreads();
    const int rows_per_y = g.rbw * 32;
    if (static_cast<int>(threadIdx.x) < min(NB * 16, rows_per_y)) {
        float2 a = red[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < kScoreWaves; ++w) { const float2 o = red[w][threadIdx.x]; merge_softmax(a.x, a.y, o.x, o.y); }
        store_partial(pstat, rows_per_y, threadIdx.x, a.x, a.y);
    }
}

// pass 2 (see col_sums_kernel): queries x keys, a lane's 4 accumulators are 4 rows (4 (lane / 16) + e) of key lane % 16.
template <typename T, int NCH, int NB>
__global__ __launch_bounds__(kScoreThreads) void narrow_col_sums_kernel(const T* __restrict__ q_text, const T* __restrict__ k_all,
                                                                        const ScoreGeom g, int sub_per_wg, const float* __restrict__ pstat,
                                                                        int nx1, float* __restrict__ colpart) {
    __shared__ MergeShared red;
    __shared__ __align__(16) float norm[64];
    constexpr int DEPTH = subtile_depth(NCH, NB);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = lane >> 4;
    const int kvh = blockIdx.y;
    q_text = of_video_elems(q_text, g.q_video); pstat = of_video(pstat, g.ws_video); colpart = of_video(colpart, g.ws_video);
    const T* k_head = of_video_elems(k_all, g.k_video) + (static_cast<size_t>(kvh) * g.S + g.vis_start) * g.dh;
    const int vb = blockIdx.x * sub_per_wg * 32;                       // visual keys [vb, ve) of this workgroup
    const int ve = min(g.n_vis, vb + sub_per_wg * 32);
    const int subs = (ve - vb + kSubKeys - 1) / kSubKeys;
    const int n = subs > wave ? (subs - wave + kScoreWaves - 1) / kScoreWaves : 0;
    auto load = [&](u32x4_t (&dst)[NCH], int t) { load_fragments<T, NCH>(dst, k_head, vb + (wave + t * kScoreWaves) * kSubKeys, ve - 1, g.dh); };
    u32x4_t k[DEPTH][NCH], q[NB][NCH];
    constexpr bool kShare = kShareQueries<NCH, NB>;
    __shared__ u32x4_t query_lds[kShare ? NB * NCH * 64 : 1];
    SharedQueries<T, NCH, NB> queries;
    if constexpr (kShare) queries.load(q_text, g, kvh);
    // a wave without keys only helps with the merge: loading its queries too made short levels in fp32 slower than the merging kernel
    // did (300 tokens, 2 heads x 64 queries of 128 elements, kernels alone: 31.5 us so, 29.9 with the merging kernel, 26.7 without)
    if (n > 0) {
        if constexpr (!kShare) load_queries<T, NCH, NB>(q, q_text, g, kvh);
#pragma unroll
        for (int d = 0; d < DEPTH - 1; ++d) load(k[d], d);
    }
    if constexpr (kShare) queries.store(query_lds);                    // the merge ends with a barrier
    const int rows = g.rbw * 32;                                       // 32 or 64; NB * 16 of them are used
    // two partials a round: with eight the kernel takes up to twice the registers, and where there is more than one workgroup per CU the
    // second one waits (fp32, 40 heads x 64 queries of 64 elements, 8 x 5000 tokens: 421 -> 407 us)
    merge_rows<2>(pstat + static_cast<size_t>(kvh) * nx1 * rows * 2, nx1, rows, 0, g.R, red, norm);
    if (kShare && n > 0) queries.take(q, query_lds);
    float cr[NB][4];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const float4 c4 = *reinterpret_cast<const float4*>(norm + b * 16 + 4 * h);       // +big for padding rows
        cr[b][0] = c4.x; cr[b][1] = c4.y; cr[b][2] = c4.z; cr[b][3] = c4.w;
    }
    walk_subtiles<NCH, DEPTH>(k, n, load, [&](const u32x4_t (&kf)[NCH], int t) {
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const f32x4_t x = narrow_chain<T, NCH>(q[b], kf);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += fast_exp2(fmaf(x[e], g.scale_log2, -cr[b][e]));
        }
        float total = (sum[0] + sum[1]) + (sum[2] + sum[3]);
        total = swap32_add(total, total);
        total = swap16_add(total, total);                              // every lane: all four lanes of its key
        const int j = vb + (wave + t * kScoreWaves) * kSubKeys + lane;
        if (lane < kSubKeys && j < ve) colpart[static_cast<size_t>(kvh) * g.n_vis + j] = total;
    });
}

// ---------------------------------------------------------------------------------------------
// scores, selection, scan, gather
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prepare_kernel(const float* __restrict__ colpart, int n_parts, int n_vis, float rows_total,
                                                      const int32_t* __restrict__ token_event, const float* __restrict__ event_weight,
                                                      int n_events, float* __restrict__ scores, int64_t ws_video) {
    colpart = of_video(colpart, ws_video); token_event = of_video_elems(token_event, n_vis);
    event_weight = of_video_elems(event_weight, n_events); scores = of_video_elems(scores, n_vis);
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n_vis) return;
    float a = 0.f;
    for (int p = 0; p < n_parts; ++p) a += colpart[static_cast<size_t>(p) * n_vis + j];
    a = a / rows_total;
    if (event_weight) {
        int e = token_event[j];
        e = e < 0 ? 0 : (e >= n_events ? n_events - 1 : e);
        a *= event_weight[e];
    }
    scores[j] = a;
}

struct Quotas { int32_t q[METOK_MAX_SEGMENTS]; };

constexpr int kSelCand = 4096;         // candidates kept in an LDS list once the first digit is fixed

// One workgroup per retention class.  Radix select of the quota-th largest key of the class: digits of up
// to 11 bits, starting at the highest bit in which the keys of the class differ.  Outputs: the threshold
// key tau and the number of tokens equal to tau that are still kept (sel_info[2 seg], [2 seg + 1];
// 0x7fffffff = every one), and per 1024-token tile the number of class members above tau (gt_count) and
// equal to it (eq_count).  The keep rule itself -- above tau, or equal and among the first `remaining`
// equal ones by index -- is applied by write_index_kernel.
// Thread t owns tokens t, t + 1024, ... (token i of a thread lies in tile i); with CACHED their keys stay
// in registers.  Attention scores share their top key bits, so a thread aggregates runs of equal digits
// before touching the LDS histogram, and once the first digit is fixed the remaining candidates (if at
// most kSelCand) move to an LDS list for the other digits.
template <bool CACHED>
__global__ __launch_bounds__(kSelThreads) void select_kernel(const float* __restrict__ scores, const int32_t* __restrict__ token_seg,
                                                             int n_vis, int n_tiles, const Quotas quotas,
                                                             int32_t* __restrict__ gt_count, int32_t* __restrict__ eq_count,
                                                             uint32_t* __restrict__ sel_info) {
    __shared__ int hist[2 * kSelThreads];      // 2048 bins: one 11-bit digit
    __shared__ int scan_scratch[17];
    __shared__ int s_digit, s_remaining, s_count, s_ncand;
    __shared__ uint32_t s_or, s_and;
    __shared__ uint32_t cand[kSelCand];
    __shared__ int cnt[2][64];
    const int seg = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int quota = quotas.q[seg];
    int32_t* my_gt = gt_count + static_cast<size_t>(seg) * n_tiles;
    int32_t* my_eq = eq_count + static_cast<size_t>(seg) * n_tiles;

    uint32_t key[CACHED ? kSelCache : 1];
    uint64_t member = 0;
    int mine = 0;
    if (CACHED) {
        // unconditional, clamped loads first so that all of them are in flight together
        int sv[kSelCache];
#pragma unroll
        for (int i = 0; i < kSelCache; ++i) {
            const int j = min(tid + i * kSelThreads, n_vis - 1);
            sv[i] = token_seg[j];
            key[i] = __float_as_uint(scores[j]);
        }
#pragma unroll
        for (int i = 0; i < kSelCache; ++i) {
            key[i] = ordered_key(__uint_as_float(key[i]));
            if (tid + i * kSelThreads < n_vis && sv[i] == seg) member |= 1ull << i;
        }
        mine = __popcll(member);
    } else {
        for (int i = 0; i < n_tiles; ++i) {
            const int j = tid + i * kSelThreads;
            mine += (j < n_vis && token_seg[j] == seg) ? 1 : 0;
        }
    }
    // f(key) for every token of the class owned by this thread
    auto for_each_key = [&](auto&& f) {
        if (CACHED) {
#pragma unroll
            for (int i = 0; i < kSelCache; ++i)
                if (member & (1ull << i)) f(key[i]);
        } else {
            for (int i = 0; i < n_tiles; ++i) {
                const int j = tid + i * kSelThreads;
                if (j < n_vis && token_seg[j] == seg) f(ordered_key(scores[j]));
            }
        }
    };
    if (tid == 0) { s_digit = 0; s_remaining = 0; s_count = 0; s_ncand = 0; s_or = 0u; s_and = 0xffffffffu; }
    int pop = 0;
    block_exclusive_scan(mine, scan_scratch, &pop);
    // bits on which the keys of the class differ: the radix digits start at the highest of them, so that the
    // first digit already separates scores that share sign, exponent and leading mantissa bits
    {
        uint32_t o = 0u, a = 0xffffffffu;
        for_each_key([&](uint32_t k) { o |= k; a &= k; });
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) { o |= __shfl_xor(o, off, 64); a &= __shfl_xor(a, off, 64); }
        if (lane == 0) { atomicOr(&s_or, o); atomicAnd(&s_and, a); }
        __syncthreads();
    }

    // keep rule: key > tau, or key == tau and fewer than `remaining` equal keys of the class precede the token
    uint32_t tau = 0;
    int remaining = 0x7fffffff;
    if (quota <= 0) {
        tau = 0xffffffffu; remaining = 0;                 // nothing is kept
    } else if (quota < pop) {
        const uint32_t differ = s_or ^ s_and;
        const int width = differ ? 32 - __clz(differ) : 0;             // the low `width` bits vary, the rest is common
        uint32_t prefix = width >= 32 ? 0u : (s_and & (0xffffffffu << width));
        int count_equal = pop;                                          // width 0: all keys are equal
        remaining = quota;
        bool use_list = false;
        // digits of up to 11 bits from the highest differing bit down (at most three rounds)
        for (int top = width; top > 0; top -= 11) {
            const int bits = top < 11 ? top : 11;
            const int shift = top - bits;
            const int bins = 1 << bits;
            const uint32_t dmask = static_cast<uint32_t>(bins - 1);
            const uint32_t hi_mask = top >= 32 ? 0u : (0xffffffffu << top);
            hist[tid] = 0; hist[tid + kSelThreads] = 0;
            __syncthreads();
            if (use_list) {
                for (int c = tid; c < s_ncand; c += kSelThreads) {
                    const uint32_t k = cand[c];
                    if ((k & hi_mask) == prefix) atomicAdd(&hist[(k >> shift) & dmask], 1);
                }
            } else {
                int run_digit = -1, run_count = 0;
                for_each_key([&](uint32_t k) {
                    if ((k & hi_mask) == prefix) {
                        const int d = static_cast<int>((k >> shift) & dmask);
                        if (d == run_digit) ++run_count;
                        else {
                            if (run_count) atomicAdd(&hist[run_digit], run_count);
                            run_digit = d; run_count = 1;
                        }
                    }
                });
                if (run_count) atomicAdd(&hist[run_digit], run_count);
            }
            __syncthreads();
            // thread t looks at digits bins-1-2t and bins-2-2t; exclusive scan = keys with a larger digit
            const int d0 = bins - 1 - 2 * tid, d1 = d0 - 1;
            const int v0 = d0 >= 0 ? hist[d0] : 0, v1 = d1 >= 0 ? hist[d1] : 0;
            int total = 0;
            const int excl = block_exclusive_scan(v0 + v1, scan_scratch, &total);
            if (excl < remaining && excl + v0 >= remaining) {
                s_digit = d0; s_remaining = remaining - excl; s_count = v0;
            } else if (excl + v0 < remaining && excl + v0 + v1 >= remaining) {
                s_digit = d1; s_remaining = remaining - excl - v0; s_count = v1;
            }
            __syncthreads();
            prefix |= static_cast<uint32_t>(s_digit) << shift;
            remaining = s_remaining;
            count_equal = s_count;
            if (!use_list && shift > 0 && count_equal <= kSelCand) {
                // the keys that still match move to the LDS list for the remaining digits
                const uint32_t fixed = 0xffffffffu << shift;
                for_each_key([&](uint32_t k) {
                    if ((k & fixed) == prefix) cand[atomicAdd(&s_ncand, 1)] = k;
                });
                use_list = true;
            }
            __syncthreads();
        }
        tau = prefix;
        if (remaining >= count_equal) remaining = 0x7fffffff;      // every token equal to the threshold is kept
    }

    if (tid == 0) {
        sel_info[2 * seg] = tau;
        sel_info[2 * seg + 1] = static_cast<uint32_t>(remaining);
    }
    // per-tile counts, tiles in groups of 64: lane i of a wave keeps the wave's counts of tile g0 + i
    for (int g0 = 0; g0 < n_tiles; g0 += 64) {
        if (tid < 128) cnt[tid >> 6][tid & 63] = 0;
        __syncthreads();
        const int g1 = min(n_tiles, g0 + 64);
        int my_gt_count = 0, my_eq_count = 0;
        auto tile_body = [&](int i, bool is_member, uint32_t k) {
            const unsigned long long gt = __ballot(is_member && k > tau), eq = __ballot(is_member && k == tau);
            if (lane == i - g0) { my_gt_count = __popcll(gt); my_eq_count = __popcll(eq); }
        };
        if (CACHED) {
#pragma unroll
            for (int i = 0; i < kSelCache; ++i)
                if (i >= g0 && i < g1) tile_body(i, (member >> i) & 1ull, key[i]);
        } else {
            for (int i = g0; i < g1; ++i) {
                const int j = tid + i * kSelThreads;
                const bool is_member = j < n_vis && token_seg[j] == seg;
                tile_body(i, is_member, is_member ? ordered_key(scores[j]) : 0u);
            }
        }
        if (my_gt_count) atomicAdd(&cnt[0][lane], my_gt_count);
        if (my_eq_count) atomicAdd(&cnt[1][lane], my_eq_count);
        __syncthreads();
        if (tid < g1 - g0) { my_gt[g0 + tid] = cnt[0][tid]; my_eq[g0 + tid] = cnt[1][tid]; }
        __syncthreads();
    }
}

// One workgroup per 1024-token tile: applies the keep rule (key above the class threshold, or equal to it and
// among the first `remaining` equal keys of the class by index), finds the position of the tile's first kept
// token from the per-class tile counts, and writes the kept index list and carried metadata in ascending order.
constexpr int kIdxThreads = 256;

__global__ __launch_bounds__(kIdxThreads) void write_index_kernel(
    const float* __restrict__ scores, const uint32_t* __restrict__ sel_info, const int32_t* __restrict__ gt_count,
    const int32_t* __restrict__ eq_count, const int32_t* __restrict__ token_seg,
    int n_vis, int n_seg, int n_tiles, int total_keep, const int32_t* __restrict__ token_event,
    const int32_t* __restrict__ orig_idx_in, int32_t* __restrict__ kept_idx, int32_t* __restrict__ token_seg_out,
    int32_t* __restrict__ token_event_out, int32_t* __restrict__ orig_idx_out,
    int64_t ws_video, int64_t keep_stride, int64_t orig_idx_in_stride, int64_t orig_idx_stride, const BatchKeep keeps) {
    __shared__ int scan_scratch[17];
    __shared__ uint32_t s_tau[METOK_MAX_SEGMENTS];
    __shared__ int s_rem[METOK_MAX_SEGMENTS], s_eq_before[METOK_MAX_SEGMENTS];
    __shared__ int tie_seg[kSelThreads];
    const int tile = blockIdx.x, tid = threadIdx.x;
    total_keep = keeps.n[blockIdx.z];
    scores = of_video_elems(scores, n_vis); token_seg = of_video_elems(token_seg, n_vis);
    token_event = of_video_elems(token_event, n_vis); orig_idx_in = of_video_elems(orig_idx_in, orig_idx_in_stride);
    sel_info = of_video(sel_info, ws_video); gt_count = of_video(gt_count, ws_video); eq_count = of_video(eq_count, ws_video);
    kept_idx = of_video_elems(kept_idx, keep_stride); token_seg_out = of_video_elems(token_seg_out, keep_stride);
    token_event_out = of_video_elems(token_event_out, keep_stride); orig_idx_out = of_video_elems(orig_idx_out, orig_idx_stride);
    // kept tokens in earlier tiles: thread s walks the tiles of class s
    int before = 0;
    for (int sg = tid; sg < n_seg; sg += kIdxThreads) {
        const uint32_t tau = sel_info[2 * sg];
        const int rem = static_cast<int>(sel_info[2 * sg + 1]);
        int eqcum = 0;
        for (int t = 0; t < tile; ++t) {
            const int eq = eq_count[static_cast<size_t>(sg) * n_tiles + t];
            const int room = rem > eqcum ? rem - eqcum : 0;
            before += gt_count[static_cast<size_t>(sg) * n_tiles + t] + (eq < room ? eq : room);
            eqcum += eq;
        }
        s_tau[sg] = tau; s_rem[sg] = rem; s_eq_before[sg] = eqcum;
    }
    int tile_off = 0;
    block_exclusive_scan(before, scan_scratch, &tile_off);      // its barriers also publish the tables above
    // four consecutive tokens per thread
    const int j0 = tile * kSelThreads + tid * 4;
    bool keep[4], tie[4];
    int sv[4];
    bool any_tie = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int j = min(j0 + u, n_vis - 1);
        sv[u] = token_seg[j];
        const uint32_t key = ordered_key(scores[j]);
        const bool ok = (j0 + u < n_vis) && sv[u] >= 0 && sv[u] < n_seg;
        const int sg = ok ? sv[u] : 0;
        keep[u] = ok && key > s_tau[sg];
        tie[u] = ok && key == s_tau[sg];
        if (tie[u] && s_rem[sg] == 0x7fffffff) { keep[u] = true; tie[u] = false; }      // every equal key is kept
        if (tie[u] && s_rem[sg] <= s_eq_before[sg]) tie[u] = false;                      // the equal keys kept lie in earlier tiles
        any_tie = any_tie || tie[u];
        tie_seg[tid * 4 + u] = tie[u] ? sg : -1;
    }
    if (__syncthreads_or(any_tie ? 1 : 0)) {
        // rank of an undecided equal key among the equal keys of its class (ties are rare; the walk is short)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (tie[u]) {
                int rank = s_eq_before[sv[u]];
                for (int q = 0; q < tid * 4 + u; ++q) rank += tie_seg[q] == sv[u] ? 1 : 0;
                keep[u] = rank < s_rem[sv[u]];
            }
        }
    }
    int mine = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) mine += keep[u] ? 1 : 0;
    int total = 0;
    int pos = tile_off + block_exclusive_scan(mine, scan_scratch, &total);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (keep[u]) {
            const int j = j0 + u;
            if (pos < total_keep) {
                kept_idx[pos] = j;
                if (token_seg_out) token_seg_out[pos] = sv[u];
                if (token_event_out) token_event_out[pos] = token_event[j];
                if (orig_idx_out) orig_idx_out[pos] = orig_idx_in ? orig_idx_in[j] : j;
            }
            ++pos;
        }
    }
    // fewer survivors than announced (a quota above its class population): the last tile pads the tail so
    // that the gather stays in bounds
    if (tile == n_tiles - 1) {
        for (int p = tile_off + total + tid; p < total_keep; p += kIdxThreads) {
            kept_idx[p] = 0;
            if (token_seg_out) token_seg_out[p] = 0;
            if (token_event_out) token_event_out[p] = 0;
            if (orig_idx_out) orig_idx_out[p] = 0;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Fast selection path: at most kFastSeg retention classes and at most kFastTiles tiles of 1024 tokens (fewer for one video
// of many classes, see one_launch_selection), one launch.
//   every workgroup     scores of its tokens from the partial column sums (skipped when scores are given)
//   the workgroup that arrives last at an atomic counter (it is the one that knows every other workgroup's scores are
//   complete; nobody waits for anybody) selects for the video: all keys in registers, per class a histogram of the
//   leading bits of (key - smallest key), the bucket of the quota-th largest key, the few keys of that bucket ranked
//   against each other, then the ascending index list of the kept tokens.
// The keep rule (key above the threshold, or equal and among the first equal keys by index) does not depend on how the
// threshold was found, so the results are the integers of the general path.
// What bounds it is latency, not work: a chain of about ten barriers and two memory round trips.  The digits start at
// the smallest key because attention scores share their leading bits: a histogram of the top 11 bits of the key itself
// left a third of the tokens in one bucket (and its atomics on one address), the shifted one leaves 20 to 200.
// Measured in kernel traces against the launches it replaces (score + histogram, candidates, index list; with 5 to 16
// classes the general path's three): 2243 tokens 30.0 -> 10.1 us, 4507 tokens with 40 partial sums each 33.4 -> 12.0 us,
// 18432 tokens in 13 classes 30.1 -> 19.2 us, eight videos of 36864 tokens 43.5 -> 31.1 us with about 20 candidates and
// 39 -> 34.5 us with about 200 (more of them in one step to rank).  Scans and extremes by DPP instead of shuffles through LDS,
// LDS made ready before the scores arrive and the events' weights requested ahead of the partial sums take another 1 to 1.3 us
// off a call (2243 tokens 33.6 -> 32.3, 5000 in fp32 37.0 -> 35.5).  One workgroup walking 36 tiles is what is left there
// (0.6 us a tile: its loads, LDS atomics and ballots).
// ---------------------------------------------------------------------------------------------
constexpr int kFastSeg = 16;
constexpr int kFastTiles = kSelCache;
constexpr int kSplitParts = 8;              // from so many partial sums per token on four threads share a token in the scoring part
constexpr int kHistWords = 8192;            // histogram bins of all classes together: 2048 per class up to 4 classes, else 512
constexpr int kListCap = 512;               // keys of the threshold buckets that are ranked against each other
constexpr int kRankStep = 8;                // list entries read from LDS together

// Which selection a call takes.  One workgroup per video walks all tiles where the general path has one per class, so with
// more than four classes the line depends on the tiles: a level of one video with 28 / 4 heads x 64 queries in 13 classes
// takes 50.5 us here and 58.8 on the general path at 12288 tokens, 63.8 and 67.3 at 20480, 71.6 and 71.9 at 24576, 83.2 and
// 79.8 at 32768, 94.0 and 88.6 at 40960; scores within 1 % beside one large one, given, need more digits here: 31.0 and 30.0
// at 20480, 36.4 and 31.1 at 24576.  The general path launches its selection per video: two or more videos are faster here
// at every size (eight of 36864 tokens in 16 classes, scores given: 37 and 190 us).
constexpr int kFastTilesManyClasses = 22;
static bool one_launch_selection(int batch, int n_seg, int n_tiles) {
    return n_seg <= kFastSeg && n_tiles <= (n_seg <= 4 || batch > 1 ? kFastTiles : kFastTilesManyClasses);
}

struct FastArgs {
    FastSel* fs;
    const float* colpart;                   // NULL: scores are given (one workgroup per video then)
    int n_parts;
    float rows_total;
    const int32_t* token_event;
    const float* event_weight;
    int n_events;
    float* scores;
    const int32_t* token_seg;
    int n_vis, n_seg;
    int32_t* kept_idx;
    int64_t keep_stride;
    int64_t ws_video;                       // bytes between the workspaces of consecutive videos
    BatchKeep keeps;
    uint16_t quota[METOK_MAX_BATCH][kFastSeg];      // at most n_vis <= 40960
};

// Values handed from one workgroup to another inside a kernel travel through device-scope accesses (they pass the
// caches that are not coherent between the chip's dies), so that no whole-cache write-back or invalidate is needed:
// the writers store, wait until their stores have completed, meet at a barrier and count their arrival; the workgroup
// that arrives last loads.
template <typename V> __device__ __forceinline__ void store_shared_between_workgroups(V* p, V v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V> __device__ __forceinline__ V load_shared_between_workgroups(const V* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Called by every thread of the workgroup after its last store: true in the workgroup that arrives last of gridDim.x.
__device__ __forceinline__ bool arrive_and_check_last(uint32_t* counter, int* s_flag) {
    __builtin_amdgcn_s_waitcnt(0);          // this thread's stores and atomics have completed
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t ticket = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_flag = ticket == gridDim.x - 1 ? 1 : 0;
    }
    __syncthreads();
    return *s_flag != 0;
}

// Histogram bins of a class lie one word further apart every 32 bins, so that the lanes of wave_find_bucket, which walk
// 32 (or 8) neighbouring bins each, read different LDS banks.
__device__ __forceinline__ int bin_slot(int bin) { return bin + (bin >> 5); }
constexpr int kHistSlots = kHistWords + kHistWords / 32;

// One wave walks the 64 * PER bins of a class from the largest digit down and returns the digit at which the running count
// reaches `need`, how many keys of that digit are still needed, how many keys the digit holds, and the count of all bins.
// A lane adds up PER neighbouring bins; then the lanes look at the bins of the one lane in which the count is reached.
template <int PER>
__device__ __forceinline__ void wave_find_bucket(const int* hist, int need, int* digit, int* rem, int* cnt, int* population) {
    static_assert(32 % PER == 0, "the bins of a lane are neighbours in LDS");
    const int lane = threadIdx.x & 63;
    const int* mine_hist = hist + bin_slot((63 - lane) * PER);      // lane 0 owns the largest digits
    int sum = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) sum += mine_hist[u];
    const int incl = wave_inclusive_scan(sum);
    *population = __builtin_amdgcn_readlane(incl, 63);
    const unsigned long long m = __ballot(incl - sum < need && incl >= need);
    const int src = m ? __ffsll(static_cast<long long>(m)) - 1 : 0;
    const int left = need - __builtin_amdgcn_readlane(incl - sum, src);      // keys needed from that lane's bins
    const int hi = (64 - src) * PER - 1;                            // the largest digit among them
    const int v = lane < PER ? hist[bin_slot(hi - lane)] : 0;
    const int incl2 = wave_inclusive_scan(v);
    const unsigned long long m2 = __ballot(incl2 - v < left && incl2 >= left);
    const int at = m2 ? __ffsll(static_cast<long long>(m2)) - 1 : 0;
    *digit = hi - at;
    *rem = left - __builtin_amdgcn_readlane(incl2 - v, at);
    *cnt = __builtin_amdgcn_readlane(v, at);
}

// What the selecting workgroup keeps in LDS.
struct SelectShared {
    int hist[kHistSlots];
    int scan[17];
    uint64_t kept[kFastTiles * 16];         // bit mask of the kept tokens of every 64-token group
    uint64_t equal[kFastTiles * 16];        // of the tokens equal to their class's threshold (only with more ties than the list holds)
    int before[kFastTiles * 16];            // kept tokens of the groups before this one
    uint64_t list[kListCap + kRankStep];    // key and, below it, the complement of the token: larger is kept first
    uint32_t lo, hi;                        // smallest and largest key
    int need[kFastSeg], cnt[kFastSeg], base[kFastSeg + 1], fill[kFastSeg];
    // a token is kept if key >> shift >= sure, and is a candidate if key >> shift == cand; 0xffffffff is met by no token (keys
    // count from the smallest one here, and no two differ by that much); the last entry is for tokens without a class
    uint2 rule[kFastSeg + 1];
};

// Adds one to hist[slot] for every lane with slot >= 0.  A wave whose lanes all meet in one bin (a class of equal scores)
// adds once instead of queueing at one address.
__device__ __forceinline__ void hist_add(int* hist, int slot) {
    const int first = __builtin_amdgcn_readfirstlane(slot);
    const bool one_bin = __ballot(slot == first) == ~0ull;
    if (slot >= 0 && (!one_bin || (threadIdx.x & 63) == 0)) atomicAdd(&hist[slot], one_bin ? 64 : 1);
}

// The selection of one video by one workgroup of 1024 threads: thread t owns tokens t, t + 1024, ... (at most K of them).
template <int K>
__device__ __forceinline__ void select_and_index(const FastArgs& a, const float* __restrict__ scores, const int32_t* __restrict__ token_seg,
                                                 FastSel* fs, int32_t* __restrict__ kept_idx, SelectShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_vis = a.n_vis, n_seg = a.n_seg;
    int n_tiles = (n_vis + kSelThreads - 1) / kSelThreads;
    const int bits = n_seg <= 4 ? 11 : 9, class_slots = bin_slot(1 << bits);

    // LDS is made ready while nothing else can be done: the scores of the other workgroups are a memory round trip away
    if (tid == 0) { sh.lo = 0xffffffffu; sh.hi = 0u; }
    if (tid <= kFastSeg) sh.rule[tid] = make_uint2(0xffffffffu, 0xffffffffu);
    if (tid < kFastSeg) { sh.fill[tid] = 0; sh.need[tid] = a.quota[blockIdx.z][tid]; sh.cnt[tid] = 0; }
    for (int i = tid; i < n_seg * class_slots; i += kSelThreads) sh.hist[i] = 0;
    // loads in rounds of up to twenty tokens, without a branch between them
    uint32_t key[K], cls[(K + 3) / 4];      // class kFastSeg: a token without a valid class, never kept
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int i = 0; i < (K + 3) / 4; ++i) cls[i] = 0u;
    constexpr int kRound = K < 20 ? K : 20;
#pragma unroll
    for (int i0 = 0; i0 < K; i0 += kRound) {
        if (i0 < n_tiles) {
            int sv[kRound];
#pragma unroll
            for (int u = 0; u < kRound; ++u) {
                const uint32_t at = static_cast<uint32_t>(min(tid + (i0 + u) * kSelThreads, n_vis - 1)) * 4u;
                key[i0 + u] = load_shared_between_workgroups(reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(scores) + at));
                sv[u] = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(token_seg) + at);
            }
#pragma unroll
            for (int u = 0; u < kRound; ++u) {
                const int i = i0 + u;
                key[i] = ordered_key(__uint_as_float(key[i]));
                const bool ok = tid + i * kSelThreads < n_vis && sv[u] >= 0 && sv[u] < n_seg;
                cls[i >> 2] |= static_cast<uint32_t>(ok ? sv[u] : kFastSeg) << (8 * (i & 3));
                lo = ok && key[i] < lo ? key[i] : lo;
                hi = ok && key[i] > hi ? key[i] : hi;
            }
        } else {
#pragma unroll
            for (int u = 0; u < kRound; ++u) { key[i0 + u] = 0u; cls[(i0 + u) >> 2] |= static_cast<uint32_t>(kFastSeg) << (8 * ((i0 + u) & 3)); }
        }
    }
    auto class_of = [&](int i) { return (cls[i >> 2] >> (8 * (i & 3))) & 0xffu; };
    // Between the phases the keys and classes count as changed: otherwise the compiler keeps the K comparisons and class
    // numbers of one phase for the next in registers it does not have.
    auto fresh = [&]() {
#pragma unroll
        for (int i = 0; i < K; ++i) asm volatile("" : "+v"(key[i]));
#pragma unroll
        for (int i = 0; i < (K + 3) / 4; ++i) asm volatile("" : "+v"(cls[i]));
        asm volatile("" : "+s"(n_tiles));
    };
    lo = wave_extreme<false>(lo); hi = wave_extreme<true>(hi);
    __syncthreads();
    if (lane == 0) { atomicMin(&sh.lo, lo); atomicMax(&sh.hi, hi); }
    __syncthreads();
    lo = sh.lo;
    const uint32_t range = sh.hi >= lo ? sh.hi - lo : 0u;
#pragma unroll
    for (int i = 0; i < K; ++i) key[i] -= lo;                       // (tokens without a class: any value, never looked at)

    // digits of `bits` bits from the highest bit of the range down, until the threshold buckets of all classes together
    // hold few enough keys, or to the last bit
    int top = range ? 32 - __clz(range) : 0, shift = 0, listed = 0;
    for (bool first = true;; first = false) {
        shift = top > bits ? top - bits : 0;
        fresh();
        if (!first) {
            for (int i = tid; i < n_seg * class_slots; i += kSelThreads) sh.hist[i] = 0;
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            if (i < n_tiles) {
                const uint32_t c = class_of(i);
                const bool in = c != kFastSeg && (first || (key[i] >> top) == sh.rule[c].y);
                const int digit = static_cast<int>((key[i] >> shift) & ((1u << bits) - 1u));
                hist_add(sh.hist, in ? static_cast<int>(c) * class_slots + bin_slot(digit) : -1);
            }
        }
        __syncthreads();
        if (wave < n_seg && (first || sh.cnt[wave] > 0)) {          // one wave per class
            const int need = sh.need[wave];
            int digit = 0, rem = 0, cnt = 0, population = 0;
            if (bits == 11) wave_find_bucket<32>(sh.hist + wave * class_slots, need, &digit, &rem, &cnt, &population);
            else            wave_find_bucket<8>(sh.hist + wave * class_slots, need, &digit, &rem, &cnt, &population);
            if (lane == 0) {
                if (first && need <= 0) { /* keeps nothing: the rule nobody meets stays */ }
                else if (first && need >= population) sh.rule[wave] = make_uint2(0u, 0xffffffffu);        // keeps everything
                else {
                    const uint32_t prefix = (first ? 0u : sh.rule[wave].y << (top - shift)) | static_cast<uint32_t>(digit);
                    sh.rule[wave] = make_uint2(prefix + 1u, prefix);
                    sh.need[wave] = rem; sh.cnt[wave] = cnt;
                }
            }
        }
        __syncthreads();
        listed = 0;
        for (int c = 0; c < n_seg; ++c) listed += sh.cnt[c];
        if (shift == 0 || listed <= kListCap) break;
        top = shift;
    }
    // One pass decides every token but the candidates; those go to a list, class by class, and are ranked against each
    // other under (key descending, index ascending).  More candidates than the list holds are equal keys of whole
    // classes (shift is 0 then) and are taken in index order below; for that the pass leaves them as a bit mask per group of
    // 64 tokens, and the tokens' classes as up to four bit planes per group where the histogram was.
    const bool ranked = listed <= kListCap;
    const int n_planes = 32 - __clz(n_seg - 1);                     // 0 for one class
    uint64_t* planes = reinterpret_cast<uint64_t*>(sh.hist);
    static_assert(sizeof(sh.hist) >= kFastTiles * 16 * 4 * sizeof(uint64_t) && kFastSeg <= 16, "four planes of every group fit the histogram");
    if (tid == 0) {
        int run = 0;
        for (int c = 0; c < n_seg; ++c) { sh.base[c] = run; run += sh.cnt[c]; }
        sh.base[n_seg] = run;
    }
    __syncthreads();
    fresh();
    constexpr int kStep = 4;                                        // rules of four tokens are read from LDS together
#pragma unroll
    for (int i0 = 0; i0 < K; i0 += kStep) {
        if (i0 < n_tiles) {
            uint2 rule[kStep];
            unsigned long long any = 0;
#pragma unroll
            for (int u = 0; u < kStep; ++u) rule[u] = sh.rule[class_of(i0 + u)];
#pragma unroll
            for (int u = 0; u < kStep; ++u) {
                const uint32_t d = key[i0 + u] >> shift;
                const bool has_class = class_of(i0 + u) != kFastSeg;
                const unsigned long long m = __ballot(has_class && d >= rule[u].x), cand = __ballot(has_class && d == rule[u].y);
                any |= cand;
                if (lane == 0) sh.kept[(i0 + u) * 16 + wave] = m;
                if (!ranked) {
                    const int g = (i0 + u) * 16 + wave;
                    if (lane == 0) sh.equal[g] = cand;
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        if (b < n_planes) {
                            const unsigned long long plane = __ballot((class_of(i0 + u) >> b) & 1u);
                            if (lane == 0) planes[4 * g + b] = plane;
                        }
                    }
                }
            }
            if (ranked && any) {
#pragma unroll
                for (int u = 0; u < kStep; ++u) {
                    const uint32_t c = class_of(i0 + u);
                    if (c != kFastSeg && (key[i0 + u] >> shift) == rule[u].y) {
                        const int p = sh.base[c] + atomicAdd(&sh.fill[c], 1);
                        if (p < kListCap) sh.list[p] = static_cast<uint64_t>(key[i0 + u]) << 32 | static_cast<uint32_t>(~(tid + (i0 + u) * kSelThreads));
                    }
                }
            }
        }
    }
    __syncthreads();
    if (ranked) {
        if (tid < sh.base[n_seg]) {
            int c = 0;
            while (c + 1 < n_seg && tid >= sh.base[c + 1]) ++c;
            // Eight entries a step: one at a time the walk is a chain of LDS round trips (about 200 candidates, eight
            // videos of 36864 tokens in one class: 47 -> 34 us for the kernel; 9216 tokens: 16.8 -> 13.6 us).
            const uint64_t own = sh.list[tid];
            const uint32_t t = ~static_cast<uint32_t>(own);
            const int end = sh.base[c + 1];
            int above = 0;
            for (int p = sh.base[c]; p < end; p += kRankStep) {
                uint64_t other[kRankStep];
#pragma unroll
                for (int u = 0; u < kRankStep; ++u) other[u] = sh.list[p + u];
#pragma unroll
                for (int u = 0; u < kRankStep; ++u) above += p + u < end && other[u] > own ? 1 : 0;
            }
            if (above < sh.need[c]) atomicOr(reinterpret_cast<unsigned long long*>(&sh.kept[t >> 6]), 1ull << (t & 63));
        }
        __syncthreads();
    } else {
        // One wave per class, a lane per run of neighbouring groups: the equal keys of the class before a lane's groups
        // by a scan over the lanes, then the lane takes its own as long as there is room.  (A pass of the workgroup over all
        // keys and a block scan per class took 4 us a class.)
        if (wave < n_seg && sh.cnt[wave] > 0) {
            constexpr int kPer = K / 4;                             // K * 16 groups on 64 lanes
            const int n_groups = n_tiles * 16;
            auto members = [&](int g) {
                uint64_t m = sh.equal[g];
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (b < n_planes) m &= ((wave >> b) & 1) ? planes[4 * g + b] : ~planes[4 * g + b];
                return m;
            };
            int mine = 0;
            for (int u = 0; u < kPer; ++u) {
                const int g = lane * kPer + u;
                if (g < n_groups) mine += __popcll(members(g));
            }
            const int incl = wave_inclusive_scan(mine);
            int room = sh.need[wave] - (incl - mine);
            for (int u = 0; u < kPer && room > 0; ++u) {
                const int g = lane * kPer + u;
                if (g >= n_groups) break;
                uint64_t take = members(g);
                const int n = __popcll(take);
                for (int drop = n - room; drop > 0; --drop) take &= ~(1ull << (63 - __clzll(static_cast<long long>(take))));      // the last ones
                room -= n;
                if (take) atomicOr(reinterpret_cast<unsigned long long*>(&sh.kept[g]), static_cast<unsigned long long>(take));
            }
        }
        __syncthreads();
    }
    int total = 0;
    const int before = block_exclusive_scan_lds(tid < n_tiles * 16 ? __popcll(sh.kept[tid]) : 0, sh.scan, &total);
    if (tid < n_tiles * 16) sh.before[tid] = before;
    __syncthreads();
    asm volatile("" : "+s"(n_tiles));
    const int total_keep = a.keeps.n[blockIdx.z];
#pragma unroll 8
    for (int i = 0; i < n_tiles; ++i) {
        const uint64_t m = sh.kept[i * 16 + wave];
        const int pos = sh.before[i * 16 + wave] + __popcll(m & ((1ull << lane) - 1ull));
        if (((m >> lane) & 1ull) && pos < total_keep) kept_idx[pos] = tid + i * kSelThreads;
    }
    // fewer survivors than announced (a quota above its class population): the tail of the list is index 0, so that the
    // gather stays in bounds
    for (int p = total + tid; p < total_keep; p += kSelThreads) kept_idx[p] = 0;
    if (tid == 0) fs->n_kept = total < total_keep ? total : total_keep;
}

template <int K>
__global__ __launch_bounds__(kSelThreads) void score_select_kernel(const FastArgs a) {
    __shared__ SelectShared sh;
    __shared__ float part[3 * kSelThreads / 4];
    __shared__ int s_last;
    const int tid = threadIdx.x;
    float* scores = of_video_elems(a.scores, a.n_vis);
    const int32_t* token_seg = of_video_elems(a.token_seg, a.n_vis);
    FastSel* fs = of_video(a.fs, a.ws_video);
    if (a.colpart) {
        // `split` threads share a token (a workgroup takes 1024 / split tokens): each adds its share of the workgroup rows'
        // partial sums in order, four loads at a time (a part past the share's last one reads that one again and is not
        // added).  With few partial sums a thread per token leaves one round of workgroups for eight videos instead of two
        // and a half, with many the loads are the longer chain.
        const float* colpart = of_video(a.colpart, a.ws_video);
        const int split = a.n_parts >= kSplitParts ? 4 : 1, tokens = kSelThreads / split;
        const int t = tid % tokens, quarter = tid / tokens;
        const int j = blockIdx.x * tokens + t, jc = min(j, a.n_vis - 1);
        const int per = (a.n_parts + split - 1) / split, p0 = quarter * per, p1 = min(a.n_parts, p0 + per);
        // the event and its weight are requested ahead of the sums: two dependent loads behind them are 0.7 us more
        float w = 1.f;
        if (quarter == 0 && a.event_weight) {
            const int32_t* token_event = of_video_elems(a.token_event, a.n_vis);
            int e = token_event[jc];
            e = e < 0 ? 0 : (e >= a.n_events ? a.n_events - 1 : e);
            w = of_video_elems(a.event_weight, a.n_events)[e];
        }
        float acc = 0.f;
        for (int p = p0; p < p1; p += 4) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = colpart[static_cast<size_t>(min(p + u, p1 - 1)) * a.n_vis + jc];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc += p + u < p1 ? v[u] : 0.f;
        }
        if (split > 1) {
            if (quarter > 0) part[(quarter - 1) * tokens + t] = acc;
            __syncthreads();
        }
        if (quarter == 0 && j < a.n_vis) {
            if (split > 1) acc = ((acc + part[t]) + part[tokens + t]) + part[2 * tokens + t];
            acc = acc / a.rows_total;
            store_shared_between_workgroups(&scores[j], a.event_weight ? acc * w : acc);
        }
        if (!arrive_and_check_last(&fs->arrive, &s_last)) return;
    }
    select_and_index<K>(a, scores, token_seg, fs, of_video_elems(a.kept_idx, a.keep_stride), sh);
}

// Metadata that the kept tokens carry, written by the first n_blocks workgroups of the kernel that moves the rows, so that
// the selecting workgroup leaves nothing but the index list (in the threads that move the rows themselves the extra
// loads cost that kernel a tenth of its rate).
struct CarryArgs {
    const FastSel* fs;
    const int32_t* token_seg;
    const int32_t* token_event;
    const int32_t* orig_idx_in;
    int32_t* token_seg_out;
    int32_t* token_event_out;
    int32_t* orig_idx_out;
    int64_t ws_video, keep_stride, orig_idx_in_stride, orig_idx_stride;
    int n_blocks;                           // 0: nothing to carry (the general selection path writes the metadata itself)
};
// entry r of a video; kept_idx is the video's own list, entries past n_kept are padding
__device__ __forceinline__ void carry_metadata(const CarryArgs& m, int video, int r, int n_keep, const int32_t* __restrict__ kept_idx, int n_vis) {
    if (r >= n_keep) return;
    const FastSel* fs = reinterpret_cast<const FastSel*>(reinterpret_cast<const char*>(m.fs) + video * m.ws_video);
    int kidx = kept_idx[r];
    kidx = kidx < 0 ? 0 : (kidx >= n_vis ? n_vis - 1 : kidx);
    const bool real = r < fs->n_kept;
    const int64_t in = static_cast<int64_t>(video) * n_vis + kidx, out = video * m.keep_stride + r;
    if (m.token_seg_out) m.token_seg_out[out] = real ? m.token_seg[in] : 0;
    if (m.token_event_out) m.token_event_out[out] = real ? m.token_event[in] : 0;
    if (m.orig_idx_out)
        m.orig_idx_out[video * m.orig_idx_stride + r] = real ? (m.orig_idx_in ? m.orig_idx_in[video * m.orig_idx_in_stride + kidx] : kidx) : 0;
}

// Source row of every output row of the compacted sequence [prefix; kept visual rows; text rows].
__global__ __launch_bounds__(256) void hidden_index_kernel(int32_t* __restrict__ src_row, int out_rows, int vis_start, int n_vis, int n_keep,
                                                           const int32_t* __restrict__ kept_idx, int video, const CarryArgs carry) {
    if (static_cast<int>(blockIdx.x) < carry.n_blocks) { carry_metadata(carry, video, blockIdx.x * 256 + threadIdx.x, n_keep, kept_idx, n_vis); return; }
    const int r = (blockIdx.x - carry.n_blocks) * 256 + threadIdx.x;
    if (r >= out_rows) return;
    int s;
    if (r < vis_start) s = r;
    else if (r < vis_start + n_keep) {
        int kidx = kept_idx[r - vis_start];
        kidx = kidx < 0 ? 0 : (kidx >= n_vis ? n_vis - 1 : kidx);
        s = vis_start + kidx;
    } else s = r - n_keep + n_vis;
    src_row[r] = s;
}

constexpr int kGatherThreads = 256;

// One 16-byte chunk per thread, non-temporal (the copy pattern that measured fastest on MI355X).
__global__ __launch_bounds__(kGatherThreads) void gather_rows_kernel(const u32x4_t* __restrict__ src, u32x4_t* __restrict__ dst,
                                                                     int64_t S, int64_t out_row_stride, int chunks_per_row, int vis_start,
                                                                     int n_vis, const int32_t* __restrict__ kept_idx, int64_t keep_stride,
                                                                     const BatchKeep keeps, const CarryArgs carry) {
    const int n_keep = keeps.n[blockIdx.z];
    const int64_t out_rows = S - n_vis + n_keep;
    src = of_video_elems(src, S * chunks_per_row); dst = of_video_elems(dst, out_row_stride * chunks_per_row);
    kept_idx = of_video_elems(kept_idx, keep_stride);
    if (static_cast<int>(blockIdx.x) < carry.n_blocks) {
        carry_metadata(carry, blockIdx.z, blockIdx.x * kGatherThreads + threadIdx.x, n_keep, kept_idx, n_vis);
        return;
    }
    // row and chunk of the workgroup's first thread once (scalar), then a 32-bit division per thread
    const int64_t first = static_cast<int64_t>(blockIdx.x - carry.n_blocks) * kGatherThreads;
    const int64_t row0 = first < 0x7fffffff ? static_cast<int64_t>(static_cast<uint32_t>(first) / static_cast<uint32_t>(chunks_per_row))
                                            : first / chunks_per_row;
    const uint32_t x = static_cast<uint32_t>(first - row0 * chunks_per_row) + threadIdx.x;
    const uint32_t dr = x / static_cast<uint32_t>(chunks_per_row);
    const int64_t r = row0 + dr;
    if (r >= out_rows) return;
    const int c = static_cast<int>(x - dr * static_cast<uint32_t>(chunks_per_row));
    int64_t s;
    if (r < vis_start) s = r;
    else if (r < static_cast<int64_t>(vis_start) + n_keep) {
        int kidx = kept_idx[r - vis_start];
        kidx = kidx < 0 ? 0 : (kidx >= n_vis ? n_vis - 1 : kidx);
        s = vis_start + kidx;
    } else s = r - n_keep + n_vis;
    __builtin_nontemporal_store(__builtin_nontemporal_load(src + s * chunks_per_row + c), dst + r * chunks_per_row + c);
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
static bool dh_supported(int dh, int dtype) {
    if (dtype == METOK_BF16) return dh == 32 || dh == 64 || dh == 128 || dh == 256;
    return dh == 32 || dh == 64 || dh == 128;
}

// Row blocks of 16 that the narrow kernels take for this shape, 0: the shape is not theirs.  bf16 rows of at most four
// chunks per lane: with eight (256 elements) fewer subtiles are on their way beside the queries (row statistics of
// 9000 keys of 256: 8.5 us above, 11.1 us here); fp32 products take sixteen times the matrix time, so there eight busy waves
// win anyway (40 heads x 64 queries x 17219 keys of 128: 208 + 210 -> 143 + 127 us).
static int narrow_blocks(const ScoreGeom& g, int nch16, bool f32) {
    return g.R > 64 || (nch16 > 4 && !f32) ? 0 : (g.R <= 16 ? 1 : (g.R <= 32 ? 2 : 4));
}

template <typename T, int NCH16, int NB>
static void launch_narrow_scores(const void* q, const void* k, const ScoreGeom& g, const ScorePlan& p, char* ws, int batch, hipStream_t st) {
    float* pstat = reinterpret_cast<float*>(ws + p.off_pstat);
    float* colpart = reinterpret_cast<float*>(ws + p.off_colpart);
    const unsigned nb = static_cast<unsigned>(batch);
    { TraceScope trace_scope(METOK_TRACE_ROW_STATS, st); hipLaunchKernelGGL((narrow_row_stats_kernel<T, NCH16, NB>), dim3(p.nx1, g.Hkv, nb), dim3(kScoreThreads), 0, st,
                       static_cast<const T*>(q), static_cast<const T*>(k), g, p.per1, pstat,
                       reinterpret_cast<uint32_t*>(ws + p.off_sel + select_general_bytes(g.n_vis)), kFastClearWords); }
    { TraceScope trace_scope(METOK_TRACE_COL_SUMS, st); hipLaunchKernelGGL((narrow_col_sums_kernel<T, NCH16, NB>), dim3(p.nx2, g.Hkv, nb), dim3(kScoreThreads), 0, st,
                       static_cast<const T*>(q), static_cast<const T*>(k), g, p.per2, pstat, p.nx1, colpart); }
}

// Whether the fp32 rows of a workgroup, at most one block per wave, are multiplied as bf16 parts.  To take a row block apart is 0.5 us of
// each pass, so it needs keys to pay.  Whole calls by graph replay, us, fp32 MFMA / parts: 14 heads on 2 x 32 queries of 64 elements,
// 5000 tokens (two subtiles a workgroup) 39.5 / 36.0, 24000 80.4 / 69.2; 28 on 4 x 64 of 128, 1500 (two) 45.9 / 42.1.  Workgroups of up
// to four row blocks have one wave with rows to a SIMD, whose steps are a chain: 12 heads on 4 x 30 of 64, 24000 (96 = subtiles x pieces
// of a row) 80.2 / 77.6; 20 on 10 x 40 of 128, 5000 (112) 61.0 / 55.2.  Below the lines, levels alone, by a chain that was a little
// shorter (one sum): 14 on 2 x 32 of 64, 1500 (one) 26.1 / 26.8, 28 on 4 x 64 of 128, 300 (one) 29.2 / 29.3; 12 on 4 x 30 of 64, 5000
// (24) 30.0 / 30.9, 20 on 10 x 40 of 128, 1500 (32) 30.3 / 32.2.
static bool split_products(const ScoreGeom& g, const ScorePlan& p, int nch) {
    return blocks_of_busiest_simd(g) > 1 ? p.per1 >= 2 : p.per1 * nch >= 96;
}

// Both passes with a workgroup's rows in the waves' RBW blocks each.  false: nothing was launched.
template <typename T, int NCH, int RBW, int SUBS>
static bool launch_staged_scores(const void* q, const void* k, const ScoreGeom& g, const ScorePlan& p, char* ws, int batch, hipStream_t st) {
    using Stage = KeyStage<T, NCH, SUBS>;
    constexpr size_t lds1 = std::max(kStageBuffers * static_cast<size_t>(Stage::kSlots) * sizeof(uint4), QueryRows<T, NCH, 1>::kLdsBytes);
    constexpr size_t lds2 = 2 * static_cast<size_t>(Stage::kSlots) * sizeof(uint4) + 2 * static_cast<size_t>(kScoreWaves) * Stage::kKeys * sizeof(float);
    static_assert(std::is_same<T, split_t>::value || std::max(lds1, lds2) <= 64 * 1024, "only the parts' kernels, which fp32 MFMA can stand in for, may not be had");
    if (!allow_lds<&row_stats_kernel<T, NCH, RBW, SUBS>>(lds1) || !allow_lds<&col_sums_kernel<T, NCH, RBW, SUBS>>(lds2)) return false;
    const int ny = g.Hkv * g.rs;
    uint32_t* clear = reinterpret_cast<uint32_t*>(ws + p.off_sel + select_general_bytes(g.n_vis));
    uint4* qfrag = reinterpret_cast<uint4*>(ws + p.off_qfrag);
    float* pstat = reinterpret_cast<float*>(ws + p.off_pstat);
    float* norm = reinterpret_cast<float*>(ws + p.off_norm);
    float* colpart = reinterpret_cast<float*>(ws + p.off_colpart);
    const unsigned nb = static_cast<unsigned>(batch);
    {
        TraceScope trace_scope(METOK_TRACE_ROW_STATS, st);
        hipLaunchKernelGGL((row_stats_kernel<T, NCH, RBW, SUBS>), dim3(p.nx1, ny, nb), dim3(kScoreThreads), lds1, st, static_cast<const T*>(q),
                           static_cast<const T*>(k), g, p.per1, pstat, qfrag, clear, kFastClearWords);
    }
    const float* unmerged = pstat;
    if (partial_bytes(g, p) > kMergeInPass2Bytes) {
        const int total_rows = ny * g.rbw * 32;
        hipLaunchKernelGGL(merge_stats_kernel, dim3((total_rows + 15) / 16, 1, nb), dim3(256), 0, st, pstat, g, p.nx1, norm);
        unmerged = nullptr;
    }
    TraceScope trace_scope(METOK_TRACE_COL_SUMS, st);
    hipLaunchKernelGGL((col_sums_kernel<T, NCH, RBW, SUBS>), dim3(p.nx2, ny, nb), dim3(kScoreThreads), lds2, st, qfrag, static_cast<const T*>(k), g, p.per2, norm, unmerged, p.nx1, colpart);
    return true;
}

template <typename T, int NCH>
static void launch_scores(const void* q, const void* k, const ScoreGeom& g, const ScorePlan& p, char* ws, int batch, hipStream_t st) {
    constexpr int RBW = NCH <= 8 ? 2 : 1;
    constexpr int SUBS = NCH <= 8 ? 2 : 1;
    constexpr int NCH16 = NCH / 2;                       // chunks per lane when four lanes share a row
    if constexpr (NCH16 <= 4 || std::is_same<T, float>::value) {
        switch (narrow_blocks(g, NCH16, std::is_same<T, float>::value)) {
            case 1: launch_narrow_scores<T, NCH16, 1>(q, k, g, p, ws, batch, st); return;
            case 2: launch_narrow_scores<T, NCH16, 2>(q, k, g, p, ws, batch, st); return;
            case 4: launch_narrow_scores<T, NCH16, 4>(q, k, g, p, ws, batch, st); return;
        }
    }
    // With at most one row block per wave the two-block pipeline would run its second chain on zeros (32 heads on 8,
    // 4 x 36928 keys: 159 -> 124 us; 14 heads on 2, 32 queries, 5064 keys in fp32: 10.4 -> 9.6 us).
    if (g.rbw > kScoreWaves) launch_staged_scores<T, NCH, RBW, SUBS>(q, k, g, p, ws, batch, st);
    else {
        if constexpr (std::is_same<T, float>::value)
            if (split_products(g, p, NCH) && launch_staged_scores<split_t, NCH, 1, SUBS>(q, k, g, p, ws, batch, st)) return;
        launch_staged_scores<T, NCH, 1, SUBS>(q, k, g, p, ws, batch, st);
    }
}

}  // namespace metok

using namespace metok;

// Workspace of ONE video of a batch of `batch` videos (the batch's videos lie one after the other).
static size_t video_workspace_bytes(int batch, int64_t S, int Hq, int Hkv, int dh, int Tq, int n_vis, int dtype) {
    if (n_vis < 0 || S < 1 || batch < 1) return 0;
    ScoreGeom g;
    ScorePlan p;
    if (Hq >= 1 && Hkv >= 1 && Tq >= 1 && Hq % Hkv == 0 && dh_supported(dh, dtype) &&
        make_geom(S, Hq, Hkv, dh, Tq, 0, n_vis, dtype, METOK_SCORE_CAUSAL_ALL, &g)) {
        plan_score(&g, n_vis, dtype, batch, &p);
        return p.total;
    }
    return round_up(select_bytes(n_vis) + inplace_bytes(S), 256);      // no attention pass (scores supplied by the caller)
}

extern "C" size_t metok_prefill_prune_workspace_bytes(int64_t S, int Hq, int Hkv, int dh, int Tq, int n_vis, int dtype) {
    return video_workspace_bytes(1, S, Hq, Hkv, dh, Tq, n_vis, dtype);
}

extern "C" size_t metok_prefill_prune_batched_workspace_bytes(int batch, int64_t S, int Hq, int Hkv, int dh, int Tq, int n_vis, int dtype) {
    if (batch < 1 || batch > METOK_MAX_BATCH) return 0;
    return static_cast<size_t>(batch) * video_workspace_bytes(batch, S, Hq, Hkv, dh, Tq, n_vis, dtype);
}

// Shared body of metok_prefill_prune, metok_prefill_prune_batched and metok_prefill_prune_static: `workspace` is the
// caller's buffer or the library's static scratch array; nothing below allocates.  Every array carries a leading
// dimension of `batch` videos (tightly packed inputs; outputs keep_stride entries / out_row_stride rows apart); every
// kernel takes the video from blockIdx.z.
static int prune_impl(int batch, const void* hidden, int64_t S, int D, int dtype,
                      const void* q_text, const void* k_all, int Hq, int Hkv, int dh, int Tq,
                      int score_mode, int vis_start, int n_vis,
                      const int32_t* token_seg, const int32_t* token_event,
                      const float* event_weight, int n_events,
                      int n_seg, const int32_t* seg_quota,
                      const int32_t* orig_idx_in, int64_t orig_idx_in_stride,
                      float* scores, int32_t* kept_idx, int64_t keep_stride, void* hidden_out, int64_t out_row_stride,
                      int32_t* token_seg_out, int32_t* token_event_out, int32_t* orig_idx_out, int64_t orig_idx_stride,
                      void* workspace, size_t workspace_bytes, void* stream) {
    if (batch < 1 || batch > METOK_MAX_BATCH) return fail(METOK_ERR_INVALID_ARG, "batch must be in [1, %d]", METOK_MAX_BATCH);
    if (dtype != METOK_F32 && dtype != METOK_BF16) return fail(METOK_ERR_INVALID_ARG, "unknown dtype %d", dtype);
    if (S < 1 || S > INT32_MAX || D < 1) return fail(METOK_ERR_INVALID_ARG, "S must be in [1, 2^31) and D positive");
    if (vis_start < 0 || n_vis < 1 || static_cast<int64_t>(vis_start) + n_vis > S)
        return fail(METOK_ERR_INVALID_ARG, "visual span [%d, %d + %d) does not fit S = %lld", vis_start, vis_start, n_vis, (long long)S);
    const size_t row_bytes = static_cast<size_t>(D) * dtype_size(dtype);
    if (row_bytes % 16) return fail(METOK_ERR_INVALID_ARG, "D * sizeof(dtype) must be a multiple of 16");
    if (!hidden || !hidden_out || !aligned16(hidden) || !aligned16(hidden_out))
        return fail(METOK_ERR_INVALID_ARG, "hidden / hidden_out NULL or not 16-byte aligned");
    if (!token_seg || !scores || !seg_quota) return fail(METOK_ERR_INVALID_ARG, "NULL pointer argument");
    if (n_seg < 1 || n_seg > METOK_MAX_SEGMENTS) return fail(METOK_ERR_INVALID_ARG, "n_seg must be in [1, %d]", METOK_MAX_SEGMENTS);
    if (!token_event && (event_weight || token_event_out)) return fail(METOK_ERR_INVALID_ARG, "token_event is NULL but needed");
    if (event_weight && n_events < 1) return fail(METOK_ERR_INVALID_ARG, "event_weight given with n_events < 1");
    BatchKeep keeps;
    int64_t max_keep = 0;
    for (int b = 0; b < METOK_MAX_BATCH; ++b) keeps.n[b] = 0;
    for (int b = 0; b < batch; ++b) {
        int64_t total_keep = 0;
        for (int s = 0; s < n_seg; ++s) {
            const int32_t q = seg_quota[static_cast<size_t>(b) * n_seg + s];
            if (q < 0 || q > n_vis) return fail(METOK_ERR_INVALID_ARG, "seg_quota[%d] = %d of video %d outside [0, n_vis]", s, q, b);
            total_keep += q;
        }
        if (total_keep > n_vis) return fail(METOK_ERR_INVALID_ARG, "quotas of video %d add up to %lld > n_vis = %d", b, (long long)total_keep, n_vis);
        keeps.n[b] = static_cast<int32_t>(total_keep);
        max_keep = total_keep > max_keep ? total_keep : max_keep;
    }
    if (max_keep > 0 && !kept_idx) return fail(METOK_ERR_INVALID_ARG, "kept_idx is NULL");
    const int64_t max_out_rows = S - n_vis + max_keep;
    if (batch > 1 && (keep_stride < max_keep || out_row_stride < max_out_rows))
        return fail(METOK_ERR_INVALID_ARG, "keep_stride = %lld / out_row_stride = %lld below the largest video's %lld kept tokens / %lld rows",
                    (long long)keep_stride, (long long)out_row_stride, (long long)max_keep, (long long)max_out_rows);
    if (batch > 1 && orig_idx_out && orig_idx_stride < max_keep)
        return fail(METOK_ERR_INVALID_ARG, "orig_idx_stride = %lld below the largest video's %lld kept tokens", (long long)orig_idx_stride, (long long)max_keep);
    if (batch > 1 && orig_idx_in && orig_idx_in_stride < n_vis)
        return fail(METOK_ERR_INVALID_ARG, "orig_idx_in_stride = %lld below n_vis = %d", (long long)orig_idx_in_stride, n_vis);
    if (batch == 1) { keep_stride = max_keep; out_row_stride = max_out_rows; orig_idx_stride = max_keep; orig_idx_in_stride = n_vis; }
    // hidden_out == hidden compacts in place (every kept row moves towards the front: source >= destination);
    // any other overlap is refused
    const bool in_place = hidden_out == hidden;
    if (!in_place) {
        const char* a0 = static_cast<const char*>(hidden); const char* a1 = a0 + static_cast<size_t>(batch) * S * row_bytes;
        const char* b0 = static_cast<const char*>(hidden_out);
        const char* b1 = b0 + (static_cast<size_t>(batch - 1) * out_row_stride + max_out_rows) * row_bytes;
        if (a0 < b1 && b0 < a1) return fail(METOK_ERR_INVALID_ARG, "hidden_out overlaps hidden without being the same buffer");
    } else {
        if (static_cast<int64_t>(row_bytes) > kInPlaceMaxRowBytes)
            return fail(METOK_ERR_UNSUPPORTED, "in-place compaction needs rows of at most %lld bytes, got %zu", (long long)kInPlaceMaxRowBytes, row_bytes);
        if (batch > 1 && out_row_stride != S)
            return fail(METOK_ERR_INVALID_ARG, "in-place compaction of a batch keeps every video where it is: out_row_stride must be S");
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    int rc;
    char* sel;
    char* inplace_ws;
    const float* colpart = nullptr;
    int n_parts = 0;
    const unsigned nb = static_cast<unsigned>(batch);
    const int64_t ws_video = static_cast<int64_t>(video_workspace_bytes(batch, S, q_text ? Hq : 0, q_text ? Hkv : 0, q_text ? dh : 0,
                                                                        q_text ? Tq : 0, n_vis, dtype));
    const int n_tiles = select_tiles(n_vis);
    const bool fast = one_launch_selection(batch, n_seg, n_tiles);      // else the general one-workgroup-per-class select
    if (q_text) {
        if (!k_all || !aligned16(q_text) || !aligned16(k_all)) return fail(METOK_ERR_INVALID_ARG, "q_text / k_all NULL or misaligned");
        if (Hq < 1 || Hkv < 1 || Hq % Hkv) return fail(METOK_ERR_INVALID_ARG, "Hq = %d must be a positive multiple of Hkv = %d", Hq, Hkv);
        if (!dh_supported(dh, dtype)) return fail(METOK_ERR_UNSUPPORTED, "head dimension %d is not supported for this dtype", dh);
        if (Tq < 1 || static_cast<int64_t>(Tq) > S - vis_start - n_vis)
            return fail(METOK_ERR_INVALID_ARG, "Tq = %d must be in [1, number of text rows = %lld]", Tq, (long long)(S - vis_start - n_vis));
        if (score_mode != METOK_SCORE_CAUSAL_ALL && score_mode != METOK_SCORE_VISUAL_ONLY)
            return fail(METOK_ERR_INVALID_ARG, "unknown score_mode %d", score_mode);
        ScoreGeom g;
        if (!make_geom(S, Hq, Hkv, dh, Tq, vis_start, n_vis, dtype, score_mode, &g)) return fail(METOK_ERR_UNSUPPORTED, "head dimension too large");
        if (static_cast<int64_t>(g.Hkv) * g.rs > 65535) return fail(METOK_ERR_UNSUPPORTED, "too many query rows");
        ScorePlan p;
        plan_score(&g, n_vis, dtype, batch, &p);
        g.q_video = static_cast<int64_t>(Hq) * Tq * dh; g.k_video = static_cast<int64_t>(Hkv) * S * dh; g.ws_video = ws_video;
        if (static_cast<int64_t>(p.total) != ws_video) return fail(METOK_ERR_DEVICE, "internal: workspace plan mismatch");
        if (!workspace || workspace_bytes < p.total * batch || !aligned16(workspace))
            return fail(METOK_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", p.total * batch, workspace_bytes);
        const int nch = chunk_count(dh, dtype);
        if (dtype == METOK_BF16) {
            switch (nch) {
                case 2: launch_scores<bf16_t, 2>(q_text, k_all, g, p, ws, batch, st); break;
                case 4: launch_scores<bf16_t, 4>(q_text, k_all, g, p, ws, batch, st); break;
                case 8: launch_scores<bf16_t, 8>(q_text, k_all, g, p, ws, batch, st); break;
                default: launch_scores<bf16_t, 16>(q_text, k_all, g, p, ws, batch, st); break;
            }
        } else {
            switch (nch) {
                case 4: launch_scores<float, 4>(q_text, k_all, g, p, ws, batch, st); break;
                case 8: launch_scores<float, 8>(q_text, k_all, g, p, ws, batch, st); break;
                default: launch_scores<float, 16>(q_text, k_all, g, p, ws, batch, st); break;
            }
        }
        if ((rc = check_launch("attention scores"))) return rc;
        sel = ws + p.off_sel;
        inplace_ws = ws + p.off_inplace;
        colpart = reinterpret_cast<const float*>(ws + p.off_colpart);
        n_parts = g.Hkv * g.rs;
        if (!fast) {
            hipLaunchKernelGGL(prepare_kernel, dim3((n_vis + 255) / 256, 1, nb), dim3(256), 0, st, colpart, n_parts, n_vis,
                               static_cast<float>(static_cast<int64_t>(Hq) * Tq), token_event, event_weight, n_events, scores, ws_video);
            if ((rc = check_launch("prepare"))) return rc;
        }
    } else {
        const size_t need = static_cast<size_t>(ws_video) * batch;
        if (!workspace || workspace_bytes < need || !aligned16(workspace))
            return fail(METOK_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", need, workspace_bytes);
        sel = ws;
        inplace_ws = ws + select_bytes(n_vis);
    }
    int32_t* gt_count = reinterpret_cast<int32_t*>(sel);
    int32_t* eq_count = reinterpret_cast<int32_t*>(sel + select_count_bytes(n_vis));
    uint32_t* sel_info = reinterpret_cast<uint32_t*>(sel + 2 * select_count_bytes(n_vis));
    CarryArgs carry = {};
    if (fast) {
        FastArgs fa;
        fa.fs = reinterpret_cast<FastSel*>(sel + select_general_bytes(n_vis));
        fa.colpart = colpart; fa.n_parts = n_parts; fa.rows_total = static_cast<float>(static_cast<int64_t>(Hq) * Tq);
        fa.token_event = token_event; fa.event_weight = event_weight; fa.n_events = n_events;
        fa.scores = scores; fa.token_seg = token_seg; fa.n_vis = n_vis; fa.n_seg = n_seg; fa.ws_video = ws_video;
        fa.kept_idx = kept_idx; fa.keep_stride = keep_stride; fa.keeps = keeps;
        for (int b = 0; b < METOK_MAX_BATCH; ++b)
            for (int c = 0; c < kFastSeg; ++c)
                fa.quota[b][c] = static_cast<uint16_t>((b < batch && c < n_seg) ? seg_quota[static_cast<size_t>(b) * n_seg + c] : 0);
        {
            // one launch is both "select" and "write index": the trace hook brackets it for either name
            TraceScope trace_select(METOK_TRACE_SELECT, st);
            TraceScope trace_index(METOK_TRACE_WRITE_INDEX, st);
            const int score_tokens = kSelThreads / (n_parts >= kSplitParts ? 4 : 1);
            const dim3 grid(colpart ? (n_vis + score_tokens - 1) / score_tokens : 1, 1, nb);
            if (n_tiles <= 4) hipLaunchKernelGGL(score_select_kernel<4>, grid, dim3(kSelThreads), 0, st, fa);
            else if (n_tiles <= 12) hipLaunchKernelGGL(score_select_kernel<12>, grid, dim3(kSelThreads), 0, st, fa);
            else hipLaunchKernelGGL(score_select_kernel<kFastTiles>, grid, dim3(kSelThreads), 0, st, fa);
        }
        if ((rc = check_launch("select"))) return rc;
        carry.n_blocks = static_cast<int>((max_keep + 255) / 256);
        carry.fs = fa.fs; carry.token_seg = token_seg; carry.token_event = token_event; carry.orig_idx_in = orig_idx_in;
        carry.token_seg_out = token_seg_out; carry.token_event_out = token_event_out; carry.orig_idx_out = orig_idx_out;
        carry.ws_video = ws_video; carry.keep_stride = keep_stride; carry.orig_idx_in_stride = orig_idx_in_stride; carry.orig_idx_stride = orig_idx_stride;
    } else {
        // the general selection takes its quotas by value: one launch per video
        {
        TraceScope trace_scope(METOK_TRACE_SELECT, st);
        for (int b = 0; b < batch; ++b) {
            Quotas quotas;
            for (int c = 0; c < METOK_MAX_SEGMENTS; ++c) quotas.q[c] = c < n_seg ? seg_quota[static_cast<size_t>(b) * n_seg + c] : 0;
            const float* sc_b = scores + static_cast<size_t>(b) * n_vis;
            const int32_t* seg_b = token_seg + static_cast<size_t>(b) * n_vis;
            auto at = [&](auto* ptr) { return reinterpret_cast<decltype(ptr)>(reinterpret_cast<char*>(ptr) + static_cast<size_t>(b) * ws_video); };
            if (n_vis <= kSelCache * kSelThreads)
                hipLaunchKernelGGL(select_kernel<true>, dim3(n_seg), dim3(kSelThreads), 0, st, sc_b, seg_b, n_vis, n_tiles, quotas,
                                   at(gt_count), at(eq_count), at(sel_info));
            else
                hipLaunchKernelGGL(select_kernel<false>, dim3(n_seg), dim3(kSelThreads), 0, st, sc_b, seg_b, n_vis, n_tiles, quotas,
                                   at(gt_count), at(eq_count), at(sel_info));
        }
        }
        if ((rc = check_launch("select"))) return rc;
        TraceScope trace_index(METOK_TRACE_WRITE_INDEX, st);
        hipLaunchKernelGGL(write_index_kernel, dim3(n_tiles, 1, nb), dim3(kIdxThreads), 0, st, scores, sel_info, gt_count, eq_count, token_seg,
                           n_vis, n_seg, n_tiles, 0, token_event, orig_idx_in, kept_idx, token_seg_out, token_event_out, orig_idx_out,
                           ws_video, keep_stride, orig_idx_in_stride, orig_idx_stride, keeps);
        if ((rc = check_launch("write index"))) return rc;
    }
    if (in_place) {
        // the row mover takes one sequence per call here: the videos of a batch go one after the other
        for (int b = 0; b < batch; ++b) {
            const int64_t out_rows = S - n_vis + keeps.n[b];
            if (out_rows == 0) continue;
            char* ws_b = inplace_ws + static_cast<size_t>(b) * ws_video;
            int32_t* src_row = reinterpret_cast<int32_t*>(ws_b);
            hipLaunchKernelGGL(hidden_index_kernel, dim3(static_cast<unsigned>((out_rows + 255) / 256) + carry.n_blocks), dim3(256), 0, st, src_row,
                               static_cast<int>(out_rows), vis_start, n_vis, keeps.n[b], kept_idx + static_cast<size_t>(b) * keep_stride, b, carry);
            if ((rc = check_launch("hidden index"))) return rc;
            RowMoveLayer layer;
            layer.k = static_cast<char*>(hidden_out) + static_cast<size_t>(b) * S * row_bytes; layer.v = nullptr; layer.idx = src_row;
            layer.n_keep = static_cast<int32_t>(out_rows);
            layer.first_item = 0; layer.tiles = 0; layer.flag_slot = 0; layer.layer_id = 0;
            rc = launch_row_moves(&layer, 1, 1, 1, 1, S, static_cast<int64_t>(row_bytes), nullptr, 0, 0, 0, nullptr, nullptr, 1,
                                  ws_b + inplace_index_bytes(S), inplace_bytes(S) - inplace_index_bytes(S), st, nullptr);
            if (rc) return rc;
        }
        return METOK_OK;
    }
    const int chunks_per_row = static_cast<int>(row_bytes / 16);
    const int64_t blocks = (max_out_rows * chunks_per_row + kGatherThreads - 1) / kGatherThreads;
    if (blocks + carry.n_blocks > 0x7fffffff) return fail(METOK_ERR_INVALID_ARG, "hidden_out too large for one launch");
    if (blocks == 0) return METOK_OK;
    { TraceScope trace_scope(METOK_TRACE_GATHER_ROWS, st); hipLaunchKernelGGL(gather_rows_kernel, dim3(static_cast<unsigned>(blocks) + carry.n_blocks, 1, nb), dim3(kGatherThreads), 0, st,
                       static_cast<const u32x4_t*>(hidden), static_cast<u32x4_t*>(hidden_out), S, out_row_stride, chunks_per_row,
                       vis_start, n_vis, kept_idx, keep_stride, keeps, carry); }
    return check_launch("gather");
}

extern "C" int metok_prefill_prune(const void* hidden, int64_t S, int D, int dtype,
                                   const void* q_text, const void* k_all, int Hq, int Hkv, int dh, int Tq,
                                   int score_mode, int vis_start, int n_vis,
                                   const int32_t* token_seg, const int32_t* token_event,
                                   const float* event_weight, int n_events,
                                   int n_seg, const int32_t* seg_quota,
                                   const int32_t* orig_idx_in,
                                   float* scores, int32_t* kept_idx, void* hidden_out,
                                   int32_t* token_seg_out, int32_t* token_event_out, int32_t* orig_idx_out,
                                   void* workspace, size_t workspace_bytes, void* stream) {
    clear_error();
    return prune_impl(1, hidden, S, D, dtype, q_text, k_all, Hq, Hkv, dh, Tq, score_mode, vis_start, n_vis, token_seg, token_event,
                      event_weight, n_events, n_seg, seg_quota, orig_idx_in, 0, scores, kept_idx, 0, hidden_out, 0, token_seg_out,
                      token_event_out, orig_idx_out, 0, workspace, workspace_bytes, stream);
}

extern "C" int metok_prefill_prune_batched(int batch, const void* hidden, int64_t S, int D, int dtype,
                                           const void* q_text, const void* k_all, int Hq, int Hkv, int dh, int Tq,
                                           int score_mode, int vis_start, int n_vis,
                                           const int32_t* token_seg, const int32_t* token_event,
                                           const float* event_weight, int n_events,
                                           int n_seg, const int32_t* seg_quota,
                                           const int32_t* orig_idx_in, int64_t orig_idx_in_stride,
                                           float* scores, int32_t* kept_idx, int64_t keep_stride,
                                           void* hidden_out, int64_t out_row_stride,
                                           int32_t* token_seg_out, int32_t* token_event_out,
                                           int32_t* orig_idx_out, int64_t orig_idx_stride,
                                           void* workspace, size_t workspace_bytes, void* stream) {
    clear_error();
    return prune_impl(batch, hidden, S, D, dtype, q_text, k_all, Hq, Hkv, dh, Tq, score_mode, vis_start, n_vis, token_seg, token_event,
                      event_weight, n_events, n_seg, seg_quota, orig_idx_in, orig_idx_in_stride, scores, kept_idx, keep_stride, hidden_out, out_row_stride,
                      token_seg_out, token_event_out, orig_idx_out, orig_idx_stride, workspace, workspace_bytes, stream);
}

// ---------------------------------------------------------------------------------------------
// metok_prefill_prune_static: the same call for callers that cannot allocate a workspace.  The scratch
// memory is a fixed array in the library's device image; every GPU holds its own copy at its own address,
// looked up once per device.  In host code the array's name is only a handle for that lookup: kernels
// and the shared body above always receive the looked-up device address.
// ---------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[METOK_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {nullptr};
}  // namespace

// Device address of this GPU's copy of `scratch` (cached after the first call on the device).
static int static_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(METOK_ERR_DEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(METOK_ERR_UNSUPPORTED, "device ordinal %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return fail(METOK_ERR_DEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return METOK_OK;
}

extern "C" size_t metok_static_scratch_bytes(void) { return METOK_STATIC_SCRATCH_BYTES; }

extern "C" int metok_prefill_prune_static(const void* hidden, int64_t S, int D, int dtype,
                                          const void* q_text, const void* k_all, int Hq, int Hkv, int dh, int Tq,
                                          int score_mode, int vis_start, int n_vis,
                                          const int32_t* token_seg, const int32_t* token_event,
                                          const float* event_weight, int n_events,
                                          int n_seg, const int32_t* seg_quota,
                                          const int32_t* orig_idx_in,
                                          float* scores, int32_t* kept_idx, void* hidden_out,
                                          int32_t* token_seg_out, int32_t* token_event_out, int32_t* orig_idx_out,
                                          void* stream) {
    clear_error();
    // the size check comes first so that an oversized request is refused before anything touches the device
    const size_t need = metok_prefill_prune_workspace_bytes(S, q_text ? Hq : 0, q_text ? Hkv : 0, q_text ? dh : 0, q_text ? Tq : 0,
                                                            n_vis, dtype);
    if (need > METOK_STATIC_SCRATCH_BYTES)
        return fail(METOK_ERR_WORKSPACE, "this shape needs %zu bytes of scratch memory, the static array holds %zu: use metok_prefill_prune "
                    "with a caller-provided workspace", need, static_cast<size_t>(METOK_STATIC_SCRATCH_BYTES));
    void* ws = nullptr;
    int rc = static_scratch(&ws);
    if (rc) return rc;
    return prune_impl(1, hidden, S, D, dtype, q_text, k_all, Hq, Hkv, dh, Tq, score_mode, vis_start, n_vis, token_seg, token_event,
                      event_weight, n_events, n_seg, seg_quota, orig_idx_in, 0, scores, kept_idx, 0, hidden_out, 0, token_seg_out,
                      token_event_out, orig_idx_out, 0, ws, METOK_STATIC_SCRATCH_BYTES, stream);
}
