// How the score passes and the selection of stage 2 lie on the chip and in the workspace: host arithmetic in plain C++, without
// HIP, so that it can be built and checked on its own.
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include "metok.h"

namespace metok {

constexpr int kScoreThreads = 512;
constexpr int kScoreWaves = kScoreThreads / 64;
constexpr int kSelThreads = 1024;      // also the tile size of the selection: tile i = tokens [1024 i, 1024 i + 1024)
constexpr int kSelCache = 40;          // keys per thread held in registers (n_vis <= 40960)

inline size_t round_up_256(size_t x) { return (x + 255) / 256 * 256; }

struct ScoreGeom {
    int64_t S;
    int Hq, Hkv, group, dh, Tq;
    int R;              // rows per kv head = group * Tq
    int rb_total;       // 32-row blocks per kv head
    int rbw;            // row blocks per workgroup (<= kScoreWaves * RBW)
    int rs;             // row splits per kv head
    int vis_start, n_vis;
    int64_t key_begin, key_end;   // keys the softmax of pass 1 normalises over (before the causal mask)
    float scale_log2;   // log2(e) / sqrt(dh)
    // a batch of videos runs as one launch, blockIdx.z = video: distances between consecutive videos
    int64_t q_video, k_video;     // elements of q_text / k_all
    int64_t ws_video;             // bytes of workspace
};

struct FastSel {
    uint32_t arrive;                        // cleared before the kernel that counts on it
    int32_t n_kept;                         // kept tokens written (the rest of the list is padding)
};
constexpr int kFastClearWords = 1;

// selection scratch: per-class tile counts above / equal to the threshold [2][METOK_MAX_SEGMENTS][n_tiles], then
// (threshold, equal keys kept) per class
inline int select_tiles(int n_vis) { return (n_vis + kSelThreads - 1) / kSelThreads; }
inline size_t select_count_bytes(int n_vis) {
    return round_up_256(static_cast<size_t>(METOK_MAX_SEGMENTS) * select_tiles(n_vis) * sizeof(int32_t));
}
inline size_t select_general_bytes(int n_vis) { return 2 * select_count_bytes(n_vis) + METOK_MAX_SEGMENTS * 2 * sizeof(uint32_t); }
// then the fast path's state.  The reserve is larger than FastSel needs, and the two words per token behind it are used by
// no kernel: they held the histograms and candidate lists of an earlier selection.  The size of a workspace is part of the
// interface (it also decides which shapes metok_prefill_prune_static takes), so it stays what it has been; row splits put their
// additional column sums there, see plan_score.
constexpr size_t kFastReserve = 34560;
static_assert(sizeof(FastSel) <= kFastReserve, "the fast path's state outgrew its reserve");
inline size_t select_bytes(int n_vis) {
    const size_t unused = round_up_256(static_cast<size_t>(n_vis < kSelCache * kSelThreads ? n_vis : kSelCache * kSelThreads) * sizeof(uint32_t));
    return select_general_bytes(n_vis) + kFastReserve + 2 * unused;
}

// In-place compaction (hidden_out == hidden): the source row of every output row as an index list, and the
// progress flags of the row mover.  Rows of at most kInPlaceMaxRowBytes keep a row inside one workgroup
// pass, so a tile has at least eight rows and the flag count is bounded by the sequence length alone.
constexpr int64_t kInPlaceMaxRowBytes = 16384;
inline size_t inplace_index_bytes(int64_t S) { return round_up_256(static_cast<size_t>(S) * sizeof(int32_t)); }
inline size_t inplace_bytes(int64_t S) {
    return inplace_index_bytes(S) + round_up_256((64 + static_cast<size_t>((S + 7) / 8)) * sizeof(uint32_t));
}

inline int chunk_count(int dh, int dtype) { return dtype == METOK_BF16 ? dh / 16 : dh / 8; }     // 16-byte chunks per lane

// Row blocks a wave keeps in registers: two while the fragments of a block take at most 32 VGPRs, else one.
inline int row_blocks_per_wave(int nch) { return nch <= 8 ? 2 : 1; }

inline bool make_geom(int64_t S, int Hq, int Hkv, int dh, int Tq, int vis_start, int n_vis, int dtype, int score_mode,
                      ScoreGeom* g) {
    g->S = S; g->Hq = Hq; g->Hkv = Hkv; g->group = Hq / Hkv; g->dh = dh; g->Tq = Tq;
    g->R = g->group * Tq;
    g->rb_total = (g->R + 31) / 32;
    const int nch = chunk_count(dh, dtype);
    if (nch > 16) return false;
    const int cap = kScoreWaves * row_blocks_per_wave(nch);
    g->rs = (g->rb_total + cap - 1) / cap;
    g->rbw = (g->rb_total + g->rs - 1) / g->rs;
    g->vis_start = vis_start; g->n_vis = n_vis;
    g->key_begin = score_mode == METOK_SCORE_VISUAL_ONLY ? vis_start : 0;
    g->key_end = score_mode == METOK_SCORE_VISUAL_ONLY ? static_cast<int64_t>(vis_start) + n_vis : S;
    g->scale_log2 = static_cast<float>(1.4426950408889634 / sqrt(static_cast<double>(dh)));
    return true;
}

struct ScorePlan {
    int nx1, nx2;                   // workgroups along the keys in pass 1 / pass 2
    int per1, per2;                 // 32-key subtiles per workgroup
    size_t off_qfrag, off_pstat, off_norm, off_colpart, off_sel, off_inplace, total;
};

// One 512-thread workgroup per CU: what the registers and LDS of the two-block kernels allow.  Two of the one-block ones
// (about 100 VGPRs, at most 64 KB) would fit; their grids were not tuned for that.
constexpr int kScoreSlots = 256;

inline void plan_grid(const ScoreGeom& g, int n_vis, int nch, int batch, size_t sel_bytes, ScorePlan* p) {
    const int ny = g.Hkv * g.rs;
    const int64_t rows_of_grid = static_cast<int64_t>(ny) * batch;          // the videos of a batch share the chip's slots
    const int nx0 = kScoreSlots / rows_of_grid < 1 ? 1 : static_cast<int>(kScoreSlots / rows_of_grid);
    auto pick = [&](int64_t subtiles, int* per) {
        int64_t nx = nx0 < subtiles ? nx0 : subtiles;
        if (nx < 1) nx = 1;
        *per = static_cast<int>((subtiles + nx - 1) / nx);
        if (*per < 1) *per = 1;
        nx = (subtiles + *per - 1) / *per;                  // smallest grid with the same critical path
        return static_cast<int>(nx < 1 ? 1 : nx);
    };
    p->nx1 = pick((g.key_end - g.key_begin + 31) / 32, &p->per1);
    p->nx2 = pick((static_cast<int64_t>(n_vis) + 31) / 32, &p->per2);
    // the partial statistics are sized for the widest pass-1 grid of either score mode, so one
    // workspace query serves both
    int64_t nx1_cap = nx0;
    const int64_t sub_all = (g.S + 31) / 32;
    if (nx1_cap > sub_all) nx1_cap = sub_all;
    size_t off = 0;
    p->off_qfrag = off;   off += static_cast<size_t>(g.Hkv) * g.rb_total * nch * 1024;
    p->off_pstat = off;   off += round_up_256(static_cast<size_t>(ny) * nx1_cap * g.rbw * 32 * 2 * sizeof(float));
    p->off_norm = off;    off += round_up_256(static_cast<size_t>(ny) * g.rbw * 32 * sizeof(float));
    p->off_colpart = off; off += round_up_256(static_cast<size_t>(ny) * n_vis * sizeof(float));
    p->off_sel = off;     off += sel_bytes;
    p->off_inplace = off; off += inplace_bytes(g.S);
    p->total = round_up_256(off);
}

// Up to here every workgroup of pass 2 merges the partial statistics of its rows for itself, above a kernel in between does it once.
// Levels, kernels alone, us, by the kernel / merged in pass 2: 28 heads on 4 x 30 queries, 224 rows x 53 to 61 partials (95 to 109 KB),
// 5000 tokens 28.8 / 27.3, 36864 64.1 / 62.5; 14 on 2 x 32 of 64 elements, 224 x 79 to 116 (138 to 203 KB), 5000 in fp32 31.6 / 30.4,
// 18432 36.7 / 35.4; 28 on 4 x 64, 448 x 58 (203 KB), 18432 54.7 / 53.4; 8 on 2 x 64 of 256, 256 x 128 (256 KB), 36864 64.4 / 62.3;
// beyond the line, 14 on 2 x 64 of 64, 448 x 116 (406 KB), 36864 56.5 / 57.6, in fp32 123.2 / 125.4.
constexpr size_t kMergeInPass2Bytes = 256 * 1024;
inline size_t partial_bytes(const ScoreGeom& g, const ScorePlan& p) { return static_cast<size_t>(p.nx1) * g.rbw * 32 * 2 * sizeof(float); }

// More than eight row blocks go two to a wave, which lets a key fragment feed two products and reads the keys once.  On short
// ranges the fixed part of a workgroup (its queries, the merge of all its rows' partial statistics, the first stage) is what takes
// the time, and half the rows in each of twice as many workgroups make it shorter: up to kSplitSubtiles subtiles a workgroup the
// rows are split until every wave has one block, up to kSplitSubtilesMerged where the whole rows' partials are more than
// kSplitMergedBytes.  One level of 28 heads on 4 x 64 queries, us whole / split: 300 tokens 26.5 / 24.1, 2243 (2 subtiles) 32.7 / 28.9, 6000
// 40.6 / 36.7, 9000 (5) 47.4 / 44.4, 15000 (8) 62.6 / 60.7, 18432 (10) 63.0 / 64.2; two videos of 4000 41.2 / 39.5, eight of 1000
// (5) 45.5 / 42.6, four of 3000 (6, merged in pass 2) 49.5 / 50.1; 14 heads on 2 x 64, 8000 tokens 34.3 / 30.8.
// Two blocks on one wave and their halves on two are the same work only where nothing is rounded: 9 to 12 blocks are three to a SIMD
// whole and two split, and half as many workgroups along the keys may be fewer than half.  What the split adds to the busiest SIMD, in
// products of a row block and a subtile over both passes, must stay below what it saves.  Levels (kernels alone) with 0 to 2 products
// more are 0.87 to 0.97 of the whole rows' time in every type; in bf16 those with 10 more are 0.96 to 0.99, with 12 0.94 to 1.05, with 16
// 1.02 to 1.07; in fp32 (both sides with fp32 MFMA, four times as long a product; split rows are now multiplied in parts), those with 4
// more are 0.97 to 1.04, with 10 1.09 to 1.16, with 24 1.26 to 1.39 (40 heads x 352 queries, 2 x 400 tokens, 64 elements: 57.9 / 80.5
// us).
// A split needs more room for the column sums and none for the two words per token that select_bytes reserves for nobody; where
// it does not fit the workspace of the whole rows, the rows stay whole.
constexpr int kSplitSubtiles = 5, kSplitSubtilesMerged = 8;
constexpr size_t kSplitMergedBytes = 64 * 1024;
constexpr int kSplitMoreBf16 = 10, kSplitMoreF32 = 3;
// Row blocks on the busiest SIMD of a workgroup: waves 0 and 4 share one.
inline int blocks_of_busiest_simd(const ScoreGeom& g) {
    auto blocks = [&](int wave) { return (g.rbw + kScoreWaves - 1 - wave) / kScoreWaves; };
    return blocks(0) + blocks(kScoreWaves / 2);
}
inline void plan_score(ScoreGeom* g, int n_vis, int dtype, int batch, ScorePlan* p) {
    const int nch = chunk_count(g->dh, dtype);
    plan_grid(*g, n_vis, nch, batch, select_bytes(n_vis), p);
    if (g->rbw <= kScoreWaves || p->per1 > (partial_bytes(*g, *p) > kSplitMergedBytes ? kSplitSubtilesMerged : kSplitSubtiles)) return;
    ScoreGeom split = *g;
    split.rs = (g->rb_total + kScoreWaves - 1) / kScoreWaves;
    split.rbw = (g->rb_total + split.rs - 1) / split.rs;
    if (static_cast<int64_t>(split.Hkv) * split.rs > 65535) return;
    ScorePlan s;
    plan_grid(split, n_vis, nch, batch, round_up_256(select_general_bytes(n_vis) + sizeof(FastSel)), &s);
    const int64_t more = static_cast<int64_t>(blocks_of_busiest_simd(split)) * (s.per1 + s.per2) - static_cast<int64_t>(blocks_of_busiest_simd(*g)) * (p->per1 + p->per2);
    if (s.total > p->total || more > (dtype == METOK_BF16 ? kSplitMoreBf16 : kSplitMoreF32)) return;
    s.total = p->total;
    *g = split; *p = s;
}

}  // namespace metok
