// Launch-plan blob shared by the host planner (plan.cpp) and the gfx950
// kernels (attn_fwd.hip). The blob is position independent: every array is
// addressed by a byte offset from the start of the blob, so the same bytes
// work in host memory and, after a plain copy, in device memory.
#pragma once

#include <stdint.h>

namespace sangam {

constexpr uint32_t kPlanMagic = 0x50414753u;  // "SGAP"
constexpr uint32_t kPlanVersion = 4;  // 4: prefill_rows may be the wide tile (256)

constexpr int kWaveRows = 32;       // query rows held by one wave (one decode block)
constexpr int kPrefillQWaves = 4;   // waves of a prefill-shaped work-group
constexpr int kPrefillQBlocks = 1;  // 32-row query blocks per prefill wave
constexpr int kPrefillRows = kWaveRows * kPrefillQBlocks * kPrefillQWaves;
// Wide prefill-shaped work-groups (head_dim 128, batches whose prefill
// launch holds no fused block decodes and only long prefill-shaped items):
// eight waves of 32 rows of one query head, 128-key stages, one work-group
// per CU; half the barriers per key of the four-wave tile.
constexpr int kWidePrefillQWaves = 8;
constexpr int kWidePrefillRows = kWaveRows * kWidePrefillQWaves;
constexpr int kWidePrefillMinRows = 1024;  // every prefill-shaped item at least this long
constexpr int kKeyAlign = 64;       // split boundaries are multiples of this many keys
constexpr int kForcedSplitLen = 8192;  // a decode context longer than this is always split
// Longest context range of one tile that reads cached (paged) rows.
constexpr int kMaxCachedRange = 8192;

// One work item of the batch (a block decode or a whole prefill).
struct ItemRec {
    int32_t q_start;     // first packed query row
    int32_t n;           // query rows
    int32_t o;           // position of the first query row (block offset)
    int32_t L;           // context length
    int32_t page_start;  // first entry of the item in page_ids
    int32_t num_splits;  // context chunks (1 = written straight to out)
    int32_t split_len;   // keys per chunk (multiple of kKeyAlign), last may be shorter
    int32_t merge_base;  // first merge row of the item, -1 when not split
    int64_t ws_o;        // float offset of num_splits x n x Hq x D floats of partial O
    int64_t ws_lse;      // float offset of num_splits x n x Hq partial LSE; merge_marks follow
    int32_t flags;       // kItemPosList or 0
    int32_t pos_start;   // first entry of the item's positions (kItemPosList)
};

// ItemRec.flags: the rows sit at the listed positions (positions[pos_start +
// r]), not at o + r; page_info[page_start + k] describes the item's page k.
constexpr int32_t kItemPosList = 1;

// page_info entry of a page of a kItemPosList item: bit s (s < 16) is set when
// slot s holds a listed position; bits 16..31 count the listed positions on
// the item's earlier pages, so the fresh row of slot s is that count plus the
// set bits below s.
constexpr int kPageInfoRowShift = 16;

// TileRec.flags: the waves of a prefill-shaped work-group hold consecutive
// query heads (q_head0 + wave, those inside the tile's GQA group) of one
// block decode instead of consecutive 32-row blocks of one head.
constexpr int32_t kTileHeadsAcross = 1;

// One work-group of an attention launch.
struct TileRec {
    int32_t item;
    int32_t kv_head;
    int32_t q_head0;   // first query head of the tile
    int32_t row0;      // first query row (local to the item)
    int32_t kv_begin;  // context range [kv_begin, kv_end)
    int32_t kv_end;
    int32_t split;     // chunk index of the context
    int32_t flags;     // kTileHeadsAcross or 0
};

// One (item, row) whose split partial results the merge kernel combines.
struct MergeRow {
    int32_t item;
    int32_t row;
};

struct PlanHeader {
    uint32_t magic;
    uint32_t version;
    uint64_t total_bytes;

    int32_t num_items;
    int32_t hq;
    int32_t hkv;
    int32_t d;
    int32_t group;      // hq / hkv
    int32_t page_size;
    float sm_scale;
    float scale_log2;   // sm_scale * log2(e): scores enter exp2 in this scale
    int64_t num_pool_pages;
    int64_t total_q;
    int64_t total_pages;

    // decode-shaped launch: items with n <= kWaveRows; one work-group holds
    // decode_qw query heads (one per wave) x decode_kw context sub-ranges
    int32_t n_decode_tiles;
    int32_t decode_qw;
    int32_t decode_kw;
    int32_t decode_nb;   // 32-key blocks per wave per stage
    // prefill-shaped launch: items with n > kWaveRows; kPrefillQWaves waves
    // of 32 rows of one query head. In a batch that holds prefills (or a
    // small decode-only batch), block decodes whose GQA group spans at least
    // kPrefillQWaves query heads run in this launch too (kTileHeadsAcross
    // tiles, n_fused_decode_tiles of n_prefill_tiles), filling its tail
    // instead of a launch of their own.
    int32_t n_prefill_tiles;
    int32_t prefill_nb;
    int32_t n_merge_rows;
    int32_t num_split_items;
    int32_t max_splits;
    int32_t prefill_rows;  // query rows per prefill-shaped tile: kPrefillRows or kWidePrefillRows
    int32_t n_fused_decode_tiles;
    int32_t mark_bytes;  // of the workspace: merge marks (0: none, merge_kernel merges)
    int64_t workspace_bytes;

    uint64_t off_items;
    uint64_t off_decode_tiles;
    uint64_t off_prefill_tiles;
    uint64_t off_merge;
    uint64_t off_positions;  // int32 positions of kItemPosList items
    uint64_t off_page_info;  // uint32 per page (page_indptr order), when any item is kItemPosList

    int32_t separate;  // 1: a launch for each kind of tile, also where one could hold both
    int32_t cus;       // compute units the plan is for (0: 256)
};

// Whether one launch holds the prefill-shaped tiles and the block decodes
// (attn_mixed_kernel): the shapes it has code for, blocks that count as int32,
// and a plan that does not ask for a launch of each kind. Those refuse the
// shapes that they have no kernel for.
inline bool one_launch(const PlanHeader& h) {
    return h.n_prefill_tiles > 0 && h.n_decode_tiles > 0 && h.decode_qw == 1 && h.decode_kw == 2 && h.decode_nb == 1 &&
           (h.prefill_rows == kPrefillRows || (h.prefill_rows == kWidePrefillRows && h.d == 128)) && !h.separate &&
           int64_t(h.n_prefill_tiles) + h.n_decode_tiles < INT32_MAX / 4;
}

// Whether split contexts are merged in a launch; else the tiles do it.
inline bool merge_launch(const PlanHeader& h) { return h.n_merge_rows > 0 && h.mark_bytes <= 0; }

// Split partials that the allocation-free forward holds.
constexpr size_t kScratchBytes = size_t(32) << 20;

// Merge marks of a split item: per 32-row block, query head and split one
// uint64 (a tile uses those of its first block and head), after the item's
// partial LSE in the workspace. Float offset, and their number of floats.
#ifdef __HIPCC__
__host__ __device__
#endif
inline int64_t merge_marks(const ItemRec& it, int hq) {
    return it.ws_lse + (int64_t(it.num_splits) * it.n * hq + 63) / 64 * 64;
}
inline int64_t merge_mark_floats(const ItemRec& it, int hq) {
    return (int64_t(it.n + kWaveRows - 1) / kWaveRows * hq * it.num_splits * 2 + 63) / 64 * 64;
}

// The tile that finishes last merges an item's S partials, given the query
// waves qw of its tiles, if no item of the plan is above this limit; else the
// plan has no marks and merge_kernel merges all. The tile reads S * qw
// partials of 16 KiB (D = 128) by itself, the launch reads all in parallel but
// costs 4 to 8 us with its gap. Measured, launch -> in the tile: 28/4 heads
// (qw 4) one decode in 8 splits 18.2 -> 17.8 us, 8 decodes in 4 19.8 -> 17.4
// and in 8 29.2 -> 30.3, 4 decodes in 12 27.6 -> 30.3; whole groups (qw 7)
// 24 decodes in 4 70 -> 63; 32/32 heads (qw 1) one decode in 12 22.3 -> 18.4
// and in 16 27.8 -> 22.2. Both ways in one call add up: 4 decodes in 3 to 14
// splits, 32/8 heads of 64, took 19.5 us with all in the launch and 21.7 us
// with the items of up to 7 splits in their tiles.
constexpr int kMaxMergeInTile = 16;
constexpr int kMaxMergePartials = 28;
constexpr int max_merge_in_tile(int qw) {
    return kMaxMergePartials / qw < kMaxMergeInTile ? kMaxMergePartials / qw : kMaxMergeInTile;
}

static_assert(sizeof(ItemRec) == 56, "ItemRec layout is part of the blob format");
static_assert(sizeof(TileRec) == 32, "TileRec layout is part of the blob format");
static_assert(sizeof(MergeRow) == 8, "MergeRow layout is part of the blob format");
static_assert(sizeof(PlanHeader) == 184, "PlanHeader layout is part of the blob format");

}  // namespace sangam
