// Internal declarations shared by the translation units of libwlb (not installed).
#pragma once
#include <cstdarg>
#include <cstddef>
#include <cstdint>

#include "wlb.h"

namespace wlb {

// Records the text returned by wlb_last_error() on this thread and passes `st` through.
wlb_status fail(wlb_status st, const char* fmt, ...);

constexpr int kGroupRows = 64;    // rows per schedule group (granularity of hull / full-range data)
constexpr int kFwdTileRows = 128; // query rows per forward / dQ work item
constexpr int kBwdKeyTile = 128;  // keys per dK/dV work item

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr int kLists = 8;         // XCDs: workgroup b runs on XCD b % 8
// Short-hull path of the forward and dQ kernels: a block of 32 rows whose visible keys, counted from
// the 32-key boundary at or below the first, span at most kShortHullKeys keys is worked on by one
// workgroup that holds those K/V rows in LDS for all query heads of the KV head.  A query tile
// takes this path when each of its four blocks qualifies.
constexpr int kShortBlockRows = 32;
constexpr int kShortHullKeys = 96;
// A dK/dV item is at most 1/kDkvSplit of the mean load of a compute unit, or kDkvMinItemStages stages where that is more: items
// this short are never split further.  Each split costs an item more to start and two partial results that are written and
// summed, so the items are coarse (kDkvCoarseSplit, kDkvCoarseStages) where the longest ones still leave the compute units
// evenly loaded: for q = 1 .. kDkvBalance at most q - 1 per compute unit are longer than 1/q of 17/16 of its mean load and
// kDkvCoarseSlack stages (what the partial results of one cost).  Only from one (key tile, KV head) per compute unit on: below
// that the splits are what fills the chip.  Fine and coarse, dK/dV: 32K tokens in documents of 8K - 32K, 32/8 heads 2245 and
// 2139 us; one of four ranks of 16K, 16/4 heads, 159 and 144; 13860 in documents of 64 - 1536, 16/4 heads, 183 and 149; and where
// the rule stays with fine items: one of eight ranks of 128K, 8/1 heads, 5456 and 5652 us, with head dimension 64 3534 and 3785;
// one document of 13719, 8/1 heads, 514 and 541.  Of 196 random calls three are more than 2 % slower than with fine items (3.5
// at most), 50 more than 2 % faster (up to 18); without the slack 43.
constexpr int kDkvSplit = 6, kDkvMinItemStages = 32;
constexpr int kDkvCoarseSplit = 2, kDkvCoarseStages = 64, kDkvCoarseSlack = 16, kDkvBalance = 8;
// workgroups per cut query tile and head in the merge kernels, and per key tile and KV head in the dK/dV fix-up (rows
// split evenly); the gangs' merges, where finding a tile's parts costs more than summing them, take fewer
constexpr int kMergeSplit = 8, kGangMergeSplit = 4;

// The public layout and the tables only the library's own kernels read.
struct PlanLayout : wlb_plan_layout {
    size_t off_key_span;       // int32 [n_key_tiles]: groups in the key tile's range
    size_t off_tile_first;     // int32 [n_fwd_tiles]: first 64-key tile the query tile visits
    // Work records of the one-workgroup-per-item launches: {query tile, first, one-past-last 64-key tile, code}, code = -1:
    // a whole tile, -2: a whole short-hull tile, else 2 * partial slot + (1: not the tile's first part)
    size_t off_row_item;       // int32 [n_fwd_tiles][4], by order rank: whole tiles only
    size_t off_row_part;       // int32 [n_fwd_tiles + row_parts_added(..)][4]: heavy tiles divided into parts (row_part_limit), longest part first, a tile's parts in turn
    size_t off_row_part_base;  // int32 [n_fwd_tiles + 1][4]: of the tile of order rank r {first record, records, first partial result, 0}; last: {records in all}
    size_t off_short_on;       // int32: 1: dkv_short_kernel does dK/dV, 0: the general kernel
    // Last, because a forward's schedule (wlb_attn_fwd_static) leaves them out.
    size_t off_dkv_item;       // int32 [dkv_max_items][8], by item: {key tile, KV head, first query head, query heads, partial slot or -1,
                               // first row group, stages, 0}
    size_t off_key_steps;      // int32 [n_key_tiles]: row blocks that see 32 keys of a tile of a short span: most | all four sums << 8
    size_t static_bytes;       // bytes counted against WLB_ATTN_FWD_STATIC_SCRATCH_BYTES
};

// compute units of the GPU (256 when none is present: layout queries on the host)
int compute_units();
// Forward and dQ run as a fixed set of workgroups, two per compute unit, in gangs of the
// G = hq / hkv query heads that share a KV head (a gang's workgroups sit on one XCD and walk the
// same K/V tiles side by side).  Number of gangs:
inline int row_gangs(int hq, int hkv, int cus) {
    const int per_xcd = (2 * cus / kLists) / (hq / hkv);
    return kLists * (per_xcd > 0 ? per_xcd : 1);
}
// Division of heavy query tiles along their keys, for launches with few items: a part holds at most kRowPartMean / 4
// of the mean work of a workgroup slot (4 / 4, 6 / 4, 8 / 4 measured at 4095 rows, 16 heads: forward + dQ 218, 203 and
// 229 us; undivided 247) and at most kRowPartMin key tiles where that is less (4 - 12: within 1 us at 2052 rows).
constexpr int kRowPartMin = 6, kRowPartMean = 6;
// None is divided unless the heaviest has kRowPartHeavy / 10 of the mean work of a compute unit: below that the launch is
// balanced as it is, heavy tiles beside light ones (one of two ranks of a 3808-token document, 32 heads: forward 80 us whole,
// 98 divided; 26624 tokens in documents of 3396, one of four ranks, 8 heads: 88 and 114).
constexpr int kRowPartHeavy = 11;
bool use_row_parts(const wlb_attn_desc& d, const PlanLayout& L);
// upper bound of the parts that divided tiles add (each is at least a slot's mean work), and of the number of divided tiles
inline int row_parts_added(const wlb_attn_desc& d, const PlanLayout& L) { return L.row_gangs * (d.hq / d.hkv) / d.hq; }
inline int row_tiles_divided(const wlb_attn_desc& d, const PlanLayout& L) {
    const int most = row_parts_added(d, L) * 4 / kRowPartMean;
    return most < L.n_fwd_tiles ? most : L.n_fwd_tiles;
}
// positions of a one-workgroup-per-item launch whose workgroups fill the compute units once (see paired_index); 0: a position's
// workgroups, one per query head, fill more than the compute units of an XCD
inline int row_first_half(const wlb_attn_desc& d) { return d.hq * kLists <= compute_units() ? compute_units() / d.hq : 0; }
// fixed cost of a query tile (loading Q, the first copies, the output) in units of one key tile's work
constexpr int kRowItemOverhead = 6;
// Default relative work share (percent) of a gang of the first half of a launch; a gang of the second half
// gets the rest.  Set from the gangs' recorded end times (wlb_plan_layout: off_gang_clock): with these shares
// the two halves end together on average.  What remains is a spread between the XCDs of a GPU (one XCD's
// gangs end several percent later than another's, the same ones in every launch), which differs from GPU to
// GPU: wlb_attn_set_gang_weights takes weights measured on the GPU at hand.
constexpr int kRowShareFirstFwd = 57, kRowShareFirstDq = 57;
// the weights in force for kernel 0 (forward) / 1 (dQ): [half of the launch][XCD]
void gang_weights(int kernel, int out[2][8]);
// Which of the two forward / dQ schedules a launch uses: gangs with fixed shares when there are fewer
// than kRowGangMaxItemsPerSlot (query tile, head) items per workgroup slot and an estimated
// kRowGangMinUnitsPerSlot key tiles of work per slot, else one workgroup per item.  The
// WLB_ATTN_SCHEDULE_* flags override.
constexpr int kRowGangMaxItemsPerSlot = 3;
constexpr int kRowGangMinUnitsPerSlot = 64;
// Query tiles are divided into parts (use_row_parts) when the items hold this many units on average: the launch that merges
// the parts takes 5 us, which at 18 units per item (8191 tokens, 8 heads: forward 43 us) is more than the better balance
// returns (47 us), at 39 (4095 rows of a 16K-token micro-batch, 16 heads) a third of it (106 -> 89 us).  Or when they fill at
// most a quarter of the workgroup slots, if the heaviest tile probably sees more than kRowPartKeys keys: twice what its rows
// see on average (a document's length, weighted by tokens) and kRowPartReach for the 128 rows' own share of the sequence (a
// tile's rows lie in several documents and, context-parallel, in distant places).  With less there is
// little or nothing to divide, and the merge launch alone costs 1.4 us (1024 tokens in documents of 1 - 64, 8/2 heads:
// forward 7.4 -> 8.8; of 64 - 384: 16.1 -> 17.5).  Of 887 random calls, forward and dQ: these leave 8 slower by more than
// 3 % and 0.5 us than undivided ones, dividing always 220; the mean time is 0.822 of the undivided one, 0.843 dividing always.
constexpr int kRowPartKeys = 704, kRowPartReach = 224;
constexpr int kRowPartMeanUnits = 24;
bool use_row_gangs(const wlb_attn_desc& d, const PlanLayout& L);
// Whether forward and dQ take two query heads to a workgroup, one workgroup to a compute unit (wlb_attn_fwd_pair.hip, wlb_attn_dq_pair.hip).  Their
// loops are faster (3 - 11 %), but nothing runs beside the start and the end of an item, so items must be long: head dimension 128, at
// least as many items as keep gangs away, and kRowPairMinItemUnits on average (forward, old / new at 34 - 73 units 1.02 - 1.07, at 20 - 26 0.99 - 1.05,
// at 13 0.88 - 1.0; at head dimension 64 0.80 - 0.93 up to 58 units; dQ at 33 - 58 units 1.025 - 1.08, at 20 - 26 0.98 - 1.08, at 13
// 0.92 - 0.98).  Or shares of kRowPairMinUnitsPerSlot units in a gang launch: a share's fixed part and the rows of short documents weigh more than in
// launches of two workgroups (documents that are long alone, 1024 - 1860 units: forward 1.09 - 1.12, at head dimension 64 0.99 - 1.035, dQ 1.095 - 1.12;
// 650: forward 0.96 - 0.995, dQ 0.93 - 0.98; 70 - 300: 0.73 - 0.99 and 0.85 - 0.99).
// There the rows of short documents must be few as well: their tiles are masked block after block, each with new maxima, which takes twice as long a
// unit (the mask and the rescaling of 64 rows at once), and being the lightest they come last, all in the last gangs.  One of 8 ranks of 131072 tokens, 8/1 heads,
// one long document and short ones, old / new of the forward (at D = 64) and of dQ: short ones of 1 - 64 tokens, 30 % of all: 0.64 (0.64), 0.81; 18 %: 0.82
// (0.81), 0.96; 8.5 %: 0.99 (0.92), 1.09; 3 %: 1.11 (0.99), 1.11; of 64 - 256, 30 %: 0.81 (0.78), 0.87; 18 %: 0.95 (0.88), 1.01; of 64 - 1536, 30 %: 0.95 (0.89), 1.0;
// 18 %: 1.04 (0.95), 1.07, and with 8/2 heads 0.95 (0.89), 0.955; of 500 - 4000, 30 %: 1.04 (0.97), 1.055.  So short_rows has a limit: at head dimension 128
// kRowPairShortRows with eight heads or more to a KV head (above it 0.81 - 0.99 of the whole pass, below it 1.01 - 1.075), kRowPairShortRowsFew with fewer;
// kRowPairShortRows64 at 64 (0.82 - 0.99 and 0.99 - 1.02).
constexpr int kRowPairMinItemUnits = 30, kRowPairMinUnitsPerSlot = 1000;
constexpr double kRowPairShortRows = 0.15, kRowPairShortRowsFew = 0.1, kRowPairShortRows64 = 0.06;
// Share of a rank's rows that probably lie in short documents beside one long: its tokens follow from what rows see on average, the others'
// mean length from the count of documents.  Documents count by how far their chunk on the rank (a rank has two chunks of each) falls short of kShortChunkRows rows.
constexpr int kShortChunkRows = 256;
double short_rows(const wlb_attn_desc& d);
bool use_row_pairs(const wlb_attn_desc& d, const PlanLayout& L);
// dQ as well: at head dimension 64 it is no faster (2546 us with two heads, 2527 as gangs of one)
inline bool use_dq_pairs(const wlb_attn_desc& d, const PlanLayout& L) { return use_row_pairs(d, L) && d.head_dim == 128; }
// share weights of its gangs: with one workgroup to a compute unit no half of the launch is slower than the other
void pair_weights(int (&weight)[2][8]);
// whether this launch sends short-hull query tiles to the short-hull kernels (only in the
// one-workgroup-per-item schedule; WLB_ATTN_NO_SHORT_PATH switches it off)
bool use_short_path(const wlb_attn_desc& d, const PlanLayout& L);
// Whether forward and dQ of the tiles that are not short-hull ones run as units that hold the keys of a block of rows in LDS for all heads
// (wlb_attn_span.hip): the ranks divide documents so that a block of 32 rows spans kSpanMinReach tokens (61, one of two ranks, measured
// 0.84 - 1.08 of the whole pass when short-hull tiles had a launch of their own), documents (2 * pairs / rows: the pair
// count has to be known) are of kSpanMaxLength tokens (old / new of forward and dQ alone at 45 - 207: 1.05 - 2.0), there are four heads or more to a KV head
// (three, which leave two of eight wavefronts idle, 36448 tokens on one of 4 ranks: 0.85 - 0.96; one: 0.4 - 0.9), and a unit's keys fit two windows or units are enough to fill half of the compute units (4 heads to a KV head, one of 8 ranks
// of 4096 tokens in documents of 1 - 160, 20 units: 0.82 - 0.95; of 32768, 158 units: 1.3).
// And no document is so long that its units, which walk its keys one window after another (0.042 us a token at head dimension 128, 0.03 at 64), end after
// the launch they replace (20 us and 0.11 us per 32 rows and 8 heads): long_tokens is at most kSpanLongBase + kSpanLongPerBlock for each of those.
// Whole pass, old / new, documents of 1 - 64 tokens and one of n: below that line (n = 1400 - 5000 of 32768 - 131072, 16/2 and 16/4 heads) 0.95 - 1.24,
// above it (n = 1200 - 5000 of 8192 - 131072) 0.67 - 1.02.
constexpr int kSpanMinReach = 96, kSpanMaxLength = 256, kSpanMaxKeys = 384, kSpanMinHeads = 4;
constexpr double kSpanLongBase = 285, kSpanLongPerBlock = 2.5;
bool use_span(const wlb_attn_desc& d, const PlanLayout& L);
// Tokens of the documents that are far longer than the others, if there are any: weighted by tokens, documents are 2 * pairs / rows long; lengths that
// are spread evenly from 1 on make that 4/3 of their mean, and what goes beyond is taken for one long document beside short ones.
double long_tokens(const wlb_attn_desc& d);
// workgroups of a launch for short-hull tiles alone (for_short_tiles): it may find none
inline unsigned short_tiles_grid(const wlb_attn_desc& d, const PlanLayout& L) {
    const int units = L.n_fwd_tiles * d.hkv * (kFwdTileRows / kShortBlockRows), most = 2 * compute_units();
    return (unsigned)(units < most ? units : most);
}
// floats of one partial result of a query tile and head: 128 x D accumulator, then 128 row sums and
// 128 reference exponents
inline size_t row_partial_floats(int head_dim) { return (size_t)kFwdTileRows * head_dim + 2 * kFwdTileRows; }
// bytes of the partial results of the query tiles that are cut at a gang boundary: two per gang and member
size_t row_partial_bytes(const wlb_attn_desc& d, const PlanLayout& L);
// dkv_short_kernel does dK/dV where no key tile is seen by more than this many 64-row groups (documents of 16 - 128 tokens:
// 121 us with 4, 119 with 6, 171 with 2, 149 with the general kernel).
constexpr int kShortSpan = 4;
// It is launched, beside the general kernel, when documents average at most kShortMeanDoc tokens and a tile of 128 keys and
// the longest documents that shape the work (2 * pairs / rows, where the pair count is known) are seen by about
// kShortSpan groups: an empty launch costs 1.5 us of a backward that may take 30.
constexpr int kShortMeanDoc = 96, kShortReach = 224;      // kShortReach = 64 * (kShortSpan - 1/2)
bool short_documents(const wlb_attn_desc& d);
bool use_short_keys(const wlb_attn_desc& d, const PlanLayout& L);
// Which of the two then does the work the schedule decides (short_keys_pay), from estimates in stages of the general kernel
// (1.2 us at D = 64, 1.7 at 128) that were fitted to 1542 random calls: the general kernel takes kGeneralStart and its longest
// item or kGeneralLoad of the mean load of a compute unit (all of them copying at once), the short one kShortStart and, at
// kShortStep.. a step, its longest wavefront or kShortLoad of a compute unit's steps.  Of 678 other random calls 24 run more
// than 3 % slower than before there was a short kernel, most by an empty launch (2 - 3 us), one by a wrong choice (49 -> 57);
// always taking the short kernel for tiles of a short span beside the general one for the others was slower in a third of
// them, by up to a factor of five.
constexpr float kGeneralStart = 18.f, kGeneralLoad = 1.45f, kEmptyLaunch = 2.f, kFixup = 2.f;
constexpr float kShortStart = 7.f, kShortStep64 = 1.0f, kShortStep128 = 1.3f, kShortLoad = 0.25f;
// bytes of the dK/dV partial results that follow delta / lse2 in the backward workspace
size_t dkv_partial_bytes(const wlb_attn_desc& d, const PlanLayout& L);

// Validates desc; on success fills the plan layout.
wlb_status check_desc(const wlb_attn_desc* d);
void plan_layout(const wlb_attn_desc& d, PlanLayout* L);

// Device-side launchers (defined in the .hip files); all asynchronous on `stream`.
wlb_status launch_plan(const wlb_attn_desc& d, const PlanLayout& L, const int32_t* q_idx,
                       const int32_t* cu_seqlens_k, char* ws, bool forward_only, void* stream);
wlb_status launch_fwd(const wlb_attn_desc& d, const PlanLayout& L, const void* q, const void* k,
                      const void* v, void* o, float* lse, char* ws, size_t off_row_partial, void* stream);
wlb_status launch_bwd(const wlb_attn_desc& d, const PlanLayout& L, const void* q, const void* k,
                      const void* v, const void* o, const float* lse, const void* d_o, void* dq,
                      void* dk, void* dv, char* ws, size_t off_delta, void* stream);

}  // namespace wlb
