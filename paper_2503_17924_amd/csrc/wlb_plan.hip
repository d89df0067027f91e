// Attention entry points of libwlb and the device-side tile scheduler.
//
// The scheduler turns (q_idx, cu_seqlens_k) into the integer tables the attention kernels
// read: for every local row the interval [lo, hi) of keys it may see (its document's start up
// to and including itself: causal inside the document, nothing outside -- paper Sections 1 and
// 3.2); for every group of 64 consecutive rows the hull of those intervals and the range every
// real row of the group sees in full; and two work lists ordered heaviest first -- query tiles
// (forward and dQ) and key tiles (dK/dV).  Kernels visit only key tiles inside a hull and
// apply the per-element mask only outside the fully visible range, which is how tiles that lie
// wholly in other documents cost nothing (the tile-level waste described in Section 5.2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "wlb_device.h"
#include "wlb_internal.h"

namespace wlb {

wlb_status check_desc(const wlb_attn_desc* d) {
    if (!d) return fail(WLB_ERR_INVALID_ARG, "attention: null desc");
    if (d->n_q < 1 || d->t_kv < 1 || d->n_docs < 1 || d->hq < 1 || d->hkv < 1)
        return fail(WLB_ERR_INVALID_ARG, "attention: n_q=%d t_kv=%d n_docs=%d hq=%d hkv=%d", d->n_q, d->t_kv,
                    d->n_docs, d->hq, d->hkv);
    if (d->hq % d->hkv != 0) return fail(WLB_ERR_INVALID_ARG, "attention: hq=%d not a multiple of hkv=%d", d->hq, d->hkv);
    if (d->visible_pairs < 0) return fail(WLB_ERR_INVALID_ARG, "attention: visible_pairs=%lld", (long long)d->visible_pairs);
    if ((d->flags & WLB_ATTN_SCHEDULE_GANGS) && (d->flags & WLB_ATTN_SCHEDULE_ITEMS))
        return fail(WLB_ERR_INVALID_ARG, "attention: both schedule flags set");
    if (!(d->scale > 0.0f) || !std::isfinite(d->scale)) return fail(WLB_ERR_INVALID_ARG, "attention: scale must be finite and > 0");
    if (d->head_dim != 64 && d->head_dim != 128)
        return fail(WLB_ERR_UNSUPPORTED, "attention: head_dim=%d (64 and 128 are built)", d->head_dim);
    const int64_t qe = (int64_t)d->n_q * d->hq * d->head_dim, ke = (int64_t)d->t_kv * d->hkv * d->head_dim;
    // tensors are addressed through 32-bit buffer descriptors: each must stay under 4 GiB, with
    // room for the offsets of the rows a last, partly filled tile would have past the end
    const int64_t q_margin = 2LL * kBwdKeyTile * d->hq * d->head_dim, k_margin = 2LL * kBwdKeyTile * d->hkv * d->head_dim;
    if (qe * 2 + q_margin >= (1LL << 32) || ke * 2 + k_margin >= (1LL << 32))
        return fail(WLB_ERR_UNSUPPORTED, "attention: a tensor of 4 GiB or more is not supported");
    if (d->flags & ~(WLB_ATTN_REUSE_PLAN | WLB_ATTN_BWD_SKIP_DELTA | WLB_ATTN_BWD_SKIP_DQ | WLB_ATTN_BWD_SKIP_DKV | WLB_ATTN_SCHEDULE_GANGS | WLB_ATTN_SCHEDULE_ITEMS | WLB_ATTN_NO_SHORT_PATH)) return fail(WLB_ERR_INVALID_ARG, "attention: unknown flag bits 0x%x", d->flags);
    return WLB_OK;
}

int compute_units() {
    static int cached = 0;          // the library runs on one kind of GPU per process
    if (cached == 0) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
        cached = cus;
    }
    return cached;
}

size_t dkv_partial_bytes(const wlb_attn_desc& d, const PlanLayout& L) {
    // one fp32 dK^T and dV^T tile per partial result
    return (size_t)L.dkv_max_partials * (2 * (size_t)kBwdKeyTile * d.head_dim * sizeof(float));
}

// Units (key tiles and the fixed cost) of an item, on average: from the caller's pair count when it gave one (a tile of
// 128 rows x 64 keys holds 8192 pairs), else from the mean document length (a tile sees about half its document:
// length / 128 key tiles), since the host does not see the mask.
static long long mean_item_units(const wlb_attn_desc& d, const PlanLayout& L) {
    return (d.visible_pairs > 0 ? d.visible_pairs / ((long long)L.n_fwd_tiles * kFwdTileRows * 64)
                                : (long long)(d.t_kv / d.n_docs / (2 * 64))) + kRowItemOverhead;
}

bool use_row_gangs(const wlb_attn_desc& d, const PlanLayout& L) {
    if (d.flags & WLB_ATTN_SCHEDULE_GANGS) return true;
    if (d.flags & WLB_ATTN_SCHEDULE_ITEMS) return false;
    const long long items = (long long)L.n_fwd_tiles * d.hq, slots = 2LL * compute_units();
    if (items >= (long long)kRowGangMaxItemsPerSlot * slots) return false;
    // and only when a slot's share is worth cutting tiles for
    return items * mean_item_units(d, L) >= (long long)kRowGangMinUnitsPerSlot * slots;
}

double short_rows(const wlb_attn_desc& d) {
    if (d.visible_pairs <= 0) return 0;           // documents alike
    const double t = d.t_kv, rest = std::max(0.0, t - std::sqrt(2.0 * (double)d.visible_pairs / d.n_q * t));
    const double chunk = rest / std::max(d.n_docs - 1, 1) * d.n_q / t / 2;
    return rest / t * std::max(0.0, 1 - chunk / kShortChunkRows);
}

bool use_row_pairs(const wlb_attn_desc& d, const PlanLayout& L) {
    if ((d.hq / d.hkv) % 2 != 0) return false;
    const long long items = (long long)L.n_fwd_tiles * d.hq, slots = 2LL * compute_units(), units = mean_item_units(d, L);
    if (use_row_gangs(d, L)) {
        const double most = d.head_dim == 64 ? kRowPairShortRows64 : d.hq / d.hkv >= 8 ? kRowPairShortRows : kRowPairShortRowsFew;
        return items * units >= (long long)kRowPairMinUnitsPerSlot * slots && short_rows(d) <= most;
    }
    return d.head_dim == 128 && items >= (long long)kRowGangMaxItemsPerSlot * slots && units >= kRowPairMinItemUnits;
}

void pair_weights(int (&weight)[2][8]) {
    for (int x = 0; x < 8; ++x) weight[0][x] = weight[1][x] = weight[0][x] + weight[1][x];
}

// Parts of tiles, in launches with few items per slot whose shares are too short for the gangs (kRowPartMeanUnits,
// kRowPartKeys).
bool use_row_parts(const wlb_attn_desc& d, const PlanLayout& L) {
    if ((d.flags & WLB_ATTN_SCHEDULE_ITEMS) || use_row_gangs(d, L) || row_tiles_divided(d, L) < 1) return false;
    const long long items = (long long)L.n_fwd_tiles * d.hq, slots = 2LL * compute_units();
    if (items >= (long long)kRowGangMaxItemsPerSlot * slots) return false;
    if (items * 4 > slots) return mean_item_units(d, L) >= kRowPartMeanUnits;
    const long long length = d.visible_pairs > 0 ? std::min<long long>(2 * (d.visible_pairs / d.n_q), d.t_kv) : d.t_kv / d.n_docs;
    return std::min<long long>(length + (long long)kRowPartReach * d.t_kv / d.n_q, d.t_kv) > kRowPartKeys;
}

// gang share weights: process-wide, set by wlb_attn_set_gang_weights (0 = not set: the defaults)
static int g_gang_weight[2][2][8];
static std::mutex g_gang_weight_mutex;

void gang_weights(int kernel, int out[2][8]) {
    std::lock_guard<std::mutex> lock(g_gang_weight_mutex);
    const int first = kernel == 0 ? kRowShareFirstFwd : kRowShareFirstDq;
    for (int h = 0; h < 2; ++h)
        for (int x = 0; x < 8; ++x)
            out[h][x] = g_gang_weight[kernel][0][0] > 0 ? g_gang_weight[kernel][h][x] : (h == 0 ? first : 100 - first);
}

bool use_short_path(const wlb_attn_desc& d, const PlanLayout& L) {
    return !(d.flags & WLB_ATTN_NO_SHORT_PATH) && !use_row_gangs(d, L);
}

double long_tokens(const wlb_attn_desc& d) {
    const double weighted = 2.0 * (double)d.visible_pairs / d.n_q, mean = (double)d.t_kv / d.n_docs;
    return std::sqrt(std::max(0.0, weighted - mean * 4 / 3) * d.t_kv);
}

bool use_span(const wlb_attn_desc& d, const PlanLayout& L) {
    const int G = d.hq / d.hkv, per = G >= 8 ? 1 : 2;                              // blocks of rows in a unit
    if (!use_short_path(d, L) || d.visible_pairs <= 0 || G < kSpanMinHeads) return false;
    if (long_tokens(d) > kSpanLongBase + kSpanLongPerBlock * L.n_blocks32 * d.hq / 8) return false;
    const long long reach = (long long)kShortBlockRows * d.t_kv / d.n_q, length = 2 * (d.visible_pairs / d.n_q);
    if (reach < kSpanMinReach || length > kSpanMaxLength) return false;
    return per * reach + length <= kSpanMaxKeys || (long long)((L.n_blocks32 + per - 1) / per) * d.hkv >= compute_units() / 2;
}

bool short_documents(const wlb_attn_desc& d) {
    if ((long long)d.n_docs * kShortMeanDoc < d.t_kv) return false;
    const long long length = d.visible_pairs > 0 ? std::min<long long>(2 * (d.visible_pairs / d.n_q), d.t_kv) : d.t_kv / d.n_docs;
    return (kBwdKeyTile + length) * d.n_q <= (long long)kShortReach * d.t_kv;
}
bool use_short_keys(const wlb_attn_desc& d, const PlanLayout& L) { return use_short_path(d, L) && short_documents(d); }

size_t row_partial_bytes(const wlb_attn_desc& d, const PlanLayout& L) {
    return (size_t)2 * L.row_gangs * (d.hq / d.hkv) * row_partial_floats(d.head_dim) * sizeof(float);
}

void plan_layout(const wlb_attn_desc& d, PlanLayout* L) {
    L->group_rows = kGroupRows;
    L->n_groups = (d.n_q + kGroupRows - 1) / kGroupRows;
    L->fwd_tile_rows = kFwdTileRows;
    L->n_fwd_tiles = (d.n_q + kFwdTileRows - 1) / kFwdTileRows;
    L->bwd_key_tile = kBwdKeyTile;
    L->n_key_tiles = (d.t_kv + kBwdKeyTile - 1) / kBwdKeyTile;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    L->off_row_lo = take(sizeof(int32_t) * d.n_q);
    L->off_row_hi = take(sizeof(int32_t) * d.n_q);
    L->off_group = take(sizeof(int32_t) * 4 * L->n_groups);
    L->off_group_real = take(sizeof(int32_t) * L->n_groups);
    L->off_fwd_order = take(sizeof(int32_t) * L->n_fwd_tiles);
    L->off_fwd_cost = take(sizeof(int32_t) * L->n_fwd_tiles);
    L->off_key_order = take(sizeof(int32_t) * L->n_key_tiles);
    L->off_key_range = take(sizeof(int32_t) * 2 * L->n_key_tiles);
    L->off_key_span = take(sizeof(int32_t) * L->n_key_tiles);
    // Items per tile are the smallest power of two that brings an item under 1/kDkvSplit of a compute
    // unit's mean load, so split tiles contribute fewer than 2 * kDkvSplit * CUs items in total.
    L->dkv_max_partials = 2 * kDkvSplit * compute_units();
    L->dkv_max_items = L->n_key_tiles * d.hkv + L->dkv_max_partials;
    L->off_key_ways = take(sizeof(int32_t) * L->n_key_tiles);
    L->off_key_item_base = take(sizeof(int32_t) * (L->n_key_tiles + 1));
    L->off_key_slot_base = take(sizeof(int32_t) * (L->n_key_tiles + 1));
    L->off_dkv_counters = take(sizeof(int32_t) * kLists);
    L->row_gangs = row_gangs(d.hq, d.hkv, compute_units());
    L->uses_gangs = use_row_gangs(d, *L) ? 1 : 0;
    L->off_fwd_prefix = take(sizeof(int64_t) * (L->n_fwd_tiles + 1));
    L->n_blocks32 = L->n_groups * (kGroupRows / kShortBlockRows);
    L->row_kernels = (use_row_pairs(d, *L) ? WLB_ROW_FWD_TWO_HEADS : 0) | (use_dq_pairs(d, *L) ? WLB_ROW_DQ_TWO_HEADS : 0) | (use_span(d, *L) ? WLB_ROW_SPAN : 0);
    L->off_block_hull = take(sizeof(int32_t) * 2 * L->n_blocks32);
    L->off_tile_short = take(sizeof(int32_t) * L->n_fwd_tiles);
    L->off_gang_clock = take(sizeof(uint64_t) * 2 * 2 * (size_t)L->row_gangs * (d.hq / d.hkv));
    L->static_bytes = off;
    L->off_tile_first = take(sizeof(int32_t) * L->n_fwd_tiles);
    L->off_row_item = take(sizeof(int32_t) * 4 * L->n_fwd_tiles);
    L->off_row_part_base = take(sizeof(int32_t) * 4 * (L->n_fwd_tiles + 1));
    L->off_row_part = take(sizeof(int32_t) * 4 * (size_t)(L->n_fwd_tiles + row_parts_added(d, *L)));
    L->off_short_on = take(sizeof(int32_t));
    L->off_dkv_item = take(sizeof(int32_t) * 8 * (size_t)L->dkv_max_items);
    L->off_key_steps = take(sizeof(int32_t) * L->n_key_tiles);
    L->plan_bytes = off;
}

// ------------------------------------------------------------------------------------------
// kernels
// ------------------------------------------------------------------------------------------
// Everything the schedule kernels read and write.
struct PlanArgs {
    const int32_t* q_idx; const int32_t* cu;
    int n_q, t_kv, n_docs, n_groups, n_tiles, n_key_tiles, hq, hkv, n_slots, row_slots, forward_only, parts, short_keys, key_run;
    float short_step, per_cu;
    int32_t* row_lo; int32_t* row_hi; int32_t* group; int32_t* group_real; int32_t* block_hull;
    int32_t* fwd_cost; int32_t* tile_first; int32_t* tile_short; int32_t* fwd_order; int32_t* row_item; int32_t* row_part; int32_t* row_part_base;
    long long* fwd_prefix;
    int32_t* key_range; int32_t* key_span; int32_t* key_ways; int32_t* key_order; int32_t* key_item_base; int32_t* key_slot_base;
    int32_t* dkv_item; int32_t* dkv_counters; int32_t* short_on; int32_t* key_steps;
};
constexpr int kGroupsPerTile = kFwdTileRows / kGroupRows;
// document starts are searched in LDS up to this many documents (a search is log2 dependent loads)
constexpr int kCuLds = 2048;

// The tokens of the rows of the groups g0, g0 + step, ... (requested before the document starts are waited for).
template <int N>
__device__ __forceinline__ void load_tokens(const PlanArgs& a, int g0, int step, int (&tok)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int row = (g0 + i * step) * kGroupRows + (int)(threadIdx.x & 63);
        tok[i] = row < a.n_q ? a.q_idx[row] : -1;
    }
}

// The groups g0, g0 + step, ... (N of them, one wavefront): per-row [lo, hi), the hulls of the two 32-row blocks, the
// group's {k_lo, k_hi, max_lo, min_hi} and its number of real rows.  hull[i] = {k_lo, k_hi, both blocks fit the
// short-hull window}; {kPadLo, 0, 1} for a group without a real row or past the end; block[i]: hull of the lane's block.
// The N groups' searches and reductions are independent chains.
template <int N>
__device__ __forceinline__ void plan_groups(const PlanArgs& a, const int32_t* cu, int g0, int step, const int (&tok)[N], int (&hull)[N][3], int2 (&block)[N]) {
    const int lane = threadIdx.x & 63;
    int d[N] = {}, lo[N], hi[N];
    // last document start <= tok (cu[0] = 0 <= tok); the step count is the same for every row
    for (int s = 1 << (31 - __clz(a.n_docs)); s > 0; s >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int m = d[i] + s;
            if (m < a.n_docs && cu[m] <= tok[i]) d[i] = m;
        }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int g = g0 + i * step, row = g * kGroupRows + lane;
        const bool real = tok[i] >= 0 && tok[i] < a.t_kv;
        lo[i] = real ? cu[d[i]] : kPadLo;
        hi[i] = real ? tok[i] + 1 : 0;
        if (row < a.n_q) { a.row_lo[row] = lo[i]; a.row_hi[row] = hi[i]; }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int g = g0 + i * step;
        const bool real = hi[i] > 0;
        // hull of each half of the wavefront (a block of 32 rows), then of the whole group
        int b_lo = lo[i], b_hi = hi[i];                  // pads carry INT_MAX / 0
        int max_lo = real ? lo[i] : 0, min_hi = real ? hi[i] : kPadLo;
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) {
            b_lo = min(b_lo, __shfl_xor(b_lo, o));
            b_hi = max(b_hi, __shfl_xor(b_hi, o));
            max_lo = max(max_lo, __shfl_xor(max_lo, o));
            min_hi = min(min_hi, __shfl_xor(min_hi, o));
        }
        const int k_lo = min(b_lo, __shfl_xor(b_lo, 32)), k_hi = max(b_hi, __shfl_xor(b_hi, 32));
        max_lo = max(max_lo, __shfl_xor(max_lo, 32));
        min_hi = min(min_hi, __shfl_xor(min_hi, 32));
        const bool fits = b_hi == 0 || b_hi - (b_lo & ~31) <= kShortHullKeys;
        hull[i][0] = k_lo; hull[i][1] = k_hi; hull[i][2] = __all(fits) ? 1 : 0;
        const int n_real = __popcll(__ballot(real));
        block[i] = make_int2(b_hi > 0 ? b_lo : 0, b_hi);
        if (g < a.n_groups) {
            if ((lane & 31) == 0) {
                const int b = g * (kGroupRows / kShortBlockRows) + (lane >> 5);
                a.block_hull[2 * b] = block[i].x;
                a.block_hull[2 * b + 1] = block[i].y;
            }
            if (lane == 0) {
                reinterpret_cast<int4*>(a.group)[g] = k_hi == 0 ? make_int4(0, 0, 0, 0) : make_int4(k_lo, k_hi, max_lo, min_hi);
                a.group_real[g] = n_real;
            }
        }
    }
}

// Sum and largest (of numbers >= 0) over a wavefront, in every lane.  Between registers: exchanges through LDS by 16 wavefronts cost the one
// workgroup that waits for them 0.1 us a step.
template <int CTRL, int ROWS>
__device__ __forceinline__ int from_lane(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false); }     // 0 where there is none
template <class Op>
__device__ __forceinline__ int over_lanes(int v, Op op) {
    v = op(v, from_lane<0x111, 0xf>(v));       // row_shr:1, 2, 4, 8
    v = op(v, from_lane<0x112, 0xf>(v));
    v = op(v, from_lane<0x114, 0xf>(v));
    v = op(v, from_lane<0x118, 0xf>(v));
    v = op(v, from_lane<0x142, 0xa>(v));       // row_bcast:15, 31
    v = op(v, from_lane<0x143, 0xc>(v));
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int lanes_sum(int v) { return over_lanes(v, [](int x, int y) { return x + y; }); }
__device__ __forceinline__ int lanes_max(int v) { return over_lanes(v, [](int x, int y) { return max(x, y); }); }

// A query tile's cost: the 64-key tiles between the ends of its hull.
struct TileCost { int first, cost; };
__device__ __forceinline__ TileCost tile_cost(int k_lo, int k_hi) {
    return k_hi > k_lo ? TileCost{k_lo / 64, (k_hi + 63) / 64 - k_lo / 64} : TileCost{0, 0};
}

// (a 64-bit division takes a third of a microsecond, and every dividend but those of enormous calls has 32 bits)
__device__ __forceinline__ unsigned long long quotient(unsigned long long x, uint32_t d) { return x >> 32 ? x / d : (uint32_t)x / d; }
// A dK/dV item is at most this many stages (row groups x heads) unless it is a single head's.
__device__ __forceinline__ int item_limit(unsigned long long total_span, const PlanArgs& a, bool coarse) {
    const uint32_t per = (uint32_t)a.n_slots * (coarse ? kDkvCoarseSplit : kDkvSplit);
    const unsigned long long least = coarse ? kDkvCoarseStages : kDkvMinItemStages;
    return (int)min(max(least, quotient(total_span * a.hq + per - 1, per)), 0x7fffffffull);
}
// Items per (key tile, KV head), the smallest power of two that brings an item under the limit, and an item's stages.
__device__ __forceinline__ int2 item_split(int span, int G, int limit) {
    int w = 1, heads = G;
    while (!(heads & 1) && span * heads > limit) { w *= 2; heads >>= 1; }
    return make_int2(span * heads, w);
}

// A query tile with more key tiles than this is divided (equally) among parts that have at most as many.  A short-hull tile
// counts as one without key tiles: its blocks' windows are all it reads, however far apart they lie.
__device__ __forceinline__ int row_part_limit(long long total_cost, int top_cost, const PlanArgs& a) {
    if ((long long)top_cost * 10 * a.n_slots < total_cost * kRowPartHeavy * a.hq) return 0x7fffffff;
    const unsigned long long units = ((unsigned long long)total_cost + (unsigned long long)a.n_tiles * kRowItemOverhead) * a.hq;
    return (int)min(max((unsigned long long)kRowPartMin, (units * kRowPartMean / 4 + a.row_slots - 1) / a.row_slots), 0x7fffffffull);
}
__device__ __forceinline__ int row_parts(int cost, int limit) { return cost > limit ? (cost + limit - 1) / limit : 1; }

// What dK/dV would have to do: the sum of the key tiles' spans and the longest, the row blocks that see 32 of a tile's keys
// (the most, and the sum over each XCD's run of tiles), and the coarse items too long for more than
// q on a compute unit.
struct KeyWork { int span, chain, load[kLists], longer[kDkvBalance]; unsigned long long total; };
__device__ __forceinline__ void clear(KeyWork& w) {              // by the threads of a workgroup
    static_assert(sizeof(KeyWork) % 4 == 0 && sizeof(KeyWork) / 4 <= 1024, "a thread per word");
    if (threadIdx.x < sizeof(KeyWork) / 4) reinterpret_cast<int*>(&w)[threadIdx.x] = 0;
}
// Whether the items may be coarse (kDkvCoarseSplit), and then whether they are, once `longer` is filled.
__device__ __forceinline__ bool coarse_items_possible(const PlanArgs& a) {
    return ((a.hq / a.hkv) & 1) == 0 && (long long)a.n_key_tiles * a.hkv >= a.n_slots;
}
// 17/16 of a compute unit's mean load and the slack, in stages: an item of x counts among the longer ones for q if (q + 1) x is more.  (Q has less than
// 4 GiB, so rows x query heads have at most 25 bits, and the stages of an item 20.)
__device__ __forceinline__ int coarse_load(const PlanArgs& a, const KeyWork& w) {
    return (int)min(quotient(17ull * w.total * a.hq, 16u * (uint32_t)a.n_slots) + kDkvCoarseSlack, 0x7fffffffull);
}
__device__ __forceinline__ bool coarse_items(const PlanArgs& a, const KeyWork& w) {
    bool even = true;
#pragma unroll
    for (int q = 0; q < kDkvBalance; ++q) even &= w.longer[q] <= q * a.n_slots;
    return even;
}
// Whether dkv_short_kernel does dK/dV.  Its wavefronts walk (row blocks x query heads of a KV head) one after another, where
// the general kernel divides a tile's heads among items; and tiles of a longer span would need the general kernel's launch
// after its own.  1024 tokens in documents of 1 - 64, dK/dV with 8 / 16 / 32 / 64 query heads on one KV head: 52 / 93 / 176 /
// 377 us there, 63 / 81 / 88 / 98 in the general kernel; 32K tokens, 16/2 heads: 108 and 136; 4096 tokens, one document of
// 1500, 8/1 heads: 176 (both launches) and 94.
__device__ __forceinline__ bool short_keys_pay(const PlanArgs& a, const KeyWork& w, int limit) {
    int load = 0;
#pragma unroll
    for (int x = 0; x < kLists; ++x) load = max(load, w.load[x]);
    const int G = a.hq / a.hkv;
    const int2 item = item_split(w.span, G, limit);              // the longest, or half of it
    const float general = kGeneralStart + fmaxf((float)item.x, kGeneralLoad * (float)w.total * a.per_cu) + (item.y > 1 ? kFixup : 0.f);
    const float steps = fmaxf((float)(w.chain * G), kShortLoad * kLists * (float)load * a.per_cu);
    return w.span <= kShortSpan && kShortStart + a.short_step * steps + kEmptyLaunch <= general;
}
// Row blocks that see a key tile's 32 keys kw0 ..: lane = 8 * (32 keys) + row block, of at most 8 from group `first` on.
static_assert(2 * kShortSpan <= 8 && kGroupRows == 2 * kShortBlockRows && kBwdKeyTile == 128, "a lane per 32 keys and row block");
__device__ __forceinline__ bool block_sees(int2 hull, int kw0) { return hull.y > hull.x && hull.x < kw0 + 32 && hull.y > kw0; }

// Sums over the tiles before a query tile: in the tiles' order (heaviest first, ties by index), and in the order of the part
// records, longest part first (short-hull tiles last).  (Records in the tiles' order put halves of heavy tiles before heavier whole ones: three of 15
// tiles of a 3808-token document on one of two ranks divided, 32 heads, forward 79 -> 98 us.)
struct RowPlace { int rank; long long cost; int part_rank, records, partials; };
__device__ __forceinline__ int part_length(int cost, int parts) { return parts == 1 ? cost : (cost + parts - 1) / parts; }
// (Each of the tile's `workers` threads calls it; they share its part records.)
__device__ __forceinline__ void put_query_tile(const PlanArgs& a, int i, int cost, int first, int is_short, int parts, const RowPlace& at, int worker, int workers) {
    int4* part = reinterpret_cast<int4*>(a.row_part) + at.records;
    for (int k = worker; parts > 1 && k < parts; k += workers)
        part[k] = make_int4(i, first + (int)((long long)cost * k / parts), first + (int)((long long)cost * (k + 1) / parts),
                            2 * (at.partials + k) + (k > 0));
    if (worker > 0) return;
    const long long before = at.cost + (long long)at.rank * kRowItemOverhead;
    a.fwd_order[at.rank] = i;
    a.fwd_prefix[at.rank] = before;
    const int4 whole = make_int4(i, first, first + cost, is_short ? -2 : -1);
    reinterpret_cast<int4*>(a.row_item)[at.rank] = whole;
    if (parts == 1) part[0] = whole;
    int4* base = reinterpret_cast<int4*>(a.row_part_base);
    base[at.rank] = make_int4(at.records, parts, at.partials, 0);
    if (at.rank == a.n_tiles - 1) a.fwd_prefix[a.n_tiles] = before + cost + kRowItemOverhead;
    if (at.part_rank == a.n_tiles - 1) base[a.n_tiles] = make_int4(at.records + parts, 0, 0, 0);
}
// One record per item, KV head major, head part minor: what a workgroup needs to begin.  (With one thread per tile they
// made the schedule of 64 KV heads 2 - 3 us longer.)
__device__ __forceinline__ void put_key_tile(const PlanArgs& a, int i, int2 range, int ways, int rank, int items_before, int slots_before, int worker, int workers) {
    const int shift = 31 - __clz(ways), G = a.hq / a.hkv, nh = G >> shift, item0 = items_before * a.hkv, slot0 = slots_before * a.hkv;
    for (int j = worker; j < a.hkv << shift; j += workers) {         // ways: a power of two
        const int hk = j >> shift, part = j & (ways - 1);
        int4* rec = reinterpret_cast<int4*>(a.dkv_item) + 2 * (size_t)(item0 + j);
        rec[0] = make_int4(i, hk, hk * G + part * nh, nh);
        rec[1] = make_int4(ways > 1 ? slot0 + j : -1, range.x, (range.y - range.x) * nh, 0);
    }
    if (worker > 0) return;
    a.key_ways[i] = ways;
    a.key_order[rank] = i;
    a.key_item_base[rank] = items_before * a.hkv;
    a.key_slot_base[rank] = slots_before * a.hkv;
    if (rank == a.n_key_tiles - 1) {
        a.key_item_base[a.n_key_tiles] = (items_before + ways) * a.hkv;
        a.key_slot_base[a.n_key_tiles] = (slots_before + (ways > 1 ? ways : 0)) * a.hkv;
    }
}

// Schedule, first launch of three: a wavefront per group of 64 rows, and the two query tiles of the workgroup.
// The three launches are bound by latency (4.7 us each on small-document inputs, a chain of dependent loads): each
// does all that needs nothing but the results of the one before.  Five launches, one per step, took 24.3 us at 32K
// tokens in 979 documents where these take 14.2, and 25.2 us where these take 18.7 at 128K tokens (CP = 8).  Sharing
// work across workgroups inside one launch (the last to arrive goes on) costs more than a launch.
__global__ void __launch_bounds__(256) plan_rows_kernel(const PlanArgs a) {
    __shared__ int s_cu[kCuLds], s_hull[4][3];
    const int wave = threadIdx.x >> 6, g = (int)blockIdx.x * 4 + wave;
    int tok[1], hull[1][3];
    int2 block[1];
    load_tokens<1>(a, g, 1, tok);
    const bool in_lds = a.n_docs <= kCuLds;
    if (in_lds) {
        for (int i = threadIdx.x; i < a.n_docs; i += 256) s_cu[i] = a.cu[i];
        __syncthreads();
    }
    if (in_lds) plan_groups<1>(a, s_cu, g, 1, tok, hull, block);
    else plan_groups<1>(a, a.cu, g, 1, tok, hull, block);
    if ((threadIdx.x & 63) == 0)
        for (int i = 0; i < 3; ++i) s_hull[wave][i] = hull[0][i];
    __syncthreads();
    const int t = (int)blockIdx.x * (4 / kGroupsPerTile) + (int)threadIdx.x;
    if ((int)threadIdx.x < 4 / kGroupsPerTile && t < a.n_tiles) {
        const int (*h)[3] = s_hull + threadIdx.x * kGroupsPerTile;
        const TileCost c = tile_cost(min(h[0][0], h[1][0]), max(h[0][1], h[1][1]));
        a.fwd_cost[t] = c.cost;
        a.tile_first[t] = c.first;
        // short-hull tile: every block of 32 rows that has a real row sees keys inside one window of
        // kShortHullKeys keys that starts at a multiple of 32
        a.tile_short[t] = h[0][2] & h[1][2];
    }
}

// Orders by a counting rank (n is at most a few thousand).  A workgroup of 1024 ranks kOrderPerBlock elements: wavefront
// w compares them with every (waves)th pair of elements, which pass through LDS in chunks, and the partial counts are
// summed in LDS.  (One element per thread kept the n^2 comparisons on very few compute units: 40 us for 1024 key
// tiles.)  item_of(j) gives an element's cost (>= 0) and a number of its own; Counts::see decides whether another one comes
// before it (ties: an earlier index) and sums; put(i, item, counts, worker, workers) receives the result: in one thread per
// element or, where much follows for an element (`shared`), in a wavefront.
constexpr int kOrderPerBlock = 64, kOrderChunk = 2048;
template <class Counts, class ItemOf, class Put>
__device__ __forceinline__ void order_block(int n, int block, bool shared, ItemOf item_of, Put put) {
    constexpr int n_seg = 1024 / kOrderPerBlock;
    __shared__ __attribute__((aligned(16))) int2 s_item[kOrderChunk];
    __shared__ Counts s_part[n_seg][kOrderPerBlock];
    __shared__ int2 s_own[kOrderPerBlock];
    const int e = threadIdx.x % kOrderPerBlock, seg = threadIdx.x / kOrderPerBlock;
    const int i = block * kOrderPerBlock + e;
    const int2 own = i < n ? item_of(i) : make_int2(0, 0);
    Counts mine{};
    for (int j0 = 0; j0 < n; j0 += kOrderChunk) {
        const int m = min(kOrderChunk, n - j0), m2 = (m + 1) & ~1;
        __syncthreads();
        // past the end: below every real one, so it never counts
        for (int j = threadIdx.x; j < m2; j += 1024) s_item[j] = j < m ? item_of(j0 + j) : make_int2(-1, -1);
        __syncthreads();
#pragma unroll 2
        for (int j = 2 * seg; j < m; j += 2 * n_seg) {
            const int4 two = *reinterpret_cast<const int4*>(&s_item[j]);
            mine.see(make_int2(two.x, two.y), own, j0 + j < i);
            mine.see(make_int2(two.z, two.w), own, j0 + j + 1 < i);
        }
    }
    s_part[seg][e] = mine;
    __syncthreads();
    if (seg == 0) {
        for (int s = 1; s < n_seg; ++s) mine.join(s_part[s][e]);
        if (!shared && i < n) put(i, own, mine, 0, 1);
        s_part[0][e] = mine;
        s_own[e] = own;
    }
    if (!shared) return;
    __syncthreads();
    for (int k = threadIdx.x >> 6; k < kOrderPerBlock; k += 1024 / 64)
        if (block * kOrderPerBlock + k < n) put(block * kOrderPerBlock + k, s_own[k], s_part[0][k], threadIdx.x & 63, 64);
}
// query tiles: cost, and the length of its longest part << kPartBits | parts (the length of a sequence with a K of less than
// 4 GiB has 19 bits in key tiles)
constexpr int kPartBits = 11;
struct RowCounts {
    RowPlace at;
    __device__ __forceinline__ void see(int2 o, int2 own, int earlier) {
        if (o.x > own.x - earlier) { at.rank += 1; at.cost += o.x; }
        if ((o.y >> kPartBits) > (own.y >> kPartBits) - earlier) {
            const int parts = o.y & ((1 << kPartBits) - 1);
            at.part_rank += 1;
            at.records += parts;
            at.partials += parts > 1 ? parts : 0;
        }
    }
    __device__ __forceinline__ void join(const RowCounts& o) {
        at.rank += o.at.rank; at.cost += o.at.cost; at.part_rank += o.at.part_rank; at.records += o.at.records; at.partials += o.at.partials;
    }
};
struct KeyCounts {                 // key tiles before this one, and their items and partial slots for one KV head
    int rank, items, slots;
    __device__ __forceinline__ void see(int2 o, int2 own, int earlier) {
        if (o.x > own.x - earlier) { rank += 1; items += o.y; slots += o.y > 1 ? o.y : 0; }
    }
    __device__ __forceinline__ void join(const KeyCounts& o) { rank += o.rank; items += o.items; slots += o.slots; }
};

// Second launch: workgroups [0, order_blocks) order the query tiles; the others find, one wavefront per key tile,
// the groups whose hull touches it.
__global__ void __launch_bounds__(1024) plan_ranges_kernel(const PlanArgs a, int order_blocks) {
    __shared__ unsigned long long s_total;
    __shared__ int s_top;
    if ((int)blockIdx.x < order_blocks) {
        int limit = 0x7fffffff;
        bool many = false;             // a tile of many parts
        if (a.parts) {
            if (threadIdx.x == 0) { s_total = 0; s_top = 0; }
            __syncthreads();
            long long sum = 0;
            int top = 0;
            for (int t = threadIdx.x; t < a.n_tiles; t += 1024) {
                const int work = a.tile_short[t] ? 0 : a.fwd_cost[t];
                sum += work;
                top = max(top, work);
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                sum += __shfl_xor(sum, o);
                top = max(top, __shfl_xor(top, o));
            }
            if ((threadIdx.x & 63) == 0 && sum) {
                atomicAdd(&s_total, (unsigned long long)sum);
                atomicMax(&s_top, top);
            }
            __syncthreads();
            limit = row_part_limit((long long)s_total, s_top, a);
            many = s_top / 16 > limit;
        }
        order_block<RowCounts>(a.n_tiles, blockIdx.x, many,
                               [&](int j) {
                                   const int cost = a.fwd_cost[j], work = a.parts && a.tile_short[j] ? 0 : cost, parts = row_parts(work, limit);
                                   return make_int2(cost, part_length(work, parts) << kPartBits | parts);
                               },
                               [&](int i, int2 own, const RowCounts& c, int worker, int workers) {
                                   put_query_tile(a, i, own.x, a.tile_first[i], a.tile_short[i], own.y & ((1 << kPartBits) - 1), c.at, worker, workers);
                               });
        return;
    }
    const int lane = threadIdx.x & 63, kt = ((int)blockIdx.x - order_blocks) * 16 + (int)(threadIdx.x >> 6);
    if (kt >= a.n_key_tiles) return;
    const int k0 = kt * kBwdKeyTile, k1 = min(k0 + kBwdKeyTile, a.t_kv);
    int first = kPadLo, last = 0;
#pragma unroll 8
    for (int g = lane; g < a.n_groups; g += 64) {
        const int2 d = *reinterpret_cast<const int2*>(a.group + 4 * g);
        if (d.y > d.x && d.x < k1 && d.y > k0) { first = min(first, g); last = max(last, g + 1); }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        first = min(first, __shfl_xor(first, o));
        last = max(last, __shfl_xor(last, o));
    }
    if (a.short_keys) {
        int2 h = make_int2(0, 0);
        const bool is_short = last && last - first <= kShortSpan;
        if (is_short && lane < 32 && (lane & 7) < 2 * (last - first)) h = reinterpret_cast<const int2*>(a.block_hull)[2 * first + (lane & 7)];
        const uint32_t seen = (uint32_t)__ballot(block_sees(h, k0 + (lane >> 3) * 32));
        const int most = max(max(__popc(seen & 0xff), __popc(seen & 0xff00)), max(__popc(seen & 0xff0000), __popc(seen & 0xff000000)));
        if (lane == 0) a.key_steps[kt] = most | __popc(seen) << 8;
    }
    if (lane == 0) {
        a.key_range[2 * kt] = last ? first : 0;
        a.key_range[2 * kt + 1] = last;
        a.key_span[kt] = last ? last - first : 0;
    }
}

// Third launch: how many items each key tile is split into, and the key tiles ordered by item cost (groups in range x
// heads per item).
__global__ void __launch_bounds__(1024) plan_key_items_kernel(const PlanArgs a) {
    __shared__ KeyWork s_work;
    if (blockIdx.x == 0 && threadIdx.x < kLists) a.dkv_counters[threadIdx.x] = 0;
    clear(s_work);
    __syncthreads();
    const int G = a.hq / a.hkv;
    {   // two wavefronts per XCD's run of key tiles
        static_assert(1024 / 64 == 2 * kLists, "wavefronts");
        const int x = (int)threadIdx.x >> 7, per = a.key_run, end = min(a.n_key_tiles, (x + 1) * per);
        int most = 0, chain = 0, load = 0;
        long long total = 0;
#pragma unroll 2
        for (int kt = x * per + (int)(threadIdx.x & 127); kt < end; kt += 128) {
            const int span = a.key_span[kt], steps = a.short_keys ? a.key_steps[kt] : 0;
            total += span;
            most = max(most, span);
            chain = max(chain, steps & 255);
            load += steps >> 8;
        }
        const int low = lanes_sum((int)(total & 0xffff)), high = lanes_sum((int)(total >> 16));
        most = lanes_max(most);
        if (a.short_keys) {
            chain = lanes_max(chain);
            load = lanes_sum(load);
        }
        if ((threadIdx.x & 63) == 0) {
            atomicAdd(&s_work.total, ((unsigned long long)high << 16) + low);
            atomicMax(&s_work.span, most);
            if (a.short_keys) {
                atomicMax(&s_work.chain, chain);
                atomicAdd(&s_work.load[x], load);
            }
        }
        __syncthreads();
    }
    int limit = item_limit(s_work.total, a, false);
    if (coarse_items_possible(a) && (long long)s_work.span * G > limit) {        // a thread per tile
        const int most = item_limit(s_work.total, a, true);
        const int load = coarse_load(a, s_work), lane = (int)threadIdx.x & 63;
        int longer[kDkvBalance] = {}, sum = 0;
        for (int kt = (int)threadIdx.x; kt < a.n_key_tiles; kt += 1024) {
            const int2 item = item_split(a.key_span[kt], G, most);
#pragma unroll
            for (int q = 0; q < kDkvBalance; ++q) longer[q] += item.x * (q + 1) > load ? item.y * a.hkv : 0;
        }
#pragma unroll
        for (int q = 0; q < kDkvBalance; ++q) {
            const int all = lanes_sum(longer[q]);
            sum = lane == q ? all : sum;
        }
        if (lane < kDkvBalance) atomicAdd(&s_work.longer[lane], sum);
        __syncthreads();
        if (coarse_items(a, s_work)) limit = most;
    }
    const bool short_on = a.short_keys && short_keys_pay(a, s_work, limit);        // every workgroup comes to the same result
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.short_on = short_on ? 1 : 0;
    order_block<KeyCounts>(a.n_key_tiles, blockIdx.x, a.hkv > 8, [&](int j) { return item_split(a.key_span[j], G, limit); },
                           [&](int i, int2 own, const KeyCounts& c, int worker, int workers) {
                               put_key_tile(a, i, make_int2(a.key_range[2 * i], a.key_range[2 * i + 1]), own.y, c.rank, c.items, c.slots, worker, workers);
                           });
}

// The whole schedule in one launch of one workgroup, for calls that one workgroup handles faster than three launches
// follow each other: up to 4096 rows (four groups per wavefront), 256 key tiles (32768 keys) and the documents the LDS holds.  At 2052 rows and 4096
// keys it takes 10.0 us (one launch per step: 17.0 in five), at 4095 rows and 16381 keys 12.5 us.
// A forward alone has no dK/dV items to order: 1031 rows with their schedule 33.1 -> 31.6 us without the key tiles, 4096 34.6 -> 32.9.
constexpr int kSmallGroups = 64, kSmallTiles = kSmallGroups / kGroupsPerTile, kSmallKeyTiles = 256;
__global__ void __launch_bounds__(1024) plan_small_kernel(const PlanArgs a) {
    __shared__ int s_cu[kCuLds];
    __shared__ int2 s_hull[kSmallGroups], s_block[2 * kSmallGroups];
    __shared__ KeyWork s_work;
    __shared__ int s_fits[kSmallGroups];
    __shared__ __attribute__((aligned(16))) int2 s_items[kSmallKeyTiles];
    const int tid = threadIdx.x, wave = tid >> 6;
    constexpr int PER = kSmallGroups / 16;
    int tok[PER], hull[PER][3];
    int2 block[PER];
    load_tokens<PER>(a, wave, 16, tok);
    for (int i = tid; i < a.n_docs; i += 1024) s_cu[i] = a.cu[i];
    clear(s_work);
    if (tid < kLists) a.dkv_counters[tid] = 0;
    __syncthreads();
    plan_groups<PER>(a, s_cu, wave, 16, tok, hull, block);
    if ((tid & 31) == 0)
#pragma unroll
        for (int i = 0; i < PER; ++i) s_block[2 * (wave + i * 16) + ((tid >> 5) & 1)] = block[i];
    if ((tid & 63) == 0)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            s_hull[wave + i * 16] = make_int2(hull[i][0], hull[i][1]);
            s_fits[wave + i * 16] = hull[i][2];
        }
    __syncthreads();
    const int G = a.hq / a.hkv;
    int2 range = make_int2(0, 0);      // of key tile tid / 4
    int key_limit = 0;
    if (!a.forward_only) {             // key tiles: four threads each
        const int kt = tid >> 2, k0 = kt * kBwdKeyTile, k1 = min(k0 + kBwdKeyTile, a.t_kv);
        int first = kPadLo, last = 0;
#pragma unroll
        for (int i = 0; i < kSmallGroups / 4; ++i) {             // groups past the end have an empty hull
            const int g = i * 4 + (tid & 3);
            const int2 h = s_hull[g];
            if (h.y > h.x && h.x < k1 && h.y > k0) { first = min(first, g); last = max(last, g + 1); }
        }
#pragma unroll
        for (int o = 2; o > 0; o >>= 1) {
            first = min(first, __shfl_xor(first, o));
            last = max(last, __shfl_xor(last, o));
        }
        if (last && kt < a.n_key_tiles) range = make_int2(first, last);
        const int span = range.y - range.x;
        int seen = 0;
        if (a.short_keys && span <= kShortSpan) {                // a thread per 32 keys
#pragma unroll
            for (int j = 0; j < 2 * kShortSpan; ++j)
                seen += j < 2 * span && block_sees(s_block[min(2 * range.x + j, 2 * kSmallGroups - 1)], k0 + (tid & 3) * 32);
        }
        int chain = seen, most = span, sum = (tid & 3) == 0 ? span : 0;
        if (a.short_keys) {
            seen += __shfl_xor(seen, 1);
            seen += __shfl_xor(seen, 2);
            if ((tid & 3) == 0 && seen) atomicAdd(&s_work.load[kt / a.key_run], seen);
        }
        sum = lanes_sum(sum);
        most = lanes_max(most);
        if (a.short_keys) chain = lanes_max(chain);
        if ((tid & 63) == 0 && sum) {
            atomicAdd(&s_work.total, (unsigned long long)sum);
            atomicMax(&s_work.span, most);
            if (a.short_keys) atomicMax(&s_work.chain, chain);
        }
        __syncthreads();
        key_limit = item_limit(s_work.total, a, false);
        if (coarse_items_possible(a) && (long long)s_work.span * G > key_limit) {        // a thread per tile and every fourth q
            static_assert(kDkvBalance % 4 == 0, "four threads per key tile");
            const int most = item_limit(s_work.total, a, true);
            const int load = coarse_load(a, s_work);
            const int2 item = kt < a.n_key_tiles ? item_split(span, G, most) : make_int2(0, 0);
#pragma unroll
            for (int q = tid & 3; q < kDkvBalance; q += 4) {
                int longer = item.x * (q + 1) > load ? item.y * a.hkv : 0;
#pragma unroll
                for (int o = 32; o > 2; o >>= 1) longer += __shfl_xor(longer, o);
                if ((tid & 63) < 4 && longer) atomicAdd(&s_work.longer[q], longer);
            }
            __syncthreads();
            if (coarse_items(a, s_work)) key_limit = most;
        }
        if ((tid & 3) == 0) {
            // past the end: a cost below every real one
            s_items[kt] = kt < a.n_key_tiles ? item_split(span, G, key_limit) : make_int2(-1, 0);
            if (kt < a.n_key_tiles) {
                a.key_range[2 * kt] = range.x;
                a.key_range[2 * kt + 1] = range.y;
                a.key_span[kt] = span;
            }
        }
    }
    {   // query tiles: a half-wavefront each, one comparison per lane
        const int t = tid >> 5, j = tid & 31;
        auto cost_of = [&](int i) __attribute__((always_inline)) {
            const int2 h0 = s_hull[kGroupsPerTile * i], h1 = s_hull[kGroupsPerTile * i + 1];
            return tile_cost(min(h0.x, h1.x), max(h0.y, h1.y));
        };
        static_assert(kSmallTiles == 32 && kGroupsPerTile == 2, "a lane of a half-wavefront per query tile");
        const TileCost own = cost_of(t), other = cost_of(j);
        const int is_short = s_fits[kGroupsPerTile * t] & s_fits[kGroupsPerTile * t + 1];
        const int other_short = s_fits[kGroupsPerTile * j] & s_fits[kGroupsPerTile * j + 1];
        const int work = a.parts && is_short ? 0 : own.cost, other_work = a.parts && other_short ? 0 : other.cost;
        const bool before = j < a.n_tiles && other.cost > own.cost - (j < t);
        int rank = before, sum = before ? other.cost : 0, total = j < a.n_tiles ? other_work : 0, top = total;
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) {
            top = max(top, __shfl_xor(top, o));
            rank += __shfl_xor(rank, o);
            sum += __shfl_xor(sum, o);
            total += __shfl_xor(total, o);
        }
        const int limit = a.parts ? row_part_limit(total, top, a) : 0x7fffffff;
        const int parts = row_parts(work, limit), other_parts = row_parts(other_work, limit);
        const bool part_before = j < a.n_tiles && part_length(other_work, other_parts) > part_length(work, parts) - (j < t);
        // records, partial results and tiles before it: at most 32 tiles and the parts added to them, in 10, 10 and 6 bits
        int places = part_before ? other_parts | (other_parts > 1 ? other_parts << 10 : 0) | 1 << 20 : 0;
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) places += __shfl_xor(places, o);
        if (t < a.n_tiles) {
            if (j == 0) {
                a.fwd_cost[t] = own.cost;
                a.tile_first[t] = own.first;
                a.tile_short[t] = is_short;
            }
            put_query_tile(a, t, own.cost, own.first, is_short, parts, RowPlace{rank, sum, places >> 20, places & 1023, (places >> 10) & 1023}, j, 32);
        }
    }
    if (a.forward_only) return;
    __syncthreads();
    if (tid == 0) *a.short_on = a.short_keys && short_keys_pay(a, s_work, key_limit) ? 1 : 0;
    {   // the key tiles' order: four threads per tile, each a quarter of the comparisons
        const int i = tid >> 2;
        const int2 own = s_items[i];
        KeyCounts c{};
#pragma unroll 4
        for (int j = 2 * (tid & 3); j < a.n_key_tiles; j += 8) {
            const int4 two = *reinterpret_cast<const int4*>(&s_items[j]);
            c.see(make_int2(two.x, two.y), own, j < i);
            c.see(make_int2(two.z, two.w), own, j + 1 < i);
        }
#pragma unroll
        for (int o = 2; o > 0; o >>= 1) {
            c.rank += __shfl_xor(c.rank, o);
            c.items += __shfl_xor(c.items, o);
            c.slots += __shfl_xor(c.slots, o);
        }
        if (i < a.n_key_tiles) put_key_tile(a, i, range, own.y, c.rank, c.items, c.slots, tid & 3, 4);
    }
}

wlb_status launch_plan(const wlb_attn_desc& d, const PlanLayout& L, const int32_t* q_idx,
                       const int32_t* cu_seqlens_k, char* ws, bool forward_only, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    auto at = [&](size_t off) { return (int32_t*)(ws + off); };
    PlanArgs a;
    a.q_idx = q_idx; a.cu = cu_seqlens_k;
    a.n_q = d.n_q; a.t_kv = d.t_kv; a.n_docs = d.n_docs; a.hq = d.hq; a.hkv = d.hkv;
    a.n_groups = L.n_groups; a.n_tiles = L.n_fwd_tiles; a.n_key_tiles = L.n_key_tiles; a.n_slots = compute_units();
    a.row_lo = at(L.off_row_lo); a.row_hi = at(L.off_row_hi);
    a.group = at(L.off_group); a.group_real = at(L.off_group_real); a.block_hull = at(L.off_block_hull);
    a.fwd_cost = at(L.off_fwd_cost); a.tile_first = at(L.off_tile_first); a.tile_short = at(L.off_tile_short);
    a.fwd_order = at(L.off_fwd_order); a.row_item = at(L.off_row_item); a.row_part = at(L.off_row_part); a.row_part_base = at(L.off_row_part_base);
    a.row_slots = std::max(1, row_parts_added(d, L) * d.hq);
    wlb_attn_desc unforced = d;        // the tables do not depend on flags that force a schedule
    unforced.flags = 0;
    a.parts = use_row_parts(unforced, L) ? 1 : 0;
    a.fwd_prefix = (long long*)(ws + L.off_fwd_prefix);
    a.key_range = at(L.off_key_range); a.key_span = at(L.off_key_span); a.key_ways = at(L.off_key_ways);
    a.key_order = at(L.off_key_order); a.key_item_base = at(L.off_key_item_base); a.key_slot_base = at(L.off_key_slot_base);
    a.dkv_counters = at(L.off_dkv_counters); a.dkv_item = at(L.off_dkv_item); a.short_on = at(L.off_short_on);
    a.key_steps = at(L.off_key_steps);
    a.forward_only = forward_only ? 1 : 0;
    a.short_keys = !forward_only && short_documents(d) ? 1 : 0;
    a.key_run = (L.n_key_tiles + kLists - 1) / kLists;
    a.per_cu = (float)d.hq / (float)a.n_slots;
    a.short_step = d.head_dim == 64 ? kShortStep64 : kShortStep128;
    if (L.n_groups <= kSmallGroups && L.n_key_tiles <= kSmallKeyTiles && d.n_docs <= kCuLds) {
        plan_small_kernel<<<1, 1024, 0, stream>>>(a);
    } else {
        const int order_blocks = (L.n_fwd_tiles + kOrderPerBlock - 1) / kOrderPerBlock;
        plan_rows_kernel<<<(L.n_groups + 3) / 4, 256, 0, stream>>>(a);
        plan_ranges_kernel<<<order_blocks + (L.n_key_tiles + 15) / 16, 1024, 0, stream>>>(a, order_blocks);
        if (!forward_only) plan_key_items_kernel<<<(L.n_key_tiles + kOrderPerBlock - 1) / kOrderPerBlock, 1024, 0, stream>>>(a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(WLB_ERR_HIP, "plan launch: %s", hipGetErrorString(e));
    return WLB_OK;
}

// ------------------------------------------------------------------------------------------
// Scratch of wlb_attn_fwd_static: the schedule tables live in this array instead of a caller's
// workspace.  Every GPU the library runs on holds its own copy, at its own address, until the
// process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the address
// that call returns (kept per device) is what kernels and every other use of the memory get.
// The stated limit counts the tables a schedule had to have when the limit was set (PlanLayout::static_bytes);
// the tables added since (52 bytes per query tile of a schedule with at least 8 bytes per row, and 16 per part added, at most one per workgroup slot)
// have room of their own.
constexpr size_t kStaticExtraBytes = WLB_ATTN_FWD_STATIC_SCRATCH_BYTES / 8 / kFwdTileRows * 52 + 1024 * 16 + 2048;
static __device__ __align__(256) unsigned char scratch[WLB_ATTN_FWD_STATIC_SCRATCH_BYTES + kStaticExtraBytes];

constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];      // device address of `scratch` on each device, once resolved
static std::mutex g_scratch_mutex;

// The current device's copy of `scratch`; resolved on the first call on that device.
static wlb_status static_scratch(char** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(WLB_ERR_HIP, "wlb_attn_fwd_static: hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(WLB_ERR_UNSUPPORTED, "wlb_attn_fwd_static: device %d (at most %d devices)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(WLB_ERR_HIP, "wlb_attn_fwd_static: hipGetSymbolAddress: %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
    }
    *out = (char*)g_scratch_ptr[dev];
    return WLB_OK;
}

// delta and the log2-scaled LSE copy, [hq][n_q] floats each
static size_t delta_bytes(const wlb_attn_desc& d) { return 2 * align_up(sizeof(float) * (size_t)d.hq * d.n_q, 256); }

}  // namespace wlb

using namespace wlb;

extern "C" wlb_status wlb_attn_workspace_size(const wlb_attn_desc* desc, size_t* fwd_bytes, size_t* bwd_bytes) {
    if (wlb_status st = check_desc(desc)) return st;
    if (!fwd_bytes || !bwd_bytes) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_workspace_size: null output");
    PlanLayout L;
    plan_layout(*desc, &L);
    *fwd_bytes = L.plan_bytes + row_partial_bytes(*desc, L);
    *bwd_bytes = L.plan_bytes + delta_bytes(*desc) + dkv_partial_bytes(*desc, L) + row_partial_bytes(*desc, L);
    return WLB_OK;
}

extern "C" wlb_status wlb_attn_set_gang_weights(int32_t kernel, const int32_t* weights) {
    if (kernel != 0 && kernel != 1) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_set_gang_weights: kernel=%d (0 = forward, 1 = dQ)", kernel);
    if (weights)
        for (int i = 0; i < 16; ++i)
            if (weights[i] < 1 || weights[i] > 1000000)
                return fail(WLB_ERR_INVALID_ARG, "wlb_attn_set_gang_weights: weight %d = %d outside [1, 10^6]", i, weights[i]);
    std::lock_guard<std::mutex> lock(g_gang_weight_mutex);
    for (int i = 0; i < 16; ++i) g_gang_weight[kernel][i / 8][i % 8] = weights ? weights[i] : 0;
    return WLB_OK;
}

extern "C" wlb_status wlb_attn_get_gang_weights(int32_t kernel, int32_t* weights_out) {
    if (kernel < 0 || kernel > 1) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_get_gang_weights: kernel %d (0 = forward, 1 = dQ)", kernel);
    if (!weights_out) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_get_gang_weights: null output");
    int w[2][8];
    gang_weights(kernel, w);
    for (int i = 0; i < 16; ++i) weights_out[i] = w[i / 8][i % 8];
    return WLB_OK;
}

extern "C" wlb_status wlb_attn_plan_layout(const wlb_attn_desc* desc, wlb_plan_layout* layout) {
    if (wlb_status st = check_desc(desc)) return st;
    if (!layout) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_plan_layout: null output");
    PlanLayout L;
    plan_layout(*desc, &L);
    *layout = L;
    return WLB_OK;
}

extern "C" wlb_status wlb_attn_plan_records(const wlb_attn_desc* desc, wlb_plan_records* records) {
    if (wlb_status st = check_desc(desc)) return st;
    if (!records) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_plan_records: null output");
    PlanLayout L;
    plan_layout(*desc, &L);
    records->uses_parts = use_row_parts(*desc, L) ? 1 : 0;
    records->max_parts = L.n_fwd_tiles + row_parts_added(*desc, L);
    records->uses_short_keys = use_short_keys(*desc, L) ? 1 : 0;
    records->short_span = kShortSpan;
    records->off_row_item = L.off_row_item;
    records->off_row_part = L.off_row_part;
    records->off_row_part_base = L.off_row_part_base;
    records->off_dkv_item = L.off_dkv_item;
    records->off_short_on = L.off_short_on;
    records->row_partial_bytes = row_partial_floats(desc->head_dim) * sizeof(float);
    records->row_partials_bytes = row_partial_bytes(*desc, L);
    return WLB_OK;
}

extern "C" wlb_status wlb_attn_plan(const wlb_attn_desc* desc, const int32_t* q_idx, const int32_t* cu_seqlens_k,
                                    void* workspace, size_t workspace_bytes, void* stream) {
    if (wlb_status st = check_desc(desc)) return st;
    if (!q_idx || !cu_seqlens_k || !workspace) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_plan: null pointer");
    PlanLayout L;
    plan_layout(*desc, &L);
    if (workspace_bytes < L.plan_bytes)
        return fail(WLB_ERR_BUFFER_TOO_SMALL, "wlb_attn_plan: workspace %zu < %zu bytes", workspace_bytes, L.plan_bytes);
    return launch_plan(*desc, L, q_idx, cu_seqlens_k, (char*)workspace, false, stream);
}

extern "C" wlb_status wlb_attn_fwd(const wlb_attn_desc* desc, const void* q, const void* k, const void* v,
                                   const int32_t* q_idx, const int32_t* cu_seqlens_k, void* o, float* lse,
                                   void* workspace, size_t workspace_bytes, void* stream) {
    if (wlb_status st = check_desc(desc)) return st;
    if (!q || !k || !v || !o || !lse || !workspace) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_fwd: null pointer");
    const bool reuse = desc->flags & WLB_ATTN_REUSE_PLAN;
    if (!reuse && (!q_idx || !cu_seqlens_k)) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_fwd: null q_idx/cu_seqlens_k");
    PlanLayout L;
    plan_layout(*desc, &L);
    const size_t need = L.plan_bytes + row_partial_bytes(*desc, L);
    if (workspace_bytes < need)
        return fail(WLB_ERR_BUFFER_TOO_SMALL, "wlb_attn_fwd: workspace %zu < %zu bytes", workspace_bytes, need);
    if (!reuse)
        if (wlb_status st = launch_plan(*desc, L, q_idx, cu_seqlens_k, (char*)workspace, false, stream)) return st;
    return launch_fwd(*desc, L, q, k, v, o, lse, (char*)workspace, L.plan_bytes, stream);
}

extern "C" wlb_status wlb_attn_fwd_static(const wlb_attn_desc* desc, const void* q, const void* k, const void* v,
                                          const int32_t* q_idx, const int32_t* cu_seqlens_k, void* o, float* lse,
                                          void* stream) {
    if (wlb_status st = check_desc(desc)) return st;
    if (!q || !k || !v || !o || !lse) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_fwd_static: null pointer");
    if (desc->flags & ~(WLB_ATTN_REUSE_PLAN | WLB_ATTN_SCHEDULE_ITEMS))
        return fail(WLB_ERR_INVALID_ARG, "wlb_attn_fwd_static: flags 0x%x (only WLB_ATTN_REUSE_PLAN and WLB_ATTN_SCHEDULE_ITEMS apply)", desc->flags);
    const bool reuse = desc->flags & WLB_ATTN_REUSE_PLAN;
    if (!reuse && (!q_idx || !cu_seqlens_k)) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_fwd_static: null q_idx/cu_seqlens_k");
    // one workgroup per (query tile, head): the schedule that leaves no partial results, so the
    // schedule tables are all the scratch the call needs
    wlb_attn_desc d = *desc;
    d.flags |= WLB_ATTN_SCHEDULE_ITEMS;
    PlanLayout L;
    plan_layout(d, &L);
    if (L.static_bytes > (size_t)WLB_ATTN_FWD_STATIC_SCRATCH_BYTES)
        return fail(WLB_ERR_UNSUPPORTED, "wlb_attn_fwd_static: the schedule of n_q=%d, t_kv=%d needs %zu bytes, the library's array holds %zu",
                    d.n_q, d.t_kv, L.static_bytes, (size_t)WLB_ATTN_FWD_STATIC_SCRATCH_BYTES);
    char* ws = nullptr;
    if (wlb_status st = static_scratch(&ws)) return st;
    if (!reuse)
        if (wlb_status st = launch_plan(d, L, q_idx, cu_seqlens_k, ws, true, stream)) return st;
    return launch_fwd(d, L, q, k, v, o, lse, ws, L.plan_bytes, stream);
}

extern "C" wlb_status wlb_attn_bwd(const wlb_attn_desc* desc, const void* q, const void* k, const void* v,
                                   const void* o, const float* lse, const void* d_o, const int32_t* q_idx,
                                   const int32_t* cu_seqlens_k, void* dq, void* dk, void* dv, void* workspace,
                                   size_t workspace_bytes, void* stream) {
    if (wlb_status st = check_desc(desc)) return st;
    if (!q || !k || !v || !o || !lse || !d_o || !dq || !dk || !dv || !workspace)
        return fail(WLB_ERR_INVALID_ARG, "wlb_attn_bwd: null pointer");
    const bool reuse = desc->flags & WLB_ATTN_REUSE_PLAN;
    if (!reuse && (!q_idx || !cu_seqlens_k)) return fail(WLB_ERR_INVALID_ARG, "wlb_attn_bwd: null q_idx/cu_seqlens_k");
    PlanLayout L;
    plan_layout(*desc, &L);
    const size_t need = L.plan_bytes + delta_bytes(*desc) + dkv_partial_bytes(*desc, L) + row_partial_bytes(*desc, L);
    if (workspace_bytes < need)
        return fail(WLB_ERR_BUFFER_TOO_SMALL, "wlb_attn_bwd: workspace %zu < %zu bytes", workspace_bytes, need);
    if (!reuse)
        if (wlb_status st = launch_plan(*desc, L, q_idx, cu_seqlens_k, (char*)workspace, false, stream)) return st;
    return launch_bwd(*desc, L, q, k, v, o, lse, d_o, dq, dk, dv, (char*)workspace, L.plan_bytes, stream);
}
