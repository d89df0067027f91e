// What the forward's kernels are launched with, shared by their translation units.
#pragma once
#include "wlb_device.h"

namespace wlb {

struct FwdParams {
    const __bf16* q; const __bf16* k; const __bf16* v;
    __bf16* o; float* lse;
    const int32_t* row_lo; const int32_t* row_hi;
    RowSched sched;            // which query tiles, heads and key ranges a workgroup works on
    float* partial;            // partial results of the tiles cut at a gang boundary
    const int32_t* row_item;   // one workgroup per item: records (PlanLayout::off_row_item, or off_row_part with row_part_base)
    const int32_t* row_part_base;     // null: whole tiles only
    int first_half;                   // see paired_index
    const int32_t* block_hull;   // short-hull path (see fwd_short_unit)
    const int32_t* tile_short;   // by query tile: a short-hull tile
    unsigned long long* gang_clock;   // [workgroup][2]: real-time counter at the start / end of a gang kernel's workgroup
    int n_q, t_kv, hq, hkv, n_tiles, n_blocks32, use_short;
    float scale_log2e, scale;
};

// Two query heads of a KV head to a workgroup (wlb_attn_fwd_pair.hip); hq / hkv is even.
void launch_fwd_pair(const FwdParams& p, int head_dim, bool gangs, unsigned grid, hipStream_t stream);

// Short documents divided among ranks (wlb_attn_span.hip).
void launch_fwd_span(const FwdParams& p, int head_dim, hipStream_t stream);

}  // namespace wlb
