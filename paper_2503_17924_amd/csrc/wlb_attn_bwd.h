// What the backward's kernels are launched with, shared by their translation units.
#pragma once
#include "wlb_device.h"

namespace wlb {

struct BwdParams {
    const __bf16* q; const __bf16* k; const __bf16* v; const __bf16* o; const __bf16* d_o;
    const float* lse; float* delta; float* lse2;
    __bf16* dq; __bf16* dk; __bf16* dv;
    const int32_t* row_lo; const int32_t* row_hi;
    const int32_t* key_order; const int32_t* key_ways; const int32_t* key_item_base; const int32_t* key_slot_base;
    const int32_t* key_range; const int32_t* short_on;   // dkv_short_kernel; null: not launched
    const int32_t* dkv_item;   // two int4 per item (PlanLayout::off_dkv_item)
    int32_t* dkv_counters;     // [8]: items of each XCD's list handed out beyond the first of every workgroup (zero before every dK/dV launch)
    float* partial;
    RowSched sched;            // dQ: which query tiles, heads and key ranges a workgroup works on
    float* row_partial;        // dQ: partial results of the tiles cut at a gang boundary
    const int32_t* row_item;   // one workgroup per item: records (PlanLayout::off_row_item, or off_row_part with row_part_base)
    const int32_t* row_part_base;     // null: whole tiles only
    int first_half;                   // see paired_index
    const int32_t* block_hull;   // short-hull path (see dq_short_unit)
    const int32_t* tile_short;   // by query tile: a short-hull tile
    unsigned long long* gang_clock;   // [workgroup][2]: real-time counter at the start / end of dq_kernel's workgroup
    int n_blocks32, use_short;
    int n_q, t_kv, hq, hkv, n_groups, n_tiles, n_key_tiles;
    float scale_log2e, scale;
};

// dQ with two query heads of a KV head to a workgroup (wlb_attn_dq_pair.hip); hq / hkv is even, head dimension 128.
void launch_dq_pair(const BwdParams& p, bool gangs, unsigned grid, hipStream_t stream);

// Short documents divided among ranks (wlb_attn_span.hip).
void launch_dq_span(const BwdParams& p, int head_dim, hipStream_t stream);

// The dK/dV launch (wlb_attn_dkv.hip).
void launch_dkv_general(const BwdParams& p, int head_dim, bool beside_short, unsigned grid, hipStream_t stream);

}  // namespace wlb
