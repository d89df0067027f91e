// Backward document-masked attention for gfx950.  The paper measures forward+backward
// latency of the attention kernel (Section 6.4) without restating the derivative; this is the
// standard one: with P = exp(scale*Q K^T - LSE) on the visible (same-document, causal) pairs
// and delta_i = <dO_i, O_i>,
//     dV = P^T dO,  dP = dO V^T,  dS = P o (dP - delta),  dQ = scale * dS K,  dK = scale * dS^T Q,
// dK/dV summed over the query heads that share a KV head.  As in all-gather context
// parallelism (Section 2.1) dK/dV hold only the calling rank's rows' contribution.
//
// No atomics, deterministic:
//   dq_kernel         query-stationary, same tiling and work schedule as the forward: S^T and dP^T
//                     per lane column, dQ^T += K^T dS^T with K^T read from LDS by transpose reads.
//                     It also forms delta[h][i] = -sum_d dO*O of its rows (stored negated: the dK/dV
//                     kernel starts its dP accumulators from it) and leaves it and a log2-scaled LSE
//                     copy (0 / +inf for padding rows) for the dK/dV kernel, which runs after it
//   delta_kernel      the same for a call that leaves dQ out (WLB_ATTN_BWD_SKIP_DQ)
//   dq_pair_kernel    (wlb_attn_dq_pair.hip) the same for two query heads at a time, in launches of long items
//   dq_merge_kernel   sums the fp32 partial dQ of query tiles cut at a gang boundary
//   dkv_kernel        (wlb_attn_dkv.hip) key-stationary: a work item owns 128 keys of one KV head and streams the row
//                     groups that can see them through LDS for some or all query heads of the KV
//                     group; dK^T, dV^T stay in registers until the single final store
//   dkv_short_kernel  the same for calls in which few rows can see any one key tile (short documents)
//   dkv_fixup_kernel  sums the fp32 partial results of key tiles whose heads were divided among
//                     several work items (heavy tiles, so that no item is a straggler)
// S and dP are recomputed in both dq_kernel and dkv_kernel (7 GEMMs for the 5 the derivative
// needs): this keeps dQ free of atomics and of an fp32 accumulation buffer.
// Q / dO / K tiles that are read both row-wise (b128) and column-wise (transpose reads) are
// stored unpadded with an XOR swizzle of their 16-byte chunks that makes both patterns
// bank-conflict free; all tiles arrive by asynchronous global->LDS copies.
#include <hip/hip_runtime.h>

#include "wlb_attn_bwd.h"
#include "wlb_attn_short.h"
#include "wlb_device.h"
#include <algorithm>
#include <type_traits>

#include "wlb_internal.h"

namespace wlb {

// ------------------------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(256) delta_kernel(const BwdParams p) {
    constexpr int LPR = D / 8;                       // lanes per (row, head)
    const size_t total = (size_t)p.n_q * p.hq;
    // gridDim.x / n_tiles workgroups share the (row, head) pairs of a query tile
    const int split = (int)gridDim.x / p.n_tiles;
    const int tile = (int)blockIdx.x / split, part = (int)blockIdx.x % split;
    if (tile >= p.n_tiles) return;
    const size_t first = (size_t)tile * kFwdTileRows * p.hq * LPR, lanes = (size_t)kFwdTileRows * p.hq * LPR;
    for (size_t off = (size_t)part * 256; off < lanes; off += (size_t)split * 256) {
        const size_t idx = first + off + threadIdx.x;
        const size_t rh = idx / LPR;                 // row * hq + head
        const int c = (int)(idx % LPR);
        const bool mine = rh < total;
        float acc = 0.f;
        if (mine) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(p.d_o + rh * D + c * 8);
            const bf16x8 b = *reinterpret_cast<const bf16x8*>(p.o + rh * D + c * 8);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc += (float)a[i] * (float)b[i];
        }
#pragma unroll
        for (int o = LPR / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
        if (mine && c == 0) {
            const int row = (int)(rh / p.hq), h = (int)(rh % p.hq);
            const bool real = p.row_hi[row] > 0;
            p.delta[(size_t)h * p.n_q + row] = real ? -acc : 0.f;
            // LSE in log2 units for the dK/dV kernel; +inf makes every probability of a padding row 0
            p.lse2[(size_t)h * p.n_q + row] = real ? p.lse[(size_t)h * p.n_q + row] * 1.4426950408889634f : INFINITY;
        }
    }
}

// ------------------------------------------------------------------------------------------
// dQ, four wavefronts x 32 rows, two workgroups per CU: K and V tiles of 64 keys arrive by
// asynchronous global->LDS copies (double buffered, one barrier per tile); per block of 32
// keys a wavefront computes S^T = K Q^T and dP^T = V dO^T (lane = its query column), forms
// dS^T = P^T o (dP^T - delta) in registers and accumulates dQ^T += K^T dS^T with K^T read
// from the same swizzled K tile by transpose reads.
// delta comes from the dO operands the wavefront holds anyway and its rows of O: a pass of its own read dO a second
// time and cost a launch (129 of 5800 us at 32K tokens with 32 query heads, 40 of 813 us in four layers of 8191
// tokens); here it is D / 16 loads
// per lane beside the copies of the first tiles (5712 -> 5629 us, 807 -> 767 us with the schedule's shorter launches).
template <int D>
__device__ __forceinline__ void dq_piece(const BwdParams& p, char* smem, const RowPiece& pc) {
    constexpr int NW = 4, BM = 128, BN = 64;
    static_assert(BM == kFwdTileRows, "tile rows must match the schedule");
    constexpr int KS = D / 16, DB = D / 32, CPR = D / 8, ROWB = D * 2, TILEB = BN * ROWB;

    const int G = p.hq / p.hkv;
    const int tile = pc.tile, hk = pc.hk;
    const int h = hk * G + pc.member;

    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int j16 = lane & 15, gi = (lane >> 4) & 1;

    const int jb = pc.jb, je = pc.je;      // this piece's 64-key tiles
    int fb = 0, fe = 0;

    const uint32_t kv_row = (uint32_t)p.hkv * D;
    const uint32_t kv_bytes = ((uint32_t)p.t_kv * kv_row - (uint32_t)hk * D) * 2u;
    BufRsrc krs, vrs;
    krs.init(p.k + (size_t)hk * D, kv_bytes);
    vrs.init(p.v + (size_t)hk * D, kv_bytes);
    TileDma<D, BN, NW> dma;
    dma.init(wave, lane, kv_row);
    const uint32_t smem_base = (uint32_t)(uintptr_t)(WLB_LDS char*)smem;
    auto tile_ptr = [&](int which) { return smem_base + (uint32_t)(which * TILEB); };
    __syncthreads();            // every wavefront has left the tiles of the piece before
    if (jb < je) {
        dma.issue(krs, tile_ptr(0), jb * BN, wave);
        dma.issue(vrs, tile_ptr(2), jb * BN, wave);
    }

    const int row = tile * BM + wave * 32 + l32;
    const bool in = row < p.n_q;
    const int rc = in ? row : p.n_q - 1;
    const int row_lo[1] = {in ? p.row_lo[rc] : kPadLo}, row_hi[1] = {in ? p.row_hi[rc] : 0};
    const int lo = row_lo[0], hi = row_hi[0];
    const bool real = hi > 0;
    // key tiles this wavefront needs no element-wise mask for: only outside [fb, fe) it masks.  Inside, the
    // rows of the wavefront's first document see every key and the rows of later documents none.
    bool other_doc[1];
    unmasked_tiles<BN>(row_lo, row_hi, fb, fe, other_doc);
    // padding rows: zero operands and LSE = +inf make P, dS and dQ exactly 0
    const float lsec = real ? p.lse[(size_t)h * p.n_q + rc] * 1.4426950408889634f : INFINITY;
    float lsec_unmasked = other_doc[0] ? INFINITY : lsec;           // inside [fb, fe): +inf switches the lane off
    float dl = 0.f;                    // -delta
    bf16x8 qf[KS], dof[KS];
    {
        const __bf16* qp = p.q + ((size_t)rc * p.hq + h) * D + half * 8;
        const __bf16* gp = p.d_o + ((size_t)rc * p.hq + h) * D + half * 8;
        const __bf16* op = p.o + ((size_t)rc * p.hq + h) * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bf16x8 a = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
            bf16x8 g = *reinterpret_cast<const bf16x8*>(gp + ks * 16);
            const bf16x8 o = *reinterpret_cast<const bf16x8*>(op + ks * 16);
#pragma unroll
            for (int i = 0; i < 8; ++i) dl = fmaf(-(float)g[i], (float)o[i], dl);
            if (!real) {
#pragma unroll
                for (int i = 0; i < 8; ++i) { a[i] = (__bf16)0.f; g[i] = (__bf16)0.f; }
            }
            qf[ks] = a; dof[ks] = g;
        }
        dl += xhalf(dl);
        if (!real) dl = 0.f;
        // the tile's first piece leaves them for the dK/dV kernel; +inf makes every probability of a padding row 0
        if (pc.first && in && half == 0) {
            p.delta[(size_t)h * p.n_q + row] = dl;
            p.lse2[(size_t)h * p.n_q + row] = lsec;
        }
    }

    int naddr[KS], taddr[DB][2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) naddr[ks] = smem_base + l32 * ROWB + swz<CPR>(l32, ks * 2 + half) * 16;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int key = t * 8 + half * 4 + (j16 >> 2);
            const int dch = db * 4 + gi * 2 + ((j16 & 3) >> 1);
            taddr[db][t] = smem_base + key * ROWB + swz<CPR>(key, dch) * 16 + (j16 & 1) * 8;
        }

    f32x16 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
    const float cs = p.scale_log2e;

    // one tile; the buffer index is a compile-time constant so that every LDS address is a
    // loop-invariant register plus an immediate
    auto tile_step = [&](int j, auto cur_tag) {
        constexpr int cur = decltype(cur_tag)::value;
        wait_vmem();
        __syncthreads();
        if (j + 1 < je) {
            dma.issue(krs, tile_ptr(cur ^ 1), (j + 1) * BN, wave);
            dma.issue(vrs, tile_ptr(2 + (cur ^ 1)), (j + 1) * BN, wave);
        }
        constexpr int kb_base = cur * TILEB, vb_base = (2 + cur) * TILEB;
        const bool partial = (j < fb) || (j >= fe);
        // S^T and dP^T of a 32-key block (two independent accumulation chains)
        // At head_dim 64, where the kernel is bound by the vector ALU, the dP accumulation starts from -delta
        // (the subtraction happens inside the first MFMA); at 128 that costs registers the kernel does not have.
        constexpr bool kDeltaInMfma = D == 64;
        auto scores = [&](int kb, f32x16& s, f32x16& dp) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = kDeltaInMfma ? dl : 0.f; }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 ka = *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(kb_base + naddr[ks] + kb * 32 * ROWB));
                const bf16x8 va = *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(vb_base + naddr[ks] + kb * 32 * ROWB));
                s = mfma32(ka, qf[ks], s);
                dp = mfma32(va, dof[ks], dp);
            }
        };
        // dS^T = P^T o (dP^T - delta), in place of s; ls = the row's LSE, or +inf to switch the lane off
        auto grads = [&](f32x16& s, const f32x16& dp, float ls) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = fast_exp2(fmaf(s[r], cs, -ls)) * (kDeltaInMfma ? dp[r] : dp[r] + dl);
        };
        // a block outside the fully visible range: rows that see none of its 32 keys (rows of another
        // document in the same wavefront) are switched off as whole lanes; the element-wise mask is
        // needed only where a row's interval cuts the block (diagonal, document edges)
        auto classify = [&](int kb, float& ls, bool& elementwise) __attribute__((always_inline)) {
            const int key0 = j * BN + kb * 32;
            const bool none = (key0 + 32 <= lo) || (key0 >= hi);
            const bool all = (key0 >= lo) && (key0 + 32 <= hi);
            elementwise = __any(!(none || all));
            ls = none ? INFINITY : lsec;
        };
        auto mask = [&](int kb, f32x16& ds) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = j * BN + kb * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
                ds[r] = (key >= lo && key < hi) ? ds[r] : 0.f;
            }
        };
        auto update = [&](int kb, const f32x16& ds) __attribute__((always_inline)) {
            bf16x8 dsf[2];
            dsf[0] = pack8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
            dsf[1] = pack8(ds[8], ds[9], ds[10], ds[11], ds[12], ds[13], ds[14], ds[15]);
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                const int koff = (kb * 32 + cc * 16) * ROWB;
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const bf16x8 a = cat4(lds_read_tr4_at(kb_base + taddr[db][0] + koff),
                                          lds_read_tr4_at(kb_base + taddr[db][1] + koff));
                    acc[db] = mfma32(a, dsf[cc], acc[db]);
                }
            }
        };
        // The vector-ALU work of a block runs beside MFMAs that do not depend on it: block 0's
        // exponentials beside block 1's score MFMAs, block 1's beside block 0's dQ update.  The mask
        // (only on a document's diagonal or edge) is a branch between those straight-line regions.
        f32x16 s0, dp0, s1, dp1;
        float ls0 = lsec_unmasked, ls1 = lsec_unmasked;
        bool em0 = false, em1 = false;
        if (partial) {
            classify(0, ls0, em0);
            classify(1, ls1, em1);
            if (!em0 && !em1) {
                // Every row sees all or none of the tile's second block.  That stays so up to the next edge of
                // a row's interval (the end of a row that sees it, the start of one still to come): the key
                // tiles from the next one up to that edge become the unmasked range, the rows that see
                // nothing switched off.  A wavefront that holds rows of two chunks of one document (or of
                // two documents) crosses the keys between them without classifying every block.
                const int key1 = j * BN + 32;
                const bool none = (key1 + 32 <= lo) || (key1 >= hi);
                int edge = none ? (lo >= key1 + 32 ? lo : kPadLo) : hi;
#pragma unroll
                for (int o = 16; o > 0; o >>= 1) edge = min(edge, __shfl_xor(edge, o));
                const int j_edge = uniform(edge / BN);
                if (j_edge > j + 1) {
                    fb = j + 1;
                    fe = j_edge;
                    lsec_unmasked = none ? INFINITY : lsec;
                }
            }
        }
        scores(0, s0, dp0);
        scores(1, s1, dp1);
        grads(s0, dp0, ls0);
        if (em0) {
            asm volatile("");   // keep the mask a branch
            mask(0, s0);
        }
        update(0, s0);
        grads(s1, dp1, ls1);
        if (em1) {
            asm volatile("");
            mask(1, s1);
        }
        update(1, s1);
    };
    for (int j = jb; j < je; j += 2) {
        tile_step(j, std::integral_constant<int, 0>{});
        if (j + 1 < je) tile_step(j + 1, std::integral_constant<int, 1>{});
    }

    if (pc.slot >= 0) {
        // part of a tile: unscaled fp32 dQ [row][d], summed by dq_merge_kernel
        float* part = p.row_partial + (size_t)pc.slot * (BM * D + 2 * BM);
        if (in) {
            const int rl = wave * 32 + l32;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int d = db * 32 + r4 * 8 + half * 4;
                    *reinterpret_cast<f32x4*>(part + (size_t)rl * D + d) =
                        f32x4{acc[db][r4 * 4 + 0], acc[db][r4 * 4 + 1], acc[db][r4 * 4 + 2], acc[db][r4 * 4 + 3]};
                }
        }
        return;
    }
    if (in) {
        __bf16* op = p.dq + ((size_t)row * p.hq + h) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int d = db * 32 + r4 * 8 + half * 4;
                bf16x4 out;
                if (real) out = pack4(acc[db][r4 * 4 + 0] * p.scale, acc[db][r4 * 4 + 1] * p.scale,
                                      acc[db][r4 * 4 + 2] * p.scale, acc[db][r4 * 4 + 3] * p.scale);
                else out = pack4(0.f, 0.f, 0.f, 0.f);
                *reinterpret_cast<bf16x4*>(op + d) = out;
            }
    }
}

// dQ: a fixed set of workgroups, each walking its gang's share of the work line (see RowSched).
template <int D>
__global__ void __launch_bounds__(256, 2) dq_kernel(const BwdParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[4 * 64 * D * 2];   // K0 | K1 | V0 | V1
    const unsigned long long t_start = wall_clock64();
    RowWalk walk;
    walk.start(p.sched, (int)blockIdx.x);
    RowPiece pc;
    while (walk.next(p.sched, pc)) dq_piece<D>(p, smem, pc);
    if (threadIdx.x == 0) {
        p.gang_clock[2 * blockIdx.x] = t_start;
        p.gang_clock[2 * blockIdx.x + 1] = wall_clock64();
    }
}

// The other schedule: one workgroup per (query tile in order, query head), heaviest first.
template <int D>
__global__ void __launch_bounds__(256, 2) dq_items_kernel(const BwdParams p) {
    constexpr int kLds = ShortDq<D>::LDS_BYTES > 4 * 64 * D * 2 ? ShortDq<D>::LDS_BYTES : 4 * 64 * D * 2;
    __shared__ __attribute__((aligned(1024))) char smem[kLds];
    const int G = p.hq / p.hkv;
    const int x = blockIdx.x & 7;
    int y = blockIdx.x >> 3;
    RowPiece pc;
    pc.member = y % G; y /= G;
    pc.hk = y % p.hkv;
    const int n_items = p.row_part_base ? ld_const(p.row_part_base + 4 * p.n_tiles) : p.n_tiles;
    int index = (y / p.hkv) * 8 + x;
    if (index >= n_items) return;
    index = paired_index(index, n_items, p.first_half, p.row_part_base != nullptr);
    // one record holds what the workgroup needs before its first copy: order, hull and flag through separate
    // tables are three dependent loads
    const int4 item = ld_const4(p.row_item + 4 * index);
    pc.tile = item.x;
    if (p.use_short && item.w == -2) {
        // a short-hull tile: its four blocks of 32 rows are units of their own (see dq_short_unit)
        constexpr int per_tile = kFwdTileRows / kShortBlockRows;
        for (int j = pc.member; j < per_tile; j += G) {
            const int blk = pc.tile * per_tile + j;
            if (blk < p.n_blocks32) dq_short_unit<D>(p, smem, blk, pc.hk);
        }
        return;
    }
    pc.jb = item.y; pc.je = item.z;
    pc.first = item.w < 0 || !(item.w & 1);
    pc.slot = item.w < 0 ? -1 : (item.w >> 1) * p.hq + pc.hk * G + pc.member;
    dq_piece<D>(p, smem, pc);
}

// The short-hull tiles of a launch whose other tiles dq_pair_items_kernel takes.
template <int D>
__global__ void __launch_bounds__(256, 2) dq_short_tiles_kernel(const BwdParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[ShortDq<D>::LDS_BYTES];
    for_short_tiles(p.row_item, p.n_tiles, p.hkv, p.n_blocks32, [&](int blk, int hk) __attribute__((always_inline)) { dq_short_unit<D>(p, smem, blk, hk); });
}

// dQ rows of 1 / SPLIT of a query tile and head; sum_of(offset) adds up the four elements at an offset of the tile's partial results.
template <int D, int SPLIT, class SumOf>
__device__ __forceinline__ void dq_merge_rows(const BwdParams& p, int tile, int h, int which, SumOf sum_of) {
    constexpr int BM = kFwdTileRows, V4 = D / 4;
    constexpr int PER = BM * V4 / SPLIT;
    for (int e = which * PER + (int)threadIdx.x; e < (which + 1) * PER; e += 256) {
        const int rl = e / V4, d4 = e % V4;
        const int row = tile * BM + rl;
        if (row >= p.n_q) continue;
        const f32x4 sum = sum_of((size_t)rl * D + d4 * 4);
        const bool real = p.row_hi[row] > 0;
        *reinterpret_cast<bf16x4*>(p.dq + ((size_t)row * p.hq + h) * D + d4 * 4) =
            real ? pack4(sum[0] * p.scale, sum[1] * p.scale, sum[2] * p.scale, sum[3] * p.scale) : pack4(0.f, 0.f, 0.f, 0.f);
    }
}

// Sums the partial dQ of a query tile that was cut at gang boundaries.  kGangMergeSplit workgroups per
// (gang, member): they act if the gang's last piece is the first part of a tile, and then take
// that part and the first piece of every later gang whose (non-empty) share begins inside the tile.  Most have two parts:
// one load after the other, where requesting four together costs registers and repeats loads (21 us against 30, 128K tokens
// on one of eight ranks).
template <int D>
__global__ void __launch_bounds__(256) dq_merge_kernel(const BwdParams p) {
    constexpr int BM = kFwdTileRows, PF = BM * D + 2 * BM;
    const RowSched& s = p.sched;
    const int job = (int)blockIdx.x / kGangMergeSplit, which = (int)blockIdx.x % kGangMergeSplit;
    const int gang = job / s.G, member = job % s.G;
    RowCut cut;
    if (!cut.find(s, gang)) return;
    auto part = [&](int slot) { return p.row_partial + ((size_t)slot * s.G + member) * PF; };
    const float* first = part(cut.first_slot());
    constexpr int CAP = 32;
    __shared__ int s_slots[CAP], s_count;
    const int n_later = gather_later_parts<CAP>(cut, s_slots, &s_count);
    dq_merge_rows<D, kGangMergeSplit>(p, cut.tile, cut.hk * s.G + member, which, [&](size_t at) __attribute__((always_inline)) {
        f32x4 sum = *reinterpret_cast<const f32x4*>(first + at);
        if (n_later <= CAP) {
            for (int i = 0; i < n_later; ++i) sum += *reinterpret_cast<const f32x4*>(part(s_slots[i]) + at);
        } else {
            cut.later_parts([&](int slot) { sum += *reinterpret_cast<const f32x4*>(part(slot) + at); });
        }
        return sum;
    });
}

// The same for tiles divided into parts: the tile of order rank job / hq, if it is one of them.
template <int D>
__global__ void __launch_bounds__(256) dq_merge_parts_kernel(const BwdParams p) {
    constexpr int PF = kFwdTileRows * D + 2 * kFwdTileRows;
    const int job = (int)blockIdx.x / kMergeSplit, which = (int)blockIdx.x % kMergeSplit;
    const int rank = job / p.hq, h = job % p.hq;
    const int4 base = ld_const4(p.row_part_base + 4 * rank);     // first record, records, first partial result
    const int n = base.y;
    if (n < 2) return;
    const float* first = p.row_partial + ((size_t)base.z * p.hq + h) * PF;
    const size_t step = (size_t)p.hq * PF;
    dq_merge_rows<D, kMergeSplit>(p, ld_const(p.sched.order + rank), h, which, [&](size_t at) __attribute__((always_inline)) {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
        for (int i0 = 0; i0 < n; i0 += 4) {                      // the loads of four parts together
            f32x4 x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = *reinterpret_cast<const f32x4*>(first + min(i0 + i, n - 1) * step + at);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i0 + i < n) sum += x[i];
        }
        return sum;
    });
}

// dK/dV of calls in which few rows can see any one key tile (documents of a few dozen tokens); the schedule decides
// between this kernel and the general one for the call as a whole.  There the general kernel walks whole
// stages of 64 rows x 128 keys of which a third holds visible pairs, and waits for each at a barrier.  Here one
// workgroup takes a key tile and KV head, and each of its four wavefronts works alone -- no barrier -- on 32 keys: it
// holds K, V, dK^T and dV^T of them and walks (query head, 32-row block that can see them), the block's Q, dO and
// per-row scalars copied into LDS of the wavefront's own.  S, P, dP and dS stay in its registers, so nothing is handed
// over, and blocks without a visible pair are never touched.  Two wavefronts per SIMD (one set of tiles each) cover each
// other's copies; one per SIMD with two sets measured slower (111 us for 104).  Bound: the copies alone take 72 us at
// 32K tokens in 979 documents, 16/2 heads (67 for the operands once at the rate of a large copy; 528 MiB are fetched past
// L2 where Q, dO, K and V have 288), the arithmetic alone 54, the kernel 104; one load per line a step ahead to warm L2 made
// it slower.  Workgroups are dealt so that neighbouring key tiles share an XCD.
// With the (then empty) general launch 130 -> 105 us there, 89 -> 62 on one of four ranks, 43 -> 35 at 8K tokens.
template <int D>
struct ShortDkv {
    static constexpr int NW = 4, ROWB = D * 2, TILE = 32 * ROWB;
    static constexpr int SMALL = 4 * 64 * 4;                       // lse2 | delta | row_lo | row_hi, 64 entries each
    static constexpr int WAVE = 2 * TILE + SMALL;              // Q tile | dO tile | scalars
};

template <int D>
__global__ void __launch_bounds__(256, 2) dkv_short_kernel(const BwdParams p) {
    using T = ShortDkv<D>;
    constexpr int KS = D / 16, DB = D / 32, CPR = D / 8, ROWB = T::ROWB, TILE = T::TILE;
    __shared__ __attribute__((aligned(1024))) char smem[T::NW * T::WAVE];
    // XCD x (workgroups b with b % 8 == x) takes a contiguous run of (key tile, KV head)
    const int jobs = p.n_key_tiles * p.hkv, per_xcd = (jobs + kLists - 1) / kLists;
    const int job = ((int)blockIdx.x % kLists) * per_xcd + (int)blockIdx.x / kLists;
    if ((int)blockIdx.x / kLists >= per_xcd || job >= jobs) return;
    if (!ld_const(p.short_on)) return;                           // the general kernel does it (short_keys_pay)
    const int kt = job / p.hkv, hk = job % p.hkv;
    const int g_first = ld_const(p.key_range + 2 * kt), span = ld_const(p.key_range + 2 * kt + 1) - g_first;

    const int G = p.hq / p.hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int j16 = lane & 15, gi = (lane >> 4) & 1;
    const float cs = p.scale_log2e;
    const int kw0 = kt * kBwdKeyTile + wave * 32, mykey = kw0 + l32;

    // the 32-row blocks that can see one of the wavefront's keys
    const int rb0 = g_first * (kGroupRows / kShortBlockRows), n_rb = span * (kGroupRows / kShortBlockRows);
    static_assert(kShortSpan * (kGroupRows / kShortBlockRows) <= 32, "a lane per row block");
    int b_lo = 0, b_hi = 0;
    if (lane < n_rb) { b_lo = p.block_hull[2 * (rb0 + lane)]; b_hi = p.block_hull[2 * (rb0 + lane) + 1]; }
    const uint32_t blocks = (uint32_t)__ballot(b_hi > b_lo && b_lo < kw0 + 32 && b_hi > kw0);
    const int steps = __popc(blocks) * G;

    const uint32_t base = uniform((uint32_t)(uintptr_t)(WLB_LDS char*)smem + (uint32_t)wave * T::WAVE);
    const uint32_t q_row_bytes = (uint32_t)p.hq * D * 2u;
    const uint32_t q_total = (uint32_t)p.n_q * q_row_bytes;
    BufRsrc q_rs, do_rs, lo_rs, hi_rs, ls_rs, dl_rs;
    q_rs.init(p.q, q_total);
    do_rs.init(p.d_o, q_total);
    lo_rs.init(p.row_lo, (uint32_t)p.n_q * 4u);
    hi_rs.init(p.row_hi, (uint32_t)p.n_q * 4u);
    // The swizzle is an XOR of chunk and row bits, tiles are 1 KiB aligned and rows 128 or 256 bytes: an instruction's
    // lane offsets and an operand's addresses are one register each, XORed with a constant (with all of them in
    // registers the kernel spills).
    constexpr int RPI = 64 / CPR, NI = 32 / RPI;                   // rows per copy instruction, instructions per tile
    int voff0 = (lane / CPR) * (int)q_row_bytes + swz<CPR>(lane / CPR, lane % CPR) * 16;
    // the copies of one step: 32 rows of Q and dO of a head (rows past n_q read as zeros) and the rows' scalars
    auto issue = [&](int rb, int h) __attribute__((always_inline)) {
        const uint32_t so = uniform((uint32_t)rb * 32u * q_row_bytes + (uint32_t)h * ROWB);
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int voff = voff0 ^ (swz<CPR>(n * RPI, 0) * 16);
            const uint32_t off = (uint32_t)(n * RPI) * q_row_bytes;
            dma_issue_1k(q_rs.r, uniform(base + n * 1024u), voff, uniform(so + off));
            dma_issue_1k(do_rs.r, uniform(base + TILE + n * 1024u), voff, uniform(so + off));
        }
        const size_t ho = (size_t)h * p.n_q;
        ls_rs.init(p.lse2 + ho, (uint32_t)p.n_q * 4u);             // per head: entries past n_q read as zeros
        dl_rs.init(p.delta + ho, (uint32_t)p.n_q * 4u);
        const uint32_t ro = uniform((uint32_t)rb * 128u), sm = uniform(base + 2 * TILE);
        dma_issue_256(ls_rs.r, sm, lane * 4, ro);
        dma_issue_256(dl_rs.r, uniform(sm + 256u), lane * 4, ro);
        dma_issue_256(lo_rs.r, uniform(sm + 512u), lane * 4, ro);
        dma_issue_256(hi_rs.r, uniform(sm + 768u), lane * 4, ro);
    };
    // query heads outermost: the wavefronts of a workgroup, whose keys the same rows see, then read those rows of a head
    // close together in time and share them in L2 (row blocks outermost: 121 us against 104 at 32K tokens, 16/2 heads)
    uint32_t left = blocks;
    int rb_n = rb0 + __ffs((int)left) - 1, h_n = hk * G;
    auto advance = [&] {
        left &= left - 1;
        if (left == 0) { left = blocks; ++h_n; }
        rb_n = rb0 + __ffs((int)left) - 1;
    };
    if (steps > 0) { issue(rb_n, h_n); advance(); }

    bf16x8 kop[KS], vop[KS];
    {
        const size_t row = ((size_t)min(mykey, p.t_kv - 1) * p.hkv + hk) * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            kop[ks] = *reinterpret_cast<const bf16x8*>(p.k + row + ks * 16);
            vop[ks] = *reinterpret_cast<const bf16x8*>(p.v + row + ks * 16);
        }
    }
    f32x16 dk[DB], dv[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dk[db][r] = 0.f; dv[db][r] = 0.f; }
    // rows read as they lie: chunk 2 ks + half of row l32; read transposed: rows qq and, with bit 5 flipped, qq + 8 (whose swizzle differs in bit 1)
    uint32_t naddr = base + l32 * ROWB + swz<CPR>(l32, half) * 16;
    const int qq = half * 4 + (j16 >> 2);
    uint32_t taddr = base + qq * ROWB + swz<CPR>(qq, gi * 2 + ((j16 & 3) >> 1)) * 16 + (j16 & 1) * 8;
    static_assert(TILE % 1024 == 0 && T::WAVE % 1024 == 0, "bit 5 of a tile's address is the swizzle's");
    const uint32_t saddr = base + 2 * TILE + half * 16;
    // the K / V operands have arrived: no compiler-visible vector load may be pending among the copies
    wait_vmem();

    auto fence = [] () __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
    for (int s = 0; s < steps; ++s) {
        wait_vmem();
        asm volatile("" : "+v"(naddr), "+v"(taddr), "+v"(voff0) :: "memory");   // (keeps the XORs inside the loop)
        // padding rows may hold anything: zero their Q and dO (rows past n_q are zeros already)
        const int my_hi = *reinterpret_cast<const WLB_LDS int*>((uintptr_t)(base + 2 * TILE + 768 + l32 * 4));
        if (__any(my_hi == 0)) {
            if (my_hi == 0) {
#pragma unroll
                for (int i = 0; i < CPR / 2; ++i) {
                    const uint32_t a = base + l32 * ROWB + (half * (CPR / 2) + i) * 16;
                    *reinterpret_cast<WLB_LDS i32x4*>((uintptr_t)a) = i32x4{0, 0, 0, 0};
                    *reinterpret_cast<WLB_LDS i32x4*>((uintptr_t)(a + TILE)) = i32x4{0, 0, 0, 0};
                }
            }
            asm volatile("" ::: "memory");
        }
        bf16x8 pk[2], ds[2];
        {
            f32x16 sc;
#pragma unroll
            for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) sc = mfma32(*reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(naddr ^ (ks * 32))), kop[ks], sc);
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                float pr[8];
#pragma unroll
                for (int r2 = 0; r2 < 2; ++r2) {
                    const int off = (cc * 2 + r2) * 32;
                    const f32x4 ls = *reinterpret_cast<const WLB_LDS f32x4*>((uintptr_t)(saddr + off));
                    const i32x4 lo = *reinterpret_cast<const WLB_LDS i32x4*>((uintptr_t)(saddr + off + 512));
                    const i32x4 hi = *reinterpret_cast<const WLB_LDS i32x4*>((uintptr_t)(saddr + off + 768));
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float e = fast_exp2(fmaf(sc[(cc * 2 + r2) * 4 + i], cs, -ls[i]));
                        pr[r2 * 4 + i] = (mykey >= lo[i] && mykey < hi[i]) ? e : 0.f;
                    }
                }
                pk[cc] = pack8(pr[0], pr[1], pr[2], pr[3], pr[4], pr[5], pr[6], pr[7]);
            }
        }
        fence();
        {
            f32x16 dp;
#pragma unroll
            for (int g8 = 0; g8 < 4; ++g8) {
                const f32x4 x = *reinterpret_cast<const WLB_LDS f32x4*>((uintptr_t)(saddr + 256 + g8 * 32));
#pragma unroll
                for (int i = 0; i < 4; ++i) dp[g8 * 4 + i] = x[i];
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) dp = mfma32(*reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)((naddr ^ (ks * 32)) + TILE)), vop[ks], dp);
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                float g[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) g[i] = (float)pk[cc][i] * dp[cc * 8 + i];
                ds[cc] = pack8(g[0], g[1], g[2], g[3], g[4], g[5], g[6], g[7]);
            }
        }
        fence();
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const uint32_t a0 = (taddr ^ (db * 64)) + cc * 16 * ROWB, a1 = (taddr ^ (db * 64 + 32)) + (cc * 16 + 8) * ROWB;
                dv[db] = mfma32(cat4(lds_read_tr4_at(a0 + TILE), lds_read_tr4_at(a1 + TILE)), pk[cc], dv[db]);
                dk[db] = mfma32(cat4(lds_read_tr4_at(a0), lds_read_tr4_at(a1)), ds[cc], dk[db]);
            }
        if (s + 1 < steps) {
            wait_lds();                                            // the tiles have been read to the end
            issue(rb_n, h_n);
            advance();
        }
    }

    // dK and dV leave as whole rows through the tiles; keys past t_kv are not stored
    wait_lds();
    asm volatile("" ::: "memory");
    const uint32_t kv_row_bytes = (uint32_t)p.hkv * D * 2u, kv_total = (uint32_t)p.t_kv * kv_row_bytes;
    const int voff = RowBlock<D>::lane_off(lane, kv_row_bytes);
    const uint32_t soff = uniform((uint32_t)kw0 * kv_row_bytes + (uint32_t)hk * ROWB);
    auto put = [&](const f32x16 (&acc)[DB], float f, __bf16* dst, uint32_t tile) __attribute__((always_inline)) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                *reinterpret_cast<WLB_LDS bf16x4*>((uintptr_t)(tile + l32 * ROWB + swz<CPR>(l32, db * 4 + r4) * 16 + half * 8)) =
                    pack4(acc[db][r4 * 4 + 0] * f, acc[db][r4 * 4 + 1] * f, acc[db][r4 * 4 + 2] * f, acc[db][r4 * 4 + 3] * f);
        asm volatile("" ::: "memory");
        RowBlock<D> rows;
        rows.from_tile(tile, lane);
        rows.store(make_buf(dst, kv_total), voff, soff, kv_row_bytes);
    };
    put(dk, p.scale, p.dk, base);
    put(dv, 1.0f, p.dv, base + TILE);
}

// Sums the partial results of the key tiles that were split into several items.
// One workgroup per (tile in order, KV head).
template <int D>
__global__ void __launch_bounds__(256) dkv_fixup_kernel(const BwdParams p) {
    constexpr int BNK = kBwdKeyTile;
    // the item counters of the dK/dV launch that has just finished go back to zero for the next one
    if (blockIdx.x == 0 && threadIdx.x < kLists) p.dkv_counters[threadIdx.x] = 0;
    const int job = (int)blockIdx.x / kMergeSplit, which = (int)blockIdx.x % kMergeSplit;
    const int hk = job % p.hkv, r = job / p.hkv;
    const int kt = p.key_order[r];
    const int ways = p.key_ways[kt];
    if (ways == 1) return;                      // one item did the whole tile and wrote dK/dV itself
    if (p.short_on && *p.short_on) return;      // dkv_short_kernel did
    const int k0 = kt * BNK, nk = min(BNK, p.t_kv - k0);
    const float* src = p.partial + (size_t)(p.key_slot_base[r] + hk * ways) * (2 * BNK * D);
    constexpr int V4 = D / 4;                   // float4 per row
    constexpr int PER = 2 * BNK * V4 / kMergeSplit;
    // The pass is bound by the latency of its loads: those of U elements and W parts (W = 8: in turns) are requested
    // together (8191 tokens, 8/2 heads: 13.8 -> 7.6 us).
    auto sum_parts = [&](auto parts_tag) __attribute__((always_inline)) {
        constexpr int W = decltype(parts_tag)::value, U = PER / 256 < 4 ? PER / 256 : 4;
        static_assert(PER % (U * 256) == 0, "elements per thread");
        for (int e0 = which * PER + (int)threadIdx.x; e0 < (which + 1) * PER; e0 += U * 256) {
            f32x4 sum[U];
#pragma unroll
            for (int u = 0; u < U; ++u) sum[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int i0 = 0; i0 < ways; i0 += W) {
                f32x4 x[U][W];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int i = 0; i < W; ++i)
                        x[u][i] = *reinterpret_cast<const f32x4*>(src + (size_t)(i0 + i) * (2 * BNK * D) + (size_t)(e0 + u * 256) * 4);
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int i = 0; i < W; ++i) sum[u] += x[u][i];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = e0 + u * 256, grad = e / (BNK * V4), rem = e % (BNK * V4);
                const int key = rem / V4, d4 = rem % V4;
                const float f = grad == 0 ? p.scale : 1.0f;
                __bf16* op = (grad == 0 ? p.dk : p.dv) + ((size_t)(k0 + key) * p.hkv + hk) * D + d4 * 4;
                if (key < nk) *reinterpret_cast<bf16x4*>(op) = pack4(sum[u][0] * f, sum[u][1] * f, sum[u][2] * f, sum[u][3] * f);
            }
        }
    };
    if (ways == 2) sum_parts(std::integral_constant<int, 2>{});
    else if (ways == 4) sum_parts(std::integral_constant<int, 4>{});
    else sum_parts(std::integral_constant<int, 8>{});        // a power of two
}

// dQ (+ merge), which leaves delta, then dK/dV (+ fix-up), all on the caller's stream.  Running dQ beside
// dK/dV on a second stream was measured: once each kernel keeps every compute unit busy to its end
// the two only get in each other's way (their workgroups cannot share a compute unit's LDS), and the
// step was 4 % slower.
wlb_status launch_bwd(const wlb_attn_desc& d, const PlanLayout& L, const void* q, const void* k,
                      const void* v, const void* o, const float* lse, const void* d_o, void* dq,
                      void* dk, void* dv, char* ws, size_t off_delta, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    BwdParams p;
    p.q = (const __bf16*)q; p.k = (const __bf16*)k; p.v = (const __bf16*)v;
    p.o = (const __bf16*)o; p.d_o = (const __bf16*)d_o; p.lse = lse;
    p.delta = (float*)(ws + off_delta);
    p.lse2 = (float*)(ws + off_delta + align_up(sizeof(float) * (size_t)d.hq * d.n_q, 256));
    p.dq = (__bf16*)dq; p.dk = (__bf16*)dk; p.dv = (__bf16*)dv;
    p.row_lo = (const int32_t*)(ws + L.off_row_lo);
    p.row_hi = (const int32_t*)(ws + L.off_row_hi);
    p.key_order = (const int32_t*)(ws + L.off_key_order);
    p.dkv_item = (const int32_t*)(ws + L.off_dkv_item);
    p.key_range = (const int32_t*)(ws + L.off_key_range);
    p.short_on = use_short_keys(d, L) ? (const int32_t*)(ws + L.off_short_on) : nullptr;
    p.key_ways = (const int32_t*)(ws + L.off_key_ways);
    p.key_item_base = (const int32_t*)(ws + L.off_key_item_base);
    p.key_slot_base = (const int32_t*)(ws + L.off_key_slot_base);
    p.dkv_counters = (int32_t*)(ws + L.off_dkv_counters);
    p.partial = (float*)(ws + off_delta + 2 * align_up(sizeof(float) * (size_t)d.hq * d.n_q, 256));
    p.sched.prefix = (const long long*)(ws + L.off_fwd_prefix);
    p.sched.order = (const int32_t*)(ws + L.off_fwd_order);
    p.sched.tile_first = (const int32_t*)(ws + L.off_tile_first);
    const bool parts = use_row_parts(d, L);
    p.first_half = row_first_half(d);
    p.row_item = (const int32_t*)(ws + (parts ? L.off_row_part : L.off_row_item));
    p.row_part_base = parts ? (const int32_t*)(ws + L.off_row_part_base) : nullptr;
    p.sched.n_tiles = L.n_fwd_tiles; p.sched.hkv = d.hkv; p.sched.G = d.hq / d.hkv; p.sched.n_gangs = L.row_gangs;
    gang_weights(1, p.sched.weight);
    p.row_partial = (float*)((char*)p.partial + dkv_partial_bytes(d, L));
    p.block_hull = (const int32_t*)(ws + L.off_block_hull);
    p.tile_short = (const int32_t*)(ws + L.off_tile_short);
    p.n_blocks32 = L.n_blocks32;
    p.gang_clock = (unsigned long long*)(ws + L.off_gang_clock) + 2 * (size_t)L.row_gangs * (d.hq / d.hkv);
    p.n_q = d.n_q; p.t_kv = d.t_kv; p.hq = d.hq; p.hkv = d.hkv;
    p.n_groups = L.n_groups; p.n_tiles = L.n_fwd_tiles; p.n_key_tiles = L.n_key_tiles;
    p.scale = d.scale;
    p.scale_log2e = d.scale * 1.4426950408889634f;

    // workgroups per query tile in the delta pass: enough to fill the GPU, at most one per 256 lanes of the tile
    const size_t tile_iters = (size_t)kFwdTileRows * d.hq * (d.head_dim / 8) / 256;
    const size_t delta_split = std::max<size_t>(1, std::min(tile_iters, (8 * (size_t)compute_units() + L.n_fwd_tiles - 1) / L.n_fwd_tiles));
    const unsigned grid_delta = (unsigned)(delta_split * L.n_fwd_tiles);
    const unsigned grid_dq = (unsigned)L.row_gangs * (unsigned)(d.hq / d.hkv);
    const unsigned grid_dq_items = (unsigned)((L.n_fwd_tiles + (parts ? row_parts_added(d, L) : 0) + 7) / 8) * 8u * (unsigned)d.hq;
    const unsigned grid_dq_parts = (unsigned)row_tiles_divided(d, L) * (unsigned)d.hq * kMergeSplit;
    const bool gangs = use_row_gangs(d, L), pairs = use_dq_pairs(d, L);
    if (gangs && pairs) pair_weights(p.sched.weight);
    // one workgroup per compute unit, each taking item after item
    const unsigned grid_dkv = (unsigned)std::min(L.dkv_max_items, compute_units());   // one workgroup per compute unit, each taking item after item
    const unsigned grid_fix = (unsigned)(L.n_key_tiles * d.hkv);
    const bool do_delta = !(d.flags & WLB_ATTN_BWD_SKIP_DELTA);
    const bool do_dq = !(d.flags & WLB_ATTN_BWD_SKIP_DQ);
    const bool do_dkv = !(d.flags & WLB_ATTN_BWD_SKIP_DKV);
    p.use_short = use_short_path(d, L) ? 1 : 0;
    const unsigned grid_short = (unsigned)((L.n_key_tiles * d.hkv + kLists - 1) / kLists) * kLists;
    auto run = [&](auto dtag) {
        constexpr int D = decltype(dtag)::value;
        if (do_dq && use_span(d, L)) {
            launch_dq_span(p, D, stream);
        } else if (do_dq && gangs) {
            if (pairs) launch_dq_pair(p, true, grid_dq / 2, stream);
            else dq_kernel<D><<<grid_dq, 256, 0, stream>>>(p);
            dq_merge_kernel<D><<<grid_dq * kGangMergeSplit, 256, 0, stream>>>(p);
        } else if (do_dq && pairs) {
            launch_dq_pair(p, false, grid_dq_items / 2, stream);           // (no parts)
            if (p.use_short) dq_short_tiles_kernel<D><<<short_tiles_grid(d, L), 256, 0, stream>>>(p);
        } else if (do_dq) {
            dq_items_kernel<D><<<grid_dq_items, 256, 0, stream>>>(p);
            if (parts) dq_merge_parts_kernel<D><<<grid_dq_parts, 256, 0, stream>>>(p);
        } else if (do_delta) {
            delta_kernel<D><<<grid_delta, 256, 0, stream>>>(p);
        }
        if (do_dkv) {
            if (p.short_on) {
                dkv_short_kernel<D><<<grid_short, 256, 0, stream>>>(p);
                launch_dkv_general(p, D, true, grid_dkv, stream);
            } else {
                launch_dkv_general(p, D, false, grid_dkv, stream);
            }
            dkv_fixup_kernel<D><<<grid_fix * kMergeSplit, 256, 0, stream>>>(p);
        }
    };
    if (d.head_dim == 128) run(std::integral_constant<int, 128>{});
    else run(std::integral_constant<int, 64>{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(WLB_ERR_HIP, "backward launch: %s", hipGetErrorString(e));
    return WLB_OK;
}

}  // namespace wlb
