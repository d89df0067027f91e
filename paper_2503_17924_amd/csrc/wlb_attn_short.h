// Short-hull units of the forward and of dQ (wlb_attn_fwd.hip and wlb_attn_bwd.hip have the arithmetic): device code that several launches share.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "wlb_attn_bwd.h"
#include "wlb_attn_fwd.h"
#include "wlb_device.h"
#include "wlb_internal.h"

namespace wlb {

// Short-hull tiles (documents of a few dozen tokens, where a tile's rows see only the keys next to
// them: the short-chunk case of paper Section 5.2).  There the general piece of work is bound by
// latency: per (tile, head) it fetches K/V, waits, and computes a handful of blocks.  A short-hull
// unit is one block of 32 rows and one KV head, run by a workgroup of the one-workgroup-per-item
// launch: it copies the (at most 96) keys the block sees into LDS
// once -- K and V, in one shot -- and its four wavefronts then work independently, one query head
// each at a time (heads w, w+4, ... of the KV head), with no further barrier.  Per head a wavefront
// loads its 32 Q rows as whole rows and passes them through a staging tile of its own into the MFMA
// operand layout (loading the operand straight from global memory would touch 32 rows x 32 bytes per
// instruction), computes the scores of the up to three 32-key blocks, the exact row maximum, the
// exponentials and O^T += V^T P^T, and sends O through the staging tile so that it leaves in whole
// rows as well.  Eight wavefronts per compute unit keep Q loads and O stores in flight; K/V
// traffic is one LDS fill per 32 rows and KV head instead of one per head.
template <int D>
struct ShortTile {
    static constexpr int KS = D / 16, DB = D / 32, CPR = D / 8, ROWB = D * 2;
    static constexpr int HULL = kShortHullKeys, NB = HULL / 32, NW = 4;
    static constexpr int STAGE = kShortBlockRows * ROWB;              // one wavefront's staging tile: 32 rows
    static constexpr int LDS_BYTES = 2 * HULL * ROWB + NW * STAGE;    // K window | V window | staging tiles
    static constexpr int RPI = 64 / CPR;                              // rows moved by one 64 x 16-byte instruction
};

template <int D, int NW = ShortTile<D>::NW>
__device__ __forceinline__ void fwd_short_unit(const FwdParams& p, char* smem, int blk, int hk) {
    using T = ShortTile<D>;
    constexpr int KS = T::KS, DB = T::DB, CPR = T::CPR, ROWB = T::ROWB, HULL = T::HULL, NB = T::NB;
    const int G = p.hq / p.hkv;
    __syncthreads();              // every wavefront has left the LDS of the unit before

    const int tid = threadIdx.x, lane = tid & 63, wave = uniform((tid >> 6) & (NW - 1));
    const int l32 = lane & 31, half = lane >> 5;
    const int j16 = lane & 15, gi = (lane >> 4) & 1;
    const int h_lo = ld_const(p.block_hull + 2 * blk), h_hi = ld_const(p.block_hull + 2 * blk + 1);
    const int row0 = blk * kShortBlockRows;
    const int row = row0 + l32;
    const bool in = row < p.n_q;
    const int rc = in ? row : p.n_q - 1;
    const uint32_t q_row = (uint32_t)p.hq * D;

    const uint32_t q_row_bytes = q_row * 2u;
    const buf_rsrc_t q_buf = make_buf(p.q, (uint32_t)p.n_q * q_row_bytes), o_buf = make_buf(p.o, (uint32_t)p.n_q * q_row_bytes);
    const int row_voff = RowBlock<D>::lane_off(lane, q_row_bytes);
    auto head_soff = [&](int hs) { return uniform((uint32_t)row0 * q_row_bytes + (uint32_t)(hk * G + hs) * ROWB); };

    if (h_hi <= h_lo) {
        // no real row in this block: O = 0, LSE = -inf for every head of the KV head
        RowBlock<D> zero;
#pragma unroll
        for (int i = 0; i < RowBlock<D>::N; ++i) zero.v[i] = i32x4{0, 0, 0, 0};
        for (int hs = wave; hs < G; hs += NW) {
            zero.store(o_buf, row_voff, head_soff(hs), q_row_bytes);
            if (in && half == 0) p.lse[(size_t)(hk * G + hs) * p.n_q + row] = -INFINITY;
        }
        __syncthreads();          // as many as in a unit with real rows (short_units_of_512)
        return;
    }
    const int kstart = h_lo & ~31;
    const int nblk = (h_hi - kstart + 31) >> 5;          // 1 .. NB (the schedule marks the tile short only then)

    const uint32_t smem_base = (uint32_t)(uintptr_t)(WLB_LDS char*)smem;
    const uint32_t stage = uniform(smem_base + 2 * HULL * ROWB + (uint32_t)wave * T::STAGE);
    const uint32_t kv_row = (uint32_t)p.hkv * D;
    const uint32_t kv_bytes = ((uint32_t)p.t_kv * kv_row - (uint32_t)hk * D) * 2u;
    BufRsrc krs, vrs;
    krs.init(p.k + (size_t)hk * D, kv_bytes);
    vrs.init(p.v + (size_t)hk * D, kv_bytes);
    TileDma<D, 32 * NW, NW> dma;                          // wavefront w copies the 32-key block w
    static_assert(TileDma<D, 32 * NW, NW>::PER * TileDma<D, 32 * NW, NW>::RPI == 32, "one 32-key block per wavefront");
    dma.init(wave, lane, kv_row);
    if (wave < nblk) {
        dma.issue(krs, smem_base, kstart, wave);
        dma.issue(vrs, smem_base + HULL * ROWB, kstart, wave);
    }

    const int lo = in ? p.row_lo[rc] : kPadLo;
    const int hi = in ? p.row_hi[rc] : 0;
    const bool real = hi > 0;

    int kaddr[KS], vaddr[DB][2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kaddr[ks] = l32 * ROWB + swz<CPR>(l32, ks * 2 + half) * 16;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int key = t * 8 + half * 4 + (j16 >> 2);
            const int dch = db * 4 + gi * 2 + ((j16 & 3) >> 1);
            vaddr[db][t] = smem_base + HULL * ROWB + key * ROWB + swz<CPR>(key, dch) * 16 + (j16 & 1) * 8;
        }
    const float cs = p.scale_log2e;

    wait_vmem();
    __syncthreads();              // the key window is in LDS; from here on the wavefronts do not meet again

#pragma nounroll
    for (int hs = wave; hs < G; hs += NW) {
        const int h = hk * G + hs;
        // this head's Q rows: whole rows into registers, then through the staging tile into the operand layout
        // (eight wavefronts per compute unit cover each other's load latency)
        {
            RowBlock<D> q_rows;
            q_rows.load(q_buf, row_voff, head_soff(hs), q_row_bytes);
            q_rows.to_tile(stage, lane);
        }
        bf16x8 qf[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(stage + kaddr[ks]));

        f32x16 s[NB];
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[b][r] = -INFINITY;
            if (b < nblk) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[b][r] = 0.f;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const bf16x8 a = *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(smem_base + kaddr[ks] + b * 32 * ROWB));
                    s[b] = mfma32(a, qf[ks], s[b]);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kstart + b * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
                    s[b][r] = (key >= lo && key < hi) ? s[b][r] : -INFINITY;
                    mx = fmaxf(mx, s[b][r]);
                }
            }
        }
        mx = fmaxf(mx, xhalf(mx));
        const float mc = (mx == -INFINITY) ? 0.f : mx * cs;
        f32x16 acc[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
        float l = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b < nblk) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float e = fast_exp2(fmaf(s[b][r], cs, -mc));
                    s[b][r] = e;
                    l += e;
                }
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    const bf16x8 pf = pack8(s[b][8 * cc + 0], s[b][8 * cc + 1], s[b][8 * cc + 2], s[b][8 * cc + 3],
                                            s[b][8 * cc + 4], s[b][8 * cc + 5], s[b][8 * cc + 6], s[b][8 * cc + 7]);
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        const int off = (b * 32 + cc * 16) * ROWB;
                        const bf16x4 v0 = lds_read_tr4_at(vaddr[db][0] + off);
                        const bf16x4 v1 = lds_read_tr4_at(vaddr[db][1] + off);
                        acc[db] = mfma32(cat4(v0, v1), pf, acc[db]);
                    }
                }
            }
        }
        const float lt = l + xhalf(l);
        const bool live = real && (lt > 0.f);
        const float inv = live ? 1.0f / lt : 0.f;
        if (__any(!live)) {                         // (0 x V is NaN where V is not finite)
            asm volatile("");                       // keep it a branch
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[db][r] = live ? acc[db][r] : 0.f;
        }
        // O rows through the staging tile (its Q rows are in registers by now): written in the
        // accumulator's layout, read back and stored as whole rows
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                *reinterpret_cast<WLB_LDS bf16x4*>((uintptr_t)(stage + l32 * ROWB + swz<CPR>(l32, db * 4 + r4) * 16 + half * 8)) =
                    pack4(acc[db][r4 * 4 + 0] * inv, acc[db][r4 * 4 + 1] * inv, acc[db][r4 * 4 + 2] * inv, acc[db][r4 * 4 + 3] * inv);
        RowBlock<D> o_rows;
        o_rows.from_tile(stage, lane);
        o_rows.store(o_buf, row_voff, head_soff(hs), q_row_bytes);
        if (in && half == 0) p.lse[(size_t)h * p.n_q + row] = live ? mx * p.scale + __logf(lt) : -INFINITY;
        wait_lds();                                 // the staging tile has been read back
    }
}

// dQ of short-hull tiles, the counterpart of the forward's short-hull kernel (same workgroup shape,
// same LDS layout: K window | V window | one staging tile per wavefront; see there).  A wavefront
// works on one query head at a time; that head's rows of Q and dO reach it as whole rows and pass
// through the staging tile into the MFMA operand layout.  All keys a row sees lie inside the window, so the wavefront has the row's whole
// P and dP and forms delta itself as sum_j P_ij dP_ij (equal to <dO_i, O_i> since O = P V), without
// reading O: first pass per 32-key block S^T, dP^T, P and X = P o dP (both kept as bf16), then
// dS^T = X - delta P and dQ^T += K^T dS^T.  delta (negated) and the log2-scaled LSE copy are left
// for the dK/dV kernel, which runs after this one.
template <int D>
struct ShortDq {
    static constexpr int NW = 4, ROWB = D * 2, HULL = kShortHullKeys, STAGE = kShortBlockRows * ROWB;
    static constexpr int LDS_BYTES = 2 * HULL * ROWB + NW * STAGE;    // K window | V window | staging tiles
};

template <int D, int NW = ShortDq<D>::NW>
__device__ __forceinline__ void dq_short_unit(const BwdParams& p, char* smem, int blk, int hk) {
    constexpr int KS = D / 16, DB = D / 32, CPR = D / 8, ROWB = D * 2;
    constexpr int HULL = kShortHullKeys, NB = HULL / 32, STAGE = kShortBlockRows * ROWB, RPI = 64 / CPR;
    const int G = p.hq / p.hkv;
    __syncthreads();              // every wavefront has left the LDS of the unit before

    const int tid = threadIdx.x, lane = tid & 63, wave = uniform((tid >> 6) & (NW - 1));
    const int l32 = lane & 31, half = lane >> 5;
    const int j16 = lane & 15, gi = (lane >> 4) & 1;
    const int h_lo = ld_const(p.block_hull + 2 * blk), h_hi = ld_const(p.block_hull + 2 * blk + 1);
    const int row0 = blk * kShortBlockRows;
    const int row = row0 + l32;
    const bool in = row < p.n_q;
    const int rc = in ? row : p.n_q - 1;
    const uint32_t q_row = (uint32_t)p.hq * D;

    const uint32_t q_row_bytes = q_row * 2u;
    const buf_rsrc_t q_buf = make_buf(p.q, (uint32_t)p.n_q * q_row_bytes), do_buf = make_buf(p.d_o, (uint32_t)p.n_q * q_row_bytes),
                     dq_buf = make_buf(p.dq, (uint32_t)p.n_q * q_row_bytes);
    const int row_voff = RowBlock<D>::lane_off(lane, q_row_bytes);
    auto head_soff = [&](int hs) { return uniform((uint32_t)row0 * q_row_bytes + (uint32_t)(hk * G + hs) * ROWB); };

    if (h_hi <= h_lo) {
        // no real row in this block: dQ = 0; delta = 0 and LSE copy = +inf keep the rows out of dK/dV
        RowBlock<D> zero;
#pragma unroll
        for (int i = 0; i < RowBlock<D>::N; ++i) zero.v[i] = i32x4{0, 0, 0, 0};
        for (int hs = wave; hs < G; hs += NW) {
            const int h = hk * G + hs;
            zero.store(dq_buf, row_voff, head_soff(hs), q_row_bytes);
            if (in && half == 0) {
                p.delta[(size_t)h * p.n_q + row] = 0.f;
                p.lse2[(size_t)h * p.n_q + row] = INFINITY;
            }
        }
        __syncthreads();          // as many as in a unit with real rows (short_units_of_512)
        return;
    }
    const int kstart = h_lo & ~31;
    const int nblk = (h_hi - kstart + 31) >> 5;

    const uint32_t smem_base = (uint32_t)(uintptr_t)(WLB_LDS char*)smem;
    const uint32_t stage = uniform(smem_base + 2 * HULL * ROWB + (uint32_t)wave * STAGE);

    const uint32_t kv_row = (uint32_t)p.hkv * D;
    const uint32_t kv_bytes = ((uint32_t)p.t_kv * kv_row - (uint32_t)hk * D) * 2u;
    BufRsrc krs, vrs;
    krs.init(p.k + (size_t)hk * D, kv_bytes);
    vrs.init(p.v + (size_t)hk * D, kv_bytes);
    TileDma<D, 32 * NW, NW> dma;                          // wavefront w copies the 32-key block w
    dma.init(wave, lane, kv_row);
    if (wave < nblk) {
        dma.issue(krs, smem_base, kstart, wave);
        dma.issue(vrs, smem_base + HULL * ROWB, kstart, wave);
    }

    const int lo = in ? p.row_lo[rc] : kPadLo;
    const int hi = in ? p.row_hi[rc] : 0;
    const bool real = hi > 0;
    int naddr[KS], taddr[DB][2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) naddr[ks] = l32 * ROWB + swz<CPR>(l32, ks * 2 + half) * 16;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int key = t * 8 + half * 4 + (j16 >> 2);
            const int dch = db * 4 + gi * 2 + ((j16 & 3) >> 1);
            taddr[db][t] = smem_base + key * ROWB + swz<CPR>(key, dch) * 16 + (j16 & 1) * 8;
        }
    const float cs = p.scale_log2e;
    // padding rows: zero operands and LSE = +inf make P, dS and dQ exactly 0 (their Q / dO may hold anything)
    auto rows_from_stage = [&](bf16x8 (&dst)[KS]) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bf16x8 a = *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(stage + naddr[ks]));
            if (!real) {
#pragma unroll
                for (int i = 0; i < 8; ++i) a[i] = (__bf16)0.f;
            }
            dst[ks] = a;
        }
    };

    wait_vmem();
    __syncthreads();              // the key window is in LDS; the wavefronts do not meet again

#pragma nounroll
    for (int hs = wave; hs < G; hs += NW) {
        const int h = hk * G + hs;
        // this head's rows of Q and dO: whole rows into registers, then through the staging tile into the
        // operand layout (eight wavefronts per compute unit cover each other's load latency)
        bf16x8 qf[KS], dof[KS];
        {
            RowBlock<D> q_rows, do_rows;
            q_rows.load(q_buf, row_voff, head_soff(hs), q_row_bytes);
            do_rows.load(do_buf, row_voff, head_soff(hs), q_row_bytes);
            q_rows.to_tile(stage, lane);
            rows_from_stage(qf);
            wait_lds();
            do_rows.to_tile(stage, lane);
            rows_from_stage(dof);
        }
        const float lse_cur = real ? p.lse[(size_t)h * p.n_q + rc] * 1.4426950408889634f : INFINITY;

        // first pass: P and X = P o dP of every block (masked entries 0), delta = sum of X over the row
        bf16x8 pk[NB][2], xk[NB][2];
        float dsum = 0.f, psum = 0.f, dsum_r = 0.f, psum_r = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b < nblk) {
                f32x16 sc, dp;
#pragma unroll
                for (int r = 0; r < 16; ++r) { sc[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const bf16x8 ka = *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(smem_base + naddr[ks] + b * 32 * ROWB));
                    const bf16x8 va = *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(smem_base + naddr[ks] + (HULL + b * 32) * ROWB));
                    sc = mfma32(ka, qf[ks], sc);
                    dp = mfma32(va, dof[ks], dp);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kstart + b * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
                    const float pr = (key >= lo && key < hi) ? fast_exp2(fmaf(sc[r], cs, -lse_cur)) : 0.f;
                    sc[r] = pr;
                    dp[r] = pr * dp[r];
                    psum += pr;
                    dsum += dp[r];
                }
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    pk[b][cc] = pack8(sc[8 * cc + 0], sc[8 * cc + 1], sc[8 * cc + 2], sc[8 * cc + 3],
                                      sc[8 * cc + 4], sc[8 * cc + 5], sc[8 * cc + 6], sc[8 * cc + 7]);
                    xk[b][cc] = pack8(dp[8 * cc + 0], dp[8 * cc + 1], dp[8 * cc + 2], dp[8 * cc + 3],
                                      dp[8 * cc + 4], dp[8 * cc + 5], dp[8 * cc + 6], dp[8 * cc + 7]);
                    // this kernel's own delta comes from the rounded X and P that dS is formed from below, so
                    // that they cancel exactly where they should (a row that sees one key: dS = 0)
#pragma unroll
                    for (int i = 0; i < 8; ++i) { dsum_r += (float)xk[b][cc][i]; psum_r += (float)pk[b][cc][i]; }
                }
            }
        }
        dsum += xhalf(dsum); psum += xhalf(psum);
        dsum_r += xhalf(dsum_r); psum_r += xhalf(psum_r);
        // delta_i = sum_j P_ij dP_ij / sum_j P_ij: the row's probabilities sum to 1 up to the rounding of
        // the stored LSE, and dividing by their actual sum keeps delta equal to dP for a row with one key
        const float delta = (real && psum_r > 0.f) ? dsum_r / psum_r : 0.f;
        if (in && half == 0) {
            p.delta[(size_t)h * p.n_q + row] = (real && psum > 0.f) ? -dsum / psum : 0.f;
            p.lse2[(size_t)h * p.n_q + row] = lse_cur;
        }
        // dS^T = X - delta P of every block, as the bf16 operand of the second pass (in place of P)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b < nblk) {
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    float ds[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) ds[i] = fmaf(-delta, (float)pk[b][cc][i], (float)xk[b][cc][i]);
                    pk[b][cc] = pack8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
                }
            }
        }
        // second pass: dQ^T += K^T dS^T
        f32x16 acc[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b < nblk) {
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    const int koff = (b * 32 + cc * 16) * ROWB;
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        const bf16x8 a = cat4(lds_read_tr4_at(taddr[db][0] + koff), lds_read_tr4_at(taddr[db][1] + koff));
                        acc[db] = mfma32(a, pk[b][cc], acc[db]);
                    }
                }
            }
        }
        // dQ rows through the staging tile (Q and dO are in registers by now), stored as whole rows
        if (__any(!real)) {                         // (0 x K is NaN where K is not finite)
            asm volatile("");                       // keep it a branch
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[db][r] = real ? acc[db][r] : 0.f;
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                *reinterpret_cast<WLB_LDS bf16x4*>((uintptr_t)(stage + l32 * ROWB + swz<CPR>(l32, db * 4 + r4) * 16 + half * 8)) =
                    pack4(acc[db][r4 * 4 + 0] * p.scale, acc[db][r4 * 4 + 1] * p.scale, acc[db][r4 * 4 + 2] * p.scale, acc[db][r4 * 4 + 3] * p.scale);
        RowBlock<D> dq_rows;
        dq_rows.from_tile(stage, lane);
        dq_rows.store(dq_buf, row_voff, head_soff(hs), q_row_bytes);
        wait_lds();                                 // the staging tile has been read back
    }
}

// A workgroup of 512 threads on the short-hull units of the blocks of rows blk0 .. blk0 + per - 1: one, f(all eight wavefronts, LDS, block), or two
// side by side, f(four wavefronts, LDS of the half, block), which meet at the same barriers (both run through two).
template <int HALF_BYTES, class F>
__device__ __forceinline__ void short_units_of_512(char* smem, int blk0, int per, F f) {
    if (per == 1) return f(std::integral_constant<int, 8>{}, smem, blk0);
    const int which = uniform((int)(threadIdx.x >> 8));
    f(std::integral_constant<int, 4>{}, smem + which * HALF_BYTES, blk0 + which);
}

}  // namespace wlb
