// Forward and dQ of short documents divided among context-parallel ranks (wlb_attn_fwd.hip and wlb_attn_bwd.hip have the arithmetic).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "wlb_acc.h"
#include "wlb_attn_bwd.h"
#include "wlb_attn_fwd.h"
#include "wlb_attn_short.h"
#include "wlb_device.h"
#include "wlb_internal.h"

namespace wlb {

// Of C ranks a block of 32 rows spans about 32 C tokens and one document: too many keys for a short-hull unit (kShortHullKeys), while the general
// kernel visits the keys of 128 rows for each of them, nearly all blocks masked, one key tile after another between barriers (4 us a tile).
// Here a unit is one or more blocks of 32 rows x one KV head: K and V of the keys that its rows see are copied into LDS, 256 at a time, for all
// query heads; then each of eight wavefronts works alone on one head and one block of rows, and on the 32-key blocks that those rows see.  With
// fewer than eight heads to a KV head a unit takes more blocks of rows.  Rows arrive and leave whole through a staging tile of 16 rows of the
// wavefront's own.  Any mask is handled (more than 256 keys in several turns, keys that none of the unit's rows sees passed over: rows of two distant
// chunks); which launches come here: use_span.  Bound: latency (a unit's
// rows and keys are requested, arrive, are worked on and leave with nothing beside them: 160 KiB of LDS hold one unit).  The blocks of short-hull tiles
// (contiguous chunks of short documents) are short-hull units in the same launch: in one of their own, 5 us each in forward and in
// dQ, a whole pass over 2320 tokens in contiguous chunks, 8/1 heads, one of 4 ranks, took 127 us for 102 here (115 without this file).
// 32768 tokens in documents of 1 - 64, 16/2 heads, before -> after, forward and dQ: one of 4 ranks 73 -> 47 and 84 -> 60 us; 36448 tokens, 8/1 heads, one of 8 ranks
// 42 -> 22 and 47 -> 27; 9000 tokens, 8/2 heads, D = 64, one of 4 ranks 20 -> 12.6 and 18 -> 14.  Contiguous chunks, 36448 tokens, 8/1 heads, one of 4 ranks,
// where a few rows of two distant chunks share a block: the whole pass 785 -> 136.  Slower: contiguous chunks of 131072 tokens, nearly all tiles short-hull
// ones, 0.92 - 1.0 (one workgroup to a compute unit, where short-hull units in a launch of their own kernel have two).
template <int D>
struct Span {
    static constexpr int NW = 8, KEYS = 32 * NW, KS = D / 16, DB = D / 32, CPR = D / 8, ROWB = D * 2;
    static constexpr int STAGE = 16 * ROWB, LDS_BYTES = 2 * KEYS * ROWB + NW * STAGE;
    static_assert(LDS_BYTES >= 2 * ShortTile<D>::LDS_BYTES && ShortTile<D>::LDS_BYTES == ShortDq<D>::LDS_BYTES, "two short-hull units");

    int lane, wave, l32, half;
    int hk, heads, blk, first_head;      // the wavefront's block of rows; -1: none
    int row, lo, hi;                     // the lane's row and its keys
    int u_lo, u_hi;                      // keys that a row of the unit sees
    uint32_t smem, stage, q_row_bytes;
    int naddr[KS], taddr[DB][2];         // operands of a 32-key block: rows as they lie, and transposed
    BufRsrc krs, vrs;
    TileDma<D, KEYS, NW> dma;

    // The workgroup's unit: its first block of rows and KV head (false: none).  Neighbouring units share keys, so they go to the same XCD.
    template <class P>
    static __device__ __forceinline__ bool unit_of(const P& p, int per, int& blk0, int& hk) {
        const int n = p.n_blocks32 / per;
        const int unit = uniform((int)(blockIdx.x % kLists) * (int)(gridDim.x / kLists) + (int)(blockIdx.x / kLists));
        blk0 = uniform(unit % n * per);
        hk = uniform(unit / n);
        return unit < n * p.hkv;
    }
    // the lane once more, where addresses of the staging tile are made from it (kept from the start they take more registers than there are)
    static __device__ __forceinline__ int lane_here() { return (int)opaque(threadIdx.x) & 63; }
    template <class P>
    __device__ __forceinline__ void init(const P& p, char* lds, int blk0, int kv_head, int per) {
        heads = min(p.hq / p.hkv, NW);
        hk = kv_head;
        lane = lane_here(); wave = uniform((int)(threadIdx.x >> 6)); l32 = lane & 31; half = lane >> 5;
        blk = blk0 + wave / heads;
        if (wave / heads >= per || blk >= p.n_blocks32) blk = -1;
        first_head = wave % heads;
        const int u_row = blk0 * kShortBlockRows + lane;   // a row of the unit (at most 64) in every lane
        const bool u_in = lane < per * kShortBlockRows && u_row < p.n_q;
        u_lo = u_in ? p.row_lo[u_row] : kPadLo;
        u_hi = u_in ? p.row_hi[u_row] : 0;
        row = blk * kShortBlockRows + l32;
        const bool in = blk >= 0 && row < p.n_q;
        if (!in) row = -1;
        lo = in ? p.row_lo[row] : kPadLo;
        hi = in ? p.row_hi[row] : 0;
        smem = (uint32_t)(uintptr_t)(WLB_LDS char*)lds;
        stage = uniform(smem + 2 * KEYS * ROWB + (uint32_t)wave * STAGE);
        q_row_bytes = (uint32_t)p.hq * ROWB;
        const int j16 = lane & 15, gi = (lane >> 4) & 1;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) naddr[ks] = l32 * ROWB + swz<CPR>(l32, ks * 2 + half) * 16;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int key = t * 8 + half * 4 + (j16 >> 2);
                taddr[db][t] = key * ROWB + swz<CPR>(key, db * 4 + gi * 2 + ((j16 & 3) >> 1)) * 16 + (j16 & 1) * 8;
            }
        const uint32_t kv_row = (uint32_t)p.hkv * D, kv_bytes = ((uint32_t)p.t_kv * kv_row - (uint32_t)hk * D) * 2u;
        krs.init(p.k + (size_t)hk * D, kv_bytes);
        vrs.init(p.v + (size_t)hk * D, kv_bytes);
        dma.init(wave, lane, kv_row);
    }
    // scalar offset of a head's first row of the wavefront's block
    __device__ __forceinline__ uint32_t head_soff(int h) const { return uniform((uint32_t)blk * (uint32_t)kShortBlockRows * q_row_bytes + (uint32_t)h * ROWB); }
    // copies of K and V of the keys from key0 on, 32 to a wavefront; every wavefront must have left the keys before
    __device__ __forceinline__ void copy_keys(int key0) const {
        if (__any(u_lo < key0 + wave * 32 + 32 && u_hi > key0 + wave * 32)) {
            BufRsrc k = krs, v = vrs;
            k.make_uniform();
            v.make_uniform();
            dma.issue(k, smem, key0, wave);
            dma.issue(v, smem + KEYS * ROWB, key0, wave);
        }
    }
    // a head's rows, and in operand layout
    __device__ __forceinline__ void load_rows(buf_rsrc_t buf, int h, RowBlock<D>& x) const { x.load(buf, RowBlock<D>::lane_off(lane_here(), q_row_bytes), head_soff(h), q_row_bytes); }
    __device__ __forceinline__ void to_operand(const RowBlock<D>& x, bf16x8 (&dst)[KS]) const {
        const int lane = lane_here(), l32 = lane & 31, half = lane >> 5;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            wait_lds();                   // what the tile held has been read
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < RowBlock<D>::N / 2; ++i) {
                const int r = i * RowBlock<D>::RPI + lane / CPR;
                *reinterpret_cast<WLB_LDS i32x4*>((uintptr_t)(stage + r * ROWB + swz<CPR>(r, lane % CPR) * 16)) = x.v[t * (RowBlock<D>::N / 2) + i];
            }
            if ((l32 >> 4) == t) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    dst[ks] = *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(stage + (l32 & 15) * ROWB + swz<CPR>(l32 & 15, ks * 2 + half) * 16));
            }
        }
    }
    // acc^T [d][row] times f to a head's rows
    __device__ __forceinline__ void store_rows(buf_rsrc_t buf, int h, const f32x16 (&acc)[DB], float f) const {
        const int lane = lane_here(), l32 = lane & 31, half = lane >> 5;
        RowBlock<D> x;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            wait_lds();
            asm volatile("" ::: "memory");
            if ((l32 >> 4) == t) {
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4)
                        *reinterpret_cast<WLB_LDS bf16x4*>((uintptr_t)(stage + (l32 & 15) * ROWB + swz<CPR>(l32 & 15, db * 4 + r4) * 16 + half * 8)) =
                            pack4(acc[db][r4 * 4 + 0] * f, acc[db][r4 * 4 + 1] * f, acc[db][r4 * 4 + 2] * f, acc[db][r4 * 4 + 3] * f);
            }
#pragma unroll
            for (int i = 0; i < RowBlock<D>::N / 2; ++i) {
                const int r = i * RowBlock<D>::RPI + lane / CPR;
                x.v[t * (RowBlock<D>::N / 2) + i] = *reinterpret_cast<const WLB_LDS i32x4*>((uintptr_t)(stage + r * ROWB + swz<CPR>(r, lane % CPR) * 16));
            }
        }
        x.store(buf, RowBlock<D>::lane_off(lane, q_row_bytes), head_soff(h), q_row_bytes);
    }
    // first key of the next window: the first 32 keys from `key` on that a row of the unit sees (kPadLo: none); the same in every wavefront
    __device__ __forceinline__ int window_from(int key) const {
        int next = u_hi > key ? max(u_lo, key) : kPadLo;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) next = min(next, __shfl_xor(next, o));
        next = uniform(next);
        return next == kPadLo ? next : next & ~31;
    }
    // f(offset in the window, first key) for the 32-key blocks of the window from key0 on that the wavefront's rows see
    template <class F>
    __device__ __forceinline__ void blocks(int key0, F f) const {
#pragma nounroll
        for (int key = key0; key < key0 + KEYS; key += 32)
            if (__any(lo < key + 32 && hi > key)) f((key - key0) * ROWB, key);
    }
    // One head to a wavefront after another: load(h) requests its rows, in front of the copies of the keys, begin(h), turn(key0) for the windows of
    // the unit's hull, end(h).
    // reset() ends the life of what a head leaves (a wavefront without a head would carry it on, in registers that the next one needs).
    template <class Reset, class Load, class Begin, class Turn, class End>
    __device__ __forceinline__ void run(int G, Reset reset, Load request, Begin begin, Turn turn, End end) const {
        const int first = window_from(0);
        const bool several = first != kPadLo && window_from(first + KEYS) != kPadLo;
        for (int h0 = 0; h0 < G; h0 += heads) {
            reset();
            const bool on = blk >= 0 && h0 + first_head < G;
            const int h = hk * G + h0 + first_head;
            const bool load = h0 == 0 || several;              // (else the window of the heads before)
            if (on) request(h);
            if (load) {
                __syncthreads();
                if (first != kPadLo) copy_keys(first);
            }
            if (on) begin(h);
#pragma nounroll
            for (int key0 = first; key0 != kPadLo; key0 = several ? window_from(key0 + KEYS) : kPadLo) {
                if (key0 > first) {
                    __syncthreads();
                    copy_keys(key0);
                }
                if (load) {
                    wait_vmem();
                    __syncthreads();
                }
                if (on) turn(key0);
            }
            if (on) end(h);
        }
    }
};

template <int D>
__global__ void __launch_bounds__(512, D == 64 ? 4 : 2) fwd_span_kernel(const FwdParams p) {
    using T = Span<D>;
    constexpr int KS = T::KS, DB = T::DB, ROWB = T::ROWB;
    __shared__ __attribute__((aligned(1024))) char smem[T::LDS_BYTES];
    const int per = T::NW / min(p.hq / p.hkv, T::NW);
    int blk0, hk;
    if (!T::unit_of(p, per, blk0, hk)) return;
    if (ld_const(p.tile_short + blk0 / (kFwdTileRows / kShortBlockRows))) {       // short-hull units are faster there, and dQ's form delta more precisely
        short_units_of_512<T::LDS_BYTES / 2>(smem, blk0, per, [&](auto waves, char* lds, int blk) __attribute__((always_inline)) {
            fwd_short_unit<D, decltype(waves)::value>(p, lds, blk, hk);
        });
        return;
    }
    T t;
    t.init(p, smem, blk0, hk, per);
    const buf_rsrc_t q_buf = make_buf(p.q, (uint32_t)p.n_q * t.q_row_bytes), o_buf = make_buf(p.o, (uint32_t)p.n_q * t.q_row_bytes);
    const float cs = p.scale_log2e;
    RowBlock<D> q_rows;
    bf16x8 qf[KS];
    f32x16 acc[DB];
    float m, l, lim;
    t.run(p.hq / p.hkv, [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RowBlock<D>::N; ++i) q_rows.v[i] = i32x4{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = bf16x8{};
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[db] = f32x16{};
        m = l = lim = 0.f;
    }, [&](int h) __attribute__((always_inline)) { t.load_rows(q_buf, h, q_rows); }, [&](int) __attribute__((always_inline)) {
        t.to_operand(q_rows, qf);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
        m = lim = -INFINITY; l = 0.f;
    }, [&](int key0) __attribute__((always_inline)) {
        t.blocks(key0, [&](int off, int key) __attribute__((always_inline)) {
            f32x16 s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) s = mfma32(*reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(t.smem + t.naddr[ks] + off)), qf[ks], s);
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = key + (r >> 2) * 8 + t.half * 4 + (r & 3);
                s[r] = (k >= t.lo && k < t.hi) ? s[r] : -INFINITY;
                mx = fmaxf(mx, s[r]);
            }
            mx = fmaxf(mx, xhalf(mx));
            if (__any(mx * cs > lim)) {   // the reference follows the maximum lazily (see fwd_piece)
                asm volatile("");
                const float m_new = fmaxf(m, mx);
                const float a = m == -INFINITY ? 0.f : fast_exp2(fmaf(m, cs, -m_new * cs));
                m = m_new;
                lim = m == -INFINITY ? -INFINITY : m * cs + 8.f;
                l *= a;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[db][r] *= a;
            }
            const float mc = m == -INFINITY ? 0.f : m * cs;
            float rs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s[r] = fast_exp2(fmaf(s[r], cs, -mc));
                rs[r & 3] += s[r];
            }
            l += (rs[0] + rs[1]) + (rs[2] + rs[3]);
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                const bf16x8 pf = pack8(s[8 * cc + 0], s[8 * cc + 1], s[8 * cc + 2], s[8 * cc + 3], s[8 * cc + 4], s[8 * cc + 5], s[8 * cc + 6], s[8 * cc + 7]);
                const uint32_t at = t.smem + T::KEYS * ROWB + off + cc * 16 * ROWB;
#pragma unroll
                for (int db = 0; db < DB; ++db) acc[db] = mfma32(cat4(lds_read_tr4_at(at + t.taddr[db][0]), lds_read_tr4_at(at + t.taddr[db][1])), pf, acc[db]);
            }
        });
    }, [&](int h) __attribute__((always_inline)) {
        const float lt = l + xhalf(l);
        const bool live = t.hi > 0 && lt > 0.f;
        const float inv = live ? 1.0f / lt : 0.f;
        if (!live) {                      // (0 x V is NaN where V is not finite)
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
        }
        t.store_rows(o_buf, h, acc, inv);
        if (t.row >= 0 && t.half == 0) p.lse[(size_t)h * p.n_q + t.row] = live ? m * p.scale + __logf(lt) : -INFINITY;
    });
}

template <int D>
__global__ void __launch_bounds__(512, 2) dq_span_kernel(const BwdParams p) {
    using T = Span<D>;
    constexpr int KS = T::KS, DB = T::DB, ROWB = T::ROWB;
    __shared__ __attribute__((aligned(1024))) char smem[T::LDS_BYTES];
    const int per = T::NW / min(p.hq / p.hkv, T::NW);
    int blk0, hk;
    if (!T::unit_of(p, per, blk0, hk)) return;
    if (ld_const(p.tile_short + blk0 / (kFwdTileRows / kShortBlockRows))) {       // short-hull units are faster there, and dQ's form delta more precisely
        short_units_of_512<T::LDS_BYTES / 2>(smem, blk0, per, [&](auto waves, char* lds, int blk) __attribute__((always_inline)) {
            dq_short_unit<D, decltype(waves)::value>(p, lds, blk, hk);
        });
        return;
    }
    T t;
    t.init(p, smem, blk0, hk, per);
    const uint32_t q_bytes = (uint32_t)p.n_q * t.q_row_bytes;
    const buf_rsrc_t q_buf = make_buf(p.q, q_bytes), do_buf = make_buf(p.d_o, q_bytes), o_buf = make_buf(p.o, q_bytes), dq_buf = make_buf(p.dq, q_bytes);
    const float cs = p.scale_log2e;
    const bool real = t.hi > 0;
    RowBlock<D> q_rows, do_rows;
    bf16x8 qf[KS], dof[KS];
    f32x16 acc[DB];
    float ls, dl;
    t.run(p.hq / p.hkv, [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RowBlock<D>::N; ++i) q_rows.v[i] = do_rows.v[i] = i32x4{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = dof[ks] = bf16x8{};
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[db] = f32x16{};
        ls = dl = 0.f;
    }, [&](int h) __attribute__((always_inline)) {
        ls = real ? p.lse[(size_t)h * p.n_q + t.row] * 1.4426950408889634f : INFINITY;      // +inf: P = 0
        t.load_rows(q_buf, h, q_rows);
        t.load_rows(do_buf, h, do_rows);
    }, [&](int h) __attribute__((always_inline)) {
        t.to_operand(q_rows, qf);
        t.load_rows(o_buf, h, q_rows);
        t.to_operand(do_rows, dof);
        bf16x8 of[KS];
        t.to_operand(q_rows, of);
        dl = 0.f;                         // -delta
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < 8; ++i) dl = fmaf(-(float)dof[ks][i], (float)of[ks][i], dl);
        dl += xhalf(dl);
        if (!real) dl = 0.f;
        if (t.row >= 0 && t.half == 0) {  // for the dK/dV kernel
            p.delta[(size_t)h * p.n_q + t.row] = dl;
            p.lse2[(size_t)h * p.n_q + t.row] = ls;
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
    }, [&](int key0) __attribute__((always_inline)) {
        t.blocks(key0, [&](int off, int key) __attribute__((always_inline)) {
            f32x16 s, dp;
#pragma unroll
            for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const uint32_t at = t.smem + t.naddr[ks] + off;
                s = mfma32(*reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)at), qf[ks], s);
                dp = mfma32(*reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(at + T::KEYS * ROWB)), dof[ks], dp);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = key + (r >> 2) * 8 + t.half * 4 + (r & 3);
                const float ds = fast_exp2(fmaf(s[r], cs, -ls)) * (dp[r] + dl);
                s[r] = (k >= t.lo && k < t.hi) ? ds : 0.f;
            }
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                const bf16x8 dsf = pack8(s[8 * cc + 0], s[8 * cc + 1], s[8 * cc + 2], s[8 * cc + 3], s[8 * cc + 4], s[8 * cc + 5], s[8 * cc + 6], s[8 * cc + 7]);
                const uint32_t at = t.smem + off + cc * 16 * ROWB;
#pragma unroll
                for (int db = 0; db < DB; ++db) acc[db] = mfma32(cat4(lds_read_tr4_at(at + t.taddr[db][0]), lds_read_tr4_at(at + t.taddr[db][1])), dsf, acc[db]);
            }
        });
    }, [&](int h) __attribute__((always_inline)) {
        if (!real) {                      // (Q and dO of padding may hold anything)
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
        }
        t.store_rows(dq_buf, h, acc, p.scale);
    });
}

static unsigned span_grid(int n_blocks32, int hq, int hkv) {
    const int per = 8 / std::min(hq / hkv, 8);
    return (unsigned)((n_blocks32 / per * hkv + kLists - 1) / kLists * kLists);
}
void launch_fwd_span(const FwdParams& p, int head_dim, hipStream_t stream) {
    const unsigned grid = span_grid(p.n_blocks32, p.hq, p.hkv);
    if (head_dim == 128) fwd_span_kernel<128><<<grid, 512, 0, stream>>>(p);
    else fwd_span_kernel<64><<<grid, 512, 0, stream>>>(p);
}
void launch_dq_span(const BwdParams& p, int head_dim, hipStream_t stream) {
    const unsigned grid = span_grid(p.n_blocks32, p.hq, p.hkv);
    if (head_dim == 128) dq_span_kernel<128><<<grid, 512, 0, stream>>>(p);
    else dq_span_kernel<64><<<grid, 512, 0, stream>>>(p);
}

}  // namespace wlb
