// dQ for two query heads of a KV head at a time (wlb_attn_bwd.hip has the derivative and the backward's other kernels).
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "wlb_acc.h"
#include "wlb_attn_bwd.h"
#include "wlb_device.h"
#include "wlb_internal.h"

namespace wlb {

// Scores with the rows' operand in accumulation registers N .. N + 3.  The vector ALU reads them at least 19 instructions later (build.py refuses
// code in which it does not).
template <int N, bool FIRST>
__device__ __forceinline__ void mfma_of_acc(f32x16& s, bf16x8 a) {
    if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], 0 ; acc" : "=&v"(s) : "v"(a), "n"(N), "n"(N + 3));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %0 ; acc" : "+v"(s) : "v"(a), "n"(N), "n"(N + 3));
}

// One workgroup = a query tile of 128 rows x two query heads, four wavefronts, one to a SIMD with its 512 registers: a wavefront takes 64 rows of
// one head, so that every K and V operand read from LDS feeds two MFMAs and the tiles in LDS serve twice the rows (dq_piece: 32 rows, two
// workgroups to a compute unit).  dQ^T fills half of the accumulation registers and the operands of Q the other half, those of dO, two sets of scores and dP the
// vector registers.  Bound: the power limit (dq_kernel: matrix pipes 70 % busy at 1.64 GHz); half the LDS reads and copies per MFMA are what is gained.
// Per launch, before -> after: 131072 tokens on one of 8 ranks, 8/1 heads 4329 -> 4014 us; 131072 tokens, one document
// of 98304 and 979 tiny ones, 16/2 heads, 48800 -> 43760; 32768 tokens, 32/8 heads 1770 -> 1711.  Where it is used: use_row_pairs.
template <int D>
__device__ __forceinline__ void dq_pair_piece(const BwdParams& p, char* smem, const RowPiece& pc) {
    constexpr int BM = kFwdTileRows, BN = 64, NU = D / 16, DB = D / 32, CH = D / 64, ROWB = D * 2, TILEB = BN * ROWB, NBUF = 4;
    constexpr int PER = TILEB / 4096, PIECES = 2 * PER;      // 1 KiB blocks of a tile that a wavefront copies; of K and V
    constexpr int HALF = 4 * CH * 1024;                      // 32 rows further
    constexpr int ACC_Q = 2 * DB * 16;                       // accumulators of dQ^T, then the operands of Q
    static_assert(D == 128, "the schedule of a block of 32 keys is laid out for 16 MFMAs a product");
    static_assert(BM == 128 && PER == 2 * CH, "a wavefront copies 16 rows");

    const int G = p.hq / p.hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5, j16 = lane & 15, gi = (lane >> 4) & 1;
    const int tile = pc.tile, hk = pc.hk, jb = pc.jb, je = pc.je;
    const int h = hk * G + 2 * pc.member + (wave >> 1);
    const int row0 = tile * BM + (wave & 1) * 64;            // the wavefront's rows
    const uint32_t smem_base = (uint32_t)(uintptr_t)(WLB_LDS char*)smem;
    auto fence = [] () __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
    auto barrier = [] () __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    wait_vmem();
    barrier();                    // every wavefront has left the tiles of the piece before

    // Copies: a wavefront takes 16 rows of every K and V tile, and its own 64 rows of Q and dO, which pass through the buffers after the first.
    const uint32_t kv_row = (uint32_t)p.hkv * ROWB, kv_total = (uint32_t)p.t_kv * kv_row;
    const uint32_t q_row = (uint32_t)p.hq * ROWB, q_total = (uint32_t)p.n_q * q_row;
    const uint32_t lane_row = (uint32_t)((lane & 7) ^ ((lane >> 4 & 1) * 4)), lane_chunk = (uint32_t)(lane >> 3) * 16u;
    BufRsrc k_rs, v_rs;
    k_rs.init(p.k, kv_total);
    v_rs.init(p.v, kv_total);
    const uint32_t voff0 = lane_row * kv_row + lane_chunk, voff1 = voff0 ^ 16u;      // of an even and an odd block of 8 rows
    const uint32_t wave_lds = smem_base + (uint32_t)(wave * PER) * 1024u, rows8 = 8u * kv_row;
    int nx = jb;                                             // the tile whose copies come next
    uint32_t nx_so = (uint32_t)(jb * BN + wave * 16) * kv_row + (uint32_t)hk * ROWB, nx_b = 0, at_so = 0, at_lds = 0;
    auto issue_piece = [&](auto k_tag) __attribute__((always_inline)) {
        constexpr int k = decltype(k_tag)::value, n = k >> 1;
        if (k == 0) {
            at_so = uniform(nx < je ? nx_so : kv_total);     // past the last tile: zeros and no memory
            at_lds = wave_lds + nx_b;
            ++nx;
            nx_so += BN * kv_row;
            nx_b = (nx_b + 2 * TILEB) & (NBUF * 2 * TILEB - 1);
        }
        const int voff = (int)(n / CH ? voff1 : voff0);
        if constexpr (k & 1) dma_issue_at<TILEB + n * 1024>(v_rs.r, at_lds, voff, at_so);
        else if constexpr (k == 0) dma_issue_at<0>(k_rs.r, at_lds, voff, at_so);
        else at_so = dma_issue_step<n * 1024>(k_rs.r, at_lds, voff, at_so, n % CH ? 128u : rows8 - 128u);
    };
    auto issue_at = [&](int k) __attribute__((always_inline)) {
        switch (k) {
            case 0: if constexpr (0 < PIECES) issue_piece(std::integral_constant<int, 0>{}); break;
            case 1: if constexpr (1 < PIECES) issue_piece(std::integral_constant<int, 1>{}); break;
            case 2: if constexpr (2 < PIECES) issue_piece(std::integral_constant<int, 2>{}); break;
            case 3: if constexpr (3 < PIECES) issue_piece(std::integral_constant<int, 3>{}); break;
            case 4: if constexpr (4 < PIECES) issue_piece(std::integral_constant<int, 4>{}); break;
            case 5: if constexpr (5 < PIECES) issue_piece(std::integral_constant<int, 5>{}); break;
            case 6: if constexpr (6 < PIECES) issue_piece(std::integral_constant<int, 6>{}); break;
            case 7: if constexpr (7 < PIECES) issue_piece(std::integral_constant<int, 7>{}); break;
        }
    };
    auto issue_tile = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < PIECES; ++k) issue_at(k);
    };
    const uint32_t qoff = lane_row * q_row + lane_chunk;
    auto copy_rows = [&](const void* rows, uint32_t lds) __attribute__((always_inline)) {
        BufRsrc rs;
        rs.init(rows, q_total);
        uint32_t so = uniform((uint32_t)row0 * q_row + (uint32_t)h * ROWB);
        for_all<8 * CH>([&](auto n) __attribute__((always_inline)) {
            const int voff = (int)(n / CH % 2 ? qoff ^ 16u : qoff);
            if constexpr (n == 0) dma_issue_at<0>(rs.r, lds, voff, so);
            else so = dma_issue_step<n * 1024>(rs.r, lds, voff, so, n % CH ? 128u : 8u * q_row - 128u);
        });
    };
    const uint32_t q_lds = uniform(smem_base + 2 * TILEB + (uint32_t)wave * TILEB), do_lds = q_lds + 4 * TILEB;
    copy_rows(p.q, q_lds);
    copy_rows(p.d_o, do_lds);
    issue_tile();

    int lo[2], hi[2];
    float lsec[2], dl[2];
    const __bf16* op[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = row0 + i * 32 + l32, rc = min(row, p.n_q - 1);
        lo[i] = row < p.n_q ? p.row_lo[rc] : kPadLo;
        hi[i] = row < p.n_q ? p.row_hi[rc] : 0;
        lsec[i] = p.lse[(size_t)h * p.n_q + rc] * 1.4426950408889634f;
        op[i] = p.o + ((size_t)rc * p.hq + h) * D + half * 8;
    }

    // Operands (wlb_acc.h): rows as they lie (row l32, chunk 2 u + half), for even and odd u; read transposed, rows qq and qq + 8 of 16 and
    // 4 columns of 32 db (lds_read_tr4)
    struct Pair { uint32_t a, b; };
    const uint32_t r0 = smem_base + (uint32_t)((l32 >> 3) * CH) * 1024u + (uint32_t)(half ^ (l32 >> 3 & 1)) * 128u + (uint32_t)(l32 & 7) * 16u, r1 = r0 ^ 64u;
    const int qq = half * 4 + (j16 >> 2), b0 = j16 >> 1 & 1;
    const uint32_t c0 = smem_base + (uint32_t)(gi * 2 + b0) * 128u + (uint32_t)(qq ^ (gi * 4)) * 16u + (j16 & 1) * 8u, c1 = (c0 ^ 128u) + CH * 1024u;
    auto rd_row = [](Pair x, int u, uint32_t at) __attribute__((always_inline)) {
        return *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(((u & 1) ? x.b : x.a) + (at + (u & 3) * 256u + (u >> 2) * 1024u)));
    };
    auto rd_col = [](Pair x, int u, uint32_t tile_at) __attribute__((always_inline)) {
        const uint32_t cc = u / DB, db = u % DB, at = tile_at + cc * (2 * CH * 1024u) + (db >> 1) * 1024u + (db & 1) * 512u;
        return cat4(lds_read_tr4_at(x.a + at), lds_read_tr4_at(x.b + at));
    };
    auto rows_of = [&](uint32_t buf) __attribute__((always_inline)) { return Pair{add_here(r0, buf), add_here(r1, buf)}; };
    auto cols_of = [&](uint32_t buf) __attribute__((always_inline)) { return Pair{add_here(c0, buf), add_here(c1, buf)}; };

    bf16x8 dof[2][NU];                // B operands of dP; those of S go to accumulation registers
    {
        bf16x8 o[2][NU];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int u = 0; u < NU; ++u) o[i][u] = *reinterpret_cast<const bf16x8*>(op[i] + u * 16);
        for_all<2 * DB>([](auto i) __attribute__((always_inline)) { acc_zero<decltype(i)::value>(u32x4{0, 0, 0, 0}); });
        wait_vmem();                  // Q and dO (the wavefront's own), the first tile, O
        asm volatile("" ::: "memory");
        const uint32_t q_at = r0 + 2 * TILEB + (uint32_t)wave * TILEB;
        const Pair xq{q_at, q_at ^ 64u}, xd{q_at + 4 * TILEB, (q_at ^ 64u) + 4 * TILEB};
        for_all<2 * NU>([&](auto n) __attribute__((always_inline)) {
            constexpr int i = decltype(n)::value / NU, u = decltype(n)::value % NU;
            const u32x4 x = __builtin_bit_cast(u32x4, rd_row(xq, u, i * HALF));
            for_all<4>([&](auto e) __attribute__((always_inline)) { acc_write<ACC_Q + decltype(n)::value * 4 + decltype(e)::value>(x[decltype(e)::value]); });
            dof[i][u] = rd_row(xd, u, i * HALF);
        });
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float x = 0.f;            // -delta
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) x = fmaf(-(float)dof[i][u][e], (float)o[i][u][e], x);
            x += xhalf(x);
            dl[i] = hi[i] > 0 ? x : 0.f;
            if (hi[i] <= 0) lsec[i] = INFINITY;           // makes every probability of a padding row 0, here and in the dK/dV kernel
        }
    }
    // the tile's first piece leaves them for the dK/dV kernel
    if (pc.first && half == 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = row0 + i * 32 + l32;
            if (row < p.n_q) {
                p.delta[(size_t)h * p.n_q + row] = dl[i];
                p.lse2[(size_t)h * p.n_q + row] = lsec[i];
            }
        }
    }
    wait_lds();
    wait_vmem();
    barrier();                        // every wavefront's part of the first tile, and Q and dO have left the buffers

    if (jb < je) {
        issue_tile();
        issue_tile();
        // Key tiles without an element-wise mask are [fb, fe); inside, the rows in `other` see nothing and are switched off as whole lanes.
        int fb, fe;
        bool other[2];
        unmasked_tiles<BN>(lo, hi, fb, fe, other);
        const float cs = p.scale_log2e;
        float ls_range[2], ls[2];     // LSE, or +inf to switch the row off: inside the range, and of the block at hand
        bool cut = false, cut_next = false;      // the block at hand, and the next, needs the element-wise mask
        // a block outside the range: whole rows off, or the mask where a row's interval cuts it; may set a new range (see dq_piece)
        auto classify = [&](int key0) __attribute__((always_inline)) {
            bool none[2], some = false;
            int edge = kPadLo;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                none[i] = (key0 + 32 <= lo[i]) || (key0 >= hi[i]);
                some = some || !(none[i] || ((key0 >= lo[i]) && (key0 + 32 <= hi[i])));
                edge = min(edge, none[i] ? (lo[i] >= key0 + 32 ? lo[i] : kPadLo) : hi[i]);
                ls[i] = none[i] ? INFINITY : lsec[i];
            }
            cut_next = __any(some);
            if (cut_next) return;
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) edge = min(edge, __shfl_xor(edge, o));
            const int j_next = key0 / BN + 1, j_edge = uniform(edge / BN);
            if (j_edge > j_next) {
                fb = uniform(j_next);
                fe = j_edge;
#pragma unroll
                for (int i = 0; i < 2; ++i) ls_range[i] = none[i] ? INFINITY : lsec[i];
            }
        };
#pragma unroll
        for (int i = 0; i < 2; ++i) ls[i] = ls_range[i] = other[i] ? INFINITY : lsec[i];
        if ((jb < fb) || (jb >= fe)) classify(jb * BN);
        cut = cut_next;

        f32x16 S[2][2], dp[2];        // scores, then P: [even and odd block of a tile][32 rows]
        u32x4 ds[2][2];               // dS as operands: [32 rows][16 keys], two values in each element
        bf16x8 ring[4];               // the A operands of the unit at hand and of the next three
        const f32x16 zero16 = {};
        float carry = 0.f;
        auto pack2 = [](float x, float y) __attribute__((always_inline)) {
            bf16x2 r;
            r[0] = (__bf16)x; r[1] = (__bf16)y;
            return opaque(__builtin_bit_cast(uint32_t, r));
        };
        auto exp_one = [&](f32x16 (&s)[2], int e) __attribute__((always_inline)) {
            const int i = e >> 4, x = e & 15;
            s[i][x] = fast_exp2(fmaf(s[i][x], cs, -ls[i]));
        };
        Pair a_row = rows_of(0), a_rown = a_row, a_col = cols_of(0);
        for_all<NU>([&](auto u) __attribute__((always_inline)) {
            const bf16x8 x = rd_row(a_row, u, 0);
            for_all<2>([&](auto i) __attribute__((always_inline)) { mfma_of_acc<ACC_Q + (i * NU + u) * 4, u == 0>(S[0][i], x); });
            fence();
        });
        acc_settle();
        fence();
#pragma unroll
        for (int u = 0; u < 3; ++u) ring[u] = rd_row(a_row, u, TILEB);
        // A block of 32 keys: 6 NU MFMAs without a gap: dP, the scores of the next block, dQ.  Beside them the exponentials (from the second half of
        // the dQ of the block before to the end of dP) and dS (beside the scores).  Operands are requested three units (of two MFMAs)
        // ahead, right behind a unit's first MFMA.  The barrier of a tile lies in its second block, in front of the first read of the next tile's K.
        constexpr int E0 = 7, EXP_SLOTS = 2 * NU - E0 + 2 * NU;      // first slot of dQ with exponentials; slots with them
        auto exp_end = [](int k) { const int e = (k * 32 + EXP_SLOTS - 2) / (EXP_SLOTS - 1); return e < 0 ? 0 : e < 32 ? e : 32; };
        auto exp_slot = [&](f32x16 (&s)[2], int k) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 32; ++e)
                if (e >= exp_end(k) && e < exp_end(k + 1)) exp_one(s, e);
        };
#pragma unroll
        for (int k = 0; k < 2 * NU - E0; ++k) exp_slot(S[0], k);
        uint32_t buf = 0;
        auto stage = [&](auto h_tag, int j) __attribute__((always_inline)) {
            constexpr int H = decltype(h_tag)::value;
            f32x16 (&sc)[2] = S[H];
            f32x16 (&sn)[2] = S[H ^ 1];
            constexpr int SY = NU - 4;              // units of dP in front of the barrier: what follows reads the next tile's K
            const uint32_t S_AT = H ? 0 : HALF, V_AT = TILEB + H * HALF, C_AT = H * HALF, N_AT = TILEB + (H ? 0 : HALF);
            for_all<NU>([&](auto u) __attribute__((always_inline)) {       // dP
                if constexpr (H == 1 && u == SY) {
                    // the next tile is complete (copied in front of the latest one), and every wavefront has left the one before this
                    wait_vmem_le<PIECES>();
                    barrier();
                    buf = (buf + 2 * TILEB) & (NBUF * 2 * TILEB - 1);
                    a_rown = rows_of(buf);
                }
                for_all<2>([&](auto i) __attribute__((always_inline)) {
                    dp[i] = mfma32(ring[u & 3], dof[i][u], u == 0 ? zero16 : dp[i]);
                    fence();
                    if constexpr (i == 0) ring[(u + 3) & 3] = u + 3 < NU ? rd_row(a_row, u + 3, V_AT) : rd_row(H ? a_rown : a_row, u + 3 - NU, S_AT);
                    fence();
                    exp_slot(sc, 2 * NU - E0 + 2 * u + i);
                    fence();
                });
            });
            for_all<NU>([&](auto u) __attribute__((always_inline)) {       // the next block's scores
                for_all<2>([&](auto i) __attribute__((always_inline)) {
                    mfma_of_acc<ACC_Q + (i * NU + u) * 4, u == 0>(sn[i], ring[u & 3]);
                    fence();
                    if constexpr (i == 0) ring[(u + 3) & 3] = u + 3 < NU ? rd_row(H ? a_rown : a_row, u + 3, S_AT) : rd_col(a_col, u + 3 - NU, C_AT);
                    else if constexpr (H == 1) issue_at(u);                // the copies of the tile after the next two
                    fence();
                    // dS = P o (dP - delta)
                    constexpr int D0 = 3, k = 2 * u + i - D0, A = (k < 0 ? 0 : k) * 32 / (2 * NU - D0), B = (k < 0 ? 0 : k + 1) * 32 / (2 * NU - D0);
                    for_all<B - A>([&](auto n) __attribute__((always_inline)) {
                        constexpr int e = A + decltype(n)::value, r = e >> 4, x = e & 15;
                        const float v = sc[r][x] * (dp[r][x] + dl[r]);
                        if constexpr (x & 1) ds[r][x >> 3][(x & 7) >> 1] = pack2(carry, v);
                        else carry = v;
                    });
                    fence();
                });
            });
            const int jn = j + H;                   // the next block's tile
            cut_next = false;
#pragma unroll
            for (int i = 0; i < 2; ++i) ls[i] = ls_range[i];
            if (__builtin_expect(cut || (jn < fb) || (jn >= fe), 0)) {
                asm volatile("");
                if (cut) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int x = 0; x < 16; x += 2) {
                            const int key = j * BN + H * 32 + (x >> 2) * 8 + half * 4 + (x & 3);
                            const uint32_t keep = (key >= lo[i] && key < hi[i] ? 0xffffu : 0u) | (key + 1 >= lo[i] && key + 1 < hi[i] ? 0xffff0000u : 0u);
                            ds[i][x >> 3][(x & 7) >> 1] &= keep;
                        }
                    asm volatile("s_nop 1");
                }
                if ((jn < fb) || (jn >= fe)) classify(jn * BN + (H ? 0 : 32));
            }
            cut = cut_next;
            for_all<NU>([&](auto u) __attribute__((always_inline)) {       // dQ
                for_all<2>([&](auto i) __attribute__((always_inline)) {
                    acc_mfma<i * DB + u % DB>(ring[u & 3], ds[i][u / DB]);
                    fence();
                    if constexpr (i == 0) ring[(u + 3) & 3] = u + 3 < NU ? rd_col(a_col, u + 3, C_AT) : rd_row(H ? a_rown : a_row, u + 3 - NU, N_AT);
                    fence();
                    if constexpr (2 * u + i >= E0) exp_slot(sn, 2 * u + i - E0);
                    fence();
                });
            });
        };
        for (int j = jb; j < je; ++j) {
            stage(std::integral_constant<int, 0>{}, j);
            stage(std::integral_constant<int, 1>{}, j);
            a_row = a_rown;
            a_col = cols_of(buf);
        }
        wait_vmem();                  // (the copies past the last tile write zeros)
    }

    acc_settle();
    for_all<2>([&](auto i_tag) __attribute__((always_inline)) {
        constexpr int i = decltype(i_tag)::value;
        const int rl = (wave & 1) * 64 + i * 32 + l32, row = tile * BM + rl;
        if (row >= p.n_q) return;
        if (pc.slot >= 0) {
            // part of a tile: unscaled fp32 dQ [row][d], summed by dq_merge_kernel
            float* part = p.row_partial + (size_t)(pc.slot + (wave >> 1)) * (BM * D + 2 * BM) + (size_t)rl * D + half * 4;
            for_all<DB * 4>([&](auto q) __attribute__((always_inline)) {
                constexpr int a = i * DB * 16 + decltype(q)::value * 4;
                *reinterpret_cast<f32x4*>(part + decltype(q)::value * 8) = f32x4{acc_read<a>(), acc_read<a + 1>(), acc_read<a + 2>(), acc_read<a + 3>()};
            });
            return;
        }
        __bf16* out = p.dq + ((size_t)row * p.hq + h) * D + half * 4;
        for_all<DB * 4>([&](auto q) __attribute__((always_inline)) {
            constexpr int a = i * DB * 16 + decltype(q)::value * 4;
            bf16x4 x = pack4(acc_read<a>() * p.scale, acc_read<a + 1>() * p.scale, acc_read<a + 2>() * p.scale, acc_read<a + 3>() * p.scale);
            if (hi[i] <= 0) x = pack4(0.f, 0.f, 0.f, 0.f);
            *reinterpret_cast<bf16x4*>(out + decltype(q)::value * 8) = x;
        });
    });
}

template <int D>
constexpr int dq_pair_lds() { return 5 * 2 * 64 * D * 2; }      // four buffers: K tile | V tile; Q passes through the second and third, dO through the next two

template <int D>
__global__ void __launch_bounds__(256, 1) dq_pair_kernel(const BwdParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[dq_pair_lds<D>()];
    const unsigned long long t_start = wall_clock64();
    RowWalk walk;
    walk.start(p.sched, (int)blockIdx.x, p.sched.G / 2);
    RowPiece pc;
    while (walk.next(p.sched, pc)) {
        if (pc.slot >= 0) pc.slot += pc.member;      // the slot of the pair's first head
        dq_pair_piece<D>(p, smem, pc);
    }
    if (threadIdx.x == 0) {
        // as the workgroups of one head each leave them
        const unsigned long long t_end = wall_clock64();
        for (int k = 0; k < 2; ++k) {
            const int b = ((walk.gang >> 3) * p.sched.G + 2 * walk.member + k) * 8 + (walk.gang & 7);
            p.gang_clock[2 * b] = t_start;
            p.gang_clock[2 * b + 1] = t_end;
        }
    }
}

// One workgroup per (query tile in order, two heads), heaviest first; whole tiles only, short-hull tiles left out (their units form delta more
// precisely, from P and dP, and are faster).
template <int D>
__global__ void __launch_bounds__(256, 1) dq_pair_items_kernel(const BwdParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[dq_pair_lds<D>()];
    const int pairs = p.hq / p.hkv / 2;
    int y = blockIdx.x >> 3;
    RowPiece pc;
    pc.member = y % pairs; y /= pairs;
    pc.hk = y % p.hkv;
    const int index = (y / p.hkv) * 8 + (blockIdx.x & 7);
    if (index >= p.n_tiles) return;
    const int4 item = ld_const4(p.row_item + 4 * index);
    if (p.use_short && item.w == -2) return;         // dq_short_tiles_kernel's
    pc.tile = item.x;
    pc.jb = item.y; pc.je = item.z;
    pc.first = true;
    pc.slot = -1;
    dq_pair_piece<D>(p, smem, pc);
}

void launch_dq_pair(const BwdParams& p, bool gangs, unsigned grid, hipStream_t stream) {
    if (gangs) dq_pair_kernel<128><<<grid, 256, 0, stream>>>(p);
    else dq_pair_items_kernel<128><<<grid, 256, 0, stream>>>(p);
}

}  // namespace wlb
