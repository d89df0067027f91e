// The forward for two query heads of a KV head at a time (wlb_attn_fwd.hip has the arithmetic and the other forward kernels).
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "wlb_acc.h"
#include "wlb_attn_fwd.h"
#include "wlb_device.h"
#include "wlb_internal.h"

namespace wlb {

// One workgroup = a query tile of 128 rows x two query heads, four wavefronts, one to a SIMD with its 512 registers: a wavefront takes 64 rows
// of one head, so that every K and V operand read from LDS feeds two MFMAs and the tiles in LDS serve twice the rows (fwd_piece: 32 rows, two
// workgroups to a compute unit).  O^T lies in accumulators named by number (wlb_acc.h).  Bound: the power limit.  A block of 32 keys takes 1480
// cycles at 1.74 GHz, 32 MFMAs of 32 cycles among them; without the checks behind it 1240, at 1.52 GHz, so that cycles saved come back as
// clock for the most part, and what counts is work: of the time the exponentials are 9 %, sums and maxima 6 %, the copies
// into LDS 5 % (this kernel has half of them).  The rare cases lie out of the way (__builtin_expect): four jumps a block cost 2 %.
// Forward before -> after: 131072 tokens on one of 8 ranks, 8/1 heads 3170 -> 2980 us, at D = 64 2112 -> 2037; 32768 tokens, 32/8 heads 1312 ->
// 1270; 16384 tokens, 32/8 heads, schedule included, 620 -> 583.  Where it is used: use_row_pairs.
// Tried: P multiplied with V a block later, so that the exponentials spread over all of a block's MFMAs (2990 -> 3100).
template <int D>
__device__ __forceinline__ void fwd_pair_piece(const FwdParams& p, char* smem, const RowPiece& pc) {
    constexpr int BM = kFwdTileRows, BN = 64, NU = D / 16, DB = D / 32, CH = D / 64, ROWB = D * 2, TILEB = BN * ROWB, NBUF = 4;
    constexpr int PER = TILEB / 4096, PIECES = 2 * PER;      // 1 KiB blocks of a tile that a wavefront copies; of K and V
    constexpr int HALF = 4 * CH * 1024;                      // 32 rows further
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

    int lo[2], hi[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = row0 + i * 32 + l32;
        lo[i] = row < p.n_q ? p.row_lo[row] : kPadLo;
        hi[i] = row < p.n_q ? p.row_hi[row] : 0;
    }
    wait_vmem();
    barrier();                    // every wavefront has left the tiles of the piece before

    // Copies: a wavefront takes 16 rows of every K and V tile, and its own 64 rows of Q, which pass through the last two buffers.
    const uint32_t kv_row = (uint32_t)p.hkv * ROWB, kv_total = (uint32_t)p.t_kv * kv_row;
    const uint32_t q_row = (uint32_t)p.hq * ROWB;
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
        else at_so = dma_issue_step<n * 1024>(k_rs.r, at_lds, voff, at_so, n % CH ? 128u : CH == 2 ? rows8 - 128u : rows8);
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
    {
        BufRsrc q_rs;
        q_rs.init(p.q, (uint32_t)p.n_q * q_row);
        const uint32_t qoff = lane_row * q_row + lane_chunk, q_lds = uniform(smem_base + 4 * TILEB + (uint32_t)wave * TILEB);
        uint32_t so = uniform((uint32_t)row0 * q_row + (uint32_t)h * ROWB);
        for_all<8 * CH>([&](auto n) __attribute__((always_inline)) {
            const int voff = (int)(n / CH % 2 ? qoff ^ 16u : qoff);
            if constexpr (n == 0) dma_issue_at<0>(q_rs.r, q_lds, voff, so);
            else so = dma_issue_step<n * 1024>(q_rs.r, q_lds, voff, so, n % CH ? 128u : CH == 2 ? 8u * q_row - 128u : 8u * q_row);
        });
    }
    issue_tile();
    issue_tile();
    for_all<2 * DB>([](auto i) __attribute__((always_inline)) { acc_zero<decltype(i)::value>(u32x4{0, 0, 0, 0}); });

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

    // Key tiles without an element-wise mask are [fb, fe); inside, rows of later documents are parked (see fwd_piece).
    int fb, fe;
    bool parked[2];
    unmasked_tiles<BN>(lo, hi, fb, fe, parked);
    const float cs = p.scale_log2e;
    constexpr float kSlack = 8.0f;       // the reference follows the row maximum lazily (see fwd_piece)
    float m[2], l[2], mc[2], lim[2], bias_base[2], bias_cur[2], bias_next[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        m[i] = -INFINITY; l[i] = 0.f; mc[i] = 0.f;
        lim[i] = parked[i] ? INFINITY : -INFINITY;
        bias_base[i] = parked[i] ? INFINITY : 0.f;
    }
    auto unpark = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            lim[i] = parked[i] ? ((m[i] == -INFINITY) ? -INFINITY : mc[i] + kSlack) : lim[i];
            parked[i] = false;
            bias_base[i] = 0.f;
        }
    };
    if (jb >= fe) unpark();
#pragma unroll
    for (int i = 0; i < 2; ++i) bias_cur[i] = bias_next[i] = bias_base[i];

    // (an addition that the compiler does not move past the branches behind the MFMAs)
    auto add_f32_here = [](float x, float y) __attribute__((always_inline)) {
        const float r = x + y;
        asm volatile("" :: "v"(r));
        return r;
    };
    // maximum of this lane's scores; the two lanes of a row are joined where the reference moves
    auto lane_max = [](const f32x16& s) __attribute__((always_inline)) {
        float mx = fmaxf(s[0], s[1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, s[r]), s[r + 1]);
        return mx;
    };
    auto mask_block = [&](f32x16 (&s)[2], int key0, float (&mx)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = key0 + (r >> 2) * 8 + half * 4 + (r & 3);
                s[i][r] = (key >= lo[i] && key < hi[i]) ? s[i][r] : -INFINITY;
            }
            mx[i] = lane_max(s[i]);
        }
    };
    auto mask_next = [&](f32x16 (&s)[2], int key0, float (&mx)[2]) __attribute__((always_inline)) {
        if (key0 >= fe * BN) unpark();
        bool none[2], cut = false;
        int edge = kPadLo;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            none[i] = (key0 + 32 <= lo[i]) || (key0 >= hi[i]);
            cut = cut || !(none[i] || ((key0 >= lo[i]) && (key0 + 32 <= hi[i])));
            edge = min(edge, none[i] ? (lo[i] >= key0 + 32 ? lo[i] : kPadLo) : hi[i]);
        }
        if (__any(cut)) {
            bias_next[0] = bias_next[1] = 0.f;
            mask_block(s, key0, mx);
            return;
        }
        // every row sees all or none of the block, and does so up to the next edge of a row's interval
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) edge = min(edge, __shfl_xor(edge, o));
        const int j_next = key0 / BN + 1, j_edge = uniform(edge / BN);
        const bool range = j_edge > j_next;
        if (range) {
            fb = uniform(j_next);
            fe = j_edge;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (range) {
                parked[i] = none[i];
                bias_base[i] = none[i] ? INFINITY : 0.f;
                lim[i] = none[i] ? INFINITY : lim[i];
            }
            bias_next[i] = none[i] ? INFINITY : 0.f;
            mx[i] = none[i] ? -INFINITY : mx[i];
        }
    };
    // moves the references up to the maxima; the factors for what has been accumulated
    auto move_reference = [&](const float (&block_mx)[2], float (&a2)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float mx = parked[i] ? -INFINITY : fmaxf(block_mx[i], xhalf(block_mx[i]));
            const float m_new = fmaxf(m[i], mx);
            const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
            const float alpha = fast_exp2(fmaf(m[i], cs, -m_use * cs));
            a2[i] = (m[i] == -INFINITY) ? 0.f : alpha;
            m[i] = m_new;
            mc[i] = m_use * cs;
            lim[i] = parked[i] ? INFINITY : ((m_new == -INFINITY) ? -INFINITY : mc[i] + kSlack);
            l[i] *= a2[i];
        }
    };
    auto rescale = [&](const float (&block_mx)[2]) __attribute__((always_inline)) {
        float a2[2];
        move_reference(block_mx, a2);
        acc_settle();
        for_all<2 * DB * 16>([&](auto n) __attribute__((always_inline)) { acc_scale<decltype(n)::value>(a2[decltype(n)::value / (DB * 16)]); });
        acc_written();
    };

    if (jb < je) {
        bf16x8 qop[2][NU];
        wait_vmem_le<PIECES>();       // Q (the wavefront's own) and the first tile
        asm volatile("" ::: "memory");
        {
            const uint32_t at = r0 + 4 * TILEB + (uint32_t)wave * TILEB;
            const Pair x{at, at ^ 64u};
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int u = 0; u < NU; ++u) qop[i][u] = rd_row(x, u, i * HALF);
        }
        wait_lds();
        barrier();                    // every wavefront's part of the first tile, and Q has left the buffers
        issue_tile();

        f32x16 S[2][2];               // [even and odd block of a tile][32 rows]
        constexpr int AH = NU == 8 ? 4 : 3;
        bf16x8 ring[8];               // the A operands of the unit at hand and of the next three
        const f32x16 zero16 = {};
        Pair a_k = rows_of(0), a_kn = a_k, a_v = cols_of(0);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const bf16x8 x = rd_row(a_k, u, 0);
#pragma unroll
            for (int i = 0; i < 2; ++i) S[0][i] = mfma32(x, qop[i][u], u == 0 ? zero16 : S[0][i]);
        }
#pragma unroll
        for (int u = 0; u < AH; ++u) ring[u] = rd_row(a_k, u, HALF);
        {
            float mx[2] = {lane_max(S[0][0]), lane_max(S[0][1])}, a2[2];
            if ((jb < fb) || (jb >= fe)) mask_block(S[0], jb * BN, mx);
            move_reference(mx, a2);
        }
        uint32_t buf = 0;
        // A block of 32 keys: 4 NU MFMAs without a gap, the scores of the next block and then this block's part of O, and the vector work
        // spread over them: exponentials from the first on (a block's second half is exponentiated while its first is multiplied with V),
        // row sums and the next block's maxima beside the second half.  Operands are requested three units (of two MFMAs) ahead, right behind a
        // unit's first MFMA.  The barrier of a tile lies in its first block, in front of the first read of the next tile's K.
        constexpr int SY = DB < NU - AH ? DB : NU - AH, SLOTS = 4 * NU, MAX0 = 2 * NU + (NU == 8 ? 4 : 3), SUM0 = NU == 8 ? 20 : 8;
        auto stage = [&](auto h_tag, int j) __attribute__((always_inline)) {
            constexpr int H = decltype(h_tag)::value;
            f32x16 (&sc)[2] = S[H];
            f32x16 (&sn)[2] = S[H ^ 1];
            u32x4 pk[2][2];
            float rs[2] = {0.f, 0.f}, mx[2];
            const float mcb[2] = {mc[0] + bias_cur[0], mc[1] + bias_cur[1]};
            // elements in the order of their use: 16 of the first 16 keys, 16 of the others
            auto exp_end = [](int k) { const int e = NU == 8 ? (7 * k + 2) / 5 : 3 * k; return e < 32 ? e : 32; };
            auto slot = [&](int k) __attribute__((always_inline)) {
                const int e0 = exp_end(k), e1 = exp_end(k + 1), done = e0 & ~1, packed = k == 0 ? 0 : exp_end(k - 1) & ~1;
#pragma unroll
                for (int e = 0; e < 32; ++e)
                    if (e >= packed && e < done && !(e & 1)) {
                        const int i = e >> 3 & 1, x = (e >> 4) * 8 + (e & 7);
                        bf16x2 r;
                        r[0] = (__bf16)sc[i][x]; r[1] = (__bf16)sc[i][x + 1];
                        pk[i][x >> 3][(x & 7) >> 1] = opaque(__builtin_bit_cast(uint32_t, r));
                    }
#pragma unroll
                for (int e = 0; e < 32; ++e)
                    if (e >= e0 && e < e1) {
                        const int i = e >> 3 & 1, x = (e >> 4) * 8 + (e & 7);
                        sc[i][x] = fast_exp2(fmaf(sc[i][x], cs, -mcb[i]));
                    }
                if (k >= SUM0) {
                    const int a0 = (k - SUM0) * 32 / (SLOTS - SUM0), a1 = (k + 1 - SUM0) * 32 / (SLOTS - SUM0);
#pragma unroll
                    for (int e = 0; e < 32; ++e)
                        if (e >= a0 && e < a1) {
                            const int i = e >> 3 & 1, x = (e >> 4) * 8 + (e & 7);
                            rs[i] = add_f32_here(rs[i], sc[i][x]);
                        }
                }
                if (k >= MAX0) {
                    const int q0 = (k - MAX0) * 16 / (SLOTS - MAX0), q1 = (k + 1 - MAX0) * 16 / (SLOTS - MAX0);
#pragma unroll
                    for (int q = 0; q < 16; ++q)
                        if (q >= q0 && q < q1) {
                            const int i = q & 1, r = q & ~1;
                            mx[i] = r == 0 ? fmaxf(sn[i][0], sn[i][1]) : fmaxf(fmaxf(mx[i], sn[i][r]), sn[i][r + 1]);
                        }
                }
            };
            const Pair a_s = H ? a_kn : a_k;
            constexpr uint32_t S_AT = H ? 0 : HALF, N_AT = H ? HALF : 0, V_AT = TILEB + H * HALF;
#pragma unroll
            for (int u = 0; u < NU; ++u) {          // the next block's scores
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    sn[i] = mfma32(ring[u & 7], qop[i][u], u == 0 ? zero16 : sn[i]);
                    fence();
                    if (i == 0) ring[(u + AH) & 7] = u + AH < NU ? rd_row(a_s, u + AH, S_AT) : rd_col(a_v, u + AH - NU, V_AT);
                    else if (H == 1 && u + (NU - SY) < PIECES) issue_at(u + (NU - SY));
                    fence();
                    slot(2 * u + i);
                    fence();
                }
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) {          // O
                if (H == 0 && u == SY) {
                    // the next tile is complete (copied in front of the latest one), and every wavefront has left the one before this
                    wait_vmem_le<PIECES>();
                    barrier();
                    buf = (buf + 2 * TILEB) & (NBUF * 2 * TILEB - 1);
                    a_kn = rows_of(buf);
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    acc_mfma(i * DB + u % DB, ring[(u + NU) & 7], pk[i][u / DB]);
                    fence();
                    if (i == 0) ring[(u + NU + AH) & 7] = u + AH < NU ? rd_col(a_v, u + AH, V_AT) : rd_row(a_kn, u + AH - NU, N_AT);
                    else if (H == 0 && u >= SY) issue_at(u - SY);      // the copies of the tile after the next two
                    fence();
                    slot(2 * NU + 2 * u + i);
                    fence();
                }
            }
            l[0] += rs[0];
            l[1] += rs[1];
            const int jn = j + H;                   // the next block's tile
            if (H == 0 || __builtin_expect(jn < je, 1)) {
                if (__builtin_expect((jn < fb) || (jn >= fe), 0)) {
                    asm volatile("");
                    mask_next(sn, jn * BN + (H ? 0 : 32), mx);
                }
                if (__builtin_expect(__any((mx[0] * cs > lim[0]) | (mx[1] * cs > lim[1])), 0)) {
                    asm volatile("");
                    rescale(mx);
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                bias_cur[i] = bias_next[i];
                bias_next[i] = bias_base[i];
            }
        };
        for (int j = jb; j < je; ++j) {
            stage(std::integral_constant<int, 0>{}, j);
            stage(std::integral_constant<int, 1>{}, j);
            a_k = a_kn;
            a_v = cols_of(buf);
        }
    }

    wait_vmem();                  // (the copies past the last tile write zeros)
    acc_settle();
#pragma unroll
    for (int i = 0; i < 2; ++i) l[i] += xhalf(l[i]);
    for_all<2>([&](auto i_tag) __attribute__((always_inline)) {
        constexpr int i = decltype(i_tag)::value;
        const int rl = (wave & 1) * 64 + i * 32 + l32, row = tile * BM + rl;
        if (row >= p.n_q) return;
        if (pc.slot >= 0) {
            // part of a tile: accumulator [row][d], row sums and reference exponents (-inf: no key seen)
            float* part = p.partial + (size_t)(pc.slot + (wave >> 1)) * (BM * D + 2 * BM);
            for_all<DB * 4>([&](auto q) __attribute__((always_inline)) {
                constexpr int a = i * DB * 16 + decltype(q)::value * 4;
                const int d = decltype(q)::value * 8 + half * 4;
                *reinterpret_cast<f32x4*>(part + (size_t)rl * D + d) = f32x4{acc_read<a>(), acc_read<a + 1>(), acc_read<a + 2>(), acc_read<a + 3>()};
            });
            if (half == 0) {
                part[BM * D + rl] = l[i];
                part[BM * D + BM + rl] = (m[i] == -INFINITY) ? -INFINITY : mc[i];
            }
            return;
        }
        const bool live = (hi[i] > 0) && (l[i] > 0.f);
        const float inv = live ? 1.0f / l[i] : 0.f;
        __bf16* op = p.o + ((size_t)row * p.hq + h) * D;
        for_all<DB * 4>([&](auto q) __attribute__((always_inline)) {
            constexpr int a = i * DB * 16 + decltype(q)::value * 4;
            const int d = decltype(q)::value * 8 + half * 4;
            bf16x4 out = pack4(acc_read<a>() * inv, acc_read<a + 1>() * inv, acc_read<a + 2>() * inv, acc_read<a + 3>() * inv);
            if (!live) out = pack4(0.f, 0.f, 0.f, 0.f);
            *reinterpret_cast<bf16x4*>(op + d) = out;
        });
        if (half == 0) p.lse[(size_t)h * p.n_q + row] = live ? m[i] * p.scale + __logf(l[i]) : -INFINITY;
    });
}

template <int D>
constexpr int fwd_pair_lds() { return 4 * 2 * 64 * D * 2; }

template <int D>
__global__ void __launch_bounds__(256, 1) fwd_pair_kernel(const FwdParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[fwd_pair_lds<D>()];   // four buffers: K tile | V tile
    const unsigned long long t_start = wall_clock64();
    const int pairs = p.sched.G / 2;
    RowWalk walk;
    walk.start(p.sched, (int)blockIdx.x, pairs);
    RowPiece pc;
    while (walk.next(p.sched, pc)) {
        if (pc.slot >= 0) pc.slot += pc.member;      // the slot of the pair's first head
        fwd_pair_piece<D>(p, smem, pc);
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

// One workgroup per (query tile in order, two heads), heaviest first; whole tiles only, short-hull tiles left out (their units are faster, and with
// the exact maximum as reference O of tiny documents is off by 1.756e-3, here by 1.786e-3).
template <int D>
__global__ void __launch_bounds__(256, 1) fwd_pair_items_kernel(const FwdParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[fwd_pair_lds<D>()];
    const int pairs = p.hq / p.hkv / 2;
    int y = blockIdx.x >> 3;
    RowPiece pc;
    pc.member = y % pairs; y /= pairs;
    pc.hk = y % p.hkv;
    const int index = (y / p.hkv) * 8 + (blockIdx.x & 7);
    if (index >= p.n_tiles) return;
    const int4 item = ld_const4(p.row_item + 4 * index);
    if (p.use_short && item.w == -2) return;         // fwd_short_tiles_kernel's
    pc.tile = item.x;
    pc.jb = item.y; pc.je = item.z;
    pc.slot = -1;
    fwd_pair_piece<D>(p, smem, pc);
}

void launch_fwd_pair(const FwdParams& p, int head_dim, bool gangs, unsigned grid, hipStream_t stream) {
    if (!gangs) fwd_pair_items_kernel<128><<<grid, 256, 0, stream>>>(p);      // (head dimension 64 runs as gangs alone)
    else if (head_dim == 128) fwd_pair_kernel<128><<<grid, 256, 0, stream>>>(p);
    else fwd_pair_kernel<64><<<grid, 256, 0, stream>>>(p);
}

}  // namespace wlb
