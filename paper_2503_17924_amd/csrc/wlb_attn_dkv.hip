// dK/dV of key tiles that many rows see (wlb_attn_bwd.hip has the derivative and the backward's other kernels).
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "wlb_acc.h"
#include "wlb_attn_bwd.h"
#include "wlb_device.h"
#include "wlb_internal.h"

namespace wlb {

// the launch's parameters once more, loaded where this is written (kept from the start they take scalar registers that the loop needs)
__device__ __forceinline__ const BwdParams& params_here() {
    auto a = (const WLB_CONST BwdParams*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return *(const BwdParams*)a;
}

// One workgroup = 128 keys x one KV head, four wavefronts, one to a SIMD with its 512 registers.  A wavefront holds K, V, dK^T and
// dV^T of 64 of the keys and takes 32 of a stage's 64 rows (stage: row group x query head), so that every operand read from LDS feeds two MFMAs;
// the two wavefronts of the same keys add up at the end of an item.  (With 32 keys a wavefront, scores and gradients in different
// wavefronts and P handed over through LDS, every MFMA needed an operand of its own, and two wavefronts a SIMD waited for LDS and
// each other at a stage's barrier: 4000 cycles a stage where the MFMAs take 2048.)  With one wavefront a SIMD the bound is the
// number of instructions it issues, an MFMA counting as two, exponentials and transposed reads as two, row-wise reads as four of 4
// cycles: 2950 cycles a stage as built, at a clock that the power limit sets 8 % lower.  Four phases of 2 NU MFMAs follow each other without a gap,
// the vector work of one stage spread over the MFMAs that do not depend on it:
//   dK of the stage before | exponentials of the first 16 rows       dP | exponentials of the other 16
//   dV | dS       S of the next stage | the copies three stages ahead
// and each operand is requested three units (of two MFMAs) ahead, right behind a unit's first MFMA: a stream of this mix takes 36 cycles an
// MFMA so, and 41 with the requests behind the exponentials, which hold LDS requests up (5326 -> 5210 us in the first call below, 2203 ->
// 2166 in the third; the clock gives back half of the cycles).  The stage's one barrier lies inside dV, in front of the
// first read of the next stage's tiles.  Per launch, before -> after: 131072 tokens on one of 8 ranks, 8/1 heads 6293 -> 5460 us, at D = 64
// 4306 -> 3492; 32768 tokens, 32/8 heads 2475 -> 2263; 65536 tokens, 8/8 heads, one of 2 ranks 1262 -> 1158; at 24 - 32 stages a
// compute unit, where loading K, V and the first stages (7 us) and adding up count as much as the stages, 80 -> 80.
// A work item is a key tile with all query heads of one KV head, or - for a tile whose work
// exceeds a threshold set by the schedule - a 1/2, 1/4 or 1/8 of those heads; such an item
// writes its dK^T / dV^T as an unscaled fp32 partial result instead of the final bf16 rows.
// SHORT: launched beside dkv_short_kernel, one of the two does the work (a kernel of its own, because the look at which one
// costs the long documents' launches 1 %).
template <int D, bool SHORT>
__global__ void __launch_bounds__(256, 1) dkv_kernel(const BwdParams args) {
    const BwdParams& p = args;
    constexpr int BNK = kBwdKeyTile, GR = kGroupRows, NU = D / 16, DB = D / 32;
    constexpr int ROWB = D * 2, TILEB = GR * ROWB, NW = 4, NBUF = 4, SMALL = 4 * GR * 4;
    static_assert(BNK == 128 && GR == 64, "tiling");

    __shared__ __attribute__((aligned(1024))) char smem[NBUF * 2 * TILEB];   // per stage buffer: Q tile | dO tile, swizzled
    __shared__ __attribute__((aligned(1024))) char small_s[NBUF * SMALL];    // per stage buffer: lse2 | delta | row_lo | row_hi
    __shared__ __attribute__((aligned(1024))) char zero_s[TILEB];            // columns of zeros, in place of a stage that the wavefront leaves out
    __shared__ int s_item;
    if (SHORT && ld_const(p.short_on)) return;                   // dkv_short_kernel has done it
    const int n_items = ld_const(p.key_item_base + p.n_key_tiles);

    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    for (int i = tid; i < TILEB / 16; i += 256) reinterpret_cast<u32x4*>(zero_s)[i] = u32x4{0, 0, 0, 0};
    wait_lds();                                                   // (in front of an item's first barrier)
    const int kb = wave & 1, rh = wave >> 1;                      // the wavefront's 64 keys and 32 rows
    const int l32 = lane & 31, half = lane >> 5, j16 = lane & 15, gi = (lane >> 4) & 1;
    const float cs = p.scale_log2e;
    const uint32_t q_row_bytes = (uint32_t)p.hq * (D * 2u), q_total = (uint32_t)p.n_q * q_row_bytes;
    const uint32_t smem_base = (uint32_t)(uintptr_t)(WLB_LDS char*)smem, small_base = (uint32_t)(uintptr_t)(WLB_LDS char*)small_s;
    const uint32_t zero_at = (uint32_t)(uintptr_t)(WLB_LDS char*)zero_s - smem_base;
    auto lds_f4 = [](uint32_t a) __attribute__((always_inline)) { return *reinterpret_cast<const WLB_LDS f32x4*>((uintptr_t)a); };
    auto lds_i4 = [](uint32_t a) __attribute__((always_inline)) { return *reinterpret_cast<const WLB_LDS i32x4*>((uintptr_t)a); };
    auto lds_i = [](uint32_t a) __attribute__((always_inline)) { return *reinterpret_cast<const WLB_LDS int*>((uintptr_t)a); };
    auto fence = [] () __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
    auto barrier = [] () __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // Tiles lie in LDS as wlb_acc.h says: with the chunks of whole rows XORed (swz) every read took an XOR as well, and the instructions that
    // a wavefront has to issue are what bounds this kernel.
    // Copies: a wavefront takes a quarter of the blocks of the Q and dO tiles and one of the four arrays of per-row scalars.
    constexpr int CH = D / 64, PER = TILEB / 1024 / NW, PIECES = 2 * PER + 1;
    static_assert(PER == 2 * CH, "a wavefront copies 16 rows");
    BufRsrc q_rs, do_rs, sm_rs;
    q_rs.init(p.q, q_total);
    do_rs.init(p.d_o, q_total);
    sm_rs.init(nullptr, (uint32_t)p.n_q * 4u);
    // lane's chunk of a block of even row / 8; of an odd one it is the neighbour
    const uint32_t voff0 = (uint32_t)((lane & 7) ^ ((lane >> 4 & 1) * 4)) * q_row_bytes + (uint32_t)(lane >> 3) * 16u, voff1 = voff0 ^ 16u;
    const uint64_t sm_array = (uint64_t)(uintptr_t)(wave == 0 ? (const void*)p.lse2 : wave == 1 ? (const void*)p.delta : wave == 2 ? (const void*)p.row_lo : (const void*)p.row_hi);
    const uint32_t sm_head = wave < 2 ? (uint32_t)p.n_q * 4u : 0u;
    // (left to the compiler as what they are: told once more that they are uniform it kept them in vector registers, one of which went to memory, and
    // the load of it waited for every copy under way)
    const uint32_t wave_lds = smem_base + (uint32_t)(wave * PER) * 1024u, wave_small = small_base + (uint32_t)wave * (GR * 4);

    // Operands: rows as they lie (row rh * 32 + l32, chunk 2 u + half), for even and odd u; read transposed, rows qq and qq + 8 of 16 and
    // 4 columns of 32 db (lds_read_tr4)
    const uint32_t row0 = smem_base + (uint32_t)((rh * 4 + (l32 >> 3)) * CH) * 1024u + (uint32_t)(half ^ (l32 >> 3 & 1)) * 128u + (uint32_t)(l32 & 7) * 16u, row1 = row0 ^ 64u;
    const int qq = half * 4 + (j16 >> 2), b0 = j16 >> 1 & 1;
    const uint32_t col0 = smem_base + (uint32_t)(rh * 4 * CH) * 1024u + (uint32_t)(gi * 2 + b0) * 128u + (uint32_t)(qq ^ (gi * 4)) * 16u + (j16 & 1) * 8u, col1 = (col0 ^ 128u) + CH * 1024u;
    struct Pair { uint32_t a, b; };
    auto rd_row = [](Pair x, int u, uint32_t tile) __attribute__((always_inline)) {
        return *reinterpret_cast<const WLB_LDS bf16x8*>((uintptr_t)(((u & 1) ? x.b : x.a) + (tile + (u & 3) * 256u + (u >> 2) * 1024u)));
    };
    auto rd_col = [](Pair x, int u, uint32_t tile) __attribute__((always_inline)) {
        const uint32_t cc = u / DB, db = u % DB, at = tile + cc * (2 * CH * 1024u) + (db >> 1) * 1024u + (db & 1) * 512u;
        return cat4(lds_read_tr4_at(x.a + at), lds_read_tr4_at(x.b + at));
    };
    auto rows_of = [&](uint32_t buf) __attribute__((always_inline)) { return Pair{add_here(row0, buf), add_here(row1, buf)}; };
    auto cols_of = [&](uint32_t buf) __attribute__((always_inline)) { return Pair{add_here(col0, buf), add_here(col1, buf)}; };
    // this lane's rows of the scalars (register layout), and its row
    auto vals_at = [&](uint32_t small_at) __attribute__((always_inline)) { return ((opaque((uint32_t)tid) >> 1) & 16) + (small_base + rh * 128 + small_at); };
    auto row_at = [&](uint32_t small_at) __attribute__((always_inline)) { return (opaque((uint32_t)tid) & 31) * 4 + (small_base + rh * 128 + small_at); };

    // Work items: tiles in order (heaviest item first), a tile's items consecutive: KV head major, head
    // part minor.  The launch is one workgroup per compute unit, and each takes item after item until
    // none is left.  Item i belongs to XCD i % 8 (workgroup b runs on XCD b % 8): the same head part of
    // neighbouring tiles then shares an XCD and its L2 copy of the Q / dO tiles.  A workgroup takes its own
    // XCD's items first, and the other XCDs' once those are gone: the XCDs of one GPU differ in speed by several
    // percent (the same ones are slower in every launch), and with one workgroup per item the hardware hands every
    // XCD the same number of them.  The first item goes by the workgroup's index, the others through one counter per XCD.
    const int list = (int)blockIdx.x % kLists;
    auto of_list = [&](int c, int n) __attribute__((always_inline)) { return (((int)gridDim.x - c + kLists - 1) / kLists + n) * kLists + c; };
  for (int item = (int)blockIdx.x; item < n_items;) {
    // one record per item: finding the tile by a search of the item bases and then its tables was a chain of a dozen
    // dependent loads in front of every item
    const BwdParams& p = params_here();
    const int4 rec0 = ld_const4(p.dkv_item + 8 * item), rec1 = ld_const4(p.dkv_item + 8 * item + 4);
    const int kt = rec0.x, hk = rec0.y, h_first = rec0.z, nh = rec0.w;   // query heads [h_first, h_first + nh)
    const int slot = rec1.x, g_first = rec1.y, t1 = rec1.z;
    const int kw0 = kt * BNK + kb * 64;

    // Stage t of the item is row group g_first + t / nh with query head h_first + t % nh.  The copies run three stages ahead; past
    // the last stage they read past the tensors' ends, that is zeros and no memory.
    int nx_left = t1, nx_h = 0;
    uint32_t nx_so = (uint32_t)g_first * (GR * q_row_bytes) + (uint32_t)h_first * ROWB + (uint32_t)(wave * 16) * q_row_bytes;
    uint32_t nx_row = (uint32_t)g_first * (GR * 4), nx_b = 0;
    uint64_t nx_sm = sm_array + (uint64_t)(uint32_t)h_first * sm_head;
    const uint32_t group_step = GR * q_row_bytes - (uint32_t)nh * ROWB, n_q_bytes = (uint32_t)p.n_q * 4u;
    const uint64_t head_back = (uint64_t)(uint32_t)nh * sm_head;
    uint32_t at_so = 0, at_lds = 0;               // of the copies at hand
    const uint32_t rows8 = 8u * q_row_bytes;
    auto issue_piece = [&](auto k_tag) __attribute__((always_inline)) {
        constexpr int k = decltype(k_tag)::value, n = k >> 1;          // block n of the wavefront's: row group n / CH, columns 64 (n % CH) on
        if constexpr (k < 2 * PER) {
            if (k == 0) {
                at_so = uniform(nx_left > 0 ? nx_so : q_total);
                at_lds = wave_lds + nx_b * (2 * TILEB);
            }
            const int voff = (int)(n / CH ? voff1 : voff0);
            if constexpr (k & 1) dma_issue_at<TILEB + n * 1024>(do_rs.r, at_lds, voff, at_so);
            else if constexpr (k == 0) dma_issue_at<0>(q_rs.r, at_lds, voff, at_so);
            else at_so = dma_issue_step<n * 1024>(q_rs.r, at_lds, voff, at_so, n % CH ? 128u : CH == 2 ? rows8 - 128u : rows8);
        } else {
            sm_rs.r[0] = (int)(uint32_t)nx_sm;
            sm_rs.r[1] = (int)(uint32_t)((nx_sm >> 32) & 0xffffu);
            sm_rs.make_uniform();
            dma_issue_256(sm_rs.r, wave_small + nx_b * SMALL, (int)((opaque((uint32_t)tid) & 63) * 4), uniform(nx_left > 0 ? nx_row : n_q_bytes));
            // the next stage (no branch: this sits between MFMAs)
            --nx_left;
            nx_b = (nx_b + 1) & (NBUF - 1);
            ++nx_h;
            const uint32_t wrap = ~(uint32_t)((nx_h - nh) >> 31);      // all ones: nx_h == nh
            nx_h &= (int)~wrap;
            nx_so += (uint32_t)ROWB + (group_step & wrap);
            nx_sm += sm_head - (head_back & (uint64_t)(int64_t)(int32_t)wrap);
            nx_row += (GR * 4u) & wrap;
        }
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
            case 8: if constexpr (8 < PIECES) issue_piece(std::integral_constant<int, 8>{}); break;
        }
    };
    auto issue_stage = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < PIECES; ++k) issue_at(k);
    };
    // K and V of the 128 keys come through the ring's third and fourth buffer (read from global memory in operand layout, 32 bytes of a
    // row at a time, they took longer than five stages)
    {
        const BwdParams& p = params_here();
        const uint32_t kv_row = (uint32_t)p.hkv * (D * 2u), kv_total = (uint32_t)p.t_kv * kv_row;
        const int lane = (int)opaque((uint32_t)tid) & 63;
        const uint32_t kvoff0 = (uint32_t)((lane & 7) ^ ((lane >> 4 & 1) * 4)) * kv_row + (uint32_t)(lane >> 3) * 16u;
        BufRsrc kv_rs;
        kv_rs.init(p.k, kv_total);
        uint32_t so = uniform((uint32_t)(kt * BNK + wave * 16) * kv_row + (uint32_t)hk * ROWB);
        const uint32_t at = wave_lds + 4 * TILEB, kv_rows8 = 8u * kv_row;
        for_all<4>([&](auto tile) __attribute__((always_inline)) {                  // 64 rows of K, 64 more, V
            if (tile == 2) kv_rs.init(p.v, kv_total);
            uint32_t block = uniform(so + (tile & 1) * 64u * kv_row);
            for_all<PER>([&](auto n) __attribute__((always_inline)) {
                const int voff = (int)(n / CH ? kvoff0 ^ 16u : kvoff0);
                constexpr int OFF = tile * TILEB + n * 1024;
                if constexpr (n == 0) dma_issue_at<OFF>(kv_rs.r, at, voff, block);
                else block = dma_issue_step<OFF>(kv_rs.r, at, voff, block, n % CH ? 128u : CH == 2 ? kv_rows8 - 128u : kv_rows8);
            });
        });
    }
#pragma nounroll
    for (int k = 0; k < 2; ++k) issue_stage();
    for_all<4 * DB>([](auto i) __attribute__((always_inline)) { acc_zero<decltype(i)::value>(u32x4{0, 0, 0, 0}); });
    bf16x8 kop[2][NU], vop[2][NU];                  // [32 keys]: the B operands of S and dP
    wait_vmem_le<2 * PIECES>();
    barrier();
    {
        const int lane = (int)opaque((uint32_t)tid) & 63, l32 = lane & 31, half = lane >> 5;
        const uint32_t at = smem_base + 4 * TILEB + (uint32_t)kb * TILEB + (uint32_t)((l32 >> 3) * CH) * 1024u + (uint32_t)(half ^ (l32 >> 3 & 1)) * 128u + (uint32_t)(l32 & 7) * 16u;
        const Pair x{at, at ^ 64u};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                kop[i][u] = rd_row(x, u, i * (4 * CH * 1024u));
                vop[i][u] = rd_row(x, u, 2 * TILEB + i * (4 * CH * 1024u));
            }
    }
    wait_lds();
    wait_vmem_le<PIECES>();       // the first stage
    barrier();                    // every wavefront has its operands
    issue_stage();
    constexpr int ACC_DK = 0, ACC_DV = 2 * DB;      // accumulator of 32 keys i and 32 columns db: + i * DB + db

    f32x16 s[2], dp[2];                             // [32 keys]
    u32x4 pk[2][2], ds[2][2];                       // P and dS as operands: [32 keys][16 rows], two values in each element
    f32x4 ls[4];
    bf16x8 ring[4];                                 // the A operands of the unit at hand and of the next three
#pragma unroll
    for (int i = 0; i < 2; ++i) ds[i][0] = ds[i][1] = u32x4{0, 0, 0, 0};
    float carry = 0.f;                              // the first of two elements of dS that are packed together
    auto pack2 = [](float x, float y) __attribute__((always_inline)) {
        bf16x2 r;
        r[0] = (__bf16)x; r[1] = (__bf16)y;
        return opaque(__builtin_bit_cast(uint32_t, r));
    };
    // Row half c = 0, 1 of S has 16 elements in this lane: 8 rows x 2 x 32 keys.  P of 16 / (2 NU) of them, in place, beside MFMA `sl` of a
    // phase's 2 NU; a pair is packed beside the MFMA after (its exponentials have a wait state).
    auto pack_p = [&](int c, int e) __attribute__((always_inline)) {      // elements e, e + 1
        const int i = e >> 3, x = c * 8 + (e & 7);
        pk[i][c][(x & 7) >> 1] = pack2(s[i][x], s[i][x + 1]);
    };
    auto exp_slot = [&](int c, int sl) __attribute__((always_inline)) {
        constexpr int N = 8 / NU;
        float arg[N];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int e = sl * N + n, i = e >> 3, x = c * 8 + (e & 7);
            arg[n] = fmaf(s[i][x], cs, -ls[x >> 2][x & 3]);
        }
        if (N == 2 && sl > 0) pack_p(c, sl * N - 2);
        if (N == 1 && sl > 0 && sl % 2 == 0) pack_p(c, sl - 2);
        if (sl == 0 && c == 1) pack_p(0, 14);
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int e = sl * N + n, i = e >> 3, x = c * 8 + (e & 7);
            s[i][x] = fast_exp2(arg[n]);
        }
    };
    // dS = P o (dP - delta), 32 elements beside the 2 NU MFMAs of a phase
    auto ds_slot = [&](int sl) __attribute__((always_inline)) {
        constexpr int N = 16 / NU;
        if (sl == 0) pack_p(1, 14);
#pragma unroll
        for (int e = sl * N; e < (sl + 1) * N; ++e) {
            const int i = e >> 4, x = e & 15;
            if (x & 1) ds[i][x >> 3][(x & 7) >> 1] = pack2(carry, s[i][x] * dp[i][x]);
            else carry = s[i][x] * dp[i][x];
        }
    };
    // Whether the wavefront's rows see any of its keys, all of them, and whether padding is among them (rows past the end count).
    struct Flags { bool live, full, pads; };
    auto flags = [&](int lo, int hi) __attribute__((always_inline)) {
        const bool real = hi > 0;
        Flags f;
        f.live = __any(real && lo < kw0 + 64 && hi > kw0);
        f.full = __all(real && lo <= kw0 && hi >= kw0 + 64);
        f.pads = __any(!real);
        return f;
    };
    // Whether a row's LSE or delta is Inf or NaN, as they are where its Q or dO is, or a K or V that it sees.  0 x Inf is not 0, so
    // such rows may meet only keys that they see: odd_stage.
    auto odd_rows = [&](int hi, int lse, int delta) __attribute__((always_inline)) {
        return (bool)__any(hi > 0 && max((uint32_t)lse & 0x7f800000u, (uint32_t)delta & 0x7f800000u) == 0x7f800000u);
    };
    // Scores of invisible pairs become -inf, rows of padding (which may hold anything) zero.  Both wavefronts of the same rows write the
    // zeros, so none waits for the other.
    auto mask = [&](uint32_t small_at) __attribute__((always_inline)) {
        const uint32_t a = vals_at(small_at);
        const int my = kw0 + ((int)opaque((uint32_t)tid) & 31);
#pragma unroll
        for (int g = 0; g < 4; g += 2) {
            i32x4 l4[2], w4[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                l4[h] = lds_i4(a + 2 * GR * 4 + (g + h) * 32);
                w4[h] = lds_i4(a + 3 * GR * 4 + (g + h) * 32);
            }
            fence();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                w4[h] -= l4[h];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e)       // one comparison: a padding row's width is 2^31 + 1, of which no key's distance falls short
                        s[i][(g + h) * 4 + e] = (uint32_t)(my + i * 32 - l4[h][e]) < (uint32_t)w4[h][e] ? s[i][(g + h) * 4 + e] : -INFINITY;
                fence();
            }
        }
    };
    auto zero_pads = [&](int hi, uint32_t buf) __attribute__((always_inline)) {
        if (hi == 0) {
            const Pair x = rows_of(buf);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const uint32_t a = ((u & 1) ? x.b : x.a) + (u & 3) * 256u + (u >> 2) * 1024u;
                *reinterpret_cast<WLB_LDS i32x4*>((uintptr_t)a) = i32x4{0, 0, 0, 0};
                *reinterpret_cast<WLB_LDS i32x4*>((uintptr_t)(a + TILEB)) = i32x4{0, 0, 0, 0};
            }
        }
        asm volatile("" ::: "memory");
    };
    auto dk_unit = [&](int u) __attribute__((always_inline)) {
        const bf16x8 a = ring[u & 3];
#pragma unroll
        for (int i = 0; i < 2; ++i) acc_mfma(ACC_DK + i * DB + u % DB, a, ds[i][u / DB]);
    };
    // dK of the stage whose Q columns are at x, without anything beside it
    auto flush_dk = [&](Pair x) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            ring[u & 3] = rd_col(x, u, 0);
            dk_unit(u);
        }
    };
    const f32x16 zero16 = {};
    // All of a stage after its scores, without anything beside it: P and dS of invisible pairs are zeros whatever the rows hold, and of the two
    // sets of 32 keys only those that one of the rows sees are added to.
    auto odd_stage = [&](Pair x_row, Pair x_col, uint32_t small_at) __attribute__((always_inline)) {
        const uint32_t a = vals_at(small_at), ra = row_at(small_at);
        const int lo = lds_i(ra + 2 * GR * 4), hi = lds_i(ra + 3 * GR * 4), my = kw0 + ((int)opaque((uint32_t)tid) & 31);
        for_all<2>([&](auto i_tag) __attribute__((always_inline)) {
            constexpr int i = decltype(i_tag)::value;
            if (!__any(hi > 0 && lo < kw0 + i * 32 + 32 && hi > kw0 + i * 32)) return;
#pragma unroll
            for (int e = 0; e < 16; ++e) dp[i][e] = __builtin_bit_cast(float, lds_i(a + GR * 4 + (e >> 2) * 32 + (e & 3) * 4));
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                dp[i] = mfma32(rd_row(x_row, u, TILEB), vop[i][u], dp[i]);
                fence();
            }
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                float pe[2], de[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const uint32_t at = a + ((e + j) >> 2) * 32 + ((e + j) & 3) * 4;
                    const int l = lds_i(at + 2 * GR * 4), w = lds_i(at + 3 * GR * 4) - l;
                    const bool seen = (uint32_t)(my + i * 32 - l) < (uint32_t)w;
                    const float pv = fast_exp2(fmaf(s[i][e + j], cs, -__builtin_bit_cast(float, lds_i(at))));
                    pe[j] = seen ? pv : 0.f;
                    de[j] = seen ? pv * dp[i][e + j] : 0.f;
                }
                pk[i][e >> 3][(e & 7) >> 1] = pack2(pe[0], pe[1]);
                ds[i][e >> 3][(e & 7) >> 1] = pack2(de[0], de[1]);
                fence();
            }
            asm volatile("s_nop 1");
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                acc_mfma(ACC_DV + i * DB + u % DB, rd_col(x_col, u, TILEB), pk[i][u / DB]);
                fence();
                acc_mfma(ACC_DK + i * DB + u % DB, rd_col(x_col, u, 0), ds[i][u / DB]);
                fence();
            }
        });
    };

    // first stage: scores
    Flags f;
    bool odd = false;
    Pair a_row = rows_of(0), a_dk = cols_of(0);     // of the stage's buffer; of the buffer of the stage whose dK is pending
    bool pending = false;                           // (none is: dS = 0, of any buffer)
    {
        const uint32_t a = row_at(0);
        const int lo = lds_i(a + 2 * GR * 4), hi = lds_i(a + 3 * GR * 4);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const bf16x8 x = rd_row(a_row, u, 0);
#pragma unroll
            for (int i = 0; i < 2; ++i) s[i] = mfma32(x, kop[i][u], u == 0 ? zero16 : s[i]);
        }
        f = flags(lo, hi);
        if (!f.full) {
            asm volatile("");
            const int lse = lds_i(a), delta = lds_i(a + GR * 4);
            mask(0);
            odd = odd_rows(hi, lse, delta);
            if (f.pads) zero_pads(hi, 0);
        }
#pragma unroll
        for (int g8 = 0; g8 < 2; ++g8) ls[g8] = lds_f4(vals_at(0) + g8 * 32);
#pragma unroll
        for (int u = 0; u < 3; ++u) ring[u] = rd_col(a_dk, u, 0);
    }
    constexpr int SY = DB < NU - 3 ? DB : NU - 3;   // dV units in front of the barrier: what follows reads the next stage's Q
    uint32_t buf = 0, small_at = 0;
    int hh = 0;
    for (int t = 0; t < t1; ++t) {
        const bool live = f.live && !odd;
        Pair a_col = cols_of(buf);
        if (live) {
            const uint32_t a_s = vals_at(small_at);
            f32x16 dl;
#pragma unroll
            for (int u = 0; u < NU; ++u) {          // dK of the stage before
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    acc_mfma(ACC_DK + i * DB + u % DB, ring[u & 3], ds[i][u / DB]);
                    fence();
                    if (i == 0) {
                        ring[(u + 3) & 3] = u + 3 < NU ? rd_col(a_dk, u + 3, 0) : rd_row(a_row, u + 3 - NU, TILEB);
                        if (u < 2) ls[2 + u] = lds_f4(a_s + (2 + u) * 32);
                        if (u >= NU - 4) {
                            const int g8 = u - (NU - 4);
                            const f32x4 x = lds_f4(a_s + GR * 4 + g8 * 32);
#pragma unroll
                            for (int e = 0; e < 4; ++e) dl[g8 * 4 + e] = x[e];
                        }
                        fence();
                    }
                    exp_slot(0, 2 * u + i);
                    fence();
                }
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) {          // dP - delta
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    dp[i] = mfma32(ring[u & 3], vop[i][u], u == 0 ? dl : dp[i]);
                    fence();
                    if (i == 0) {
                        ring[(u + 3) & 3] = u + 3 < NU ? rd_row(a_row, u + 3, TILEB) : rd_col(a_col, u + 3 - NU, TILEB);
                        fence();
                    }
                    exp_slot(1, 2 * u + i);
                    fence();
                }
            }
#pragma unroll
            for (int u = 0; u < SY; ++u) {          // dV, first part
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    acc_mfma(ACC_DV + i * DB + u % DB, ring[u & 3], pk[i][u / DB]);
                    fence();
                    if (i == 0) {
                        ring[(u + 3) & 3] = rd_col(a_col, u + 3, TILEB);
                        fence();
                    }
                    ds_slot(2 * u + i);
                    fence();
                }
            }
        } else {
            // none of the wavefront's pairs is visible here, or rows are odd: the pending dK while its rows are still in LDS, then zeros
            // times zeros (the rows of a stage that the wavefront does not see may hold anything)
            if (pending) flush_dk(a_dk);
            if (f.live) {
                asm volatile("");
                odd_stage(a_row, a_col, small_at);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                ds[i][0] = ds[i][1] = pk[i][0] = pk[i][1] = u32x4{0, 0, 0, 0};
                s[i] = dp[i] = zero16;
            }
            carry = 0.f;
#pragma unroll
            for (int u = SY; u < SY + 3; ++u) ring[u & 3] = bf16x8{};
            a_col = cols_of(zero_at - TILEB);
        }
        // The next stage's copies are complete (issued in front of the latest ones), and every wavefront has left the buffer of the
        // stage before this one.
        wait_vmem_le<PIECES>();
        barrier();
        const uint32_t buf_n = (buf + 2 * TILEB) & (NBUF * 2 * TILEB - 1), small_n = (small_at + SMALL) & (NBUF * SMALL - 1);
        a_row = rows_of(buf_n);
        int lo, hi;
        {
            const uint32_t a = row_at(small_n);
            lo = lds_i(a + 2 * GR * 4); hi = lds_i(a + 3 * GR * 4);
        }
#pragma unroll
        for (int u = SY; u < NU; ++u) {             // dV, second part
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                acc_mfma(ACC_DV + i * DB + u % DB, ring[u & 3], pk[i][u / DB]);
                fence();
                if (i == 0) {
                    ring[(u + 3) & 3] = u + 3 < NU ? rd_col(a_col, u + 3, TILEB) : rd_row(a_row, u + 3 - NU, 0);
                    fence();
                } else {
                    issue_at(u - SY);                 // the copies of the stage after the next two, a piece per unit
                    fence();
                }
                ds_slot(2 * u + i);
                fence();
            }
        }
        a_dk = cols_of(live ? buf : zero_at);
        pending = live;
        const uint32_t a_sn = vals_at(small_n);
#pragma unroll
        for (int u = 0; u < NU; ++u) {              // the next stage's scores (after the last stage: of zeros, not used)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                s[i] = mfma32(ring[u & 3], kop[i][u], u == 0 ? zero16 : s[i]);
                fence();
                if (i == 0) {
                    ring[(u + 3) & 3] = u + 3 < NU ? rd_row(a_row, u + 3, 0) : rd_col(a_dk, u + 3 - NU, 0);
                    if (u == 1 || u == 2) ls[u - 1] = lds_f4(a_sn + (u - 1) * 32);
                } else if (u + (NU - SY) < PIECES) issue_at(u + (NU - SY));
                fence();
            }
        }
        if (++hh == nh) hh = 0;
        if (hh == 0) f = flags(lo, hi);             // other rows
        odd = false;
        if (!f.full) {
            asm volatile("");
            const uint32_t a = row_at(small_n);
            const int lse = lds_i(a), delta = lds_i(a + GR * 4);
            mask(small_n);
            odd = odd_rows(hi, lse, delta);
            if (f.pads) zero_pads(hi, buf_n);
        }
        buf = buf_n;
        small_at = small_n;
    }
    if (pending) flush_dk(a_dk);

    // The two wavefronts of the same keys add up through LDS, dV and then dK: every wavefront leaves its accumulators ([32 keys and columns]
    // [4 columns][lane] x 16 bytes, lanes XORed so that whole rows are read without bank conflicts), and every thread takes 4 columns
    // of a row at a time, so that rows leave whole.
    wait_vmem();                  // (the copies past the last stage write zeros)
    acc_settle();
    int next = 0;
    if (tid == 0) next = of_list(list, atomicAdd(params_here().dkv_counters + list, 1));      // (its answer comes meanwhile)
    constexpr uint32_t ACC_BYTES = 2 * DB * 4096;   // of a wavefront and gradient
    auto finish = [&](auto first, bool of_k) __attribute__((always_inline)) {
        const int l = (int)opaque((uint32_t)tid), lane = l & 63;
        __syncthreads();          // every wavefront has left what is overwritten
        const uint32_t mine = smem_base + (uint32_t)wave * ACC_BYTES + (uint32_t)(lane ^ (lane >> 5) * 8) * 16u;
        for_all<8>([&](auto x) __attribute__((always_inline)) {
            const uint32_t at = mine ^ (x * 16u);
            for_all<2 * DB * 4 / 8>([&](auto y) __attribute__((always_inline)) { acc_to_lds<first + y * 8 + x, (y * 8 + x) * 1024>(at); });
        });
        wait_lds();
        __syncthreads();
        const BwdParams& p = params_here();
        const float f = of_k ? p.scale : 1.0f;
        __bf16* const dst = of_k ? p.dk : p.dv;
        float* const part = p.partial + (size_t)max(slot, 0) * (2 * BNK * D) + (of_k ? 0 : BNK * D);     // [dK | dV][key][d], unscaled
        // thread: columns 4 c .. of key k + 8 j (D = 128)
        constexpr int V4 = D / 4, STEP = 256 / V4;
        const int c = l % V4, k0 = (l & 255) / V4;
        const uint32_t quad = (uint32_t)(c >> 3) * 4u + (uint32_t)(c >> 1 & 3), hf = (uint32_t)(c & 1);
        const uint32_t total = (uint32_t)p.t_kv * (uint32_t)p.hkv * ROWB;
        const buf_rsrc_t out = make_buf(dst, total);                     // (keys past t_kv are not stored)
        const uint32_t key_bytes = (uint32_t)p.hkv * ROWB;
        const int voff = k0 * (int)key_bytes + c * 8;
        const uint32_t soff0 = (uint32_t)(kt * BNK) * key_bytes + (uint32_t)hk * ROWB;
        float* const po = part + (size_t)k0 * D + c * 4;
        constexpr int U = 8;                          // rows whose loads are requested together
#pragma nounroll
        for (int j0 = 0; j0 < BNK / STEP; j0 += U) {
            f32x4 x[U], y[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int k = k0 + (j0 + j) * STEP;  // of the tile's 128: wavefronts k / 64 and k / 64 + 2, 32 keys k / 32 % 2
                const uint32_t at = smem_base + (uint32_t)(k >> 6) * ACC_BYTES + ((uint32_t)(k >> 5 & 1) * (DB * 4) + quad) * 1024u
                                    + (hf * 32u + (((uint32_t)k & 31u) ^ (hf * 8u) ^ (quad & 7u))) * 16u;
                x[j] = lds_f4(at);
                y[j] = lds_f4(at + 2 * ACC_BYTES);
            }
            fence();
            if (slot >= 0) {
#pragma unroll
                for (int j = 0; j < U; ++j) *reinterpret_cast<f32x4*>(po + (size_t)(j0 + j) * (STEP * D)) = x[j] + y[j];
            } else {
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    x[j] += y[j];
                    const bf16x4 r = pack4(x[j][0] * f, x[j][1] * f, x[j][2] * f, x[j][3] * f);
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(__attribute__((ext_vector_type(2))) unsigned, r), out, voff,
                                                          (int)uniform(soff0 + (uint32_t)(j0 + j) * STEP * key_bytes), 0);
                }
            }
        }
    };
    finish(std::integral_constant<int, ACC_DV * 4>{}, false);
    finish(std::integral_constant<int, ACC_DK * 4>{}, true);
    if (tid == 0) {
        for (int k = 1; k < kLists && next >= n_items; ++k) {
            const int c = (list + k) % kLists;
            next = of_list(c, atomicAdd(params_here().dkv_counters + c, 1));
        }
        s_item = next;
    }
    __syncthreads();              // (and every wavefront has left the LDS)
    item = uniform(s_item);
  }   // next item
}

void launch_dkv_general(const BwdParams& p, int head_dim, bool beside_short, unsigned grid, hipStream_t stream) {
    if (head_dim == 128 && beside_short) dkv_kernel<128, true><<<grid, 256, 0, stream>>>(p);
    else if (head_dim == 128) dkv_kernel<128, false><<<grid, 256, 0, stream>>>(p);
    else if (beside_short) dkv_kernel<64, true><<<grid, 256, 0, stream>>>(p);
    else dkv_kernel<64, false><<<grid, 256, 0, stream>>>(p);
}

}  // namespace wlb
