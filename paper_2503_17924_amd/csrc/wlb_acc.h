// Accumulators that a kernel names by number, and other statements of kernels that run one wavefront to a SIMD.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "wlb_device.h"

namespace wlb {

// Layout of the tiles in LDS of these kernels.
// Tiles of rows x D that operands are read from both row-wise and transposed lie in LDS as blocks of 1 KiB: 8 rows x 64 columns, block
// (row / 8) * CH + column / 64.  Of a block's 64 chunks of 16 bytes the one of row r and chunk column c is number
// ((c & 7) ^ (r >> 3 & 1)) * 8 + ((r & 7) ^ (c >> 1 & 1) * 4).  Both ways to read a tile are then free of bank conflicts, and an operand's place
// is one of two registers plus a constant.

// The accumulators of such a kernel fill half or all of the accumulation registers (AGPRs), and the compiler does not keep such a
// set in place through a loop with branches (it copies and spills all of it).  They are therefore registers by number, 16 to an
// accumulator, named in the statements below and declared as written by each; build.py refuses code in which the compiler
// touches one on its own account.  What an accumulating MFMA leaves is read by that accumulator's next one (which the hardware orders)
// and, after acc_settle(), by acc_to_lds, acc_read and acc_scale; what acc_write and acc_scale leave, by MFMAs some
// instructions later (acc_written() where none lie between).
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
#define WLB_ACC_ALL \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", \
    "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", \
    "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", \
    "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63", \
    "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79", \
    "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95", \
    "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111", \
    "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127", \
    "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143", \
    "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159", \
    "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175", \
    "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191", \
    "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", \
    "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223", \
    "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239", \
    "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255"
// Two wait states must lie between a vector instruction and an MFMA that reads what it wrote, and the compiler does not put them in front of a
// statement of ours.  As built, operands come from LDS or were packed some instructions before; build.py refuses code in which that is not so.
template <int I>
__device__ __forceinline__ void acc_mfma(bf16x8 a, u32x4 b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %3, a[%0:%1] ; acc" ::"n"(I * 16), "n"(I * 16 + 15), "v"(a), "v"(b) : WLB_ACC_ALL);
}
template <int I>
__device__ __forceinline__ void acc_zero(u32x4 zeros) {      // 0 x 0 + 0: an instruction where writing the registers takes sixteen
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %2, 0 ; acc" ::"n"(I * 16), "n"(I * 16 + 15), "v"(zeros) : WLB_ACC_ALL);
}
// registers 4 Q .. 4 Q + 3 to LDS at addr + OFF; complete after wait_lds()
template <int Q, int OFF>
__device__ __forceinline__ void acc_to_lds(uint32_t addr) {
    asm volatile("ds_write_b128 %0, a[%1:%2] offset:%3 ; acc" ::"v"(addr), "n"(4 * Q), "n"(4 * Q + 3), "n"(OFF) : "memory");
}
__device__ __forceinline__ void acc_settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }
// the same with an index that is a constant once loops are unrolled
__device__ __forceinline__ void acc_mfma(int i, bf16x8 a, u32x4 b) {
    switch (i) {
        case 0: acc_mfma<0>(a, b); break;
        case 1: acc_mfma<1>(a, b); break;
        case 2: acc_mfma<2>(a, b); break;
        case 3: acc_mfma<3>(a, b); break;
        case 4: acc_mfma<4>(a, b); break;
        case 5: acc_mfma<5>(a, b); break;
        case 6: acc_mfma<6>(a, b); break;
        case 7: acc_mfma<7>(a, b); break;
        case 8: acc_mfma<8>(a, b); break;
        case 9: acc_mfma<9>(a, b); break;
        case 10: acc_mfma<10>(a, b); break;
        case 11: acc_mfma<11>(a, b); break;
        case 12: acc_mfma<12>(a, b); break;
        case 13: acc_mfma<13>(a, b); break;
        case 14: acc_mfma<14>(a, b); break;
        case 15: acc_mfma<15>(a, b); break;
    }
}
// f(integral_constant 0), ..., f(integral_constant N - 1)
template <class F, int... I>
__device__ __forceinline__ void for_all(std::integer_sequence<int, I...>, F f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void for_all(F f) { for_all(std::make_integer_sequence<int, N>{}, f); }
// keeps what is derived from x where it is written (as loop invariants such values take more registers than there are)
__device__ __forceinline__ uint32_t opaque(uint32_t x) { asm volatile("" : "+v"(x)); return x; }
__device__ __forceinline__ uint32_t add_here(uint32_t x, uint32_t uniform_y) {
    uint32_t r;
    asm volatile("v_add_u32 %0, %1, %2" : "=v"(r) : "s"(uniform_y), "v"(x));
    return r;
}
// dma_issue_1k to lds + OFF; the second form at soff + step, which it returns (the addition fills the wait state after a write to m0)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int OFF>
__device__ __forceinline__ void dma_issue_at(const i32x4& rsrc, uint32_t lds, int voff, uint32_t soff) {
    asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff), "n"(OFF) : "memory", "m0", "scc");
}
template <int OFF>
__device__ __forceinline__ uint32_t dma_issue_step(const i32x4& rsrc, uint32_t lds, int voff, uint32_t soff, uint32_t step) {
    uint32_t so;
    asm volatile("s_add_u32 m0, %1, %6\n\ts_add_u32 %0, %4, %5\n\tbuffer_load_dwordx4 %2, %3, %0 offen lds"
                 : "=&s"(so) : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff), "s"(step), "n"(OFF) : "memory", "m0", "scc");
    return so;
}
#pragma clang diagnostic pop
// register N as a value, after acc_settle()
template <int N>
__device__ __forceinline__ float acc_read() {
    float x;
    asm volatile("v_accvgpr_read_b32 %0, a[%1] ; acc" : "=v"(x) : "n"(N));
    return x;
}
// register N times f, after acc_settle() and in front of acc_written()
template <int N>
__device__ __forceinline__ void acc_scale(float f) {
    float x;
    asm volatile("v_accvgpr_read_b32 %0, a[%2] ; acc\n\tv_mul_f32 %0, %0, %1\n\tv_accvgpr_write_b32 a[%2], %0 ; acc" : "=&v"(x) : "v"(f), "n"(N) : WLB_ACC_ALL);
}
// in front of the first MFMA that reads it by some instructions
template <int N>
__device__ __forceinline__ void acc_write(uint32_t x) {
    asm volatile("v_accvgpr_write_b32 a[%0], %1 ; acc" ::"n"(N), "v"(x) : WLB_ACC_ALL);
}
__device__ __forceinline__ void acc_written() { asm volatile("s_nop 3" ::: "memory"); }

}  // namespace wlb
