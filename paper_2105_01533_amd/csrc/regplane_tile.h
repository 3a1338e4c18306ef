// Register-plane form of the fused phase/permutation pass (Sec. 3.2), for
// gfx950 (device code; included by mono_regplane.hip).
//
// A wave owns a tile of 2048 entries: lane l holds entries l + 64 j, j =
// 0..31, as 32-bit bit-planes (bit j of plane q = qubit q of entry j).  The
// planes live in VGPRs v100 .. v100 + nq + 2 for the whole run: the compiler
// is capped below v80 (amdgpu_num_vgpr), so it never allocates v80 and above,
// and only the inline assembly here touches them.  A gate names its planes by
// index at run time, so the plane registers are addressed with the GPR
// indexing mode (the low byte of M0 is added to the register number of the
// operands that M0's bits 12-15 enable), with no LDS round trip.
//
// Register map (fixed, assembly only):
//   v80        P  -- eighth-turn accumulator, weight 4 (one bit per entry)
//   v81, v82   Q  -- weight-2 counter, 2 bits
//   v83..v85   R  -- weight-1 counter, 3 bits
//   v86..v94   temporaries; v95 prefetch address, v96 prefetch target
//   v97        the lane number (kept here, it costs the compiler no register)
//   v100 + q   plane q; plane nq is all ones, nq + 1 scratch, nq + 2 zero.
// An eighth-turn op adding k where x holds adds x (k & 1) to R, x ((k >> 1) &
// 1) to Q and x (k >> 2) to P, so the entry's count is R + 2 Q + 4 P mod 8.
//
// What bounds the pass is the latency of one wave's instruction stream: at
// most two waves share a SIMD (the planes' registers), each in order.  So the
// interpreter spends as few instructions as it can on each op.  Its program
// (RpBlock, see sim_internal.h) is read with scalar loads, a 64-byte block
// ahead into the SGPRs the current block does not use, and every operand field
// is an index with its operand-enable bits in the form M0 holds them, so
// that one scalar move or shift both unpacks and selects it: a CNOT is four
// instructions, a Toffoli six.  A block holds ops of one shape; its first word
// is the distance from the block handlers' base to the instruction that starts
// with its first op, so a partly filled block runs no padding and a dispatch
// is six instructions.  Read with v_readlane and padded to quads, the same
// programs took 25 ns per CNOT, 31 per Toffoli and 102 per gate of adders (short
// segments) of one wave; they take 11, 15 and 16 (2^16 entries).  Turn ops do
// not break the stream either: their conditions are flipped into capture
// planes and their fractions added eight at a time (random mix of 24 qubits: 68
// ns per gate, 41 without the capture planes, 26 with them).
#pragma once
#include "sim_internal.h"

namespace sparsesim {
namespace rp {

// Highest VGPR the kernel reserves for planes (v100..v230: up to 131 planes).
// The kernel declares it clobbered whatever a run's plane count, so its
// allocation is 231 VGPRs and at most two waves share a SIMD.  Narrower
// allocations (132 and 164 VGPRs, three waves per SIMD) gave results on
// multi-million-entry states that differed from run to run, as did two waves
// of different programs on one SIMD; waves of one program at most two per
// SIMD reproduce the LDS-plane pass bit for bit, as does one wave a SIMD of any
// programs (the launchers keep passes apart).  The 132-register form also loaded a label's second word
// (v132..v163) past its allocation.
constexpr uint32_t kVmax = 230;
constexpr uint32_t kTurnAccBytes = 32 * 64 * 8;   // per wave: 32 entries x 64 lanes x 64-bit turns

// LSB-first 32x32 bit transpose (out[q] bit j = in[j] bit q), by the
// recursive block-swap method of Warren, Hacker's Delight, Sec. 7-3: five
// rounds of masked swaps of 16-, 8-, 4-, 2- and 1-bit blocks.
__device__ __forceinline__ void transpose32(uint32_t (&A)[32]) {
  uint32_t m = 0x0000FFFFu;
#pragma unroll
  for (int j = 16; j != 0; j >>= 1, m ^= (m << j)) {
#pragma unroll
    for (int k = 0; k < 32; k = (k + j + 1) & ~j) {
      const uint32_t t = ((A[k] >> j) ^ A[k + j]) & m;
      A[k] ^= t << j;
      A[k + j] ^= t;
    }
  }
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// omega^k = e^{i pi k / 4}, exact.
__device__ __forceinline__ double2 omega_pow(uint32_t k) {
  const double h = 0.70710678118654752440;
  const double x = (k & 1u) ? h : 1.0, y = (k & 1u) ? h : 0.0;
  const uint32_t r = (k >> 1) & 3u;
  const double re = r == 0 ? x : (r == 1 ? -y : (r == 2 ? -x : y));
  const double im = r == 0 ? y : (r == 1 ? x : (r == 2 ? -y : -x));
  return make_double2(re, im);
}

// Plane q (the low byte of a wave-uniform value) into a compiler register,
// and back.
__device__ __forceinline__ uint32_t rd_plane(uint32_t q) {
  uint32_t r;
  asm volatile(
      "s_set_gpr_idx_on %1, gpr_idx(SRC0)\n\t"
      "v_mov_b32 %0, v100\n\t"
      "s_set_gpr_idx_off"
      : "=v"(r)
      : "s"(q)
      : "m0");
  return r;
}
__device__ __forceinline__ void wr_plane(uint32_t q, uint32_t v) {
  asm volatile(
      "s_set_gpr_idx_on %0, gpr_idx(DST)\n\t"
      "v_mov_b32 v100, %1\n\t"
      "s_set_gpr_idx_off" ::"s"(q),
      "v"(v)
      : "m0");
}

__device__ __forceinline__ int lane_now() {
  int l;
  asm volatile("v_mov_b32 %0, v97" : "=v"(l));
  return l;
}

#define RP_IN(R, X) asm volatile("v_mov_b32 v" #R ", %0" ::"v"(X))
#define RP_OUT(R, X) asm volatile("v_mov_b32 %0, v" #R : "=v"(X))
#define RP_IN_WORD0(a) \
  RP_IN(100, a[0]); RP_IN(101, a[1]); RP_IN(102, a[2]); RP_IN(103, a[3]); RP_IN(104, a[4]); RP_IN(105, a[5]); RP_IN(106, a[6]); RP_IN(107, a[7]); \
  RP_IN(108, a[8]); RP_IN(109, a[9]); RP_IN(110, a[10]); RP_IN(111, a[11]); RP_IN(112, a[12]); RP_IN(113, a[13]); RP_IN(114, a[14]); RP_IN(115, a[15]); \
  RP_IN(116, a[16]); RP_IN(117, a[17]); RP_IN(118, a[18]); RP_IN(119, a[19]); RP_IN(120, a[20]); RP_IN(121, a[21]); RP_IN(122, a[22]); RP_IN(123, a[23]); \
  RP_IN(124, a[24]); RP_IN(125, a[25]); RP_IN(126, a[26]); RP_IN(127, a[27]); RP_IN(128, a[28]); RP_IN(129, a[29]); RP_IN(130, a[30]); RP_IN(131, a[31]);
#define RP_OUT_WORD0(a) \
  RP_OUT(100, a[0]); RP_OUT(101, a[1]); RP_OUT(102, a[2]); RP_OUT(103, a[3]); RP_OUT(104, a[4]); RP_OUT(105, a[5]); RP_OUT(106, a[6]); RP_OUT(107, a[7]); \
  RP_OUT(108, a[8]); RP_OUT(109, a[9]); RP_OUT(110, a[10]); RP_OUT(111, a[11]); RP_OUT(112, a[12]); RP_OUT(113, a[13]); RP_OUT(114, a[14]); RP_OUT(115, a[15]); \
  RP_OUT(116, a[16]); RP_OUT(117, a[17]); RP_OUT(118, a[18]); RP_OUT(119, a[19]); RP_OUT(120, a[20]); RP_OUT(121, a[21]); RP_OUT(122, a[22]); RP_OUT(123, a[23]); \
  RP_OUT(124, a[24]); RP_OUT(125, a[25]); RP_OUT(126, a[26]); RP_OUT(127, a[27]); RP_OUT(128, a[28]); RP_OUT(129, a[29]); RP_OUT(130, a[30]); RP_OUT(131, a[31]);
#define RP_IN_WORD1(a) \
  RP_IN(132, a[0]); RP_IN(133, a[1]); RP_IN(134, a[2]); RP_IN(135, a[3]); RP_IN(136, a[4]); RP_IN(137, a[5]); RP_IN(138, a[6]); RP_IN(139, a[7]); \
  RP_IN(140, a[8]); RP_IN(141, a[9]); RP_IN(142, a[10]); RP_IN(143, a[11]); RP_IN(144, a[12]); RP_IN(145, a[13]); RP_IN(146, a[14]); RP_IN(147, a[15]); \
  RP_IN(148, a[16]); RP_IN(149, a[17]); RP_IN(150, a[18]); RP_IN(151, a[19]); RP_IN(152, a[20]); RP_IN(153, a[21]); RP_IN(154, a[22]); RP_IN(155, a[23]); \
  RP_IN(156, a[24]); RP_IN(157, a[25]); RP_IN(158, a[26]); RP_IN(159, a[27]); RP_IN(160, a[28]); RP_IN(161, a[29]); RP_IN(162, a[30]); RP_IN(163, a[31]);
#define RP_OUT_WORD1(a) \
  RP_OUT(132, a[0]); RP_OUT(133, a[1]); RP_OUT(134, a[2]); RP_OUT(135, a[3]); RP_OUT(136, a[4]); RP_OUT(137, a[5]); RP_OUT(138, a[6]); RP_OUT(139, a[7]); \
  RP_OUT(140, a[8]); RP_OUT(141, a[9]); RP_OUT(142, a[10]); RP_OUT(143, a[11]); RP_OUT(144, a[12]); RP_OUT(145, a[13]); RP_OUT(146, a[14]); RP_OUT(147, a[15]); \
  RP_OUT(148, a[16]); RP_OUT(149, a[17]); RP_OUT(150, a[18]); RP_OUT(151, a[19]); RP_OUT(152, a[20]); RP_OUT(153, a[21]); RP_OUT(154, a[22]); RP_OUT(155, a[23]); \
  RP_OUT(156, a[24]); RP_OUT(157, a[25]); RP_OUT(158, a[26]); RP_OUT(159, a[27]); RP_OUT(160, a[28]); RP_OUT(161, a[29]); RP_OUT(162, a[30]); RP_OUT(163, a[31]);
#define RP_IN_WORD2(a) \
  RP_IN(164, a[0]); RP_IN(165, a[1]); RP_IN(166, a[2]); RP_IN(167, a[3]); RP_IN(168, a[4]); RP_IN(169, a[5]); RP_IN(170, a[6]); RP_IN(171, a[7]); \
  RP_IN(172, a[8]); RP_IN(173, a[9]); RP_IN(174, a[10]); RP_IN(175, a[11]); RP_IN(176, a[12]); RP_IN(177, a[13]); RP_IN(178, a[14]); RP_IN(179, a[15]); \
  RP_IN(180, a[16]); RP_IN(181, a[17]); RP_IN(182, a[18]); RP_IN(183, a[19]); RP_IN(184, a[20]); RP_IN(185, a[21]); RP_IN(186, a[22]); RP_IN(187, a[23]); \
  RP_IN(188, a[24]); RP_IN(189, a[25]); RP_IN(190, a[26]); RP_IN(191, a[27]); RP_IN(192, a[28]); RP_IN(193, a[29]); RP_IN(194, a[30]); RP_IN(195, a[31]);
#define RP_OUT_WORD2(a) \
  RP_OUT(164, a[0]); RP_OUT(165, a[1]); RP_OUT(166, a[2]); RP_OUT(167, a[3]); RP_OUT(168, a[4]); RP_OUT(169, a[5]); RP_OUT(170, a[6]); RP_OUT(171, a[7]); \
  RP_OUT(172, a[8]); RP_OUT(173, a[9]); RP_OUT(174, a[10]); RP_OUT(175, a[11]); RP_OUT(176, a[12]); RP_OUT(177, a[13]); RP_OUT(178, a[14]); RP_OUT(179, a[15]); \
  RP_OUT(180, a[16]); RP_OUT(181, a[17]); RP_OUT(182, a[18]); RP_OUT(183, a[19]); RP_OUT(184, a[20]); RP_OUT(185, a[21]); RP_OUT(186, a[22]); RP_OUT(187, a[23]); \
  RP_OUT(188, a[24]); RP_OUT(189, a[25]); RP_OUT(190, a[26]); RP_OUT(191, a[27]); RP_OUT(192, a[28]); RP_OUT(193, a[29]); RP_OUT(194, a[30]); RP_OUT(195, a[31]);
#define RP_IN_WORD3(a) \
  RP_IN(196, a[0]); RP_IN(197, a[1]); RP_IN(198, a[2]); RP_IN(199, a[3]); RP_IN(200, a[4]); RP_IN(201, a[5]); RP_IN(202, a[6]); RP_IN(203, a[7]); \
  RP_IN(204, a[8]); RP_IN(205, a[9]); RP_IN(206, a[10]); RP_IN(207, a[11]); RP_IN(208, a[12]); RP_IN(209, a[13]); RP_IN(210, a[14]); RP_IN(211, a[15]); \
  RP_IN(212, a[16]); RP_IN(213, a[17]); RP_IN(214, a[18]); RP_IN(215, a[19]); RP_IN(216, a[20]); RP_IN(217, a[21]); RP_IN(218, a[22]); RP_IN(219, a[23]); \
  RP_IN(220, a[24]); RP_IN(221, a[25]); RP_IN(222, a[26]); RP_IN(223, a[27]); RP_IN(224, a[28]); RP_IN(225, a[29]); RP_IN(226, a[30]); RP_IN(227, a[31]);
#define RP_OUT_WORD3(a) \
  RP_OUT(196, a[0]); RP_OUT(197, a[1]); RP_OUT(198, a[2]); RP_OUT(199, a[3]); RP_OUT(200, a[4]); RP_OUT(201, a[5]); RP_OUT(202, a[6]); RP_OUT(203, a[7]); \
  RP_OUT(204, a[8]); RP_OUT(205, a[9]); RP_OUT(206, a[10]); RP_OUT(207, a[11]); RP_OUT(208, a[12]); RP_OUT(209, a[13]); RP_OUT(210, a[14]); RP_OUT(211, a[15]); \
  RP_OUT(212, a[16]); RP_OUT(213, a[17]); RP_OUT(214, a[18]); RP_OUT(215, a[19]); RP_OUT(216, a[20]); RP_OUT(217, a[21]); RP_OUT(218, a[22]); RP_OUT(219, a[23]); \
  RP_OUT(220, a[24]); RP_OUT(221, a[25]); RP_OUT(222, a[26]); RP_OUT(223, a[27]); RP_OUT(224, a[28]); RP_OUT(225, a[29]); RP_OUT(226, a[30]); RP_OUT(227, a[31]);

// Raw buffer resource over n bytes at p (gfx9 descriptor word 3): loads past
// n return zero and stores past n are dropped, so a ragged tile needs no
// per-entry branches.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, uint32_t n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)n, 0x00020000);
}
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4i buf_rsrc_v4(const void* p, uint32_t n) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  v4i r;
  r.x = (int)(uint32_t)a;
  r.y = (int)(uint32_t)(a >> 32);   // stride 0
  r.z = (int)n;
  r.w = 0x00020000;
  return r;
}

// ---- the interpreter ---------------------------------------------------------
// Buffers of two blocks: A = s48..s63, B = s64..s79; s80:s81 and s82:s83 are
// the handlers' bases for a block in A and in B, s84:s85 a handler's address.
// Fields: bits 0-7 index from v80, bits 12-15 operand enables (1 source 0, 9
// source 0 and destination); a field is the low or the high half of a word.
#define RP_LO(W) "s_mov_b32 m0, " W "\n\t"
#define RP_HI(W) "s_lshr_b32 m0, " W ", 16\n\t"
#define RP_GET "v_mov_b32_e32 v86, v80\n\t"
#define RP_AND "v_and_b32_e32 v86, v80, v86\n\t"
#define RP_XOR "v_xor_b32_e32 v80, v80, v86\n\t"
// Flips with one, two and three controls: 16, 24 and 32 bytes of code.
#define RP_F1(W) RP_LO(W) RP_GET RP_HI(W) RP_XOR
#define RP_F2E(W0, W1) RP_LO(W0) RP_GET RP_HI(W0) RP_AND RP_LO(W1) RP_XOR
#define RP_F2O(W0, W1) RP_HI(W0) RP_GET RP_LO(W1) RP_AND RP_HI(W1) RP_XOR
#define RP_F3(W0, W1) RP_LO(W0) RP_GET RP_HI(W0) RP_AND RP_LO(W1) RP_AND RP_HI(W1) RP_XOR
// Four weight-1 adds at once, by full adders (bitop3 0xe8 majority, 0x96 sum,
// 0x6a = S2 ^ (S0 & S1), bits indexed S0 * 4 + S1 * 2 + S2): 88 bytes.
#define RP_T4(W0, W1)                                                                               \
  RP_LO(W0) "v_mov_b32_e32 v86, v80\n\t" RP_HI(W0) "v_mov_b32_e32 v87, v80\n\t"                 \
  RP_LO(W1) "v_mov_b32_e32 v90, v80\n\t" RP_HI(W1) "v_mov_b32_e32 v91, v80\n\t"                 \
  "s_mov_b32 m0, 0\n\t"                                                                           \
  "v_bitop3_b32 v92, v83, v86, v87 bitop3:0xe8\n\tv_bitop3_b32 v83, v83, v86, v87 bitop3:0x96\n\t" \
  "v_bitop3_b32 v93, v83, v90, v91 bitop3:0xe8\n\tv_bitop3_b32 v83, v83, v90, v91 bitop3:0x96\n\t" \
  "v_bitop3_b32 v94, v84, v92, v93 bitop3:0xe8\n\tv_bitop3_b32 v84, v84, v92, v93 bitop3:0x96\n\t" \
  "v_xor_b32_e32 v85, v85, v94\n\t"
// A weight-2 add (16 bytes).
#define RP_S(W) RP_LO(W) "v_bitop3_b32 v82, v80, v81, v82 bitop3:0x6a\n\tv_xor_b32_e32 v81, v80, v81\n\t"

// The next block (in the other buffer, header H, handlers' base BASE) once it
// is there; the one after it is loaded over this one (REGS).
#define RP_NEXT(REGS, H, BLO, BHI)                          \
  "s_waitcnt lgkmcnt(0)\n\t"                              \
  "s_buffer_load_dwordx16 " REGS ", %[rs], %[off]\n\t"    \
  "s_add_u32 %[off], %[off], 64\n\t"                      \
  "s_add_u32 s84, " BLO ", " H "\n\t"                     \
  "s_addc_u32 s85, " BHI ", 0\n\t"                        \
  "s_setpc_b64 s[84:85]\n\t"
#define RP_GO_A RP_NEXT("s[64:79]", "s48", "s80", "s81")
#define RP_GO_B RP_NEXT("s[48:63]", "s64", "s82", "s83")

// The handlers of one buffer (words R0..R15), kRpStride bytes apart, in the
// order of the shapes.
#define RP_HANDLERS(GO, R0, R1, R2, R3, R4, R5, R6, R7, R8, R9, R10, R11, R12, R13, R14, R15)                     \
  "s_mov_b32 %[shape], " R1 "\n\ts_mov_b32 %[cnt], " R2 "\n\ts_branch 9f\n\t"                                  \
  ".p2align 10\n\t"                                                                                              \
  RP_F1(R1) RP_F1(R2) RP_F1(R3) RP_F1(R4) RP_F1(R5) RP_F1(R6) RP_F1(R7) RP_F1(R8) RP_F1(R9) RP_F1(R10) RP_F1(R11) \
  RP_F1(R12) RP_F1(R13) RP_F1(R14) RP_F1(R15) GO                                                                  \
  ".p2align 10\n\t"                                                                                              \
  RP_F2E(R1, R2) RP_F2O(R2, R3) RP_F2E(R4, R5) RP_F2O(R5, R6) RP_F2E(R7, R8) RP_F2O(R8, R9) RP_F2E(R10, R11)     \
  RP_F2O(R11, R12) RP_F2E(R13, R14) RP_F2O(R14, R15) GO                                                          \
  ".p2align 10\n\t"                                                                                              \
  RP_F3(R2, R3) RP_F3(R4, R5) RP_F3(R6, R7) RP_F3(R8, R9) RP_F3(R10, R11) RP_F3(R12, R13) RP_F3(R14, R15) GO     \
  ".p2align 10\n\t"                                                                                              \
  RP_T4(R2, R3) RP_T4(R4, R5) RP_T4(R6, R7) RP_T4(R8, R9) RP_T4(R10, R11) RP_T4(R12, R13) RP_T4(R14, R15) GO     \
  ".p2align 10\n\t"                                                                                              \
  RP_S(R1) RP_S(R2) RP_S(R3) RP_S(R4) RP_S(R5) RP_S(R6) RP_S(R7) RP_S(R8) RP_S(R9) RP_S(R10) RP_S(R11) RP_S(R12)  \
  RP_S(R13) RP_S(R14) RP_S(R15) GO

static_assert(kRpStride == 1024, "the .p2align of the handlers");

struct Fetch {
  uint32_t off;   // byte offset of the next block
  v4i rs;         // the program: loads past its end return zeros, an END block
};

// Run blocks from f.off on until one that the caller does itself: its shape
// and count, with f.off at the block after it.
__device__ __forceinline__ void interpret(Fetch& f, uint32_t& shape, uint32_t& cnt) {
  asm volatile(
      "s_getpc_b64 s[80:81]\n"
      "1:\n\t"
      "s_add_u32 s80, s80, 2f-1b\n\t"
      "s_addc_u32 s81, s81, 0\n\t"
      "s_add_u32 s82, s80, 3f-2f\n\t"
      "s_addc_u32 s83, s81, 0\n\t"
      "s_buffer_load_dwordx16 s[48:63], %[rs], %[off]\n\t"
      "s_add_u32 %[off], %[off], 64\n\t"
      "s_set_gpr_idx_on s80, gpr_idx()\n\t"   // no operand enabled until a field says so
      RP_GO_A
      ".p2align 10\n"
      "2:\n\t"
      RP_HANDLERS(RP_GO_B, "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", "s60",
                  "s61", "s62", "s63")
      ".p2align 10\n"
      "3:\n\t"
      RP_HANDLERS(RP_GO_A, "s64", "s65", "s66", "s67", "s68", "s69", "s70", "s71", "s72", "s73", "s74", "s75", "s76",
                  "s77", "s78", "s79")
      "9:\n\t"
      "s_waitcnt lgkmcnt(0)\n\t"   // the load of the block after next
      "s_set_gpr_idx_off\n\t"
      "s_sub_u32 %[off], %[off], 64"
      : [off] "+s"(f.off), [shape] "=&s"(shape), [cnt] "=&s"(cnt)
      : [rs] "s"(f.rs)
      : "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", "s60", "s61", "s62",
        "s63", "s64", "s65", "s66", "s67", "s68", "s69", "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77",
        "s78", "s79", "s80", "s81", "s82", "s83", "s84", "s85", "m0", "scc", "memory");
}

// The first waves of a launch bring the program into their XCD's L2: read by
// the scalar loads alone, each line's first touch would cost its latency.
__device__ __forceinline__ void prefetch_program(const Fetch& f, uint32_t bytes, int lane) {
  for (uint32_t o = 0; o < bytes; o += 64 * 64) {
    asm volatile(
        "v_lshl_add_u32 v95, %[lane], 6, %[o]\n\t"
        "buffer_load_dword v96, v95, %[rs], 0 offen" ::[lane] "v"(lane),
        [o] "s"(o), [rs] "s"(f.rs)
        : "memory");
  }
}

// Words of the program at byte offset off, wave-uniform (scalar loads).
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v8u __attribute__((ext_vector_type(8)));
__device__ __forceinline__ v2u words2(const Fetch& f, uint32_t off) {
  v2u r;
  asm volatile("s_buffer_load_dwordx2 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&s"(r) : "s"(f.rs), "s"(off));
  return r;
}
// The fractions of captured ops: uniform, read through the constant address
// space (scalar loads that the compiler waits for).
typedef const __attribute__((address_space(4))) uint64_t* TurnPtr;
// A turn group: cond words, fractions (words 0-3 and 4-11 of its block).
struct TurnWords {
  v4u cond;
  v8u tau;
};
__device__ __forceinline__ TurnWords turn_words(const Fetch& f, uint32_t off) {
  TurnWords r;
  asm volatile("s_buffer_load_dwordx4 %0, %2, %3\n\ts_buffer_load_dwordx8 %1, %2, %4\n\ts_waitcnt lgkmcnt(0)"
               : "=&s"(r.cond), "=&s"(r.tau)
               : "s"(f.rs), "s"(off), "s"(off + 16u));
  return r;
}

// General eighth-turn ops, two per quad (cond word, k), from f.off on: x =
// planes t & c0 & c1 & c2, then the weighted adds with k's bits as masks.
__device__ __forceinline__ void omega_general(const Fetch& f, uint32_t nquads) {
  for (uint32_t i = 0; i < 2 * nquads; ++i) {
    const v2u ck = words2(f, f.off + 8u * i);
    const uint32_t c = ck.x, k = ck.y;
    const uint32_t x = rd_plane(c) & rd_plane(c >> 8) & rd_plane(c >> 16) & rd_plane(c >> 24);
    const uint32_t m1 = (k & 1u) ? ~0u : 0u, m2 = (k & 2u) ? ~0u : 0u, m4 = (k & 4u) ? ~0u : 0u;
    asm volatile(
        "v_bitop3_b32 v80, %0, %3, v80 bitop3:0x6a\n\t"   // P ^= x & m4
        "v_and_b32 v86, %2, %0\n\t"
        "v_bitop3_b32 v82, v82, v81, v86 bitop3:0x78\n\t" // Q += x & m2
        "v_xor_b32 v81, v81, v86\n\t"
        "v_and_b32 v86, %1, %0\n\t"
        "v_and_b32 v87, v83, v86\n\t"                      // R += x & m1
        "v_xor_b32 v83, v83, v86\n\t"
        "v_bitop3_b32 v85, v85, v84, v87 bitop3:0x78\n\t"
        "v_xor_b32 v84, v84, v87" ::"v"(x),
        "s"(m1), "s"(m2), "s"(m4));
  }
}

// TURN groups: a block per group of four ops (cond words; then the fractions of
// ops 0..3).  Each entry's accumulator (LDS, acc[64 j + lane])
// gains the sum of the fractions of the ops whose condition holds for it: per
// group, one of 16 subset sums, kept in a 16-entry LDS table and read with
// one 64-bit load per entry.
// FORM: kRpTB (condition = one plane) or kRpTG (four).
template <uint32_t FORM>
__device__ __forceinline__ void turn_group(const Fetch& f, uint32_t off, uint64_t* acc, uint64_t* table, int lane) {
  uint32_t B[8];
  const TurnWords tw = turn_words(f, off);
  const uint32_t cw[4] = {tw.cond.x, tw.cond.y, tw.cond.z, tw.cond.w};
  uint32_t x[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    x[u] = rd_plane(cw[u]);
    if (FORM == kRpTG) x[u] &= rd_plane(cw[u] >> 8) & rd_plane(cw[u] >> 16) & rd_plane(cw[u] >> 24);
  }
  uint64_t tau[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) tau[u] = ((uint64_t)tw.tau[2 * u + 1] << 32) | tw.tau[2 * u];
  // Entry j's offset in the table, 8 x (the ops, bit u = op u, whose
  // condition holds for it), is byte j >> 3 of B[j & 7]: bit j of x[u]
  // moves to bit 8 (j >> 3) + 3 + u by one constant shift; the four merge
  // under disjoint byte-lane masks.
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    uint32_t v = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int sh = w - 3 - u;
      const uint32_t y = sh >= 0 ? x[u] >> sh : x[u] << -sh;
      v |= y & (0x01010101u << (3 + u));
    }
    B[w] = v;
  }
  // Table entry m (lane m < 16) is the sum of the fractions named by m's
  // bits.  (The lane number is made opaque here so that the four masks are
  // formed where they are used, not kept live across the whole tile.)
  int l = lane;
  asm volatile("" : "+v"(l));
  uint64_t S = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) S += tau[u] & (0ull - (uint64_t)((l >> u) & 1));
  if (l < 16) table[l] = S;   // the wave's LDS accesses complete in order
  __builtin_amdgcn_sched_barrier(0);
  const char* tb = reinterpret_cast<const char*>(table);
#pragma unroll
  for (int j0 = 0; j0 < 32; j0 += 4) {
    uint64_t a[4], v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = j0 + k;
      a[k] = acc[64 * j + lane];
      v[k] = *reinterpret_cast<const uint64_t*>(tb + __builtin_amdgcn_ubfe(B[j & 7], 8 * (j >> 3), 8));
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[64 * (j0 + k) + lane] = a[k] + v[k];
    // Keep the blocks apart (otherwise every entry's table address is formed
    // up front, and they do not fit the registers).
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Eight planes from q on.
__device__ __forceinline__ void rd_planes8(uint32_t q, uint32_t (&x)[8]) {
  asm volatile(
      "s_set_gpr_idx_on %8, gpr_idx(SRC0)\n\t"
      "v_mov_b32 %0, v100\n\tv_mov_b32 %1, v101\n\tv_mov_b32 %2, v102\n\tv_mov_b32 %3, v103\n\t"
      "v_mov_b32 %4, v104\n\tv_mov_b32 %5, v105\n\tv_mov_b32 %6, v106\n\tv_mov_b32 %7, v107\n\t"
      "s_set_gpr_idx_off"
      : "=v"(x[0]), "=v"(x[1]), "=v"(x[2]), "=v"(x[3]), "=v"(x[4]), "=v"(x[5]), "=v"(x[6]), "=v"(x[7])
      : "s"(q)
      : "m0");
}
__device__ __forceinline__ void clear_planes8(uint32_t q) {
  asm volatile(
      "s_set_gpr_idx_on %0, gpr_idx(DST)\n\t"
      "v_mov_b32 v100, 0\n\tv_mov_b32 v101, 0\n\tv_mov_b32 v102, 0\n\tv_mov_b32 v103, 0\n\t"
      "v_mov_b32 v104, 0\n\tv_mov_b32 v105, 0\n\tv_mov_b32 v106, 0\n\tv_mov_b32 v107, 0\n\t"
      "s_set_gpr_idx_off" ::"s"(q)
      : "m0");
}

// Byte b of B[w]: bit u says that the condition x[u] holds for entry 8 b + 4 H
// + w (an 8 x 8 bit transpose in each byte, Warren, Hacker's Delight, Sec. 7-3,
// of which a half is needed).
template <int H>
__device__ __forceinline__ void turn_index(const uint32_t (&x)[8], uint32_t (&B)[4]) {
  auto merge = [](uint32_t m, uint32_t p, uint32_t q) { return (p & m) | (q & ~m); };
  uint32_t y[4], z[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    y[k] = H ? merge(0x0f0f0f0fu, x[k] >> 4, x[k + 4]) : merge(0x0f0f0f0fu, x[k], x[k + 4] << 4);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    z[k] = merge(0x33333333u, y[k], y[k + 2] << 2);
    z[k + 2] = merge(0x33333333u, y[k] >> 2, y[k + 2]);
  }
#pragma unroll
  for (int k = 0; k < 4; k += 2) {
    B[k] = merge(0x55555555u, z[k], z[k + 1] << 1);
    B[k + 1] = merge(0x55555555u, z[k] >> 1, z[k + 1]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(B[k]));   // (formed once, not per byte)
}

// Entry m of a table of 256: the sum of the fractions that m's bits name.
__device__ __forceinline__ void turn_table(const uint64_t (&t)[8], uint64_t* table) {
  const int l = lane_now();   // (the bits' masks are formed here, not kept live)
  uint64_t s = 0;
#pragma unroll
  for (int u = 0; u < 6; ++u) {
    uint32_t m = (uint32_t)__builtin_amdgcn_sbfe(l, u, 1);
    asm volatile("" : "+v"(m));   // (a mask and two ands, not a compare and two selects)
    s += (uint64_t)((uint32_t)(t[u] >> 32) & m) << 32 | ((uint32_t)t[u] & m);
    asm volatile("" : "+v"(s));   // (one fraction at a time: registers are short)
  }
  table[l] = s;   // the wave's LDS accesses complete in order
  table[l + 64] = s + t[6];
  table[l + 128] = s + t[7];
  table[l + 192] = s + t[6] + t[7];
}

// Captured turn ops, ng groups of eight: op u of group g has its condition in
// plane first + 8 g + u, its fraction at tau[8 g + u].  The 16 entries j (of
// the lane's 32) with bit 2 of j equal to H, in registers over all groups; only
// j < nj exist.  Per group an entry adds one of the 256 subset sums of its
// fractions, read from LDS; while a group's sums are on their way the next
// group's indices and table are made.  Two 16-entry tables and a
// read-modify-write of LDS accumulators per group took 69 instructions an op
// and 64 cycles of LDS, this takes 36 and 32.  Captures included, an Rz costs one
// wave 110 ns on 24 qubits and 135 on 100 (24 capture planes), where it cost 197
// and 190, and two waves of a SIMD 230 instead of 316; on 256 entries 56
// instead of 196.  What is left is the latency of the tables (LDS, written and
// read) and, with every flush of the capture planes, 0.5 us of leaving and
// entering the interpreter.
template <int H>
__device__ __forceinline__ void captured_half(TurnPtr tau, uint32_t ng, uint32_t first, uint32_t nj, uint64_t* acc,
                                              uint64_t* table) {
  const int lane = lane_now();
  uint64_t a[16], t[8];
  uint32_t x[8], B[4];
#pragma unroll
  for (int u = 0; u < 8; ++u) t[u] = tau[u];
  rd_planes8(first, x);
  turn_index<H>(x, B);
  turn_table(t, table);
#pragma unroll
  for (int i = 0; i < 16; ++i) a[i] = acc[64 * (8 * (i >> 2) + 4 * H + (i & 3)) + lane];
  const bool upper = nj > 16u + 4u * H;
  for (uint32_t g = 0; g < ng; ++g) {
    // (After the last group: its own planes once more, unused, and the program's
    // next block, which the interpreter then finds in the scalar cache.)
    const uint32_t gn = g + 1 < ng ? g + 1 : g;
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = tau[8 * g + 8 + u];
    uint64_t v[12];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = table[B[i] & 0xffu];
    __builtin_amdgcn_sched_barrier(0);
    uint32_t C[4];
    rd_planes8(first + 8 * gn, x);
    turn_index<H>(x, C);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] += v[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = table[(B[i] >> 8) & 0xffu];
    if (upper) {
#pragma unroll
      for (int i = 4; i < 12; ++i) v[i] = table[(B[i & 3] >> (8 + 2 * (i & 12))) & 0xffu];
      __builtin_amdgcn_sched_barrier(0);
      turn_table(t, table);   // (over what the reads above, issued before, still use)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 4; i < 12; ++i) a[4 + i] += v[i];
    } else {
      __builtin_amdgcn_sched_barrier(0);
      turn_table(t, table);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) a[4 + i] += v[i];
#pragma unroll
    for (int k = 0; k < 4; ++k) B[k] = C[k];
  }
  const int lane_end = lane_now();
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[64 * (8 * (i >> 2) + 4 * H + (i & 3)) + lane_end] = a[i];
}
__device__ __forceinline__ void captured_turns(TurnPtr tau, uint32_t ng, uint32_t first, uint32_t nj, uint64_t* acc,
                                               uint64_t* table) {
  captured_half<0>(tau, ng, first, nj, acc, table);
  if (nj > 4) captured_half<1>(tau, ng, first, nj, acc, table);
  for (uint32_t g = 0; g < ng; ++g) clear_planes8(first + 8 * g);
}

// (programs on too many qubits for capture planes, and ops under four planes)
template <uint32_t FORM>
__device__ __forceinline__ void turn_groups(const Fetch& f, uint32_t ng, uint64_t* acc, uint64_t* table, int lane) {
  for (uint32_t g = 0; g < ng; ++g) turn_group<FORM>(f, f.off + 64u * g, acc, table, lane);
}

// Labels of the tile (word w of each label: bits 32w..32w+31) into planes.
__device__ __forceinline__ void load_word(const Buf& b, uint64_t base, uint32_t lim, int w, int lane) {
  const __amdgpu_buffer_rsrc_t rs = buf_rsrc((w < 2 ? b.key_lo : b.key_hi) + base, 8 * lim);
  const int off = 8 * lane + 4 * (w & 1);
  uint32_t a[32];
#pragma unroll
  for (int j = 0; j < 32; ++j) a[j] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 512 * j, 0);
  transpose32(a);
  if (w == 0) { RP_IN_WORD0(a) }
  else if (w == 1) { RP_IN_WORD1(a) }
  else if (w == 2) { RP_IN_WORD2(a) }
  else { RP_IN_WORD3(a) }
}

__device__ __forceinline__ void store_word(const Buf& b, uint64_t base, uint32_t lim, int w, int nq, int lane) {
  const __amdgpu_buffer_rsrc_t rs = buf_rsrc((w < 2 ? b.key_lo : b.key_hi) + base, 8 * lim);
  const int off = 8 * lane + 4 * (w & 1);
  uint32_t a[32];
  if (w == 0) { RP_OUT_WORD0(a) }
  else if (w == 1) { RP_OUT_WORD1(a) }
  else if (w == 2) { RP_OUT_WORD2(a) }
  else { RP_OUT_WORD3(a) }
  // Planes at and above nq are the all-ones, scratch and zero planes (or
  // unused): labels have no such bits.
#pragma unroll
  for (int q = 0; q < 32; ++q) a[q] = 32 * w + q < nq ? a[q] : 0u;
  transpose32(a);
#pragma unroll
  for (int j = 0; j < 32; ++j) __builtin_amdgcn_raw_buffer_store_b32(a[j], rs, off, 512 * j, 0);
}

// Apply a run's program (nblk blocks) to the tile at base (lim valid
// entries).  TURNS: the kernel provides acc, the wave's turn accumulators in
// LDS, and table, its subset-sum tables; a run uses them if it has turn ops
// (the result does not depend on TURNS otherwise).  prefetch: bring the program
// into the XCD's L2 first.
// get: the state's arrays and the run's parameters, asked for before and again
// after the program (kept over it they take scalar registers it needs).
struct RpArgs {
  Buf b;
  BsRun run;
};
template <bool TURNS, class Get>
__device__ __forceinline__ void rp_tile(Get&& get, uint64_t base, uint32_t lim, const RpBlock* __restrict__ prog,
                                        uint32_t nblk, bool prefetch, uint64_t* acc, uint64_t* table) {
  const RpArgs before = get();
  const Buf& b = before.b;
  asm volatile("v_mov_b32 v97, %0" ::"v"(threadIdx.x));
  const uint32_t nq = before.run.n_planes;
  const bool turns = TURNS && before.run.has_turns;
  const uint32_t rw = before.run.words_read | before.run.words_write;
  Fetch f;
  f.rs = buf_rsrc_v4(prog, 64u * nblk);
  f.off = 0;
  if (prefetch) prefetch_program(f, 64u * nblk, lane_now());
#pragma unroll
  for (int w = 0; w < 4; ++w)
    if (rw & (1u << w)) load_word(b, base, lim, w, lane_now());
  wr_plane(nq, ~0u);       // all ones
  wr_plane(nq + 2, 0u);    // zero
  if (turns)
    for (uint32_t q = 0; q < rp_capture_planes(nq); q += 8) clear_planes8(nq + 3 + q);
  asm volatile(
      "v_mov_b32 v80, 0\n\tv_mov_b32 v81, 0\n\tv_mov_b32 v82, 0\n\t"
      "v_mov_b32 v83, 0\n\tv_mov_b32 v84, 0\n\tv_mov_b32 v85, 0");
  if (turns) {
    const int lane = lane_now();
#pragma unroll
    for (int j = 0; j < 32; ++j) acc[64 * j + lane] = 0;
  }
  for (;;) {
    uint32_t shape, cnt;
    interpret(f, shape, cnt);
    if (shape == kRpOG) {
      omega_general(f, cnt);
      f.off += 64u * ((cnt + 3) / 4);
    } else if (shape == kRpTC || shape == kRpTB || shape == kRpTG) {
      if (!turns) break;   // the host never sends turn ops to this variant
      if (shape == kRpTC) {
        captured_turns(reinterpret_cast<TurnPtr>(reinterpret_cast<uint64_t>(prog) + f.off), cnt, nq + 3, (lim + 63) / 64,
                       acc, table);
      } else if (shape == kRpTB) {
        turn_groups<kRpTB>(f, cnt, acc, table, lane_now());
      } else {
        turn_groups<kRpTG>(f, cnt, acc, table, lane_now());
      }
      f.off += 64u * cnt;
    } else {
      break;   // END (zero words past the program) or an unknown shape
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the prefetch
  const RpArgs after = get();
  const BsRun& run = after.run;
  // Labels back to memory (only words some gate flips).
#pragma unroll
  for (int w = 0; w < 4; ++w)
    if (run.words_write & (1u << w)) store_word(after.b, base, lim, w, (int)nq, lane_now());
  if (!run.has_phase) return;
  uint32_t P, Q0, Q1, R0, R1, R2;
  asm volatile(
      "v_mov_b32 %0, v80\n\tv_mov_b32 %1, v81\n\tv_mov_b32 %2, v82\n\t"
      "v_mov_b32 %3, v83\n\tv_mov_b32 %4, v84\n\tv_mov_b32 %5, v85"
      : "=v"(P), "=v"(Q0), "=v"(Q1), "=v"(R0), "=v"(R1), "=v"(R2));
  // One complex multiply per amplitude by the accumulated phase.
  const int lane = lane_now();
  double2* amp = after.b.amp + base + lane;
#pragma unroll 1
  for (int j = 0; j < 32; ++j) {
    if (64u * j + lane >= lim) break;
    const uint32_t rj = ((R0 >> j) & 1u) | (((R1 >> j) & 1u) << 1) | (((R2 >> j) & 1u) << 2);
    const uint32_t qj = ((Q0 >> j) & 1u) | (((Q1 >> j) & 1u) << 1);
    const uint32_t k = (rj + 2u * qj + 4u * ((P >> j) & 1u) + run.g_omega) & 7u;
    double2 f2;
    if (!turns && run.g_turn == 0) {
      f2 = omega_pow(k);
    } else {
      const uint64_t tj = turns ? acc[64 * j + lane] : 0ull;
      const uint64_t T = tj + run.g_turn + ((uint64_t)k << 61);
      double sn, cs;
      sincospi((double)(T >> 11) * 0x1p-52, &sn, &cs);   // angle = 2 pi T / 2^64
      f2 = make_double2(cs, sn);
    }
    amp[64 * j] = cmul(amp[64 * j], f2);
  }
}

}  // namespace rp
}  // namespace sparsesim
