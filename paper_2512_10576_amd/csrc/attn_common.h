// What the attention kernels share: vector types, gathers from memory straight into LDS, the two LDS access patterns of
// an entry's row, and the form in which partial results travel.
#pragma once
#include "ess_internal.h"
#include <utility>

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// Partial results travel from the partial-attention kernels to the merge kernel as fp16: they are
// softmax-normalised (|value| <= the largest entry value), fp16 keeps 11 bits of them while the merged
// output is rounded to bf16's 8, and the traffic between the two kernels, which is most of what both
// cost beyond their tile loops, is halved.  The split weights (log-sum-exp) stay fp32.
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

constexpr float kLazyMax = 8.0f;
constexpr int TRP = 1024;                        // latent row pitch in LDS
constexpr int F8_PIECES = 41;                    // 16-byte pieces of a quantised entry (648 bytes and 8 of padding)
constexpr int F8_PITCH = F8_PIECES * 16;         // 656

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {      // one v_cvt_pk_bf16_f32, round to nearest even
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));
}

__device__ __forceinline__ uint32_t lds_addr_of(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// 64 lanes x 16 bytes from `gptr` (per lane) to LDS address `lds_dst` + 16 * lane (lds_dst wave-uniform)
// The statement writes m0 and says so (m0 is reserved: the compiler never keeps a value of its own there across
// statements, but the clobber makes the write visible to it; clang warns about reserved registers in clobber lists).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const void* gptr, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(gptr), "s"(lds_dst) : "memory", "m0");
}
// the same from a wave-uniform base and a byte offset per lane.  A memory instruction may read a scalar register five wait
// states after a vector ALU instruction wrote it, not earlier, and the compiler's hazard logic does not look into asm
// statements.  LANES: the base comes straight from v_readlane, and the five are in the statement.  Without, it has been through
// scalar arithmetic (or a kernel argument), which needs none; in k_attn_partial_tr, bound by what its one wave per SIMD issues, they
// cost 2 % (48 x 2 quantised ragged rows 87.9 us against 86.0).  tests/test_abi.py counts the states in all instances of both kernels.
template <bool LANES = false>
__device__ __forceinline__ void dma16_base(const void* base, uint32_t off, uint32_t lds_dst) {
  if constexpr (LANES)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds_dst) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds_dst) : "memory", "m0");
}
// the same for the first F8_PIECES lanes only (a quantised entry); all lanes are active before and after.  The execution
// mask is set inside the statement: a branch around it would cut the pinned order of the loop into pieces.
template <bool LANES = false>
__device__ __forceinline__ void dma16_entry(const void* base, uint32_t off, uint32_t lds_dst) {
  if constexpr (LANES)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 2\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1"
                 : : "v"(off), "s"(base), "s"(lds_dst), "s"((1ull << 41) - 1) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1"
                 : : "v"(off), "s"(base), "s"(lds_dst), "s"((1ull << 41) - 1) : "memory", "m0");
}
#pragma clang diagnostic pop

template <int N>
__device__ __forceinline__ void wait_vmcnt() {     // vmcnt <= N, other counters untouched
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// The 256 output accumulators of a wave (16 blocks of 32 value columns x 32 heads, 16 registers each) live in
// AGPRs a0..a255 under fixed names, outside the compiler's register allocation: every access is an asm statement
// that names them by number.  (Left to the allocator -- as MFMA builtins, or as asm operands with the "a"
// constraint -- they are copied around or spilled, because the rare rescale multiplies them with vector ALU
// instructions and the loop leaves no spare 16-register tuple.)  The kernels that do this are compiled with
// -amdgpu-mfma-vgpr-form, which keeps the results of the compiler's own MFMAs (the first product) in VGPRs, and
// the AGPR file is claimed as a whole (see AgprHold below), so that the compiler has no use for AGPRs of its own:
// tests/test_abi.py checks in the generated code that nothing but these statements names one and that nothing is
// spilled.
// The compiler's hazard logic does not look into asm statements, and an MFMA that directly follows the vector ALU
// instruction producing one of its VGPR operands was seen to read the register's previous contents: an MFMA
// marked WAIT carries wait states inside its own statement, where no scheduling can separate them from it.
// The compiler must keep its hands off the AGPRs that these statements use behind its back.  It is told that they
// are taken: eight 32-register values with the "a" constraint are defined at the start of the kernel (by an empty
// statement) and passed through empty statements (agpr_fence) at the top of every tile iteration and at the end, so
// they are live throughout and fill the AGPR file -- the allocator has no AGPR left for a temporary or a spill of
// its own, and the launch reserves all 256.  What the values "hold" is of no interest to the compiler's code.
typedef float floatx32 __attribute__((ext_vector_type(32)));
struct AgprHold { floatx32 d0, d1, d2, d3, d4, d5, d6, d7; };
// (the comments inside the statements mark the claimed stretch in the generated code, for the test that reads it)
__device__ __forceinline__ void agpr_claim(AgprHold& h) {
  asm volatile("; ess_agpr_claim" : "=a"(h.d0), "=a"(h.d1), "=a"(h.d2), "=a"(h.d3), "=a"(h.d4), "=a"(h.d5), "=a"(h.d6), "=a"(h.d7));
}
__device__ __forceinline__ void agpr_fence(AgprHold& h) {
  asm volatile("; ess_agpr_fence" : "+a"(h.d0), "+a"(h.d1), "+a"(h.d2), "+a"(h.d3), "+a"(h.d4), "+a"(h.d5), "+a"(h.d6), "+a"(h.d7));
}
__device__ __forceinline__ void agpr_release(AgprHold& h) {
  asm volatile("; ess_agpr_release" : "+a"(h.d0), "+a"(h.d1), "+a"(h.d2), "+a"(h.d3), "+a"(h.d4), "+a"(h.d5), "+a"(h.d6), "+a"(h.d7));
}
template <int VB, bool WAIT>
__device__ __forceinline__ void pv_mfma(const bf16x8& a, const bf16x8& b) {
  if constexpr (WAIT)
    asm volatile("s_nop 7\n\tv_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" : : "v"(a), "v"(b), "n"(16 * VB), "n"(16 * VB + 15));
  else
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" : : "v"(a), "v"(b), "n"(16 * VB), "n"(16 * VB + 15));
}
template <int R> __device__ __forceinline__ void acc_zero1() { asm volatile("v_accvgpr_write_b32 a[%0], 0" : : "n"(R)); }
template <int R> __device__ __forceinline__ void acc_scale1(float alpha) {
  float t;
  asm volatile("v_accvgpr_read_b32 %0, a[%2]\n\ts_nop 0\n\tv_mul_f32 %0, %0, %1\n\ts_nop 0\n\tv_accvgpr_write_b32 a[%2], %0" : "=&v"(t) : "v"(alpha), "n"(R));
}
template <int R> __device__ __forceinline__ float acc_read1() {
  float t;
  asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(t) : "n"(R));
  return t;
}
template <int... R> __device__ __forceinline__ void acc_zero_seq(std::integer_sequence<int, R...>) { (acc_zero1<R>(), ...); }
template <int... R> __device__ __forceinline__ void acc_scale_seq(float alpha, std::integer_sequence<int, R...>) { (acc_scale1<R>(alpha), ...); }
__device__ __forceinline__ void acc_zero() { acc_zero_seq(std::make_integer_sequence<int, 256>{}); }
// every register of a lane belongs to the lane's head: all scale by the lane's alpha
__device__ __forceinline__ void acc_scale(float alpha) { acc_scale_seq(alpha, std::make_integer_sequence<int, 256>{}); }
// the 16 registers of block VB: rows (value columns) 32 VB + 8q + 4hh + i at index 4q + i
template <int VB, int... I>
__device__ __forceinline__ void acc_read_block(float (&o)[16], std::integer_sequence<int, I...>) { ((o[I] = acc_read1<16 * VB + I>()), ...); }

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v lds_short4v;
typedef unsigned uint2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int tr_swz(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

__device__ __forceinline__ bf16x8 tr_frag(uint32_t addr_lo, uint32_t addr_hi) {
  const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_short4v*>(addr_lo));
  const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_short4v*>(addr_hi));
  typedef short short8v __attribute__((ext_vector_type(8)));
  const short8v x = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, x);
}

// max / sum over the two lanes that hold one head (l and l ^ 32), result in both
__device__ __forceinline__ float pair_max(float x) {
  uint2v a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(a.x), __uint_as_float(a.y));
}
__device__ __forceinline__ float pair_sum(float x) {
  uint2v a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(a.x) + __uint_as_float(a.y);
}

}  // namespace
