// What the attention kernels of this library share beyond gfx950.hpp: the constants of the softmax, operands from LDS, and the
// matrix instructions and LDS reads in assembly of the kernels whose loops are pipelined by hand.
#pragma once
#include <hip/hip_runtime.h>

#include "gfx950.hpp"

namespace tasp {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kRescaleGap = 8.0f;   // the running max is only raised when it grew by more than 2^8
constexpr float kNegBig = -1.0e30f;

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}
// A operand of Y^T E: 32 columns of Y (rows of Y^T) by 16 rows of Y, from two transposing reads
// eight rows apart.
__device__ inline bf16x8 lds_tr8(const unsigned char* lo, const unsigned char* hi) {
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)const_cast<unsigned char*>(lo));
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)const_cast<unsigned char*>(hi));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// LDS operand reads whose wait is placed by hand.  A read is volatile assembly (issued in program
// order), and the fragment reaches its matrix instruction only behind a wait until at most N
// younger LDS instructions are outstanding (LDS instructions of a wavefront complete in order, so
// extra ones the compiler adds only make a wait stricter).  That wait is part of the
// matrix instruction's own asm statement (TASP_MFMA_ASM).
template <int IMM>
__device__ __forceinline__ void lds_read_b128(u32x4& d, unsigned addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(IMM));
}
template <int IMM>
__device__ __forceinline__ void lds_read_tr_b64(u32x2& d, unsigned addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(IMM));
}

// Matrix instructions as volatile assembly: they stay in program order, which is the schedule, and
// the register classes are fixed: score tiles in VGPRs (the softmax reads them), O^T and the Q
// fragments in AGPRs.  The compiler does not know these are matrix instructions, so the wait states
// it would insert are placed by hand (the fence_* helpers):
//   matrix result -> vector ALU / accvgpr read: 12 wait states;  vector ALU result -> matrix operand: 2.
// Dependent matrix instructions on the same accumulator need none.
// ACC: O^T and the Q fragments live in AGPRs (needed when a wave owns two strips; with one strip
// everything fits the 256 VGPRs of a wave that shares its SIMD, and using any AGPR would make the
// compiler split that budget in half).
// W >= 0: the instruction's fragment `a` comes from LDS reads in flight, and the wait for it (at most
// W younger LDS instructions outstanding) sits in the same asm statement: a wait in a statement of
// its own that names the fragment makes the compiler put a wait state between the two (it has to
// assume that any asm statement forwards its result like a sub-dword write).  W < 0: no wait.
#define TASP_MFMA_ASM(W, ...)                                                                   \
  do {                                                                                          \
    if constexpr ((W) >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\t" __VA_ARGS__, "n"((W) < 0 ? 0 : (W))); \
    else asm volatile(__VA_ARGS__, "n"(0));                                                     \
  } while (0)
template <bool ACC, int W = -1>
__device__ __forceinline__ void mfma_s_first(f32x16& d, const u32x4& a, const u32x4& b) {
  if constexpr (ACC) TASP_MFMA_ASM(W, "v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
  else TASP_MFMA_ASM(W, "v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
template <bool ACC, int W = -1>
__device__ __forceinline__ void mfma_s(f32x16& d, const u32x4& a, const u32x4& b) {
  if constexpr (ACC) TASP_MFMA_ASM(W, "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
  else TASP_MFMA_ASM(W, "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
// score tile: readable by the vector ALU after this point (placed at least one matrix instruction after the last one that wrote it)
__device__ __forceinline__ void fence_s(f32x16& a, f32x16& b) { asm volatile("s_nop 15" : "+v"(a), "+v"(b)); }
// P fragment: written by the vector ALU, read by matrix instructions after this point
__device__ __forceinline__ void fence_p(u32x4& f) { asm volatile("s_nop 1" : "+v"(f)); }

}  // namespace
}  // namespace tasp
