// What the bf16 attention kernels share (internal to libaspd): how pages come into LDS and lie there, and the pieces of the
// running softmax.
#pragma once

#include "attn_common.h"

namespace {

// ---------------------------------------------------------------------------------------------
// Pages and queries go from global memory straight into LDS, 16 bytes per lane: lane l's to byte lds + 16 l, so that one
// instruction fills 1024 consecutive bytes (the rows of a page as they follow each other in the cache).  Assembly because
// behind the builtin the compiler makes every later LDS read wait for all such loads in flight; the kernels count which
// of them have to be there.  A statement reads no vector register but the offsets, and writes none.  It brings its own
// wait states: one behind the write of m0, and five in front of the load for a base that a vector instruction has
// written, as the reload of a spilled scalar register is; the compiler does not see that a memory instruction in here
// reads it.
// ---------------------------------------------------------------------------------------------
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // (m0 is reserved; in the code as built nothing else uses it)
__device__ __forceinline__ void load_to_lds(const void* base /* uniform */, uint32_t offset, uint32_t lds /* uniform */) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base)
               : "memory", "m0");
}
// Four bytes per lane.
__device__ __forceinline__ void load4_to_lds(const void* base /* uniform */, uint32_t offset, uint32_t lds /* uniform */) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(offset), "s"(base)
               : "memory", "m0");
}
// A page of one KV head (D = 128: 4096 bytes, D = 64: 2048), `offset`: per load, within its 1024 bytes.  The constant
// offset of such a load counts on either side.  NT: non-temporal.
template <int D, bool NT>
__device__ __forceinline__ void page_to_lds(const void* base /* uniform */, const uint32_t (&offset)[D / 32],
                                            uint32_t lds /* uniform */) {
#define ASPD_PAGE_LOAD(NTS)                                                                                            \
  if constexpr (D == 128)                                                                                              \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %5" NTS                                    \
                 "\n\tglobal_load_lds_dwordx4 %2, %5 offset:1024" NTS "\n\tglobal_load_lds_dwordx4 %3, %5 offset:2048" NTS \
                 "\n\tglobal_load_lds_dwordx4 %4, %5 offset:3072" NTS ::"s"(lds),                                      \
                 "v"(offset[0]), "v"(offset[1]), "v"(offset[D / 32 - 2]), "v"(offset[D / 32 - 1]), "s"(base)           \
                 : "memory", "m0");                                                                                    \
  else                                                                                                                 \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %3" NTS                                    \
                 "\n\tglobal_load_lds_dwordx4 %2, %3 offset:1024" NTS ::"s"(lds), "v"(offset[0]), "v"(offset[1]), "s"(base) \
                 : "memory", "m0")
  if constexpr (NT) {
    ASPD_PAGE_LOAD(" nt");
  } else {
    ASPD_PAGE_LOAD("");
  }
#undef ASPD_PAGE_LOAD
}
#pragma clang diagnostic pop
// All but the youngest N of the wave's vector memory operations have arrived.
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// LDS operands by byte address.
__device__ __forceinline__ bf16x8 lds_operand(uint32_t at) {
  return *(const __attribute__((address_space(3))) bf16x8*)(uintptr_t)at;
}
__device__ __forceinline__ s16x4 lds_operand_transposed(uint32_t at) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)at);
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}

// Owner tags through the scalar (constant) path, for the kernels whose waves fetch pages cooperatively: the address is
// the same for the whole wave, and scalar loads are counted apart from the vector loads, whose count those kernels wait
// on for pages (a vector load of tags among them would have to be waited for together with every group of pages sent
// before it).
typedef u32x4 __attribute__((aligned(4))) u32x4_a4;
__device__ __forceinline__ u32x4 load_tags_uniform(const uint8_t* p /* same in all lanes, 4-byte aligned */) {
  return *(const __attribute__((address_space(4))) u32x4_a4*)(uintptr_t)p;
}
// A pointer every lane holds, as a value the compiler knows to be the same in all of them.
__device__ __forceinline__ const uint8_t* uniform_ptr(const uint8_t* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const uint8_t*)(((uint64_t)hi << 32) | lo);
}
// A word through the scalar path, of an array that no kernel writes while this one runs.
__device__ __forceinline__ int load_word_uniform(const int32_t* p /* same in all lanes */) {
  return *(const __attribute__((address_space(4))) int32_t*)(uintptr_t)p;
}

// Largest of eight scores in four instructions.  Written as assembly because fmaxf() makes the compiler
// quiet a possible signalling NaN in every operand first (one more instruction each: 11 instead of 4);
// scores are MFMA results or -inf and never NaN here, and the three-operand
// maximum returns a number whenever one operand is a number.
// The operands are usually MFMA results, and a vector instruction that reads one too soon after the MFMA
// was issued gets the old register contents: the hardware does not interlock, the compiler pads with
// wait states for the instructions it emits itself, and it does not look into assembly.  So the block
// brings its own wait states (16: more than the 8-pass MFMA used here needs) and is ONE statement, so
// that no MFMA can be scheduled between them and the reads.
__device__ __forceinline__ float max8(const float (&x)[8]) {
  float r1, r2, m;
  asm("s_nop 15\n\t"
      "v_max3_f32 %0, %3, %4, %5\n\t"
      "v_max3_f32 %1, %6, %7, %8\n\t"
      "v_max3_f32 %2, %9, %10, %0\n\t"
      "v_max_f32 %2, %1, %2"
      : "=&v"(r1), "=&v"(r2), "=&v"(m)
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]));
  return m;
}

// A lane's value combined with that of the lane 32 further (both get the result), without LDS.
template <typename F>
__device__ __forceinline__ float over_halves(float v, F combine) {
  const unsigned b = __builtin_bit_cast(unsigned, v);
  const auto x = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  const unsigned x0 = x[0], x1 = x[1];  // (the compiler takes element 0 for a bit cast of x[1] itself)
  return combine(__builtin_bit_cast(float, x0), __builtin_bit_cast(float, x1));
}

// A lane's value combined with that of the lanes 16 / 32 further (every lane gets the result), without LDS.
template <typename F>
__device__ __forceinline__ float over_quarters(float v, F combine) {
  const unsigned b = __builtin_bit_cast(unsigned, v);
  const auto x = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  const unsigned x0 = x[0], x1 = x[1];  // (the compiler takes element 0 for a bit cast of x[1] itself)
  return over_halves(combine(__builtin_bit_cast(float, x0), __builtin_bit_cast(float, x1)), combine);
}

}  // namespace
