// Device code shared by the kernels in which every column of a stripe takes
// part (the prefill product and the batched decode): a wave expands one
// 64-row bitmap word of 16 columns at a time from LDS straight into the
// operand registers of v_mfma_f32_32x32x16_f16.
//
// The word records. For every stripe, group of 16 (padded) columns and
// bitmap word, spdp_encode lays out one record of 160 bytes on the device:
// the 16 columns' words (64 bits each) and, per column, the byte offset of
// the word's first value from the start of the group's chunk (a chunk: four
// groups, 64 columns, whose values are one contiguous run). A wave reads its
// record with three scalar loads; the words serve as rank masks and as
// select masks, the offsets as the ranks' base, so no popcount of the
// column's earlier words is left to the loop.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdint>

#include "chunks.h"

namespace spdp_dev {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRecBytes = 160;
constexpr int kChunkRecBytes = kChunkGroups * 4 * kRecBytes;

// Pointers into the constant address space: reads through them are scalar
// loads.
template <class T>
using const_ptr = const __attribute__((address_space(4))) T*;

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
// Global -> LDS DMA (lane l's bytes land at lds + 16 l), as assembly so that
// the compiler does not order LDS reads of other buffers behind it; the
// waits are explicit. A vector memory instruction needs 5 wait states after
// a VALU write of an SGPR it reads, which the compiler does not insert for
// assembly: s_nop 4.
__device__ __forceinline__ void dma16(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "{m0}"(lds) : "memory");
}

struct WordRec {
  uint64_t w[kGroupCols];
  uint32_t off[kGroupCols / 2];  // two byte offsets per dword
};

__device__ __forceinline__ void load_rec(const_ptr<unsigned char> p, WordRec& m) {
  const const_ptr<uint64_t> pw = (const_ptr<uint64_t>)p;
#pragma unroll
  for (int c = 0; c < kGroupCols; ++c) m.w[c] = pw[c];
  const const_ptr<uint32_t> po = (const_ptr<uint32_t>)(p + 8 * kGroupCols);
#pragma unroll
  for (int c = 0; c < kGroupCols / 2; ++c) m.off[c] = po[c];
}

// The lane's value of column c of the record's word: the one at the column's
// offset plus the word's masked popcount below the lane (every lane reads; a
// lane whose bit is clear reads a neighbour, dropped by the select).
// `base2`: half the LDS byte address of the chunk's values, in a VGPR (the
// popcounts accumulate onto it).
__device__ __forceinline__ uint32_t gather_column(const WordRec& m, int c, uint32_t base2) {
  const uint32_t off = (c & 1) ? m.off[c / 2] >> 16 : m.off[c / 2] & 0xFFFFu;
  const uint32_t rank =
      __builtin_amdgcn_mbcnt_hi((uint32_t)(m.w[c] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m.w[c], base2));
  return *(const __attribute__((address_space(3))) uint16_t*)(uintptr_t)((rank << 1) + off);
}

// the lane's value where its bit of the word is set, else 0 (assembly: the
// compiler would shift before the select and lose the shift-or)
__device__ __forceinline__ uint32_t select_word(uint32_t v, uint64_t mask) {
  uint32_t r;
  asm("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "v"(v), "s"(mask));
  return r;
}

// The two 32x32x16 operands of the word's rows 0-31 and 32-63: lane l holds
// row l mod 32 and columns 8 (l / 32) .. + 7. The selects leave lane = row
// with a column pair per register; swapping the upper half of the pair j
// register with the lower half of the pair j + 4 one gives both operands.
struct Operands {
  uint32_t p[8];  // rows 0-31: 0..3, rows 32-63: 4..7
  __device__ __forceinline__ half8 rows(int i) const {
    return __builtin_bit_cast(half8, u32x4{p[4 * i], p[4 * i + 1], p[4 * i + 2], p[4 * i + 3]});
  }
};
// pairs j and j + 4 of the record's word
__device__ __forceinline__ void select_pairs(const WordRec& m, const uint32_t (&v)[kGroupCols], int j, Operands& o) {
  const uint32_t a = select_word(v[2 * j], m.w[2 * j]) | (select_word(v[2 * j + 1], m.w[2 * j + 1]) << 16);
  const uint32_t b = select_word(v[2 * j + 8], m.w[2 * j + 8]) | (select_word(v[2 * j + 9], m.w[2 * j + 9]) << 16);
  const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  o.p[j] = s[0];
  o.p[j + 4] = s[1];
}

}  // namespace spdp_dev
