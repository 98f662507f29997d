// Device code shared by the kernels whose operands travel packed (gfx950).
#pragma once
#include "agent_access.h"
#include "cell_kernels.h"

namespace acrobat {
namespace {

// Keeps a kernel argument in scalar registers: loaded again where it is used, it would cost the chain of a level 200 cycles.
// (The address space is named because the compiler can no longer see it.)
#define ACROBAT_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ ACROBAT_GLOBAL T* keep(T* p) {
  ACROBAT_GLOBAL T* g = (ACROBAT_GLOBAL T*)p;
  asm volatile("" : "+s"(g));
  return g;
}
// base[byte / sizeof(T)]: a scalar base and a 32-bit offset take one vector register where a pointer takes two
template <class T>
__device__ __forceinline__ ACROBAT_GLOBAL T& at_byte(ACROBAT_GLOBAL T* base, unsigned byte) {
  return *(ACROBAT_GLOBAL T*)((ACROBAT_GLOBAL char*)base + byte);
}
// Loads, stores and matrix instructions stay on their side: the scheduler would request the steps of a block in an order of
// its own, and the first matrix instruction then waits for the last of them.
__device__ __forceinline__ void hold_order() { __builtin_amdgcn_sched_barrier(0x4); }

// The two terms of a state, hi in the lower half
__device__ __forceinline__ unsigned split_state(const float h) {
  const float x = h * kStateScale;
  const _Float16 hi = (_Float16)x;
  const _Float16 lo = (_Float16)__builtin_fmaf(h, kStateScale, -(float)hi);
  return (unsigned)__builtin_bit_cast(unsigned short, hi) | (unsigned)__builtin_bit_cast(unsigned short, lo) << 16;
}
// Lane q of a quad holds unit 4 i + q of a row; it gets the word that it stores: hi terms 0 1, hi 2 3, lo 0 1, lo 2 3.
__device__ __forceinline__ unsigned quad_word(const unsigned w, const int lane) {
  const unsigned even = (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0x88, 0xF, 0xF, true);  // lanes 0 2 0 2
  const unsigned odd = (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0xDD, 0xF, 0xF, true);   // lanes 1 3 1 3
  return __builtin_amdgcn_perm(odd, even, lane & 2 ? 0x07060302u : 0x05040100u);
}

// Unit 16 jb + eu of a tree node's states goes to its place (see packed_kernels.hip); to < 0: nobody reads it.  The four
// lanes of a quad hold four units of one node.
__device__ __forceinline__ void store_tree_place(const __amdgpu_buffer_rsrc_t operand, float* const cells, const int H, const int to,
                                                 const int jb, const int eu, const int lane, const float h, const float c) {
  const unsigned word = quad_word(split_state(h), lane);
  if (to < 0) return;
  const unsigned row = (unsigned)(to >> 1) & 15u, side_block = 2u * (unsigned)(to >> 5) + ((unsigned)to & 1u);
  const unsigned in_place = 2048u * (jb >> 1) + 8u * (jb & 1) + 512u * (eu & 2) + 256u * (eu >> 2) + 4u * (eu & 1);
  __builtin_amdgcn_raw_buffer_store_b32(word, operand, (int)(side_block * (64u * H) + 16u * row + in_place), 0, 0);
  cells[(size_t)side_block * (16u * H) + 256u * jb + 16u * row + eu] = c;
}

}  // namespace
}  // namespace acrobat
