// fp32 operands as two fp16 terms for the fp16 matrix cores (device code, gfx950).
#pragma once
#include <hip/hip_runtime.h>

namespace acrobat {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

// exact reciprocal of a power of two with a normal reciprocal
__device__ __forceinline__ float inverse_power(float s) { return __uint_as_float((254u << 23) - __float_as_uint(s)); }

// A split operand is exact to 2^-23 of itself where its row (column, in the MV-RNN kernel) lifts it above 2^-3, which is
// 2^-17 of the largest, and to half the smallest fp16 number, 2^-25 over the scale, below that.  A sum of K products of
// operands whose inverse scales have the product f is then off by some sqrt(K) 2^-11 f from what small operands lose, and
// no sum of the other errors can hide that where small operands meet large ones (a feature of 1e9 with a weight of 1e-9
// beside features and weights of order one).  The gates' own rounding is 2^-24, so sums with f above this limit - the
// largest elements of the two rows have a product of 2^13 or more - are computed in fp32.
constexpr float kLargestUnit = 0x1p-16f;

// power of two that lifts m > 0 to [2^14, 2^15); any power of two does where that one is out of range
__device__ __forceinline__ float scale_for(float m) {
  const int e = (int)(__float_as_uint(m) >> 23);
  if (e == 255) return 1.0f;  // an infinity in the row: its products are computed again in fp32
  const int s = 268 - e;
  return __uint_as_float((unsigned)(s > 253 ? 253 : s) << 23);
}

__device__ __forceinline__ void split4(const floatx4 x, const float s, half4& hi, half4& lo) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    hi[e] = (_Float16)(x[e] * s);
    lo[e] = (_Float16)__builtin_fmaf(x[e], s, -(float)hi[e]);
  }
}

// The same for the eight k of a matrix operand, eight instructions per four elements: the scaled element and its
// remainder are rounded straight into their half of a packed register.  (The pairs are interleaved because a half written
// by one instruction must not be read by the next.)
__device__ __forceinline__ void split4_packed(const floatx4 x, const float s, unsigned (&hi)[2], unsigned (&lo)[2]) {
  asm("v_fma_mixlo_f16 %0, %4, %8, 0\n\t"
      "v_fma_mixlo_f16 %1, %6, %8, 0\n\t"
      "v_fma_mixhi_f16 %0, %5, %8, 0\n\t"
      "v_fma_mixhi_f16 %1, %7, %8, 0\n\t"
      "v_fma_mixlo_f16 %2, %4, %8, -%0 op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixlo_f16 %3, %6, %8, -%1 op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixhi_f16 %2, %5, %8, -%0 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixhi_f16 %3, %7, %8, -%1 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\t"
      "s_nop 1"
      : "=&v"(hi[0]), "=&v"(hi[1]), "=&v"(lo[0]), "=&v"(lo[1])
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(s));
}
__device__ __forceinline__ void split8(const floatx4 x0, const floatx4 x1, const float s, half8& hi, half8& lo) {
  unsigned h0[2], l0[2], h1[2], l1[2];
  split4_packed(x0, s, h0, l0);
  split4_packed(x1, s, h1, l1);
  hi = __builtin_bit_cast(half8, uintx4{h0[0], h0[1], h1[0], h1[1]});
  lo = __builtin_bit_cast(half8, uintx4{l0[0], l0[1], l1[0], l1[1]});
}

// largest of the four lanes i, i + 16, i + 32, i + 48, in all of them
__device__ __forceinline__ float largest_of_quarters(const float m) {
  const unsigned u = __float_as_uint(m);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned v = __float_as_uint(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ __forceinline__ float largest(const floatx4 v, const float m) {
  return fmaxf(m, fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))));
}

// A 32-k step of 16 rows on its way into the layout of a matrix operand.  A matrix instruction wants lane l to hold row
// l % 16, but a load whose neighbouring lanes are in different rows fetches 37 KB/us per compute unit where one whose lanes
// read whole cache lines, eight lanes each, fetches 126 (pieces of 64 bytes: 65).  So a step is requested line by line - half
// h: lane l, row 8 h + l / 8, 16 bytes number l % 8 -, split where it arrives and turned through 2 KB of LDS that belong to
// the wavefront (the LDS serves a wavefront's instructions in order: no barrier, and the next step may be written as soon
// as the reads of this one have been issued).  A row in LDS is the 32 hi terms, then the 32 lo terms, in 16-byte units
// swizzled so that neither side has bank conflicts.
constexpr int kTurnFloats = 512;
__device__ __forceinline__ void turn_write(float* const tile, const int lane, const floatx4 (&lines)[2], const float s0,
                                           const float s1) {
  const int wr = lane >> 3, p = lane & 7;
  const int at = 32 * wr + 2 * (p >> 2) + 4 * ((p & 3) ^ (wr >> 1));
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");  // (for the compiler only: no instruction)
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    unsigned hi[2], lo[2];
    split4_packed(lines[h], h ? s1 : s0, hi, lo);
    // (row 8 h + l / 8: the swizzle of the second half is that of the first with the halves of a row exchanged)
    *reinterpret_cast<uintx2*>(tile + 256 * h + (h ? at ^ 16 : at)) = uintx2{hi[0], hi[1]};
    *reinterpret_cast<uintx2*>(tile + 256 * h + (h ? at : at ^ 16)) = uintx2{lo[0], lo[1]};
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
}
// lane l: row l % 16, k = 4 (l / 16) + 0 .. 3 and 16 more
__device__ __forceinline__ void turn_read(const float* const tile, const int lane, half8& hi, half8& lo) {
  const int li = lane & 15, at = 32 * li + 4 * ((lane >> 4) ^ (li >> 1));
  hi = *reinterpret_cast<const half8*>(tile + at);
  lo = *reinterpret_cast<const half8*>(tile + (at ^ 16));
}
// largest over the eight lanes that hold one line, in all of them
__device__ __forceinline__ float largest_of_line(float m) {
  m = fmaxf(m, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(m), 0xB1, 0xF, 0xF, true)));   // lane ^ 1
  m = fmaxf(m, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(m), 0x4E, 0xF, 0xF, true)));   // lane ^ 2
  return fmaxf(m, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(m), 0x141, 0xF, 0xF, true)));  // the other four
}

}  // namespace
}  // namespace acrobat
