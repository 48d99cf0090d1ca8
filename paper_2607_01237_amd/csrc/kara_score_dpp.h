// Reductions over the 16 lanes of a DPP row, shared by the scoring kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace kara {
namespace {

// Reductions over the 16 lanes of a row by DPP butterflies (quad swaps,
// then half-row and row mirrors).  Every lane ends with the same value:
// each step combines two equal partial results, in either order.
template <class Op>
__device__ __forceinline__ float dpp_reduce16(float v, Op op) {
  v = op(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false)));
  v = op(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false)));
  v = op(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x141, 0xF, 0xF, false)));
  v = op(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x140, 0xF, 0xF, false)));
  return v;
}
__device__ __forceinline__ float dpp_sum16(float v) {
  return dpp_reduce16(v, [](float x, float y) { return x + y; });
}

// One DPP step over 8 values at once (the leading s_nop covers the values' last
// writes before the block).  Written as instructions because the compiler keeps
// a separate DPP move per step, and in IEEE mode adds a quieting max before
// every fmaxf.
#define S1_DPP8(OP, PAT)                                                                               \
  asm volatile("s_nop 1\n\t"                                                                           \
               OP " %0, %0, %0 " PAT "\n\t" OP " %1, %1, %1 " PAT "\n\t" OP " %2, %2, %2 " PAT "\n\t"  \
               OP " %3, %3, %3 " PAT "\n\t" OP " %4, %4, %4 " PAT "\n\t" OP " %5, %5, %5 " PAT "\n\t"  \
               OP " %6, %6, %6 " PAT "\n\t" OP " %7, %7, %7 " PAT                                        \
               : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]),     \
                 "+v"(v[7]))
// Reduce-scatter over the 16 lanes of a row: every lane's v[i] combined,
// lane li ending with index li's result.  Four butterfly steps, each
// keeping half of the values: lanes li and li ^ 8 (a rotation by 8), then
// li and 7 - li within each half (the half mirror), then the quad swaps
// li ^ 2 and li ^ 1.  A lane keeps the half its bit names and sends the
// other, so each step combines only the values that stay: 45 instructions
// against 64 for every lane's full result.
// (each step is one asm statement that starts with the wait states a DPP
// read needs after the VALU writes of its sources, which all precede it)
template <bool MAX, int K, int PATTERN>
__device__ __forceinline__ void s1_rs_step(float (&keep)[8], const float (&send)[8]) {
  // PATTERN: 0 row_ror:8, 1 row_half_mirror, 2 quad_perm:[2,3,0,1], 3 quad_perm:[1,0,3,2]
#define S1_OPS(OP, PAT)                                                                                     \
  if constexpr (K == 8)                                                                                     \
    asm volatile("s_nop 1\n\t"                                                                              \
                 OP " %0, %8, %0 " PAT "\n\t" OP " %1, %9, %1 " PAT "\n\t" OP " %2, %10, %2 " PAT "\n\t"    \
                 OP " %3, %11, %3 " PAT "\n\t" OP " %4, %12, %4 " PAT "\n\t" OP " %5, %13, %5 " PAT "\n\t"  \
                 OP " %6, %14, %6 " PAT "\n\t" OP " %7, %15, %7 " PAT                                     \
                 : "+v"(keep[0]), "+v"(keep[1]), "+v"(keep[2]), "+v"(keep[3]), "+v"(keep[4]), "+v"(keep[5]), \
                   "+v"(keep[6]), "+v"(keep[7])                                                             \
                 : "v"(send[0]), "v"(send[1]), "v"(send[2]), "v"(send[3]), "v"(send[4]), "v"(send[5]),     \
                   "v"(send[6]), "v"(send[7]));                                                             \
  else if constexpr (K == 4)                                                                                \
    asm volatile("s_nop 1\n\t"                                                                              \
                 OP " %0, %4, %0 " PAT "\n\t" OP " %1, %5, %1 " PAT "\n\t" OP " %2, %6, %2 " PAT "\n\t"     \
                 OP " %3, %7, %3 " PAT                                                                      \
                 : "+v"(keep[0]), "+v"(keep[1]), "+v"(keep[2]), "+v"(keep[3])                               \
                 : "v"(send[0]), "v"(send[1]), "v"(send[2]), "v"(send[3]));                                 \
  else if constexpr (K == 2)                                                                                \
    asm volatile("s_nop 1\n\t" OP " %0, %2, %0 " PAT "\n\t" OP " %1, %3, %1 " PAT                           \
                 : "+v"(keep[0]), "+v"(keep[1])                                                             \
                 : "v"(send[0]), "v"(send[1]));                                                             \
  else                                                                                                      \
    asm volatile("s_nop 1\n\t" OP " %0, %1, %0 " PAT : "+v"(keep[0]) : "v"(send[0]))
  if constexpr (MAX) {
    if constexpr (PATTERN == 0) S1_OPS("v_max_f32_dpp", "row_ror:8 row_mask:0xf bank_mask:0xf");
    else if constexpr (PATTERN == 1) S1_OPS("v_max_f32_dpp", "row_half_mirror row_mask:0xf bank_mask:0xf");
    else if constexpr (PATTERN == 2) S1_OPS("v_max_f32_dpp", "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf");
    else S1_OPS("v_max_f32_dpp", "quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf");
  } else {
    if constexpr (PATTERN == 0) S1_OPS("v_add_f32_dpp", "row_ror:8 row_mask:0xf bank_mask:0xf");
    else if constexpr (PATTERN == 1) S1_OPS("v_add_f32_dpp", "row_half_mirror row_mask:0xf bank_mask:0xf");
    else if constexpr (PATTERN == 2) S1_OPS("v_add_f32_dpp", "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf");
    else S1_OPS("v_add_f32_dpp", "quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf");
  }
#undef S1_OPS
}
template <bool MAX>
__device__ __forceinline__ float reduce_scatter16(const float (&v)[16], int li) {
  float keep[8], send[8];
  const bool h3 = (li & 8) != 0, h2 = (li & 4) != 0, h1 = (li & 2) != 0, h0 = (li & 1) != 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    keep[k] = h3 ? v[8 + k] : v[k];
    send[k] = h3 ? v[k] : v[8 + k];
  }
  s1_rs_step<MAX, 8, 0>(keep, send);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float a = keep[k], b = keep[4 + k];
    keep[k] = h2 ? b : a;
    send[k] = h2 ? a : b;
  }
  s1_rs_step<MAX, 4, 1>(keep, send);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float a = keep[k], b = keep[2 + k];
    keep[k] = h1 ? b : a;
    send[k] = h1 ? a : b;
  }
  s1_rs_step<MAX, 2, 2>(keep, send);
  {
    const float a = keep[0], b = keep[1];
    keep[0] = h0 ? b : a;
    send[0] = h0 ? a : b;
  }
  s1_rs_step<MAX, 1, 3>(keep, send);
  return keep[0];
}

// max of three, with no quieting of its operands
__device__ __forceinline__ float s1_max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Eight values per lane combined over the 16 lanes of a row: lane li ends
// with value li & 7 (both halves of the row).  A rotation by 8 of every
// value, then the three halving steps above.
template <bool MAX>
__device__ __forceinline__ float reduce_scatter8(float (&v)[8], int li) {
  if constexpr (MAX) {
    S1_DPP8("v_max_f32_dpp", "row_ror:8 row_mask:0xf bank_mask:0xf");
  } else {
    S1_DPP8("v_add_f32_dpp", "row_ror:8 row_mask:0xf bank_mask:0xf");
  }
  float keep[8], send[8];
  const bool h2 = (li & 4) != 0, h1 = (li & 2) != 0, h0 = (li & 1) != 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    keep[k] = h2 ? v[4 + k] : v[k];
    send[k] = h2 ? v[k] : v[4 + k];
  }
  s1_rs_step<MAX, 4, 1>(keep, send);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float a = keep[k], b = keep[2 + k];
    keep[k] = h1 ? b : a;
    send[k] = h1 ? a : b;
  }
  s1_rs_step<MAX, 2, 2>(keep, send);
  {
    const float a = keep[0], b = keep[1];
    keep[0] = h0 ? b : a;
    send[0] = h0 ? a : b;
  }
  s1_rs_step<MAX, 1, 3>(keep, send);
  return keep[0];
}
#undef S1_DPP8

}  // namespace
}  // namespace kara
