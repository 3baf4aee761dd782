// Transposed fragment reads from LDS (gfx950's ds_read_b64_tr_b16): the operand of a
// bfloat16 matrix instruction wants 8 consecutive k of one row per lane, and a tile
// whose rows are contiguous at each k holds them 8 lines apart.  In a group of 16
// lanes, lane l passes the address of four consecutive rows 4 (l % 4) .. + 3 at line
// l / 4, and receives row l at those four lines.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sq {

typedef __bf16 tr_bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 tr_bf16x8 __attribute__((ext_vector_type(8)));
typedef short tr_s4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ tr_bf16x4 lds_tr4(const void* p) {
  typedef __attribute__((address_space(3))) tr_s4* lds_ptr;
  return __builtin_bit_cast(tr_bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p));
}

// 8 consecutive k per lane: p0 / p1 are this lane's addresses for the first and last four
__device__ __forceinline__ tr_bf16x8 lds_tr8(const void* p0, const void* p1) {
  const tr_bf16x4 a = lds_tr4(p0), b = lds_tr4(p1);
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

}  // namespace sq
