// Small pieces shared by the matrix-core kernels of the front end and the
// prompt scorer.
#pragma once

#include "spot_internal.h"

namespace spot {
namespace mc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;

// c + A B: lane l holds 8 consecutive k of row l%16 of A (column l%16 of B)
// from k = 8(l/16), and rows 4(l/16) ..+3 of column l%16 of c.
__device__ __forceinline__ f32x4 mfma(const u32x4& a, const u32x4& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Two floats -> packed BF16, round to nearest even.
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2_t));
}

// 16 bytes per lane, global -> LDS, lane l's at dst + 16 l.
__device__ __forceinline__ void load_lds(const void* src, unsigned char* dst) {
  __builtin_amdgcn_global_load_lds(src, (lds_void*)dst, 16, 0, 0);
}

// s_waitcnt: at most VM vector loads outstanding, every LDS access done.
template <int VM>
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | 0x0070);
}

}  // namespace mc
}  // namespace spot
