// Device helpers of the kernels that multiply FP32 values on the BF16 matrix
// cores, each value split into three BF16 parts.
#pragma once
#include "internal.hpp"

namespace plnmf {

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Buffer loads from a view with an offset past its range return zeros without
// touching memory.  With a scalar offset the range check uses the range less
// that offset, so scalar offsets are only used where they lie inside the view.
constexpr uint32_t kOutside = 0x80000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_view(const void* base, int64_t bytes) {
  const int64_t n = bytes < 0 ? 0 : (bytes > 0x7fffffff ? 0x7fffffff : bytes);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)n, 0x00020000);
}
__device__ __forceinline__ uintx4 ld16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ unsigned ld4(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
}

__device__ __forceinline__ unsigned hi_halves(unsigned lo, unsigned hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x07060302);
}
__device__ __forceinline__ unsigned lo_halves(unsigned lo, unsigned hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x05040100);
}

// Eight FP32 values into their three BF16 parts, packed: the value rounded to the
// nearest BF16, the rest rounded likewise, and what remains, which seven bits hold
// (exact for magnitudes from 2^-110 up; below, BF16 runs out of exponent and the
// last bits go: 2^-13 of the value at 1e-37).  With rounded parts, the middle of
// either sign, the products that the kernels leave out, xm yl + xl ym + xl yl, are
// at most 2^-24 of x y (RMS 5.3e-9; with a high part cut to BF16 four times that).
// Infinities, NaN and values above the largest BF16 leave NaN in a part.
__device__ __forceinline__ void split8(const unsigned (&x)[8], uintx4& ph, uintx4& pm, uintx4& pl) {
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const float x0 = __uint_as_float(x[2 * q]), x1 = __uint_as_float(x[2 * q + 1]);
    const unsigned h = __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{x0, x1}), bf16x2));
    ph[q] = h;
    const floatx2 r = {x0 - __uint_as_float(h << 16), x1 - __uint_as_float(h & 0xffff0000u)};
    const unsigned m = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf16x2));
    pm[q] = m;
    const float l0 = r[0] - __uint_as_float(m << 16);
    const float l1 = r[1] - __uint_as_float(m & 0xffff0000u);
    pl[q] = hi_halves(__float_as_uint(l0), __float_as_uint(l1));
  }
}

}  // namespace plnmf
