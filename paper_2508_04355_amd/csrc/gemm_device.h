// Device side of the fp32 and general bf16 product kernels: types, LDS layout of an operand tile, the pieces of an fp32
// value (see gemm_kernels.hip).
#pragma once
#include "scan_device.h"

namespace gecc {
namespace {

typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) double f64x4_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;

constexpr int THREADS = 256;
constexpr float TINY = 0x1p-110f;

// smallest magnitude of the nonzero values seen, as an integer that has their order (zero: the largest one)
struct Least {
  uint32_t v = 0xffffffffu;
  static __device__ __forceinline__ uint32_t of(float x) { return (__float_as_uint(x) << 1) - 1u; }
  __device__ __forceinline__ void see(float x0, float x1) { v = min(min(v, of(x0)), of(x1)); }
  __device__ __forceinline__ bool tiny() const { return v < of(TINY); }
};

// LDS of one operand: PIECES planes of tile[row][BK] bf16; the 16-byte chunks of a row are XOR-swizzled so
// that neither the 16 rows a fragment read touches nor the 16 rows a transposed store writes meet in a bank (measured for
// both row lengths with the bank conflict counter: none; by row / 4 instead, rows of 64 bytes, a fragment read takes 8 cycles for
// 4 and a transposed store 16 for 8)
template <int BK> __device__ __forceinline__ int lds_at(int row, int chunk) {
  return row * (BK * 2) + ((chunk ^ ((row / 2) & (BK / 8 - 1))) << 4);
}

// two neighbouring k-values of a row -> their PIECES packed pairs
__device__ __forceinline__ void split2(float x0, float x1, uint32_t (&p)[3]) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const f32x2_t x = {x0, x1};
    p[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));   // round to nearest even
    x0 -= __uint_as_float(p[q] << 16);
    x1 -= __uint_as_float(p[q] & 0xffff0000u);
  }
}

// sum over the 16 lanes of a row of lanes, in every one of them
__device__ __forceinline__ float row16_sum(float x) {
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xf, 0xf, false));   // row_ror:8
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x124, 0xf, 0xf, false));   // row_ror:4
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x122, 0xf, 0xf, false));   // row_ror:2
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x121, 0xf, 0xf, false));   // row_ror:1
  return x;
}

}  // namespace
}  // namespace gecc
