// Packed MFMA operands of the sweep products (gemm_pk.hip): for each block of
// 16 rows, each 32 elements of K and each part, the KiB that one wave reads as
// an operand of v_mfma_f32_16x16x32_bf16 (lane l holds row l % 16, elements
// 8 (l / 16) .. + 7 of the 32).  BF16 elements have one part, FP32 elements
// three BF16 parts that hold all their bits.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include "nnc_device.h"

namespace nnc {

template <typename T> struct PkElem {  // BF16
  static constexpr int NP = 1;   // parts
  static constexpr int KB = 32;  // elements along K of one block
};
template <> struct PkElem<float> {
  static constexpr int NP = 3;
  static constexpr int KB = 32;
};
template <> struct PkElem<double> {
  static constexpr int NP = 1;
  static constexpr int KB = 8;
};

// The parts of four consecutive elements.  (Never contracted with the product
// that an element comes from: its parts are then those of the rounded element
// in every kernel, and a result does not depend on which of them wrote it.)
template <int NP>
__device__ __forceinline__ void cut_parts(const float (&v)[4], uint2 (&o)[NP]) {
#pragma clang fp contract(off)
  if constexpr (NP == 1) {
    bf16x4 t;
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = (bf16)v[e];
    o[0] = __builtin_bit_cast(uint2, t);
  } else {
    // Each of the first two parts is what is left rounded to 8 significant bits:
    // the differences are exact, the third part leaves nothing, and what the
    // products below leave out (gemm_pk.hip) has either sign.
    typedef float float2v __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    uint32_t w[3][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float r0 = v[2 * h], r1 = v[2 * h + 1];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        w[p][h] = __builtin_bit_cast(uint32_t, __builtin_convertvector(float2v{r0, r1}, bf16x2));
        r0 -= __uint_as_float(w[p][h] << 16);
        r1 -= __uint_as_float(w[p][h] & 0xffff0000u);
      }
    }
    // An element that rounds past the largest finite one is cut off there instead.
    // An infinite one is 1, 0 and itself: the third part meets only first parts,
    // which are zero or not as their elements are, so infinity times a number is
    // infinite and times zero NaN, as for the elements themselves.  (As the first
    // part it met the zero second and third parts of every short number.)
    const float big = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
    if (__builtin_expect(big >= 0x1.ffp127f, 0)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t t[3] = {__float_as_uint(v[e]) & 0xffff0000u, 0u, 0u};
        if (fabsf(v[e]) == INFINITY) {
          t[2] = t[0];
          t[0] = (t[0] & 0x80000000u) | 0x3f800000u;
        } else if (fabsf(v[e]) >= 0x1.ffp127f) {
          const float r = v[e] - __uint_as_float(t[0]);
          t[1] = __float_as_uint(r) & 0xffff0000u;
          t[2] = __float_as_uint(r - __uint_as_float(t[1]));
        } else {
          continue;
        }
#pragma unroll
        for (int p = 0; p < 3; ++p)
          w[p][e / 2] = e & 1 ? (w[p][e / 2] & 0xffffu) | (t[p] & 0xffff0000u) : (w[p][e / 2] & 0xffff0000u) | t[p] >> 16;
      }
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) o[p] = make_uint2(w[p][0], w[p][1]);
  }
}

// Byte offset of element (row, col) of part 0 of an operand with kt blocks
// along K; part p is p KiB on.
template <typename T>
__device__ __forceinline__ long long packed_offset(int row, int col, int kt) {
  using E = PkElem<T>;
  constexpr int LANE = E::KB / 4;  // elements of one lane
  return ((long long)(row >> 4) * kt + col / E::KB) * (E::NP * 1024) + col % E::KB / LANE * 256 + (row & 15) * 16 +
         col % LANE * (16 / LANE);
}

// Four consecutive elements (row, col .. col + 3), col a multiple of 4, into a
// packed operand.
template <typename T, typename A>
__device__ __forceinline__ void put_packed(void* base, int row, int col, int kt, const A (&v)[4]) {
  char* o = (char*)base + packed_offset<T>(row, col, kt);
  if constexpr (sizeof(T) == 8) {
    *(double2*)o = make_double2(v[0], v[1]);
    *(double2*)(o + 256) = make_double2(v[2], v[3]);  // the next lane group's pair
  } else {
    constexpr int NP = PkElem<T>::NP;
    uint2 t[NP];
    cut_parts<NP>(v, t);
#pragma unroll
    for (int p = 0; p < NP; ++p) *(uint2*)(o + p * 1024) = t[p];
  }
}

}  // namespace nnc
