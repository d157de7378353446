// fp32 matrix products on the bf16 matrix cores without giving up fp32 precision.
//
// An fp32 number is the exact sum of three bf16 numbers: x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0),
// x2 = x - x0 - x1 (8 + 8 + 8 bits of significand, round to nearest, so |x1| <= 2^-9 |x| and |x2| <= 2^-17 |x| up to the
// rounding of the exponent).  A product is then the sum of nine bf16 products, each exact in fp32; the six of them that
// matter are taken and the three that are left out (x1 y2, x2 y1, x2 y2) sum to at most 2^-25 |x y|, half the rounding
// of one fp32 operation.  Sums are fp32 as before.  Measured on MI355X against double precision (K = 512, 131,072 dot
// products of normal numbers): relative error 3.4e-7 this way, 4.1e-7 with v_mfma_f32_16x16x4_f32; taking eight
// products instead of six changes no digit of that.  A bf16 MFMA does sixteen times the work of an fp32 one per cycle
// (2,040 against 140 TFLOP/s measured), so six of them are 2.4 times as fast.
// The splitting and the choice of products are those of G. Henry, P. T. P. Tang and A. Heinecke, "Leveraging the bfloat16
// Artificial Intelligence Datatype For Higher-Precision Computations" (ARITH 2019).
// Parts below 1e-38 may be flushed.  A number that is infinite, or that rounds to infinity in bf16 (finite magnitudes above
// 3.38e38), has a part inf - inf: every sum it enters is NaN, where fp32 products give an infinity or even a finite number.
// So a kernel that uses split operands looks at its finished sums and takes each NaN among them once more, as a plain fp32 sum
// over the operands as they are (a sum that is NaN in fp32, too, ends at its first NaN term).
#pragma once
#include <hip/hip_runtime.h>

namespace tgnn {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// the three parts of two numbers, packed {a | b << 16}
__device__ __forceinline__ void split_pair(float a, float b, unsigned& q0, unsigned& q1, unsigned& q2) {
  q0 = __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{a, b}), bf16x2));
  a -= __uint_as_float(q0 << 16);
  b -= __uint_as_float(q0 & 0xffff0000u);
  q1 = __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{a, b}), bf16x2));
  a -= __uint_as_float(q1 << 16);
  b -= __uint_as_float(q1 & 0xffff0000u);
  q2 = __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{a, b}), bf16x2));
}

// the three parts of one MFMA operand run: eight consecutive k of one row or column
struct Split8 {
  bf16x8 p[3];
};
__device__ __forceinline__ Split8 split8(const floatx4& lo, const floatx4& hi) {
  uintx4 q[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = i < 2 ? lo[2 * i] : hi[2 * i - 4], b = i < 2 ? lo[2 * i + 1] : hi[2 * i - 3];
    unsigned q0, q1, q2;
    split_pair(a, b, q0, q1, q2);
    q[0][i] = q0; q[1][i] = q1; q[2][i] = q2;
  }
  Split8 s;
#pragma unroll
  for (int p = 0; p < 3; ++p) s.p[p] = __builtin_bit_cast(bf16x8, q[p]);
  return s;
}

// Which parts meet in product t of the six, smallest first.
constexpr int SPLIT_TERMS = 6;
__host__ __device__ constexpr int split_ta(int t) { return t == 0 ? 0 : t == 1 ? 2 : t == 2 ? 1 : t == 3 ? 0 : t == 4 ? 1 : 0; }
__host__ __device__ constexpr int split_tb(int t) { return t == 0 ? 2 : t == 1 ? 0 : t == 2 ? 1 : t == 3 ? 1 : t == 4 ? 0 : 0; }

}  // namespace tgnn
