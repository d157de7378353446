// Device helpers: sine/cosine of a double-precision argument, row copies.
#pragma once
#include <hip/hip_runtime.h>

namespace tgnn {

// sin and cos of `arg`.  The argument of the time encoding, w * dt + b, reaches ~1e6 rad, where one float
// ulp is a quarter of a radian; so the argument is formed and reduced to [-pi/4, pi/4] in double, and only
// the polynomial is evaluated in float.  The two polynomials' coefficients are those of sinf / cosf in the Cephes
// mathematical library (S. L. Moshier, single/sinf.c).  On [-pi/4, pi/4] the polynomials are within 2.7e-9 (sine) and
// 1.1e-10 (cosine) of the functions, with their roundings to float within 4.6e-8 and 7.4e-8
// (tests/test_device_math.py).
__device__ __forceinline__ void sincos_reduced(double arg, float& s, float& c) {
  // j = arg * 2/pi rounded to the nearest integer, by adding and taking off 1.5 * 2^52 (round-to-nearest mode): the
  // sum's low mantissa bits then are j's low bits in two's complement, which gives the quadrant j mod 4 without a
  // double -> integer conversion (the 64-bit one is a dozen double-precision instructions).  |arg| < 2^51.
  const double magic = 6755399441055744.0;
  const double t = fma(arg, 0.63661977236758134308, magic);     // 2/pi
  const int q = __double2loint(t) & 3;
  const double j = t - magic;
  double r = fma(-j, 1.57079632679489655800e+00, arg);          // pi/2 high part
  r = fma(-j, 6.12323399573676603587e-17, r);                   // pi/2 low part
  const float x = (float)r, x2 = x * x;
  const float sp = x + x * x2 * (-1.6666654611e-1f + x2 * (8.3321608736e-3f + x2 * (-1.9515295891e-4f)));
  const float cp = 1.0f - 0.5f * x2 +
                   x2 * x2 * (4.166664568298827e-2f + x2 * (-1.388731625493765e-3f + x2 * 2.443315711809948e-5f));
  s = (q & 1) ? cp : sp;
  c = (q & 1) ? sp : cp;
  if (q & 2) s = -s;
  if ((q + 1) & 2) c = -c;
}

__device__ __forceinline__ float time_enc(double delta, float w, float b) {
  float s, c;
  sincos_reduced(fma((double)w, delta, (double)b), s, c);
  return c;
}

// Brings the kernel's explicit arguments into the scalar cache, all lines of them at once; `args`: the kernel's own parameters,
// all of them, in their order.  (The values are not used, and have come in when the asm block ends.)  The argument block is
// cold, and wherever the compiler first needs a field of it is a miss of its own: with several hundred bytes of arguments a
// chain of them.  What lies behind the explicit arguments (block and grid sizes) is there only in kernels that use it; GRID asks for
// its first word through the pointer that makes it be there.
template <class... Args> constexpr int kernarg_bytes() {   // (each argument at its alignment)
  size_t at = 0;
  ((at = (at + alignof(Args) - 1) / alignof(Args) * alignof(Args) + sizeof(Args)), ...);
  return (int)at;
}
// lines 0 .. 2 and so on, and the word behind the arguments, as one block
#define TGNN_WARM_3 "s_load_dword %0, %16, 0x0\n\ts_load_dword %1, %16, 0x40\n\ts_load_dword %2, %16, 0x80\n\t"
#define TGNN_WARM_5 TGNN_WARM_3 "s_load_dword %3, %16, 0xc0\n\ts_load_dword %4, %16, 0x100\n\t"
#define TGNN_WARM_6 TGNN_WARM_5 "s_load_dword %5, %16, 0x140\n\t"
#define TGNN_WARM_8 TGNN_WARM_6 "s_load_dword %6, %16, 0x180\n\ts_load_dword %7, %16, 0x1c0\n\t"
#define TGNN_WARM_13 TGNN_WARM_8 "s_load_dword %8, %16, 0x200\n\ts_load_dword %9, %16, 0x240\n\ts_load_dword %10, %16, 0x280\n\t" \
                     "s_load_dword %11, %16, 0x2c0\n\ts_load_dword %12, %16, 0x300\n\t"
#define TGNN_WARM(LOADS)                                                                                                        \
  asm volatile(LOADS "s_waitcnt lgkmcnt(0)"                                                                                     \
               : "=&s"(d[0]), "=&s"(d[1]), "=&s"(d[2]), "=&s"(d[3]), "=&s"(d[4]), "=&s"(d[5]), "=&s"(d[6]), "=&s"(d[7]), "=&s"(d[8]), \
                 "=&s"(d[9]), "=&s"(d[10]), "=&s"(d[11]), "=&s"(d[12]), "=&s"(d[13]), "=&s"(d[14]), "=&s"(d[15])                \
               : "s"(p), "s"(behind))
template <bool GRID, class... Args> __device__ __forceinline__ void warm_kernarg_lines() {
#ifdef __HIP_DEVICE_COMPILE__
  constexpr int LINES = (kernarg_bytes<Args...>() + 63) / 64;
  static_assert(LINES == 3 || LINES == 5 || LINES == 6 || LINES == 8 || LINES == 13, "spelled out above");
  static_assert(!GRID || LINES == 8, "spelled out below");
  const auto p = __builtin_amdgcn_kernarg_segment_ptr();
  auto behind = p;
  if constexpr (GRID) behind = __builtin_amdgcn_implicitarg_ptr();
  unsigned d[16];
  if constexpr (LINES == 3) TGNN_WARM(TGNN_WARM_3);
  if constexpr (LINES == 5) TGNN_WARM(TGNN_WARM_5);
  if constexpr (LINES == 6) TGNN_WARM(TGNN_WARM_6);
  if constexpr (LINES == 8 && !GRID) TGNN_WARM(TGNN_WARM_8);
  if constexpr (LINES == 8 && GRID) TGNN_WARM(TGNN_WARM_8 "s_load_dword %8, %17, 0x0\n\t");
  if constexpr (LINES == 13) TGNN_WARM(TGNN_WARM_13);
#endif
}
#undef TGNN_WARM
#undef TGNN_WARM_3
#undef TGNN_WARM_5
#undef TGNN_WARM_6
#undef TGNN_WARM_8
#undef TGNN_WARM_13
template <class... Args> __device__ __forceinline__ void warm_kernargs(const Args&...) { warm_kernarg_lines<false, Args...>(); }
template <class... Args> __device__ __forceinline__ void warm_kernargs_and_grid(const Args&...) { warm_kernarg_lines<true, Args...>(); }

// x plus what the DPP control `CTRL` brings in from another lane of the row of 16
template <int CTRL> __device__ __forceinline__ float dpp_add(float x) {
  return x + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}

// One wavefront copies n floats (dst, src aligned to VEC floats, n % VEC == 0) and appends nz zeros.
template <int VEC>
__device__ __forceinline__ void wave_copy(float* __restrict__ dst, const float* __restrict__ src, int n, int nz,
                                          int lane) {
  if (VEC == 4) {
    for (int i = lane; i < n / 4; i += 64)
      reinterpret_cast<float4*>(dst)[i] = reinterpret_cast<const float4*>(src)[i];
  } else if (VEC == 2) {
    for (int i = lane; i < n / 2; i += 64)
      reinterpret_cast<float2*>(dst)[i] = reinterpret_cast<const float2*>(src)[i];
  } else {
    for (int i = lane; i < n; i += 64) dst[i] = src[i];
  }
  for (int i = lane; i < nz; i += 64) dst[n + i] = 0.f;
}

__device__ __forceinline__ void wave_zero(float* __restrict__ dst, int n, int lane) {
  for (int i = lane; i < n; i += 64) dst[i] = 0.f;
}

}  // namespace tgnn
