// Device helpers of the pivoted eliminations: pivot keys, wave-wide maxima and
// reciprocals, shared by the Gauss-Jordan inversions and the banded one.
#pragma once
#include <hip/hip_runtime.h>

#include <cfloat>

namespace fsi {

constexpr int kNoRow = 0x7fffffff;

// DPP move of a double to a fresh register (full EXEC, every row written)
template <int CTRL>
__device__ __forceinline__ double mov_dpp_f64(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// DPP move of a double (full EXEC); rows outside ROWS keep their own value
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ double dpp_f64(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, ROWS, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double readlane_f64(double x, int l) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double readlane(double x, int l) { return readlane_f64(x, l); }
__device__ __forceinline__ float readlane(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
// DPP controls: quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_ror 4, row_ror 8,
// row_bcast 15 (lane 15 of each row into the next row), row_bcast 31 (lane 31
// into rows 2 and 3)
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppRor4 = 0x124, kDppRor8 = 0x128;
constexpr int kDppBcast15 = 0x142, kDppBcast31 = 0x143;

// Pivot keys.  A candidate row i with entry a in the pivot column is keyed
// by |a| with its lowest 13 mantissa bits replaced by 8191 - i (rows are
// below 8192): keys order by |a| to 39 significant bits, then by the lowest
// row, and a plain fmax reduces them (positive doubles order as their bit
// patterns).  A non-finite |a| keys as the largest finite double, which
// fails the step; rows that are not candidates carry -1.
constexpr long long kKeyMask = (1LL << 13) - 1;
__device__ __forceinline__ double pivot_key(double a, int i) {
  double x = fabs(a);
  if (!(x <= DBL_MAX)) x = DBL_MAX;   // NaN or infinite
  return __longlong_as_double((__double_as_longlong(x) & ~kKeyMask) | (kKeyMask - i));
}
__device__ __forceinline__ int key_row(double k) {
  return (int)(kKeyMask - (__double_as_longlong(k) & kKeyMask));
}
__device__ __forceinline__ double key_value(double k) {
  return __longlong_as_double(__double_as_longlong(k) & ~kKeyMask);
}

// max of two pivot keys.  Keys are never NaN, so with RAW the plain
// instruction is used (fmax first quiets possible signalling NaNs of both
// operands); the asm statement limits the scheduler, so kernels whose panel
// already fills most registers keep fmax.
template <bool RAW>
__device__ __forceinline__ double key_max(double a, double b) {
  if constexpr (RAW) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
  } else {
    return fmax(a, b);
  }
}

// wave-wide maximum of a key, the same value in every lane: DPP inside each
// row of 16 lanes, then row broadcasts carry the running maximum into the
// last row, whose lane 63 is read.  Requires all 64 lanes active.
template <bool RAW>
__device__ __forceinline__ double wave_max(double v) {
  v = key_max<RAW>(v, mov_dpp_f64<kDppXor1>(v));
  v = key_max<RAW>(v, mov_dpp_f64<kDppXor2>(v));
  v = key_max<RAW>(v, mov_dpp_f64<kDppRor4>(v));
  v = key_max<RAW>(v, mov_dpp_f64<kDppRor8>(v));
  v = key_max<RAW>(v, dpp_f64<kDppBcast15, 0xA>(v));   // rows 1, 3: max with rows 0, 2
  v = key_max<RAW>(v, dpp_f64<kDppBcast31, 0xC>(v));   // rows 2, 3: max with row 1
  return readlane_f64(v, 63);
}

// 1 / a from the hardware reciprocal refined by two Newton steps: within an
// ulp of the rounded quotient for 2^-1021 <= |a| <= 2^1021 (outside that range
// the result may be 0 or NaN; such a pivot leaves the block unusable anyway)
__device__ __forceinline__ double recip(double a) {
  double x = __builtin_amdgcn_rcp(a);
  x = fma(x, fma(-a, x, 1.0), x);
  x = fma(x, fma(-a, x, 1.0), x);
  return x;
}

// 1 / a in single precision: the hardware reciprocal and one Newton step
__device__ __forceinline__ float recip(float a) {
  float x = __builtin_amdgcn_rcpf(a);
  return fmaf(x, fmaf(-a, x, 1.0f), x);
}

typedef double dx4 __attribute__((ext_vector_type(4)));
typedef float fx4 __attribute__((ext_vector_type(4)));

// The 16x16x4 matrix-core product of each element type.  Operand layouts are
// the same (A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k); the output
// tile differs: the FP64 instruction holds D[i][j] in lane j + 16 (i % 4),
// register i / 4, the FP32 one in lane j + 16 (i / 4), register i % 4.
template <typename T>
struct Mfma16;
template <>
struct Mfma16<double> {
  typedef dx4 acc;
  static __device__ __forceinline__ acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int kq) { return r * 4 + kq; }
};
template <>
struct Mfma16<float> {
  typedef fx4 acc;
  static __device__ __forceinline__ acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int kq) { return kq * 4 + r; }
};

}  // namespace fsi
