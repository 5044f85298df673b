// FP64 tile products on v_mfma_f64_4x4x4_4b, the FP64 matrix instruction that
// reaches the part's FP64 rate.  Register-only loops on one card, TFLOP/s at 1
// and at 2..8 wavefronts per SIMD, by independent accumulators:
//                      1            2            4            8
//   4x4x4_4b       61, 77       76, 77       77, 77       77, 77
//   16x16x4        68, 73-74    67, 71-72    60, 66-68    49, 59-60
// An accumulator of the wide form is four registers a lane, so a tile of several
// units has the larger counts.
//
// One instruction forms four independent 4 x 4 products (blocks b) over four
// contraction indices; lane l = j + 4 b + 16 k holds A_b[j][k] and B_b[k][j],
// and lane j + 4 b + 16 i receives D_b[i][j].  A 16 x 16 x 4 product (A 16
// rows x 4, B 4 x 16 columns, both with lane l = x + 16 k as for the 16 x 16
// instruction) is four of them: with the quads of A's rows rotated by r, lane
// quad b multiplies A's row quad (b + r) % 4 by B's column quad b, and r = 0..3
// cover the sixteen 4 x 4 blocks.  Accumulator r of lane quad b then holds row
// quad (b + r) % 4 (element row 4 ((b + r) % 4) + l / 16, column l % 16);
// unrot4 brings a tile into the 16 x 16 instruction's layout (register q =
// row 4 q + l / 16, column l % 16).
#pragma once
#include <hip/hip_runtime.h>

namespace gk {

// four independent accumulators (no register tuple)
struct m4d {
  double r0, r1, r2, r3;
};

// the value of lane quad (b + R) % 4 of the same row of 16 lanes
template <int R>
__device__ __forceinline__ double quad_rot(double v) {
  if (R == 0) return v;
  const unsigned long long u = __double_as_longlong(v);
  constexpr int ctrl = 0x120 + 16 - 4 * (R == 0 ? 1 : R);   // row_ror by 16 - 4 R lanes
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(u & 0xffffffffu), ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), ctrl, 0xf, 0xf, true);
  return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ void quad_rots(double v, double (&r)[4]) {
  r[0] = v;
  r[1] = quad_rot<1>(v);
  r[2] = quad_rot<2>(v);
  r[3] = quad_rot<3>(v);
}
// acc += A B for one 16 x 16 x 4 step; ar: the rotations of A, b: B
__device__ __forceinline__ void mma4(const double (&ar)[4], double b, m4d& acc) {
  acc.r0 = __builtin_amdgcn_mfma_f64_4x4x4f64(ar[0], b, acc.r0, 0, 0, 0);
  acc.r1 = __builtin_amdgcn_mfma_f64_4x4x4f64(ar[1], b, acc.r1, 0, 0, 0);
  acc.r2 = __builtin_amdgcn_mfma_f64_4x4x4f64(ar[2], b, acc.r2, 0, 0, 0);
  acc.r3 = __builtin_amdgcn_mfma_f64_4x4x4f64(ar[3], b, acc.r3, 0, 0, 0);
}
// v[q] = row 4 q + l / 16, column l % 16
__device__ __forceinline__ void unrot4(const m4d& a, double (&v)[4]) {
  const int b = (int)(threadIdx.x >> 2) & 3;
  const double t0 = (b & 1) ? a.r3 : a.r0, t1 = (b & 1) ? a.r0 : a.r1, t2 = (b & 1) ? a.r1 : a.r2,
               t3 = (b & 1) ? a.r2 : a.r3;
  v[0] = (b & 2) ? t2 : t0;
  v[1] = (b & 2) ? t3 : t1;
  v[2] = (b & 2) ? t0 : t2;
  v[3] = (b & 2) ? t1 : t3;
}

}  // namespace gk
