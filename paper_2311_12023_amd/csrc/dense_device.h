// Device helpers of the kernels that keep a small dense fp64 matrix in the registers of one workgroup, and of others that
// index register arrays by compile-time constants.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace lq {

// f(0), f(1), .. f(N - 1) (or downwards) with the index a compile-time constant, so that register arrays keep constant
// subscripts however large the body is.
template <int N, class F>
__device__ __forceinline__ void for_each_block(F&& f) {
  if constexpr (N > 0) { for_each_block<N - 1>(f); f(std::integral_constant<int, N - 1>{}); }
}
template <int N, class F>
__device__ __forceinline__ void for_each_block_down(F&& f) {
  if constexpr (N > 0) { f(std::integral_constant<int, N - 1>{}); for_each_block_down<N - 1>(f); }
}

// Pair a of a round of the parallel Jacobi method (circle method: round < n-1, a < n/2, so both sums stay below 2(n-1) and
// one conditional subtraction replaces the modulo); p < q.
__device__ inline void circle_pair(int a, int round, int n, int& p, int& q) {
  if (a == 0) { p = n - 1; q = round; }
  else {
    p = round + a; if (p >= n - 1) p -= n - 1;
    q = round - a + (n - 1); if (q >= n - 1) q -= n - 1;
  }
  if (p > q) { const int t = p; p = q; q = t; }
}

// Descending order of the values, NaN last, equal ones by index: a total order, so that counting what stands before each gives
// every rank once.
template <typename T>
__device__ __forceinline__ bool sorts_before(T a, int ia, T b, int ib) {
  return a == b || (a != a && b != b) ? ia < ib : a > b || b != b;
}

template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, false);     // every lane has a source: no old value
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
constexpr int XOR1 = 0xB1, XOR2 = 0x4E, XOR7 = 0x141, XOR15 = 0x140;   // quad_perm, quad_perm, row_half_mirror, row_mirror

__device__ __forceinline__ double lane_value(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane), __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// Sum over the 64 lanes, the same in all of them.
__device__ __forceinline__ double wave_sum(double x) {
  x += dpp_move<XOR1>(x);
  x += dpp_move<XOR2>(x);
  x += dpp_move<XOR7>(x);
  x += dpp_move<XOR15>(x);
  return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}

// 1/x for normal x: the hardware seed (about 23 bits) times 1 + e + e^2, e = 1 - x seed.  1/sqrt(x): its seed and two Newton steps.
__host__ __device__ __forceinline__ double rcp64(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  const double r = __builtin_amdgcn_rcp(x), e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
#else
  return 1.0 / x;
#endif
}
__device__ __forceinline__ double rsqrt64(double x) {
  double r = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x;
  r = fma(r, fma(-h * r, r, 0.5), r);
  return fma(r, fma(-h * r, r, 0.5), r);
}

// The two points of the next round of the eigenvalue search, as parts of the interval: around the zero of the secant through
// the ends' values flo 2^elo and fhi 2^ehi, q to either side, or thirds where there is no secant to take (not wanted, an end's
// value not known, which 0 says, or a zero outside).
struct SearchPoints { double a, b; bool secant; };
__host__ __device__ __forceinline__ SearchPoints search_points(double flo, int elo, double fhi, int ehi, bool wanted, double q) {
  const double ratio = ldexp(flo * rcp64(fhi), elo - ehi), at = ratio * rcp64(ratio - 1.0);
  const bool secant = wanted && flo != 0.0 && fhi != 0.0 && at >= 0.0 && at <= 1.0;     // false for NaN
  return {secant ? fmax(at - q, 0.5 * at) : 1.0 / 3, secant ? fmin(at + q, 0.5 + 0.5 * at) : 2.0 / 3, secant};
}

}  // namespace lq
