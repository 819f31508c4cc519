// Small complex helpers for device code (FP32 and FP64).
#pragma once
#include <hip/hip_runtime.h>

namespace lbs {

template <typename T>
struct cx {
  T x, y;
};

template <typename T>
__device__ __forceinline__ cx<T> mk(T a, T b) {
  return cx<T>{a, b};
}
template <typename T>
__device__ __forceinline__ cx<T> operator+(cx<T> a, cx<T> b) {
  return cx<T>{a.x + b.x, a.y + b.y};
}
template <typename T>
__device__ __forceinline__ cx<T> operator-(cx<T> a, cx<T> b) {
  return cx<T>{a.x - b.x, a.y - b.y};
}
template <typename T>
__device__ __forceinline__ cx<T> operator*(cx<T> a, cx<T> b) {
  return cx<T>{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__device__ __forceinline__ cx<T> operator*(T s, cx<T> a) {
  return cx<T>{s * a.x, s * a.y};
}
__device__ __forceinline__ float tfma(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}
__device__ __forceinline__ double tfma(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}
// a * b + c in four fused multiply-adds, x = a.x b.x + (c.x - a.y b.y),
// y = a.x b.y + (c.y + a.y b.x): the step of a complex Horner scheme
template <typename T>
__device__ __forceinline__ cx<T> cfma(cx<T> a, cx<T> b, cx<T> c) {
  return cx<T>{tfma(a.x, b.x, tfma(-a.y, b.y, c.x)),
               tfma(a.x, b.y, tfma(a.y, b.x, c.y))};
}
template <typename T>
__device__ __forceinline__ cx<T> cinv(cx<T> a) {
  T d = T(1) / (a.x * a.x + a.y * a.y);
  return cx<T>{a.x * d, -a.y * d};
}
template <typename T>
__device__ __forceinline__ cx<T> cpow(cx<T> z, int n) {
  cx<T> r{T(1), T(0)};
  while (n) {
    if (n & 1) r = r * z;
    z = z * z;
    n >>= 1;
  }
  return r;
}

// sum_j w_j log x_j for squared distances x_j (x = 0: -inf; x = +inf: +inf
// with INF, which the sums over points of the sphere do without: 3% of them):
// x = 2^k m with m in [sqrt(1/2), sqrt(2)), and with s = (m - 1) / (m + 1)
//   log m = 2 atanh(s) = 2 s + s R(s^2) = f - s (f - R),  f = m - 1 (exact),
// where R's coefficients interpolate sum_{j >= 1} 2 z^j / (2 j + 1) at the
// Chebyshev points of [0, (3 - sqrt(8))^2] (5e-18 of log m).  The powers of
// two and the log m are summed apart, which keeps the rounding of the sum no
// larger than with the library's log.  About 32 FP64 instructions a term
// against the library's 110: 2000 sources at 1e5 targets 0.57 -> 0.22 ms.
template <bool INF = false>
struct LogSums {
  double k = 0.0, t = 0.0;
  __device__ __forceinline__ void add(double w, double x) {
    const int e = __builtin_amdgcn_frexp_exp(x * 1.4142135623730951) - 1;
    const double m = __builtin_amdgcn_ldexp(x, -e);
    const double f = m - 1.0, g = m + 1.0;
    double r = __builtin_amdgcn_rcp(g);
    const double d = __builtin_fma(-g, r, 1.0);
    r = __builtin_fma(__builtin_fma(d, d, d), r, r);
    const double s = f * r, z = s * s;
    double q = 0.14617807153417325;
    q = __builtin_fma(q, z, 0.15331611722055008);
    q = __builtin_fma(q, z, 0.1818289243253687);
    q = __builtin_fma(q, z, 0.22222211089379496);
    q = __builtin_fma(q, z, 0.28571428626253836);
    q = __builtin_fma(q, z, 0.3999999999989889);
    q = __builtin_fma(q, z, 0.666666666666667);
    const double l = __builtin_fma(-s, __builtin_fma(-q, z, f), f);
    // (classes +-0 and +inf: f is -1 or +inf there)
    const bool edge = INF ? __builtin_amdgcn_class(x, 0x260) : x == 0.0;
    const double lim = INF ? __builtin_copysign(__builtin_inf(), f) : -__builtin_inf();
    t = __builtin_fma(w, edge ? lim : l, t);
    k = __builtin_fma(w, (double)e, k);
  }
  __device__ __forceinline__ double value() const {
    return __builtin_fma(k, 0.6931471805599453, t);
  }
};

using LogSum = LogSums<>;

// Sums of 32 values over the 64 lanes: at each step a lane gives half of its
// values away and adds the partner's other half (32 shuffles; 192 one value
// at a time); lanes 2 i and 2 i + 1 return value i's sum.
// (N: values kept; a recursion, so that every index is static)
template <int N = 16>
__device__ __forceinline__ double lane_sums32(double (&v)[32], int lane) {
  const bool up = lane & (2 * N);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double give = up ? v[i] : v[i + N], keep = up ? v[i + N] : v[i];
    v[i] = keep + __shfl_xor(give, 2 * N, 64);
  }
  if constexpr (N > 1) return lane_sums32<N / 2>(v, lane);
  else return v[0] + __shfl_xor(v[0], 1, 64);
}

}  // namespace lbs
