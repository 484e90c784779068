// Short DFTs of one sequence held in the registers of a lane (lengths 8, 16,
// 32, 64), forward, natural order in and out.
#pragma once
#include <hip/hip_runtime.h>

#include "fft_lds.h"

namespace hvk {

// exp(-2 pi i m / 64) by compile-time Taylor series of the angle reduced to
// [0, pi/4].
struct W64Table {
  float c[64], s[64];
};
constexpr double taylor_cos(double x) {
  double t = 1.0, r = 1.0;
  for (int n = 1; n < 12; ++n) {
    t *= -x * x / ((2 * n - 1) * (2 * n));
    r += t;
  }
  return r;
}
constexpr double taylor_sin(double x) {
  double t = x, r = x;
  for (int n = 1; n < 12; ++n) {
    t *= -x * x / ((2 * n) * (2 * n + 1));
    r += t;
  }
  return r;
}
constexpr W64Table make_w64() {
  W64Table t{};
  const double step = 6.283185307179586476925 / 64;
  for (int m = 0; m < 64; ++m) {
    const int oct = m / 8, q = m % 16, r = q <= 8 ? q : 16 - q;  // angle within the quadrant, folded at pi/4
    const double c = taylor_cos(r * step), s = taylor_sin(r * step);
    const double cq = q <= 8 ? c : s, sq = q <= 8 ? s : c;  // of angle q * step in [0, pi/2)
    const int quad = oct / 2;
    const double cc = quad == 0 ? cq : quad == 1 ? -sq : quad == 2 ? -cq : sq;
    const double ss = quad == 0 ? sq : quad == 1 ? cq : quad == 2 ? -sq : -cq;
    t.c[m] = (float)cc;
    t.s[m] = (float)(-ss);
  }
  return t;
}

// N = N1 * N2: DFTs of length N2 over x[n1 + N1 n2], twiddles, DFTs of length
// N1.  Elements are consumed in the order n1 = 0, 1, ..., so loads issued in
// that order are waited for a group at a time.
template <int N>
__device__ inline void reg_fft(float2* x) {
  if constexpr (N <= 16) {
    dft_reg<N, -1>(x);
  } else {
    constexpr int N2 = 8, N1 = N / N2;
    constexpr W64Table tw = make_w64();
    float2 a[N1][N2];
#pragma unroll
    for (int n1 = 0; n1 < N1; ++n1) {
#pragma unroll
      for (int n2 = 0; n2 < N2; ++n2) a[n1][n2] = x[n1 + N1 * n2];
      dft_reg<N2, -1>(a[n1]);
#pragma unroll
      for (int k2 = 1; k2 < N2; ++k2) {
        const int m = n1 * k2 * (64 / N);
        if (n1 > 0) a[n1][k2] = c2::mul(a[n1][k2], make_float2(tw.c[m], tw.s[m]));
      }
    }
#pragma unroll
    for (int k2 = 0; k2 < N2; ++k2) {
      float2 b[N1];
#pragma unroll
      for (int n1 = 0; n1 < N1; ++n1) b[n1] = a[n1][k2];
      dft_reg<N1, -1>(b);
#pragma unroll
      for (int k1 = 0; k1 < N1; ++k1) x[k2 + N2 * k1] = b[k1];
    }
  }
}

}  // namespace hvk
