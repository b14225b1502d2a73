// Complex FP64 DFTs of a line held in one lane's registers: fully unrolled,
// mixed radix, compile-time roots of unity.
//
// A 1-D pass of the 2D operator as a DFT-matrix GEMM in split FP16 needs, per
// value, more vector instructions for the operand splits alone (about 8) than
// the whole FFT line costs in FP64 (432 instructions for 32 points: 13.5 per
// value, two values per complex point), and FP64 vector instructions issue at
// the FP32 rate on this chip. So the passes run here without matrix cores, in
// FP64 throughout.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

namespace qcoll {
namespace {

// ------------------------------------------------- compile-time roots of unity

// sin and cos of x in [0, pi/4] by their Taylor series (constant expressions;
// the terms after the last one kept are below 2^-60).
constexpr double taylor_sin(double x) {
  double s = 0.0;
  for (int k = 21; k >= 3; k -= 2) s = (s + 1.0) * (-x * x / (k * (k - 1)));
  return x + x * s;
}
constexpr double taylor_cos(double x) {
  double s = 0.0;
  for (int k = 22; k >= 2; k -= 2) s = (s + 1.0) * (-x * x / (k * (k - 1)));
  return 1.0 + s;
}

struct Root {
  double c, s;
};

// exp(2 pi i k / n), the angle reduced to the first octant in integers.
constexpr Root unit_root(int k, int n) {
  const int m = ((k % n) + n) % n;
  const int quarter = 4 * m / n, rem = 4 * m - quarter * n;   // angle = (quarter + rem / n) pi / 2
  const double half_pi = 1.5707963267948966192;
  double c = 0.0, s = 0.0;
  if (2 * rem > n) {
    const double x = half_pi * (n - rem) / n;
    c = taylor_sin(x);
    s = taylor_cos(x);
  } else {
    const double x = half_pi * rem / n;
    c = taylor_cos(x);
    s = taylor_sin(x);
  }
  if (quarter == 0) return {c, s};
  if (quarter == 1) return {-s, c};
  if (quarter == 2) return {-c, -s};
  return {s, -c};
}

template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// (r, i) *= exp(2 pi i K / N)
template <int K, int N>
__device__ __forceinline__ void rotate(double& r, double& i) {
  constexpr int k = ((K % N) + N) % N;
  if constexpr (k == 0) {
  } else if constexpr (2 * k == N) {
    r = -r;
    i = -i;
  } else if constexpr (4 * k == N) {
    const double t = r;
    r = -i;
    i = t;
  } else if constexpr (4 * k == 3 * N) {
    const double t = r;
    r = i;
    i = -t;
  } else if constexpr ((8 * k) % N == 0) {   // odd eighths: |c| = |s| = sqrt(1/2)
    constexpr Root w = unit_root(k, N);
    constexpr double h = 0.70710678118654752440;
    const double p = w.c > 0 ? r : -r, q = w.c > 0 ? i : -i;      // c r, c i over h
    const double u = w.s > 0 ? r : -r, v = w.s > 0 ? i : -i;
    r = (p - v) * h;
    i = (q + u) * h;
  } else {
    constexpr Root w = unit_root(k, N);
    const double t = fma(w.c, r, -(w.s * i));
    i = fma(w.c, i, w.s * r);
    r = t;
  }
}

constexpr int first_radix(int n) {
  if (n % 4 == 0) return 4;
  for (int p = 2; p * p <= n; ++p)
    if (n % p == 0) return p;
  return n;
}

// x[k] <- sum_n x[n] exp(2 pi i SG n k / N), natural order in and out.
template <int N, int SG>
__device__ __forceinline__ void dft(double (&r)[N], double (&i)[N]) {
  if constexpr (N == 1) {
  } else if constexpr (N == 2) {
    const double a = r[0], b = i[0];
    r[0] = a + r[1];
    i[0] = b + i[1];
    r[1] = a - r[1];
    i[1] = b - i[1];
  } else if constexpr (N == 4) {
    const double ar = r[0] + r[2], ai = i[0] + i[2], br = r[0] - r[2], bi = i[0] - i[2];
    const double cr = r[1] + r[3], ci = i[1] + i[3], dr = r[1] - r[3], di = i[1] - i[3];
    r[0] = ar + cr;
    i[0] = ai + ci;
    r[2] = ar - cr;
    i[2] = ai - ci;
    // SG i (dr + i di) = -SG di + i SG dr
    r[1] = SG > 0 ? br - di : br + di;
    i[1] = SG > 0 ? bi + dr : bi - dr;
    r[3] = SG > 0 ? br + di : br - di;
    i[3] = SG > 0 ? bi - dr : bi + dr;
  } else if constexpr (first_radix(N) == N) {   // odd prime: real cosine and sine sums over symmetric pairs
    constexpr int H = (N - 1) / 2;
    double ar[H], ai[H], br[H], bi[H];
    double sr = r[0], si = i[0];
    static_for<H>([&](auto I) {
      constexpr int k = I + 1;
      ar[I] = r[k] + r[N - k];
      ai[I] = i[k] + i[N - k];
      br[I] = r[k] - r[N - k];
      bi[I] = i[k] - i[N - k];
      sr += ar[I];
      si += ai[I];
    });
    const double x0 = r[0], y0 = i[0];
    r[0] = sr;
    i[0] = si;
    static_for<H>([&](auto Mm) {
      constexpr int m = Mm + 1;
      double er = x0, ei = y0, fr = 0.0, fi = 0.0;
      static_for<H>([&](auto I) {
        constexpr Root w = unit_root(m * (I + 1), N);
        er = fma(w.c, ar[I], er);
        ei = fma(w.c, ai[I], ei);
        if constexpr (I == 0) {
          fr = w.s * br[I];
          fi = w.s * bi[I];
        } else {
          fr = fma(w.s, br[I], fr);
          fi = fma(w.s, bi[I], fi);
        }
      });
      // + SG i (fr + i fi)
      r[m] = SG > 0 ? er - fi : er + fi;
      i[m] = SG > 0 ? ei + fr : ei - fr;
      r[N - m] = SG > 0 ? er + fi : er - fi;
      i[N - m] = SG > 0 ? ei - fr : ei + fr;
    });
  } else {
    // n = A n2 + n1, k = k2 + B k1
    constexpr int A = first_radix(N), B = N / A;
    double ur[A][B], ui[A][B];
    static_for<A>([&](auto N1) {
      static_for<B>([&](auto N2) {
        ur[N1][N2] = r[A * N2 + N1];
        ui[N1][N2] = i[A * N2 + N1];
      });
      dft<B, SG>(ur[N1], ui[N1]);
      static_for<B>([&](auto K2) { rotate<SG * N1 * K2, N>(ur[N1][K2], ui[N1][K2]); });
    });
    static_for<B>([&](auto K2) {
      double vr[A], vi[A];
      static_for<A>([&](auto N1) {
        vr[N1] = ur[N1][K2];
        vi[N1] = ui[N1][K2];
      });
      dft<A, SG>(vr, vi);
      static_for<A>([&](auto K1) {
        r[K2 + B * K1] = vr[K1];
        i[K2 + B * K1] = vi[K1];
      });
    });
  }
}

// Order LDS accesses of one wavefront (they execute in order; this keeps the
// compiler from moving one across).
__device__ __forceinline__ void lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace
}  // namespace qcoll
