// Complex FP64 DFTs of a line held in one lane's registers: fully unrolled,
// mixed radix, compile-time roots of unity.
//
// A 1-D pass of the 2D operator as a DFT-matrix GEMM in split FP16 needs, per
// value, more vector instructions for the operand splits alone (about 8) than
// the whole FFT line costs in FP64 (388 instructions for 32 points: 12 per
// point, six per value), and FP64 vector instructions issue at
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

// (p, m) <- a + w b, a - w b with w = exp(2 pi i K / N): six FMAs, w b formed as
// c (1 + i t) b with t = s / c (or s (t + i) b with t = c / s where |s| > |c|) and
// its factor c folded into the two sums. With radix 4 as two such steps a line of 32
// points takes 388 instructions; rotations ahead of plain butterflies took 432. The
// BPR(3,4,3) step of 4096 cells of 32 x 32: 494 -> 466 us.
template <int K, int N>
__device__ __forceinline__ void butterfly(double ar, double ai, double br, double bi, double& pr, double& pi,
                                          double& mr, double& mi) {
  constexpr int k = ((K % N) + N) % N;
  if constexpr (4 * k % N == 0) {   // w = 1, i, -1, -i
    rotate<K, N>(br, bi);
    pr = ar + br;
    pi = ai + bi;
    mr = ar - br;
    mi = ai - bi;
  } else {
    constexpr Root w = unit_root(k, N);
    constexpr double ac = w.c < 0 ? -w.c : w.c, as = w.s < 0 ? -w.s : w.s;
    constexpr bool by_c = 8 * k % N == 0 || ac > as;
    constexpr double scale = by_c ? w.c : w.s;
    double yr, yi;
    if constexpr (8 * k % N == 0) {   // |c| = |s|
      constexpr bool same = (w.c > 0) == (w.s > 0);
      yr = same ? br - bi : br + bi;
      yi = same ? bi + br : bi - br;
    } else if constexpr (by_c) {
      constexpr double t = w.s / w.c;
      yr = fma(-t, bi, br);
      yi = fma(t, br, bi);
    } else {
      constexpr double t = w.c / w.s;
      yr = fma(t, br, -bi);
      yi = fma(t, bi, br);
    }
    pr = fma(scale, yr, ar);
    pi = fma(scale, yi, ai);
    mr = fma(-scale, yr, ar);
    mi = fma(-scale, yi, ai);
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
    });
    static_for<B>([&](auto K2) {
      double vr[A], vi[A];
      if constexpr (A == 2) {
        butterfly<SG * K2, N>(ur[0][K2], ui[0][K2], ur[1][K2], ui[1][K2], r[K2], i[K2], r[K2 + B], i[K2 + B]);
        return;
      }
      // x0 + w^2 x2, x1 + w^2 x3 and their differences, then the sums with w and i w.
      // (Odd B: fewer instructions as well, but 2000 cells of 48 points took 337 us
      // instead of 330, of 20 points 51.7 instead of 50.9.)
      if constexpr (A == 4 && B % 2 == 0) {
        double cr, ci, dr, di;
        butterfly<SG * 2 * K2, N>(ur[0][K2], ui[0][K2], ur[2][K2], ui[2][K2], vr[0], vi[0], vr[1], vi[1]);
        butterfly<SG * 2 * K2, N>(ur[1][K2], ui[1][K2], ur[3][K2], ui[3][K2], cr, ci, dr, di);
        butterfly<SG * K2, N>(vr[0], vi[0], cr, ci, r[K2], i[K2], r[K2 + 2 * B], i[K2 + 2 * B]);
        butterfly<SG * (K2 + B), N>(vr[1], vi[1], dr, di, r[K2 + B], i[K2 + B], r[K2 + 3 * B], i[K2 + 3 * B]);
        return;
      }
      static_for<A>([&](auto N1) { rotate<SG * N1 * K2, N>(ur[N1][K2], ui[N1][K2]); });
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
