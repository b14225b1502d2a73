// Classical spectral method (section 3.3): Q_hat_k as the direct double sum over
// l + m = k (modulo N, the collocation reading of the fast method) of
// beta(l, m) f_hat_l f_hat_m with a dense table of kernel modes, O(N^4) per cell
// in 2D. FP64 throughout, one launch.
//
// Two symmetries leave a quarter of the sum. f is real and beta(-l, -m) =
// beta(l, m), so Q_hat(-k) is the conjugate of Q_hat(k): rows k1 = 0 .. N/2 are
// computed. And (l, m), (m, l) multiply the same product: for an output row k1
// the pairs of rows {m1, k1 - m1} are taken once, with the weight beta(l, m) +
// beta(m, l) (a row paired with itself keeps its own weights).
//
// A workgroup holds C cells in LDS, [mode][cell]; thread (j, c) works on cell c.
// The transforms are register FFTs (fft_reg.hpp), thread j taking line j. In the
// sum thread j owns half an output row, N/2 modes (k1, h N/2 + i): row 0 and row
// N/2 have only their first half, so there are N such tasks (and the two real
// modes (0, N/2) and (N/2, N/2), summed over all threads). Per pair of rows a
// thread reads the row l1 into registers once, each f_hat_m once, and runs N x N/2
// products from registers: 2 N LDS reads for N^2 / 2 products, where reading
// both factors of every product bound the direct form (about 19 TB/s from LDS).
//
// What bounds it: FP64 vector issue, 6 instructions per product (7.1 M wavefront
// instructions for 4096 cells of 16 x 16, 15 us; one wavefront per SIMD, so LDS and
// L2 latencies add). 4096 cells of 16 x 16: 35 us (180 for the direct form over all
// modes and both orders), 16384: 98 (640); 4096 of 24 x 24: 155 (960); 1 cell of 16 x
// 16: 31 (89).

#include <hip/hip_runtime.h>

#include <cstdint>

#include "classical_args.hpp"
#include "fft_reg.hpp"
#include "kernels_common.hpp"

namespace qcoll {
namespace {

// Workgroups of 16 cells (8 above 20 points: 16 would be two wavefronts on a SIMD, whose
// registers hold less than a line needs) or, for more workgroups, of 4. Up to 16 points
// and above 20, wide from a wide workgroup for every CU on (16 x 16: 4096 cells 37 us with
// 4, 34 with 16; 512 cells 32 and 33). The wide form of 18 and 20 points spills (47 and 94
// registers), but its rounds hold 16 cells per CU where those of the narrow form, one
// wavefront per SIMD, hold 8: a wide round takes 1.15 narrow ones at 18 points and 1.8 at
// 20. So 18 points are wide from the second narrow round on (2000 cells 49 us with 4, 56
// with 16; 2500 cells 93 and 57) and 20 points where the number of narrow rounds is even
// (2500 cells 106 and 89, 4500 cells 158 and 174, 8192 cells 216 and 204).
static bool classical_wide(const ClassicalArgs& a) {
  const int64_t narrow_rounds = (a.cells + 8 * a.cus - 1) / (8 * a.cus);
  if (a.N == 18) return narrow_rounds > 1;
  if (a.N == 20) return narrow_rounds % 2 == 0;
  return a.cells >= 16 * static_cast<int64_t>(a.cus);
}

template <int N, int C>
struct Classical {
  static constexpr int n = N * N, H = N / 2, P = N / 2 + 1;   // P pairs of rows per output row
  static constexpr int W = classical_row(N);                  // doubles per weight row (N/2, even)
  static constexpr int kThreads = N * C;
  static constexpr int kLdsBytes = n * C * 16 + 2 * N * C * 8;
};

template <int N, int C>
__global__ __launch_bounds__(N* C) void classical_kernel(ClassicalArgs a) {
  using K = Classical<N, C>;
  constexpr int n = K::n, H = K::H;
  extern __shared__ double2 A[];                           // [mode][cell]
  double* part = reinterpret_cast<double*>(A + n * C);     // [2][N][C]
  const int c = threadIdx.x % C, j = threadIdx.x / C;
  const int k1 = (j + 1) / 2, h = j == 0 || j == N - 1 ? 0 : (j + 1) & 1;   // this thread's half row
  for (int64_t c0 = static_cast<int64_t>(blockIdx.x) * C; c0 < a.cells; c0 += static_cast<int64_t>(gridDim.x) * C) {
    const bool live = c0 + c < a.cells;
    const int64_t base = (live ? c0 + c : c0) * n;
    double xr[N], xi[N];
    // ---- forward: row j along the last axis, then column j along the first, normalised
#pragma unroll
    for (int v = 0; v < N; ++v) {
      xr[v] = static_cast<double>(a.f[base + j * N + v]);
      xi[v] = 0.0;
    }
    dft<N, -1>(xr, xi);
#pragma unroll
    for (int v = 0; v < N; ++v) A[(j * N + v) * C + c] = make_double2(xr[v], xi[v]);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < N; ++v) {
      const double2 z = A[(v * N + j) * C + c];
      xr[v] = z.x;
      xi[v] = z.y;
    }
    dft<N, -1>(xr, xi);
#pragma unroll
    for (int v = 0; v < N; ++v) A[(v * N + j) * C + c] = make_double2(xr[v] * (1.0 / n), xi[v] * (1.0 / n));
    __syncthreads();
    // ---- the double sum
    double ar[H], ai[H];
#pragma unroll
    for (int i = 0; i < H; ++i) ar[i] = ai[i] = 0.0;
    const double* wt = a.weights + static_cast<int64_t>(j) * (K::P * N * K::W);
    int m1 = (k1 + 1) / 2;
#pragma unroll 1
    for (int p = 0; p < K::P; ++p) {
      const int l1 = k1 - m1 < 0 ? k1 - m1 + N : k1 - m1;
      // row l1 rotated by h N/2: register i holds mode l2 = i + h N/2
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int l2 = (i + h * H) % N;
        const double2 z = A[(l1 * N + l2) * C + c];
        xr[i] = z.x;
        xi[i] = z.y;
      }
      const double2* mrow = A + m1 * N * C + c;
      static_for<N>([&](auto M2) {
        constexpr int m2 = M2;
        const double2 fm = mrow[m2 * C];
        double wv[K::W];
#pragma unroll
        for (int i = 0; i < K::W; i += 2) {
          const double2 w2 = *reinterpret_cast<const double2*>(wt + m2 * K::W + i);
          wv[i] = w2.x;
          wv[i + 1] = w2.y;
        }
        static_for<H>([&](auto I) {
          constexpr int i = I, l = (i - m2 + N) % N;   // mode k2 = i + h N/2, l2 = k2 - m2
          const double ur = wv[i] * fm.x, ui = wv[i] * fm.y;
          ar[i] = fma(xr[l], ur, fma(-xi[l], ui, ar[i]));
          ai[i] = fma(xr[l], ui, fma(xi[l], ur, ai[i]));
        });
      });
      wt += N * K::W;
      m1 = m1 + 1 == N ? 0 : m1 + 1;
    }
    // the real modes (0, N/2) and (N/2, N/2): thread j sums over m1 = j
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int l1 = ((e ? H : 0) - j + N) % N;
      const double* wx = a.extra + (e * N + j) * N;
      double s = 0.0;
#pragma unroll
      for (int m2 = 0; m2 < N; ++m2) {
        const double2 fm = A[(j * N + m2) * C + c], fl = A[(l1 * N + (H - m2 + N) % N) * C + c];
        s = fma(wx[m2], fma(fl.x, fm.x, -(fl.y * fm.y)), s);
      }
      part[(e * N + j) * C + c] = s;
    }
    __syncthreads();   // the spectrum has been read: Q_hat takes its place
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int k2 = h * H + i;
      A[(k1 * N + k2) * C + c] = make_double2(ar[i], ai[i]);
      // rows 0 and N/2: the mirrored half
      if ((j == 0 || j == N - 1) && i > 0) A[(k1 * N + N - i) * C + c] = make_double2(ar[i], -ai[i]);
    }
    if (j < 2) {
      double s = 0.0;
#pragma unroll
      for (int v = 0; v < N; ++v) s += part[(j * N + v) * C + c];
      A[((j ? H : 0) * N + H) * C + c] = make_double2(s, 0.0);
    }
    __syncthreads();
    // ---- inverse: column j along the first axis (rows k1 > N/2 are conjugates), then row j
#pragma unroll
    for (int v = 0; v < N; ++v) {
      const double2 z = v <= H ? A[(v * N + j) * C + c] : A[((N - v) * N + (j == 0 ? 0 : N - j)) * C + c];
      xr[v] = z.x;
      xi[v] = v <= H ? z.y : -z.y;
    }
    dft<N, 1>(xr, xi);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < N; ++v) A[(v * N + j) * C + c] = make_double2(xr[v], xi[v]);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < N; ++v) {
      const double2 z = A[(j * N + v) * C + c];
      xr[v] = z.x;
      xi[v] = z.y;
    }
    dft<N, 1>(xr, xi);
    if (!a.conserve) {
      if (live) {
        float* Qo = reinterpret_cast<float*>(a.q) + base + j * N;
#pragma unroll
        for (int v = 0; v < N; ++v) Qo[v] = static_cast<float>(xr[v]);
      }
    } else {   // FP64 projection: moments over the cell's N threads
      const double v1 = -a.L + a.dv * j;
      double m[4] = {0, 0, 0, 0};
#pragma unroll
      for (int v = 0; v < N; ++v) {
        const double v2 = -a.L + a.dv * v;
        m[0] += xr[v];
        m[2] += v2 * xr[v];
        m[3] += (v1 * v1 + v2 * v2) * xr[v];
      }
      m[1] = v1 * m[0];
      __syncthreads();   // A is free
      double* red = reinterpret_cast<double*>(A);
#pragma unroll
      for (int i = 0; i < 4; ++i) red[(i * N + j) * C + c] = m[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        m[i] = 0.0;
        for (int v = 0; v < N; ++v) m[i] += red[(i * N + v) * C + c];
      }
      double lam[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        lam[i] = a.gram_inv[i * 4 + 0] * m[0] + a.gram_inv[i * 4 + 1] * m[1] + a.gram_inv[i * 4 + 2] * m[2] +
                 a.gram_inv[i * 4 + 3] * m[3];
      if (live) {
        double* Qo = reinterpret_cast<double*>(a.q) + base + j * N;
#pragma unroll
        for (int v = 0; v < N; ++v) {
          const double v2 = -a.L + a.dv * v;
          Qo[v] = xr[v] - (lam[0] + lam[1] * v1 + lam[2] * v2 + lam[3] * (v1 * v1 + v2 * v2));
        }
      }
    }
    __syncthreads();   // the next group rewrites A
  }
}

template <int N, int C>
int launch_nc(const ClassicalArgs& args, hipStream_t stream) {
  constexpr int kLds = Classical<N, C>::kLdsBytes;
  static_assert(kLds <= 160 * 1024, "LDS of a CU");
  if (kLds > 64 * 1024) {   // above the default limit of dynamic LDS
    static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(classical_kernel<N, C>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, kLds) == hipSuccess;
    if (!ok) return -3;
  }
  const int64_t groups = (args.cells + C - 1) / C;
  const int64_t blocks = groups < 4096 ? groups : 4096;
  hipLaunchKernelGGL((classical_kernel<N, C>), dim3(static_cast<unsigned>(blocks)), dim3(N * C), kLds, stream, args);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

template <int N>
int launch_n(const ClassicalArgs& args, hipStream_t stream) {
  return classical_wide(args) ? launch_nc<N, (N > 20 ? 8 : 16)>(args, stream) : launch_nc<N, 4>(args, stream);
}

}  // namespace

int launch_classical(const ClassicalArgs& args, hipStream_t stream) {
  if (args.cells <= 0) return 0;
  switch (args.N) {
    case 4: return launch_n<4>(args, stream);
    case 6: return launch_n<6>(args, stream);
    case 8: return launch_n<8>(args, stream);
    case 10: return launch_n<10>(args, stream);
    case 12: return launch_n<12>(args, stream);
    case 14: return launch_n<14>(args, stream);
    case 16: return launch_n<16>(args, stream);
    case 18: return launch_n<18>(args, stream);
    case 20: return launch_n<20>(args, stream);
    case 22: return launch_n<22>(args, stream);
    case 24: return launch_n<24>(args, stream);
    default: return -1;
  }
}

}  // namespace qcoll
