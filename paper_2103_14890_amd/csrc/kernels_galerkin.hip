// Dealiased (Galerkin) variant of Q_h on 2D grids (section 3.3, eqs. (VAR) and
// (ode) without wrap-around): the operator is evaluated on the grid of
// nf = 3n/2 points per axis with the filters restricted to the active modes of
// the n grid, between a trigonometric interpolation of f (n -> nf) and a
// restriction of Q back to the active n-grid modes (nf -> n). Both are separable
// real matrices, applied along each axis in FP64.
//
// The two products of a cell run on the FP64 matrix instructions, straight from
// registers: an accumulator register v of tile kt holds row 16 kt + 4 v + k on lanes
// 16 k .. 16 k + 15, so with the first product formed transposed, T^t = X^t M^t, its
// accumulators are, register for register, the A operand of the second, T M^t.
// A wavefront computes 16 rows of the result, a workgroup one cell after another; the
// matrix stays in registers (a wavefront's own rows of it in LDS), and each column tile
// of a field is loaded while the one before it is used.
//
// 4096 cells of 32 x 32 (48 x 48 fine): both kernels 245 -> 91 us (interpolation 33,
// restriction 57) against a form with the products as FP64 vector loops over LDS, which
// its LDS reads bounded (24 bytes per two FMAs). What bounds them now: the fine fields'
// traffic (54 and 109 MB, 12 and 24 us at 4.6 TB/s) and 120 matrix instructions of 64
// cycles per cell (13 us each), which four cells per workgroup overlap only in part.
// Without loading ahead the restriction took 107 us, with 2048 workgroups (two cells
// for each load of the matrix) 81.

#include <hip/hip_runtime.h>

#include <cstdint>

#include "galerkin_args.hpp"
#include "kernels_common.hpp"

namespace qcoll {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Values [16 tile + lane % 16][4 s + lane / 16] of a row-major matrix m [rows][cols]
// of 16 KT columns at most, zero outside.
template <int KT>
__device__ __forceinline__ void load_tile(const double* m, int rows, int cols, int tile, int lane,
                                          double (&x)[4 * KT]) {
  const int r = 16 * tile + (lane & 15);
#pragma unroll
  for (int s = 0; s < 4 * KT; ++s) {
    const int k = 4 * s + (lane >> 4);
    const bool in = r < rows && k < cols;
    const double v = m[in ? r * cols + k : 0];
    x[s] = in ? v : 0.0;
  }
}

// Column tile ct of a cell's field x [n][n], as load_tile holds rows.
template <int KT, class X>
__device__ __forceinline__ void load_columns(const X* x, int n, int ct, int lane, X (&col)[4 * KT]) {
  const int c = 16 * ct + (lane & 15);
#pragma unroll
  for (int s = 0; s < 4 * KT; ++s) {
    const int k = 4 * s + (lane >> 4);
    const bool in = k < n && c < n;
    const X v = x[in ? k * n + c : 0];
    col[s] = in ? v : X(0);
  }
}

// The result's rows 16 w .. 16 w + 15 of M X M^t: X is a cell's field [n][n], M is
// [m][n] (mine: its rows of tile w, in LDS, value s of lane l at 64 s + l; all: those
// of every tile); KT, MT: tiles of 16 that hold n and m. col: column tile 0 of X on
// entry, of the next cell's field on return (each tile is loaded while the one before
// it is used). out[t][v]: row 16 w + 4 v + lane / 16, column 16 t + lane % 16.
template <int KT, int MT, class X>
__device__ __forceinline__ void two_sided(const X* x, const X* next, int n, int lane, const double* mine,
                                          const double (&all)[MT][4 * KT], X (&col)[4 * KT], d4 (&out)[MT]) {
#pragma unroll
  for (int t = 0; t < MT; ++t) out[t] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ct = 0; ct < KT; ++ct) {
    X ahead[4 * KT];
    load_columns<KT>(ct + 1 < KT ? x : next, n, ct + 1 < KT ? ct + 1 : 0, lane, ahead);
    __builtin_amdgcn_sched_barrier(0);
    d4 t = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4 * KT; ++s) t = mfma(static_cast<double>(col[s]), mine[64 * s + lane], t);
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int j = 0; j < MT; ++j) out[j] = mfma(t[v], all[j][4 * ct + v], out[j]);
#pragma unroll
    for (int s = 0; s < 4 * KT; ++s) col[s] = ahead[s];
  }
}

// f_fine = I f I^T with I = interp [nf][n].
template <int CT, int RT>
__global__ __launch_bounds__(64 * RT, 2) void galerkin_interp_kernel(GalerkinArgs a) {
  const int n = a.n, nf = a.nf, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __shared__ double rows[RT][4 * CT * 64];
  double all[RT][4 * CT];
  load_tile<CT>(a.interp, nf, n, w, lane, all[0]);
#pragma unroll
  for (int s = 0; s < 4 * CT; ++s) rows[w][64 * s + lane] = all[0][s];
#pragma unroll
  for (int j = 0; j < RT; ++j) load_tile<CT>(a.interp, nf, n, j, lane, all[j]);
  const int64_t size = static_cast<int64_t>(n) * n, first = blockIdx.x;   // (grid: no more workgroups than cells)
  float col[4 * CT];
  load_columns<CT>(a.f + first * size, n, 0, lane, col);
  for (int64_t cell = first; cell < a.cells; cell += gridDim.x) {
    d4 out[RT];
    const int64_t next = cell + gridDim.x < a.cells ? cell + gridDim.x : cell;
    two_sided<CT, RT>(a.f + cell * size, a.f + next * size, n, lane, rows[w], all, col, out);
    float* ff = a.f_fine + cell * static_cast<int64_t>(nf) * nf;
#pragma unroll
    for (int j = 0; j < RT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * w + 4 * v + (lane >> 4), c = 16 * j + (lane & 15);
        if (r < nf && c < nf) ff[r * nf + c] = static_cast<float>(out[j][v]);
      }
  }
}

// Q = R Q_fine R^T with R = restrict_ [n][nf]; then the FP64 projection onto
// the complement of (1, v, |v|^2) on the n grid when conserve is set.
template <int CT, int RT>
__global__ __launch_bounds__(64 * CT, CT > 2 ? 1 : 2) void galerkin_restrict_kernel(GalerkinArgs a) {
  __shared__ double red[2][CT][4];
  const int n = a.n, nf = a.nf, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __shared__ double rows[CT][4 * RT * 64];
  double all[CT][4 * RT];
  load_tile<RT>(a.restrict_, n, nf, w, lane, all[0]);
#pragma unroll
  for (int s = 0; s < 4 * RT; ++s) rows[w][64 * s + lane] = all[0][s];
#pragma unroll
  for (int j = 0; j < CT; ++j) load_tile<RT>(a.restrict_, n, nf, j, lane, all[j]);
  const int64_t size = static_cast<int64_t>(nf) * nf, first = blockIdx.x;   // (grid: no more workgroups than cells)
  double col[4 * RT];
  load_columns<RT>(a.q_fine + first * size, nf, 0, lane, col);
  int turn = 0;   // the half of `red` that no wavefront may still be reading
  for (int64_t cell = first; cell < a.cells; cell += gridDim.x, turn ^= 1) {
    d4 out[CT];
    const int64_t next = cell + gridDim.x < a.cells ? cell + gridDim.x : cell;
    two_sided<RT, CT>(a.q_fine + cell * size, a.q_fine + next * size, nf, lane, rows[w], all, col, out);
    const int64_t base = cell * static_cast<int64_t>(n) * n;
    if (!a.conserve) {
      float* Qo = reinterpret_cast<float*>(a.q) + base;
#pragma unroll
      for (int j = 0; j < CT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * w + 4 * v + (lane >> 4), c = 16 * j + (lane & 15);
          if (r < n && c < n) Qo[r * n + c] = static_cast<float>(out[j][v]);
        }
      continue;
    }
    double m[4] = {0, 0, 0, 0};   // (rows and columns from n on are zero)
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double v1 = -a.L + a.dv * (16 * w + 4 * v + (lane >> 4)), v2 = -a.L + a.dv * (16 * j + (lane & 15));
        const double q = out[j][v];
        m[0] += q;
        m[1] += v1 * q;
        m[2] += v2 * q;
        m[3] += (v1 * v1 + v2 * v2) * q;
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) m[i] = wave_sum(m[i]);
    if constexpr (CT > 1) {
      if (lane == 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[turn][w][i] = m[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        m[i] = red[turn][0][i];
#pragma unroll
        for (int k = 1; k < CT; ++k) m[i] += red[turn][k][i];
      }
    }
    double lam[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      lam[i] = a.gram_inv[i * 4 + 0] * m[0] + a.gram_inv[i * 4 + 1] * m[1] + a.gram_inv[i * 4 + 2] * m[2] +
               a.gram_inv[i * 4 + 3] * m[3];
    double* Qo = reinterpret_cast<double*>(a.q) + base;
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * w + 4 * v + (lane >> 4), c = 16 * j + (lane & 15);
        const double v1 = -a.L + a.dv * r, v2 = -a.L + a.dv * c;
        if (r < n && c < n) Qo[r * n + c] = out[j][v] - (lam[0] + lam[1] * v1 + lam[2] * v2 + lam[3] * (v1 * v1 + v2 * v2));
      }
  }
}

template <int CT, int RT>
int launch_tiles(const GalerkinArgs& args, bool restriction, hipStream_t stream) {
  // four workgroups per compute unit, up to 16 points eight (4096 cells of 16 points:
  // 247 us for the call with four, 239 with eight)
  constexpr int64_t kMax = CT == 1 ? 2048 : 1024;
  const unsigned blocks = static_cast<unsigned>(args.cells < kMax ? args.cells : kMax);
  if (restriction)
    hipLaunchKernelGGL((galerkin_restrict_kernel<CT, RT>), dim3(blocks), dim3(64 * CT), 0, stream, args);
  else
    hipLaunchKernelGGL((galerkin_interp_kernel<CT, RT>), dim3(blocks), dim3(64 * RT), 0, stream, args);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// Tiles of 16 that hold n and nf = 3 n / 2 (n up to 40).
int launch_galerkin(const GalerkinArgs& args, bool restriction, hipStream_t stream) {
  if (args.cells <= 0) return 0;
  const int ct = (args.n + 15) / 16, rt = (args.nf + 15) / 16;
  if (ct == 1 && rt == 1) return launch_tiles<1, 1>(args, restriction, stream);
  if (ct == 1 && rt == 2) return launch_tiles<1, 2>(args, restriction, stream);
  if (ct == 2 && rt == 2) return launch_tiles<2, 2>(args, restriction, stream);
  if (ct == 2 && rt == 3) return launch_tiles<2, 3>(args, restriction, stream);
  if (ct == 3 && rt == 4) return launch_tiles<3, 4>(args, restriction, stream);
  return -1;
}

}  // namespace

int launch_galerkin_interp(const GalerkinArgs& args, hipStream_t stream) {
  return launch_galerkin(args, false, stream);
}

int launch_galerkin_restrict(const GalerkinArgs& args, hipStream_t stream) {
  return launch_galerkin(args, true, stream);
}

}  // namespace qcoll
