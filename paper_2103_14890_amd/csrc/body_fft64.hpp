// Per-cell body of the 2D FX16 plans on grids of N = 4 R points per axis, R = 9
// .. 16 (36, 40, .. 64): one workgroup of four wavefronts per cell, FP64 FFTs in
// registers. Shared by the single-plan and the batched kernels; the dataflow is
// that of body_fft.hpp.
//
// A thread holds R points at a time (a whole 64-point line would take 256
// registers). A 2D transform is three register steps with two exchanges of the
// field through LDS:
//   1. wavefront n0 = k2 mod 4, lane = row k1: R-point FFT over k2 = 4 n1 + n0,
//      times w^(n0 k0) (the same for the whole wavefront: scalar operands);
//   2. thread (k0, r0): 4 x 4 points, the 4-point FFT over n0 -> columns
//      y = k0 + R j, and the 4-point FFT over k1 = r0 + R i -> a, times w^(r0 a)
//      (three roots per lane, held in registers);
//   3. wavefront a, lane = column y: R-point FFT over r0 -> rows x = a + 4 b.
// The forward transform of f is the same flow backwards. The spectrum stays in
// the registers of step 1 and the gain in those of step 3, so a transform moves
// four fields through LDS (two written, two read) and its filter from L2. The
// filters are even, m(-k) = m(k): wavefront 3 reads the entries of wavefront 1
// with rows and registers reversed, which leaves three quarters of the table.
//
// What bounds it: FP64 vector issue and the LDS exchanges, in about equal parts
// (64 points, per transform and thread: 160 + 60 FFT and twiddle instructions in
// step 1, 176 in step 2, 160 in step 3, 64 for the filter, 16 for the gain; 256
// KB of LDS traffic per cell and transform, 2048 cycles of a CU's LDS). Two cells
// per CU (67 KB of LDS, 256 registers) overlap the one with the other. 4000 cells
// of 64 x 64 (hard spheres, M = 8): 0.96 ms, the split-FP16 matrix form 1.32 ms; 48
// x 48: 0.66 and 1.23 ms.
#pragma once

#include "fft_reg.hpp"
#include "kernels_common.hpp"

namespace qcoll {
namespace {

template <int R>
struct Fft64 {
  static constexpr int N = 4 * R, S = N + 1;               // LDS row stride (odd: column access without conflicts)
  static constexpr int kField = 4 * R * S;                 // complex values
  static constexpr int kLdsBytes = kField * 16 + 32 * 8;   // and the reduction slots
};

// Sum over the workgroup of K values per thread, in wavefront order.
template <int K>
__device__ __forceinline__ void block_sum4(double* x, double* red) {
#pragma unroll
  for (int i = 0; i < K; ++i) x[i] = wave_sum(x[i]);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int i = 0; i < K; ++i) red[w * 4 + i] = x[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < K; ++i) x[i] = red[i] + red[4 + i] + red[8 + i] + red[12 + i];
}

// Grid sizes 4 R with a body.
#define QCOLL_FFT64_SIZES(X) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

// Epilogue: float Q, single-stage update, or (single-plan launches only, SINGLE) RK
// stage; the plans of these kernels have neither the projection nor a Galerkin grid.
// Thread (w, lane) holds rows w + 4 b of column `lane`. Whole rows are stored at a
// time; results and stage slots are streamed past the L2 (non-temporal), so that they
// do not evict the filters that all cells share.
template <int R, bool SINGLE>
__device__ __forceinline__ void finish_rows(const KernelArgs& a, int64_t cell, double (&q)[R], int w, double* red) {
  constexpr int N = 4 * R;
  int lane = threadIdx.x & 63;
  // per-cell addresses and velocities, not hoisted out of the cell loop
  asm volatile("" : "+v"(lane), "+s"(w) : "v"(q[0]));
  const bool in = lane < N;
  const int c = in ? lane : 0;
  const int64_t base = cell * static_cast<int64_t>(N * N);
  const int kind = a.out_kind;
  if (kind == 0) {
    float* Qc = reinterpret_cast<float*>(a.q) + base;
    if (in)
#pragma unroll
      for (int b = 0; b < R; ++b) __builtin_nontemporal_store(static_cast<float>(q[b]), &Qc[(w + 4 * b) * N + c]);
    return;
  }
  const double v2 = -a.L + a.dv * c;
  auto v1 = [&](int b) { return -a.L + a.dv * (w + 4 * b); };
  const float* fc = a.f + base;
  float fv[R];
#pragma unroll
  for (int b = 0; b < R; ++b) {
    const float x = fc[(w + 4 * b) * N + c];
    fv[b] = in ? x : 0.0f;
  }
  int bad = 0;
  bool last = true;
  if (SINGLE && (kind == 3 || kind == 5)) {
    // stage l of the penalised IMEX RK step (finish_cell<3>); fv holds F_{l-1}, q its Q
    int sch = a.rk_scheme - 1, l = a.rk_stage;
    asm volatile("" : "+s"(sch), "+s"(l));   // the tableau is read here, per cell
    const int St = sch == 0 ? 3 : 5;
    const bool both = kind == 5;   // the last two stages of BPR(3,4,3)
    last = l == St || both;
    const double* At5 = kRkAt[1][4];
    const double* Dd5 = kRkD[1][4];
    const double A55 = kRkA[1][4][4];
    const double* At = kRkAt[sch][l - 1];
    const double* Ai = kRkA[sch][l - 1];
    const double* Dd = kRkD[sch][l - 1];
    float* fnp = a.rk_fn + base;
    // moments of f^n: summed by stage 2, whose input is f^n, kept for the later stages
    double s[4] = {0, 0, 0, 0};
    double* mp = a.rk_mom + cell * 4;
    if (l == 2) {
#pragma unroll
      for (int b = 0; b < R; ++b) {
        const double x = static_cast<double>(fv[b]);
        s[0] += x;
        s[1] += v1(b) * x;
        s[2] += v2 * x;
        s[3] += (v1(b) * v1(b) + v2 * v2) * x;
      }
      block_sum4<4>(s, red);
      if (threadIdx.x < 4) mp[threadIdx.x] = red[threadIdx.x] + red[4 + threadIdx.x] + red[8 + threadIdx.x] + red[12 + threadIdx.x];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] = mp[i];
    }
    const double rho = s[0] * a.dv * a.dv, u1 = s[1] / s[0], u2 = s[2] / s[0];
    const double Tm = 0.5 * (s[3] / s[0] - u1 * u1 - u2 * u2);
    const double nu = rho, k = a.dt_eps;
    const double cM = rho / (2.0 * 3.14159265358979323846 * Tm);
    const double rden = 1.0 / (1.0 + Ai[l - 1] * k * nu), rden5 = 1.0 / (1.0 + A55 * k * nu);
    const double* ec = exp_consts();
    const double e2 = exp_nonpos(-(v2 - u2) * (v2 - u2) / (2.0 * Tm), ec);
    const double vr = -a.L + a.dv * (w + 4 * (lane % R));   // the factor of row w + 4 (lane mod R)
    const double e1 = exp_nonpos(-(vr - u1) * (vr - u1) / (2.0 * Tm), ec);
#pragma unroll
    for (int b = 0; b < R; ++b) {
      const int o = (w + 4 * b) * N + c;
      const double fnv = static_cast<double>(fnp[o]);
      const double M = cM * __shfl(e1, b) * e2;
      double t1 = Ai[l - 1] * M, t2 = 0.0, w1 = A55 * M, w2 = 0.0;
#pragma unroll
      for (int m = 1; m <= 4; ++m) {
        if (m >= l) break;   // uniform
        const double Fm = m == 1 ? fnv
                          : (m == l - 1 ? static_cast<double>(fv[b])
                                        : static_cast<double>(__builtin_nontemporal_load(&a.rk_work[(m - 2) * a.rk_stride + base + o])));
        t1 += Dd[m - 1] * (M - Fm);
        if (both) w1 += Dd5[m - 1] * (M - Fm);
        if (At[m - 1] != 0.0) {   // (the same terms in stages 4 and 5 of BPR(3,4,3))
          const double Qm =
              m == l - 1 ? q[b] : static_cast<double>(__builtin_nontemporal_load(&a.rk_work[(St - 3 + m) * a.rk_stride + base + o]));
          t2 += At[m - 1] * Qm;
          if (both) w2 += At5[m - 1] * Qm;
        }
      }
      float Fl = static_cast<float>((fnv + k * (nu * t1 + t2)) * rden);
      if (both) Fl = static_cast<float>((fnv + k * (nu * (w1 + Dd5[3] * (M - static_cast<double>(Fl))) + w2)) * rden5);
      if (!in) continue;
      if (last) {
        bad |= !(fabsf(Fl) <= 3.0e38f);
        __builtin_nontemporal_store(Fl, &fnp[o]);
      } else {
        __builtin_nontemporal_store(Fl, &a.rk_work[(l - 2) * a.rk_stride + base + o]);
        __builtin_nontemporal_store(static_cast<float>(q[b]), &a.rk_work[(St - 3 + (l - 1)) * a.rk_stride + base + o]);
      }
    }
  } else {   // kind 2: single-stage update in place
    double rho[1] = {0.0};
#pragma unroll
    for (int b = 0; b < R; ++b) rho[0] += static_cast<double>(fv[b]);
    block_sum4<1>(rho, red);
    const double k = a.scheme == 1 ? a.dt_eps / (1.0 + a.dt_eps * (rho[0] * a.dv * a.dv)) : a.dt_eps;
    float* fw = const_cast<float*>(a.f) + base;
#pragma unroll
    for (int b = 0; b < R; ++b) {
      const float nv = static_cast<float>(static_cast<double>(fv[b]) + k * q[b]);
      if (!in) continue;
      bad |= !(fabsf(nv) <= 3.0e38f);
      __builtin_nontemporal_store(nv, &fw[(w + 4 * b) * N + c]);
    }
  }
  if (last && a.status) {
    double n[1] = {0.0};
    n[0] = __any(bad) ? 1.0 : 0.0;
    __syncthreads();
    if (lane == 0) red[16 + w] = n[0];
    __syncthreads();
    if (threadIdx.x == 0) a.status[cell] = red[16] + red[17] + red[18] + red[19] > 0.0 ? 1 : 0;
  }
}

// Work items first, first + stride, ...: a cell, or with a.split = S > 1 part
// i mod S of cell i / S. Part p takes the transforms p, p + S, ... of the list
// (loss, gain 0, gain 1, ...), leaves its sums in a.split_ws and counts itself on
// the cell's counter; the workgroup that arrives last adds the parts in order and
// runs the epilogue. No workgroup waits for another.
template <int R, bool SINGLE>
__device__ __forceinline__ void fft64_body(const KernelArgs& a, int64_t first, int64_t stride, double2* lds) {
  using F = Fft64<R>;
  constexpr int N = F::N, S = F::S;
  double* red = reinterpret_cast<double*>(lds + F::kField);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int parts = a.split;
  constexpr int kPer = (R * R + 3) / 4;   // step-2 threads per wavefront
  for (int64_t item = first; item < a.cells * parts; item += stride) {
    const int64_t cell = parts > 1 ? item / parts : item;
    const int part = parts > 1 ? static_cast<int>(item - cell * parts) : 0;
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int c = lane < N ? lane : N - 1;
    const int p2 = w * kPer + lane;
    const bool on2 = R == 16 || (lane < kPer && p2 < R * R);
    const int k0 = on2 ? p2 / R : 0, r0 = on2 ? p2 % R : 0;
    const float* fc = a.f + cell * static_cast<int64_t>(N * N);
    const double* twu = a.tw + w * 32;                                  // w^(w j), j < R
    double fr[R], fi[R];
    // ---- forward
    {
#pragma unroll
      for (int b = 0; b < R; ++b) {
        fr[b] = static_cast<double>(fc[(w + 4 * b) * N + c]);
        fi[b] = 0.0;
      }
      dft<R, -1>(fr, fi);
      __syncthreads();   // the previous cell's last reads
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const double cj = twu[2 * j], sj = -twu[2 * j + 1];
        if (lane < N)
          lds[(w * R + j) * S + lane] = make_double2(fma(cj, fr[j], -(sj * fi[j])), fma(cj, fi[j], sj * fr[j]));
      }
      __syncthreads();
      double yr[4][4], yi[4][4];   // [a][j]
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double2 z = lds[(i * R + r0) * S + k0 + R * j];
          yr[i][j] = z.x;
          yi[i][j] = z.y;
        }
      __syncthreads();
      {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          double br[4] = {yr[0][j], yr[1][j], yr[2][j], yr[3][j]}, bi[4] = {yi[0][j], yi[1][j], yi[2][j], yi[3][j]};
          dft<4, -1>(br, bi);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            yr[i][j] = br[i];
            yi[i][j] = bi[i];
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          dft<4, -1>(yr[i], yi[i]);
#pragma unroll
          for (int n0 = 0; n0 < 4; ++n0) {
            const double cj = a.tw[(n0 * 16 + k0) * 2], sj = -a.tw[(n0 * 16 + k0) * 2 + 1];
            const double2 z = make_double2(fma(cj, yr[i][n0], -(sj * yi[i][n0])), fma(cj, yi[i][n0], sj * yr[i][n0]));
            if (on2) lds[(n0 * R + k0) * S + r0 + R * i] = z;
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const double2 z = lds[(w * R + j) * S + c];
        fr[j] = z.x;
        fi[j] = z.y;
      }
      dft<R, -1>(fr, fi);
    }
    double tc[3], ts[3];   // w^(r0 a), a = 1 .. 3
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      tc[i] = a.tw[((i + 1) * 16 + r0) * 2];
      ts[i] = a.tw[((i + 1) * 16 + r0) * 2 + 1];
    }
    double gain[R];
#pragma unroll
    for (int b = 0; b < R; ++b) gain[b] = 0.0;
    // this wavefront's rows of the filter table [entry][k2 class 0, 1, 2][n1][64]
    const int64_t entry = 3 * R * 64;
    const double2* ft = reinterpret_cast<const double2*>(a.filt) + (w < 3 ? w * R : R + R - 1) * 64;
    const int row = w < 3 ? 64 : -64;
    const unsigned lx = w < 3 ? lane : (lane == 0 ? 0 : (lane < N ? N - lane : 0));
#pragma unroll 1
    for (int e = part; e <= a.P; e += parts) {
      const int q = e == 0 ? a.P : e - 1;
      double zr[R], zi[R];
      {
        const double2* m = ft + q * entry;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const double2 mv = m[j * row + static_cast<int>(lx)];
          zr[j] = fma(mv.x, fr[j], -(mv.y * fi[j]));
          zi[j] = fma(mv.x, fi[j], mv.y * fr[j]);
        }
      }
      dft<R, 1>(zr, zi);
      const double* tu = twu;
      asm volatile("" : "+s"(tu));   // scalar loads here, not scalar registers held through the loop
      __syncthreads();               // the field has been read
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const double cj = tu[2 * j], sj = tu[2 * j + 1];
        const double2 z = j == 0 ? make_double2(zr[0], zi[0])
                                 : make_double2(fma(cj, zr[j], -(sj * zi[j])), fma(cj, zi[j], sj * zr[j]));
        if (lane < N) lds[(w * R + j) * S + lane] = z;
      }
      __syncthreads();
      double yr[4][4], yi[4][4];   // [n0][i]
#pragma unroll
      for (int n0 = 0; n0 < 4; ++n0)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double2 z = lds[(n0 * R + k0) * S + r0 + R * i];
          yr[n0][i] = z.x;
          yi[n0][i] = z.y;
        }
      __syncthreads();
      {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          double br[4] = {yr[0][i], yr[1][i], yr[2][i], yr[3][i]}, bi[4] = {yi[0][i], yi[1][i], yi[2][i], yi[3][i]};
          dft<4, 1>(br, bi);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            yr[j][i] = br[j];
            yi[j][i] = bi[j];
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {   // column y = k0 + R j
          dft<4, 1>(yr[j], yi[j]);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double cj = i ? tc[i - 1] : 1.0, sj = i ? ts[i - 1] : 0.0;
            const double2 z = i == 0 ? make_double2(yr[j][0], yi[j][0])
                                     : make_double2(fma(cj, yr[j][i], -(sj * yi[j][i])), fma(cj, yi[j][i], sj * yr[j][i]));
            if (on2) lds[(i * R + r0) * S + k0 + R * j] = z;
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const double2 z = lds[(w * R + j) * S + c];
        zr[j] = z.x;
        zi[j] = z.y;
      }
      dft<R, 1>(zr, zi);
      if (e == 0) {   // the loss field: -f L
#pragma unroll
        for (int b = 0; b < R; ++b) gain[b] = fma(-static_cast<double>(fc[(w + 4 * b) * N + c]), zr[b], gain[b]);
      } else {
#pragma unroll
        for (int b = 0; b < R; ++b) gain[b] = fma(zr[b], zi[b], gain[b]);
      }
    }
    if (parts > 1) {
      double* mine = a.split_ws + ((cell * parts + part) * 4 + w) * 1024;
#pragma unroll
      for (int b = 0; b < R; ++b) mine[b * 64 + lane] = gain[b];
      __threadfence();   // the part is visible device-wide before it is counted
      __syncthreads();
      if (threadIdx.x == 0) red[20] = atomicAdd(&a.split_cnt[cell], 1) == parts - 1 ? 1.0 : 0.0;
      __syncthreads();
      if (red[20] == 0.0) continue;   // workgroup-uniform
      __threadfence();   // the other parts' results are read after their counts
#pragma unroll
      for (int b = 0; b < R; ++b) gain[b] = 0.0;
      for (int j = 0; j < parts; ++j) {
        const double* pj = a.split_ws + ((cell * parts + j) * 4 + w) * 1024;
#pragma unroll
        for (int b = 0; b < R; ++b) gain[b] += pj[b * 64 + lane];
      }
      if (threadIdx.x == 0) a.split_cnt[cell] = 0;   // zero for the next launch
    }
    finish_rows<R, SINGLE>(a, cell, gain, w, red);
  }
}

}  // namespace
}  // namespace qcoll
