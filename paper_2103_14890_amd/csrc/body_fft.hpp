// Per-cell body of the 2D FX16 plans on grids of up to 32 points per axis: one
// wavefront per cell, FP64 FFTs in registers. Shared by the single-plan and the
// batched kernels.
//
// Dataflow (section 3.3): forward DFT of f -> f_hat; for every packed filter
// m_q the inverse DFT of m_q f_hat, whose real and imaginary parts are the two
// real fields g and h of a pair of directions (their product is the gain
// contribution); the inverse DFT of l f_hat is the loss field; Q = gain - f L.
//
// A lane holds one whole line of a transform (N complex values), so that both
// 1-D passes of a transform are register FFTs and one transposition through LDS
// between them is the only exchange. A line needs G = 16 or 32 lanes' worth of
// lines, so a wavefront runs T = 64 / G transforms at a time, transform slot t on
// lanes t G .. t G + G - 1; the slots' gain sums are added once per cell.
//
// The filters are real-even pairs, m(-k) = m(k), and f_hat(-k) is the conjugate
// of f_hat(k): a lane of a row k1 < 0 computes the conjugate of its row from the
// entries of row -k1 (with conj m), and the reader of the transposition takes
// conjugates of those rows (a sign folded into the second pass). So the filter
// table and the spectrum hold half of the rows.
//
// What bounds it: FP64 vector issue. Per pair of 32-point transforms a lane issues
// 930 FP64 instructions (2 x 387 FFT, 124 filter, 32 gain), 64 lane swaps and 31
// sign flips, against about 1660 vector instructions and 192 MFMAs of the
// split-FP16 matrix form. 4096 cells of 32 x 32 (hard spheres, M = 8) take 54.5 M
// wavefront instructions, 117-128 us at the 2.2-2.4 ns per instruction that two
// wavefronts on a SIMD reach; measured 140 us, the matrix form 216 us.
#pragma once

#include "fft_reg.hpp"
#include "kernels_common.hpp"

namespace qcoll {
namespace {

// Swap the odd 16-lane rows (the upper 32 lanes) of a with the even rows (the
// lower 32 lanes) of b.
__device__ __forceinline__ void swap16(double& a, double& b) {
  const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(x), static_cast<unsigned>(y), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(x >> 32), static_cast<unsigned>(y >> 32),
                                                   false, false);
  a = __hiloint2double(static_cast<int>(hi[0]), static_cast<int>(lo[0]));
  b = __hiloint2double(static_cast<int>(hi[1]), static_cast<int>(lo[1]));
}
__device__ __forceinline__ void swap32(double& a, double& b) {
  const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap(static_cast<unsigned>(x), static_cast<unsigned>(y), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(static_cast<unsigned>(x >> 32), static_cast<unsigned>(y >> 32),
                                                   false, false);
  a = __hiloint2double(static_cast<int>(hi[0]), static_cast<int>(lo[0]));
  b = __hiloint2double(static_cast<int>(hi[1]), static_cast<int>(lo[1]));
}

// Flip the sign of x where `mask` has the sign bit.
__device__ __forceinline__ double flip(double x, int mask) {
  return __hiloint2double(__double2hiint(x) ^ mask, __double2loint(x));
}

template <int NN>
struct FftGrid {
  static constexpr int G = NN > 16 ? 32 : 16;        // lanes per transform
  static constexpr int T = 64 / G;                   // transforms at a time
  static constexpr int H = NN / 2 + 1;               // rows kept of the spectrum and the filters (k1 = 0 .. N/2)
  // The transposition goes through LDS one real component at a time; above 28
  // points also 16 registers at a time (a 2 x 2 block swap between registers
  // and lanes first), so that eight wavefronts fit a CU's 160 KB.
  static constexpr bool CHUNK = NN > 28;
  static constexpr int XS = CHUNK ? 65 : T * NN + 1; // odd: the column reads fall on distinct banks
  static constexpr int XD = (CHUNK ? 16 : NN) * XS;
  // the layout of the epilogue: slot t holds rows t V .. t V + V - 1 of its column
  static constexpr int N = G, V = (NN + T - 1) / T;
  __device__ static int row(int v, int lane) { return V * (lane / G) + v; }
  __device__ static int col(int lane) { return lane & (G - 1); }
  static constexpr int kFh = 2 * NN * H;             // doubles
  static constexpr int kWaveBytes = ((kFh + (XD > V * 64 ? XD : V * 64)) * 8 + 15) / 16 * 16;
};

template <int NN, int W>
constexpr int fft_round_bytes() {
  using F = FftGrid<NN>;
  return (F::kFh + NN * 64 + 2 + W * F::XD) * 8;
}

// Transpose within each transform slot: lane r holds line r, register v its
// point v; afterwards lane c holds point c of every line, register = line.
template <int NN>
__device__ __forceinline__ void transpose(double (&x)[NN], double* buf, int lane) {
  using F = FftGrid<NN>;
  const int t = lane / F::G, r = lane & (F::G - 1);
  if constexpr (F::CHUNK) {
    double y[32];
#pragma unroll
    for (int v = 0; v < 32; ++v) y[v] = v < NN ? x[v] : 0.0;
    // 2 x 2 blocks: afterwards lane (t, rb, r0), register (c1, c0) holds line
    // 16 c1 + r0, point 16 rb + c0
#pragma unroll
    for (int v = 0; v < 16; ++v) swap16(y[v], y[v + 16]);
    const int rd = (r & 15) * F::XS + 32 * t + (r & 16);
#pragma unroll
    for (int c1 = 0; c1 < 2; ++c1) {
#pragma unroll
      for (int v = 0; v < 16; ++v) buf[v * F::XS + lane] = y[16 * c1 + v];
      lds_fence();
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (16 * c1 + j < NN) x[16 * c1 + j] = buf[rd + j];
      lds_fence();
    }
  } else {
    const int wr = r < NN ? t * NN + r : F::T * NN;
    const int rd = (r < NN ? r : 0) * F::XS + t * NN;
#pragma unroll
    for (int v = 0; v < NN; ++v) buf[v * F::XS + wr] = x[v];
    lds_fence();
#pragma unroll
    for (int j = 0; j < NN; ++j) x[j] = buf[rd + j];
    lds_fence();
  }
}

// The epilogue of an output kind chosen at run time: float Q, single-stage update, or
// (single-plan launches only) RK stage; the plans of these kernels have neither the
// projection nor a Galerkin grid.
template <class LY, bool SINGLE>
__device__ __forceinline__ void finish_any(const KernelArgs& a, int64_t cell, const float* fv, double* q, int lane) {
  if (a.out_kind == 0) finish_cell<0, LY>(a, cell, fv, q, lane);
  else if (!SINGLE || a.out_kind == 2) finish_cell<2, LY>(a, cell, fv, q, lane);
  else if constexpr (SINGLE) {
    if (a.out_kind == 3) finish_cell<3, LY>(a, cell, fv, q, lane);
    else finish_cell<5, LY>(a, cell, fv, q, lane);
  }
}

// Cells first, first + stride, ... (per wavefront). lds: this wavefront's
// FftGrid<NN>::kWaveBytes. With `split` (wavefront-uniform) the four wavefronts
// of a workgroup share each cell's transforms: every wavefront computes the
// spectrum, wavefront wv takes the groups of T transforms wv, wv + 4, ...; the
// partial sums meet in LDS and wavefront 0 adds them in the order 0, 1, 2, 3.
//
// W > 0, few cells: the W wavefronts of a workgroup take the groups of a cell in turn
// and add to one gain in LDS, group after group, so the results are bitwise those of
// one wavefront per cell. lds: the workgroup's fft_round_bytes<NN, W>.
template <int NN, bool SINGLE, int W = 0>
__device__ __forceinline__ void fft_body(const KernelArgs& a, int64_t first, int64_t stride, bool split, int wv,
                                         double* lds) {
  using F = FftGrid<NN>;
  constexpr int G = F::G, T = F::T, H = F::H, V = F::V;
  double2* fh = reinterpret_cast<double2*>(lds);   // f_hat[k2][k1], k1 = 0 .. N/2
  double* acc = lds + F::kFh;                      // W > 0: the gain, [v][lane], and the group whose turn it is
  int* turn = reinterpret_cast<int*>(acc + NN * 64);
  double* buf = W > 0 ? acc + NN * 64 + 2 + wv * F::XD : lds + F::kFh;
  const int g0 = split ? wv : 0, gs = split ? 4 : 1;
  for (int64_t cell = first; cell < a.cells; cell += stride) {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int t = lane / G, r = lane & (G - 1);
    const int c = r < NN ? r : 0;
    const float* fc = a.f + cell * static_cast<int64_t>(NN * NN);
    double xr[NN], xi[NN];
    auto load_f64 = [&] {
#pragma unroll
      for (int v = 0; v < NN; ++v) {
        xr[v] = static_cast<double>(fc[v * NN + c]);
        xi[v] = 0.0;
      }
    };
    if constexpr (W == 0) {
      // ---- forward: along axis 0 (lane = column), transpose, along axis 1 (lane = row k1)
      load_f64();
      // Above 16 points the conjugate, by the inverse transform, with zeros that the
      // compiler does not fold: the form with W > 0 runs these very instructions, rounding
      // for rounding.
      constexpr int SG = NN > 16 ? 1 : -1;
      if constexpr (SG > 0) {
#pragma unroll
        for (int v = 0; v < NN; ++v) asm volatile("" : "+v"(xi[v]));
      }
      dft<NN, SG>(xr, xi);
      transpose<NN>(xr, buf, lane);
      transpose<NN>(xi, buf, lane);
      dft<NN, SG>(xr, xi);
      if (lane < H) {
#pragma unroll
        for (int v = 0; v < NN; ++v) fh[v * H + lane] = make_double2(xr[v], SG > 0 ? -xi[v] : xi[v]);
      }
      lds_fence();
    }

    double gain[NN];
#pragma unroll
    for (int v = 0; v < NN; ++v) gain[v] = 0.0;
    const int kap = r < H ? r : (r < NN ? NN - r : 0);                       // the row's partner in 0 .. N/2
    const int neg = (r >= H && r < NN) ? static_cast<int>(0x80000000u) : 0;  // conjugate row
    // The filter values of a group come from L2 at once, the spectrum from LDS one
    // batch of four ahead of its use (the scheduling barriers keep the batches apart:
    // all loads together would spill the gain).
    constexpr int B = 4, NB = (NN + B - 1) / B;
    double2 m[NB][B];
    auto load_m = [&](int b, int g) {
      const int q = g * T + t;
      const unsigned off = static_cast<unsigned>(((q < a.P ? q : a.P) * (NN * H) + kap) * 16);
      const char* ft = reinterpret_cast<const char*>(a.filt);
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const int v = b * B + j;
        if (v < NN && v != NN / 2) m[b][j] = *reinterpret_cast<const double2*>(ft + v * H * 16 + off);
      }
    };
    // the spectrum times the filters of group g
    auto filter = [&](int g) {
      double2 z[NB][B];
      auto load_z = [&](int b) {
#pragma unroll
        for (int j = 0; j < B; ++j) {
          const int v = b * B + j;
          if (v < NN && v != NN / 2) z[b][j] = fh[v * H + kap];
        }
      };
#pragma unroll
      for (int b = 0; b < NB; ++b) load_m(b, g);
      load_z(0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if (b + 1 < NB) load_z(b + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < B; ++j) {
          const int v = b * B + j;
          if (v >= NN) continue;
          if (v == NN / 2) {   // no Nyquist content in any filter
            xr[v] = xi[v] = 0.0;
            continue;
          }
          const double my = flip(m[b][j].y, neg);
          xr[v] = fma(m[b][j].x, z[b][j].x, -(my * z[b][j].y));
          xi[v] = fma(m[b][j].x, z[b][j].y, my * z[b][j].x);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto transform = [&](int g) {
      filter(g);
      dft<NN, 1>(xr, xi);
      transpose<NN>(xr, buf, lane);
      transpose<NN>(xi, buf, lane);
#pragma unroll
      for (int v = H; v < NN; ++v) xi[v] = -xi[v];
      dft<NN, 1>(xr, xi);
    };
    const int full = a.P / T;   // groups of gain transforms only; the group after them ends with the loss
    int g = g0;
    if constexpr (W > 0) {
      // The forward transform (its conjugate: the inverse transform of real values) goes
      // through the loop as well: few cells run each piece of code a few times, and the
      // instructions fetched for it would take as long as the transform (one cell of 24
      // points, hard spheres, M = 8: 17.8 us with a forward transform of its own, 14.4 so;
      // with many wavefronts per SIMD the shared loop is 7 % slower).
      g = -1;
#pragma unroll 1
      for (;;) {
        if (g < 0) load_f64();
        else filter(g);
        const int sign = g < 0 ? 0 : static_cast<int>(0x80000000u);
        dft<NN, 1>(xr, xi);
        transpose<NN>(xr, buf, lane);
        transpose<NN>(xi, buf, lane);
#pragma unroll
        for (int v = H; v < NN; ++v) xi[v] = flip(xi[v], sign);
        dft<NN, 1>(xr, xi);
        if (g < 0) {
          if (lane < H && wv == 0) {
#pragma unroll
            for (int v = 0; v < NN; ++v) fh[v * H + lane] = make_double2(xr[v], -xi[v]);
          }
          if (threadIdx.x == 0) *turn = 0;
          __syncthreads();
          g = wv;
          if (g > full) break;
          continue;
        }
        // The turn of a group is over when its wavefront has added it; the wavefronts of
        // a workgroup are resident together, so every wait ends.
        while (__hip_atomic_load(turn, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != g) __builtin_amdgcn_s_sleep(1);
        if (g > 0) {
#pragma unroll
          for (int v = 0; v < NN; ++v) gain[v] = acc[v * 64 + lane];
        } else {
#pragma unroll
          for (int v = 0; v < NN; ++v) gain[v] = 0.0;
        }
        if (g == full) break;
#pragma unroll
        for (int v = 0; v < NN; ++v) acc[v * 64 + lane] = fma(xr[v], xi[v], gain[v]);
        __hip_atomic_store(turn, g + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        g += W;
        if (g > full) break;
      }
    } else {
#pragma unroll 1
      for (; g < full; g += gs) {
        transform(g);
#pragma unroll
        for (int v = 0; v < NN; ++v) gain[v] = fma(xr[v], xi[v], gain[v]);
      }
    }
    if (g == full) {   // wavefront-uniform
      if constexpr (W == 0) transform(full);
      const int q = full * T + t;
      const bool is_gain = q < a.P, is_loss = q == a.P;   // (neither: an idle slot)
      constexpr int C = 8;
      float fl[2][C];
      auto load_f = [&](int b) {
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const int v = b * C + j;
          if (v < NN) fl[b & 1][j] = fc[v * NN + c];
        }
      };
      load_f(0);
#pragma unroll
      for (int b = 0; b * C < NN; ++b) {
        if ((b + 1) * C < NN) load_f(b + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const int v = b * C + j;
          if (v >= NN) continue;
          asm volatile("" : "+v"(fl[b & 1][j]));   // loaded by every lane, selected below
          const double x = is_loss ? -static_cast<double>(fl[b & 1][j]) : 0.0;
          gain[v] = fma(xr[v], is_gain ? xi[v] : x, gain[v]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // The cell's values for the epilogue are on their way while the slots are added.
    const bool ends = W > 0 ? g == full : !split || wv == 0;
    float fv[V];
    if (ends && (a.out_kind == 2 || a.out_kind == 3 || a.out_kind == 5)) {
      load_cell<F>(a, cell, lane, fv, static_cast<float>(gain[0]));
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) fv[v] = 0.0f;
    }
    // ---- add the slots: lane (t, c) keeps rows t V .. t V + V - 1 of column c
    double sum[V];
    if constexpr (T == 2) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        double p = gain[v], s = v + V < NN ? gain[v + V] : 0.0;
        swap32(p, s);
        sum[v] = p + s;
      }
    } else {
      double half[2 * V];
#pragma unroll
      for (int v = 0; v < 2 * V; ++v) {
        double p = v < NN ? gain[v] : 0.0, s = v + 2 * V < NN ? gain[v + 2 * V] : 0.0;
        swap32(p, s);
        half[v] = p + s;
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        double p = half[v], s = half[v + V];
        swap16(p, s);
        sum[v] = p + s;
      }
    }
    if (split) {
      double* part = buf;
#pragma unroll
      for (int v = 0; v < V; ++v) part[v * 64 + lane] = sum[v];
      __syncthreads();
      if (wv == 0) {
#pragma unroll
        for (int k = 1; k < 4; ++k)
#pragma unroll
          for (int v = 0; v < V; ++v) sum[v] += part[k * (F::kWaveBytes / 8) + v * 64 + lane];
      }
    }
    if (ends) {
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (F::row(v, lane) >= NN || r >= NN) sum[v] = 0.0;
      finish_any<F, SINGLE>(a, cell, fv, sum, lane);
    }
    if (split || W > 0) __syncthreads();   // the buffers are rewritten by the next cell
  }
}

// Many cells of up to 16 points per axis: a cell per transform slot (four cells per
// wavefront). The slots then share no forward transform and no sums, and no slot
// idles in the last group: 1.7 times fewer instructions per cell at P = 8, 1.3 times
// at P = 20. It needs four cells' spectra in LDS (two wavefronts per SIMD) and runs a
// cell's transforms one after another, so small batches keep the form above. Each
// cell's sums are formed in the order of that form, (s0 + s2) + (s1 + s3) with s_t the
// transforms q = t mod 4, so the results are bitwise equal. Output kinds 0 and 2.
// The filter values of a transform are loaded at once and the spectrum in batches of
// four (loads next to their use: 10000 cells of 16 x 16 took 60 us instead of 41). 16 x 16, M = 16, Maxwell:
// 8192 cells 39.8 -> 28.9 us, 10000 47.5 -> 37.1; hard spheres, M = 8: 8192 cells
// 63.1 -> 55.6; 8 x 8, hard spheres, M = 8: 20000 cells 65.4 -> 51.8.
template <int NN>
struct FftCells {
  using F = FftGrid<NN>;
  static constexpr int kFh = 4 * 2 * NN * F::H;   // doubles
  static constexpr int kWaveBytes = ((kFh + F::XD) * 8 + 15) / 16 * 16;
};

template <int NN>
__device__ __forceinline__ void fft_cells_body(const KernelArgs& a, int64_t first, int64_t stride, int64_t end,
                                               double* lds) {
  using F = FftGrid<NN>;
  static_assert(F::T == 4, "four slots of 16 lanes");
  constexpr int H = F::H, V = F::V;
  double2* fh = reinterpret_cast<double2*>(lds);   // f_hat[k2][slot][k1]
  double* buf = lds + FftCells<NN>::kFh;
  for (int64_t c4 = first; 4 * c4 < end; c4 += stride) {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int t = lane >> 4, r = lane & 15;
    const int c = r < NN ? r : 0;
    const bool live = 4 * c4 + t < end;
    const int64_t cell = live ? 4 * c4 + t : end - 1;
    const float* fc = a.f + cell * static_cast<int64_t>(NN * NN) + c;
    double xr[NN], xi[NN];
#pragma unroll
    for (int v = 0; v < NN; ++v) {
      xr[v] = static_cast<double>(fc[v * NN]);
      xi[v] = 0.0;
    }
    dft<NN, -1>(xr, xi);
    transpose<NN>(xr, buf, lane);
    transpose<NN>(xi, buf, lane);
    dft<NN, -1>(xr, xi);
    if (r < H) {
#pragma unroll
      for (int v = 0; v < NN; ++v) fh[(v * 4 + t) * H + r] = make_double2(xr[v], xi[v]);
    }
    lds_fence();
    const int kap = r < H ? r : (r < NN ? NN - r : 0);
    const int neg = (r >= H && r < NN) ? static_cast<int>(0x80000000u) : 0;
    double s[NN], pair[NN], sum[NN];   // one class of transforms, s0 + s2 or s1 + s3, and the total
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {
      const int cls = k < 2 ? 2 * k : 2 * k - 3;   // 0, 2, 1, 3
#pragma unroll
      for (int v = 0; v < NN; ++v) s[v] = 0.0;
#pragma unroll 1
      for (int q = cls; q <= a.P; q += 4) {
        const char* ft = reinterpret_cast<const char*>(a.filt) + static_cast<int64_t>(q) * (NN * H * 16);
        const unsigned off = static_cast<unsigned>(kap * 16);
        double2 m[NN];
#pragma unroll
        for (int v = 0; v < NN; ++v)
          if (v != NN / 2) m[v] = *reinterpret_cast<const double2*>(ft + v * H * 16 + off);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int B = 4;
        double2 z[2][B];
        auto load_z = [&](int b) {
#pragma unroll
          for (int j = 0; j < B; ++j)
            if (b * B + j < NN && b * B + j != NN / 2) z[b & 1][j] = fh[((b * B + j) * 4 + t) * H + kap];
        };
        load_z(0);
#pragma unroll
        for (int b = 0; b * B < NN; ++b) {
          load_z(b + 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < B; ++j) {
            const int v = b * B + j;
            if (v >= NN) continue;
            if (v == NN / 2) {   // no Nyquist content in any filter
              xr[v] = xi[v] = 0.0;
              continue;
            }
            const double my = flip(m[v].y, neg);
            xr[v] = fma(m[v].x, z[b & 1][j].x, -(my * z[b & 1][j].y));
            xi[v] = fma(m[v].x, z[b & 1][j].y, my * z[b & 1][j].x);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        dft<NN, 1>(xr, xi);
        transpose<NN>(xr, buf, lane);
        transpose<NN>(xi, buf, lane);
#pragma unroll
        for (int v = H; v < NN; ++v) xi[v] = -xi[v];
        dft<NN, 1>(xr, xi);
        if (q < a.P) {   // wavefront-uniform
#pragma unroll
          for (int v = 0; v < NN; ++v) s[v] = fma(xr[v], xi[v], s[v]);
        } else {         // the loss transform
#pragma unroll
          for (int v = 0; v < NN; ++v) s[v] = fma(xr[v], -static_cast<double>(fc[v * NN]), s[v]);
        }
      }
      if (k == 0 || k == 2) {
#pragma unroll
        for (int v = 0; v < NN; ++v) pair[v] = s[v];
      } else if (k == 1) {
#pragma unroll
        for (int v = 0; v < NN; ++v) sum[v] = pair[v] + s[v];
      } else {
#pragma unroll
        for (int v = 0; v < NN; ++v) sum[v] = sum[v] + (pair[v] + s[v]);
      }
    }
    // ---- epilogue: lane (t, r) holds column r of its cell
    const bool in = live && r < NN;
    if (a.out_kind == 0) {
      float* Qc = reinterpret_cast<float*>(a.q) + cell * static_cast<int64_t>(NN * NN) + c;
      if (in)
#pragma unroll
        for (int v = 0; v < NN; ++v) Qc[v * NN] = static_cast<float>(sum[v]);
      continue;
    }
    float fv[NN];
    double p[4] = {0.0, 0.0, 0.0, 0.0};   // partial sums of rho as the lanes of the other form hold them
#pragma unroll
    for (int v = 0; v < NN; ++v) {
      fv[v] = fc[v * NN];
      p[v / V] += r < NN ? static_cast<double>(fv[v]) : 0.0;
    }
    double rho = (p[0] + p[2]) + (p[1] + p[3]);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) rho += __shfl_xor(rho, o);
    rho = rho * a.dv * a.dv;
    const double kk = a.scheme == 1 ? a.dt_eps / (1.0 + a.dt_eps * rho) : a.dt_eps;
    float* fw = const_cast<float*>(fc);
    int bad = 0;
#pragma unroll
    for (int v = 0; v < NN; ++v) {
      const float nv = static_cast<float>(static_cast<double>(fv[v]) + kk * sum[v]);
      if (in) {
        bad |= !(fabsf(nv) <= 3.0e38f);
        fw[v * NN] = nv;
      }
    }
    const unsigned long long any = __ballot(bad);
    if (a.status && live && r == 0) a.status[cell] = (any >> (16 * t)) & 0xffff ? 1 : 0;
  }
}

// Grid sizes with a body: every even size up to 32.
#define QCOLL_FFT_SIZES(X) X(4) X(6) X(8) X(10) X(12) X(14) X(16) X(18) X(20) X(22) X(24) X(26) X(28) X(30) X(32)

// LDS of a wavefront for grid size n.
inline int fft_wave_bytes(int n) {
  switch (n) {
#define QCOLL_FFT_BYTES(N) \
  case N: return FftGrid<N>::kWaveBytes;
    QCOLL_FFT_SIZES(QCOLL_FFT_BYTES)
#undef QCOLL_FFT_BYTES
    default: return 0;
  }
}

}  // namespace
}  // namespace qcoll
