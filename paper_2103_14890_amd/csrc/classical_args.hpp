// Argument block of the classical (direct-sum) kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace qcoll {

// Doubles per row of pair weights: N/2 rounded up to an even count (16-byte loads).
constexpr int classical_row(int N) { return (N / 2 + 1) & ~1; }

// Classical spectral method (section 3.3, eqs. (CF1)/(ode) summed directly): FP64,
// one workgroup per group of cells. Task j = 0 .. N - 1 owns the output modes
// (k1, h N/2 + i), i < N/2, with k1 = (j + 1) / 2 and h = 0 for j = 0 and j = N - 1,
// else (j + 1) mod 2. weights[j][p][m2][i]: weight of f_l f_m for the row pair p = 0
// .. N/2, m1 = (k1 + 1) / 2 + p, l = k - m (all modulo N): beta(l, m) + beta(m, l)
// for two different rows, beta(l, m) where l1 = m1, zero for the pair p = N/2 of an
// odd k1 (it is the pair p = 0). extra[e][m1][m2] = beta(k - m, m) of the modes
// k = (0, N/2) and (N/2, N/2).
struct ClassicalArgs {
  const float* f = nullptr;     // [cells][N][N]
  void* q = nullptr;            // [cells][N][N] float, or double with the projection
  int64_t cells = 0;
  int N = 0;
  int cus = 256;                // compute units
  const double* weights = nullptr;  // [N][N/2 + 1][N][classical_row(N)]
  const double* extra = nullptr;    // [2][N][N]
  int conserve = 0;
  double gram_inv[16] = {};
  double L = 0, dv = 0;
};
int launch_classical(const ClassicalArgs& args, hipStream_t stream);

}  // namespace qcoll
