// Single-plan launches of the 2D FX16 plans on grids of up to 32 points per
// axis (the per-cell body is in body_fft.hpp), gfx950.

#include <hip/hip_runtime.h>

#include <cstdint>

#include "body_fft.hpp"

namespace qcoll {
namespace {

// Lines of up to 16 points leave room for three wavefronts per SIMD, longer
// ones (two lines' worth of registers and the gain) for two.
template <int N>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(N > 16 ? 2 : 3))) void fft_kernel(KernelArgs a) {
  extern __shared__ double lds[];
  const int wpb = blockDim.x >> 6, w = threadIdx.x >> 6;
  fft_body<N, true>(a, static_cast<int64_t>(blockIdx.x) * wpb + w, static_cast<int64_t>(gridDim.x) * wpb, false, 0,
              lds + w * (FftGrid<N>::kWaveBytes / 8));
}

template <int N>
int launch_n(const KernelArgs& args, dim3 grid, dim3 block, hipStream_t stream) {
  constexpr int kWave = FftGrid<N>::kWaveBytes;
  static_assert(8 * kWave <= 160 * 1024, "eight wavefronts share a CU's LDS");
  if (8 * kWave > 64 * 1024) {   // above the default limit of dynamic LDS
    static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(fft_kernel<N>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 8 * kWave) == hipSuccess;
    if (!ok) return -3;
  }
  hipLaunchKernelGGL(fft_kernel<N>, grid, block, kWave * (block.x / 64), stream, args);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// A workgroup of four wavefronts per cell.
template <int N>
__global__ __launch_bounds__(256, 2) void fft_round_kernel(KernelArgs a) {
  extern __shared__ double lds[];
  fft_body<N, true, 4>(a, blockIdx.x, gridDim.x, false, threadIdx.x >> 6, lds);
}

template <int N>
int launch_round(const KernelArgs& args, hipStream_t stream) {
  constexpr int kLds = fft_round_bytes<N, 4>();
  static_assert(2 * kLds <= 160 * 1024, "two workgroups share a CU's LDS");
  if (kLds > 64 * 1024) {
    static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(fft_round_kernel<N>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, kLds) == hipSuccess;
    if (!ok) return -3;
  }
  const int64_t blocks = args.cells < args.max_blocks ? args.cells : args.max_blocks;
  hipLaunchKernelGGL(fft_round_kernel<N>, dim3(static_cast<unsigned>(blocks)), dim3(256), kLds, stream, args);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// Cells 0 .. full - 1 four to a wavefront (the first `blocks` workgroups), the rest
// one to a wavefront.
template <int N>
__global__ __launch_bounds__(256, 2) void fft_cells_kernel(KernelArgs a, int64_t full, int blocks) {
  extern __shared__ double lds[];
  const int w = threadIdx.x >> 6;
  const int b = static_cast<int>(blockIdx.x);
  double* mine = lds + w * (FftCells<N>::kWaveBytes / 8);
  if (b < blocks)
    fft_cells_body<N>(a, static_cast<int64_t>(b) * 4 + w, static_cast<int64_t>(blocks) * 4, full, mine);
  else
    fft_body<N, true>(a, full + static_cast<int64_t>(b - blocks) * 4 + w,
                      static_cast<int64_t>(gridDim.x - blocks) * 4, false, 0, mine);
}

template <int N>
int launch_cells(const KernelArgs& args, int64_t full, hipStream_t stream) {
  static_assert(FftCells<N>::kWaveBytes >= FftGrid<N>::kWaveBytes, "both forms run in one kernel");
  constexpr int kLds = 4 * FftCells<N>::kWaveBytes;
  if (kLds > 64 * 1024) {
    static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(fft_cells_kernel<N>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, kLds) == hipSuccess;
    if (!ok) return -3;
  }
  // The two parts share the grid cap, two thirds for the first: with the default cap of
  // 12 workgroups per CU its workgroups walk their cells in whole rounds of 8 (100000 cells
  // of 16 x 16, Maxwell, M = 16: 268 us; 1916 workgroups beside a second part of 132 took
  // 281). A cap of one leaves none for a second part: all cells then go four to a wavefront.
  if (args.max_blocks < 2) full = args.cells;
  const int64_t most = args.max_blocks / 3 * 2 > 1 ? args.max_blocks / 3 * 2 : 1;
  int64_t blocks = (full + 15) / 16, rest = (args.cells - full + 3) / 4;
  if (blocks > most) blocks = most;
  if (rest > args.max_blocks - blocks) rest = args.max_blocks - blocks;
  hipLaunchKernelGGL(fft_cells_kernel<N>, dim3(static_cast<unsigned>(blocks + rest)), dim3(256), kLds, stream, args,
                     full, static_cast<int>(blocks));
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// Four cells per wavefront from whole rounds of one such wavefront per SIMD on. What
// is left over joins them where it would take longer a cell per wavefront: with G + 1
// passes for each of its cells (G groups of four of the P + 1 transforms) against P + 2
// for a round of `unit` cells, from a ratio of 0.3 on alone and of 0.23 on beside other
// rounds (measured on 4 to 16 points and P = 1 to 20; the lines are where neither side
// gains). Alone, one and four cells per wavefront: 12 x 12, Maxwell, M = 8 (P = 4), 2048
// cells 9.5 and 10.0 us, 3500 cells 14.4 and 10.1; 16 x 16, hard spheres, M = 8 (P =
// 20), 3000 cells 26.9 and 34.9, 3500 34.7 and 35.1. Beside a round: the former 7000
// cells 18.1 and 14.6, the latter 6000 cells 42.7 and 53.0, 7000 50.5 and 53.3, 12000
// 80.7 and 79.4. Returned: the number of cells that go four to a wavefront.
int64_t cells_of_four(const KernelArgs& args) {
  if (args.n > 16 || (args.out_kind != 0 && args.out_kind != 2)) return 0;
  const int64_t unit = 16 * static_cast<int64_t>(args.cus), G = args.P / 4 + 1;
  const int64_t full = args.cells / unit * unit, left = args.cells - full;
  return 100 * left * (1 + G) >= (full > 0 ? 23 : 30) * unit * (args.P + 2) ? args.cells : full;
}

// Few cells: four wavefronts per cell while one such workgroup per compute unit holds
// them all, and two where a cell has enough transforms for its wavefronts (P >= 4). One
// and four wavefronts per cell, one cell: 32 points, hard spheres, M = 8 (P = 20) 37.8
// and 23.8 us; 24 points, Maxwell, M = 4 (P = 2) 9.8 and 9.6, 200 cells 13.5 and 10.0. 300
// cells: 24 points, P = 20, 39.0 and 23.5; 28 points, P = 4, 20.2 and 17.6, P = 3, 16.5
// and 17.3; 20 points, P = 4, 13.8 and 12.4, P = 3, 11.3 and 12.1. (Two wavefronts per
// cell beyond that: 700 cells of 32 points, Maxwell, M = 16, 28.6 -> 31.)
bool few_cells(const KernelArgs& args) {
  return args.n > 16 && args.cells <= static_cast<int64_t>(args.P >= 4 ? 2 : 1) * args.cus;
}

}  // namespace

bool own_workgroups_fft(const KernelArgs& args) { return cells_of_four(args) > 0 || few_cells(args); }

int launch_fft(const KernelArgs& args, hipStream_t stream) {
  if (args.cells <= 0) return 0;
  const int wpb = args.waves_per_block;
  int64_t blocks = (args.cells + wpb - 1) / wpb;
  if (blocks > args.max_blocks) blocks = args.max_blocks;
  const dim3 grid(static_cast<unsigned>(blocks)), block(64 * wpb);
  if (const int64_t full = cells_of_four(args); full > 0) {
    switch (args.n) {
      case 4: return launch_cells<4>(args, full, stream);
      case 6: return launch_cells<6>(args, full, stream);
      case 8: return launch_cells<8>(args, full, stream);
      case 10: return launch_cells<10>(args, full, stream);
      case 12: return launch_cells<12>(args, full, stream);
      case 14: return launch_cells<14>(args, full, stream);
      case 16: return launch_cells<16>(args, full, stream);
      default: break;
    }
  }
  if (few_cells(args)) {
    switch (args.n) {
      case 18: return launch_round<18>(args, stream);
      case 20: return launch_round<20>(args, stream);
      case 22: return launch_round<22>(args, stream);
      case 24: return launch_round<24>(args, stream);
      case 26: return launch_round<26>(args, stream);
      case 28: return launch_round<28>(args, stream);
      case 30: return launch_round<30>(args, stream);
      case 32: return launch_round<32>(args, stream);
      default: break;
    }
  }
  switch (args.n) {
#define QCOLL_FFT_LAUNCH(N) \
  case N: return launch_n<N>(args, grid, block, stream);
    QCOLL_FFT_SIZES(QCOLL_FFT_LAUNCH)
#undef QCOLL_FFT_LAUNCH
    default: return -4;
  }
}

}  // namespace qcoll
