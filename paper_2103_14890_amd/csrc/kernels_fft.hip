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

}  // namespace

int launch_fft(const KernelArgs& args, hipStream_t stream) {
  if (args.cells <= 0) return 0;
  const int wpb = args.waves_per_block;
  int64_t blocks = (args.cells + wpb - 1) / wpb;
  if (blocks > args.max_blocks) blocks = args.max_blocks;
  const dim3 grid(static_cast<unsigned>(blocks)), block(64 * wpb);
  switch (args.n) {
#define QCOLL_FFT_LAUNCH(N) \
  case N: return launch_n<N>(args, grid, block, stream);
    QCOLL_FFT_SIZES(QCOLL_FFT_LAUNCH)
#undef QCOLL_FFT_LAUNCH
    default: return -4;
  }
}

}  // namespace qcoll
