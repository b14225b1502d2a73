// Single-plan launches of the 2D FX16 plans on grids of 36, 40, .. 64 points per
// axis (the per-cell body is in body_fft64.hpp), gfx950.

#include <hip/hip_runtime.h>

#include <cstdint>

#include "body_fft64.hpp"

namespace qcoll {
namespace {

template <int R>
__global__ __launch_bounds__(256, 2) void fft64_kernel(KernelArgs a) {
  extern __shared__ double2 lds[];
  fft64_body<R, true>(a, blockIdx.x, gridDim.x, lds);
}

template <int R>
int launch_r(const KernelArgs& args, dim3 grid, hipStream_t stream) {
  constexpr int kLds = Fft64<R>::kLdsBytes;
  if (kLds > 64 * 1024) {   // above the default limit of dynamic LDS
    static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(fft64_kernel<R>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, kLds) == hipSuccess;
    if (!ok) return -3;
  }
  hipLaunchKernelGGL(fft64_kernel<R>, grid, dim3(256), kLds, stream, args);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace

int launch_fft64(const KernelArgs& args, hipStream_t stream) {
  if (args.cells <= 0) return 0;
  KernelArgs a = args;
  a.split = 1;   // one workgroup per cell; the split form runs in the batched kernel
  int64_t blocks = a.cells;
  if (blocks > a.max_blocks) blocks = a.max_blocks;
  const dim3 grid(static_cast<unsigned>(blocks));
  switch (a.n) {
#define QCOLL_FFT64_LAUNCH(R) \
  case 4 * R: return launch_r<R>(a, grid, stream);
    QCOLL_FFT64_SIZES(QCOLL_FFT64_LAUNCH)
#undef QCOLL_FFT64_LAUNCH
    default: return -4;
  }
}

}  // namespace qcoll
