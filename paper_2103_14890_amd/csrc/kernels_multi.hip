// Batched launch over several plans: cells of different velocity grids (and
// arithmetic variants) in one grid. The operator is cell-local (section 3.3),
// so every cell runs exactly the code of its single-plan launch and the
// results are bitwise equal to separate launches. Workgroups are assigned to
// slots by contiguous ranges; a workgroup finds its slot with a short scan of
// the slot table (at most kMaxSlots2 entries) and then walks its slot's cells:
// one cell per wavefront on 16x16 and 32x32 tiles, one cell per workgroup of
// four wavefronts on the 64-point grids (the tile-64 body).

#include <hip/hip_runtime.h>

#include <cstdint>

#include "body_fft.hpp"
#include "body_fft64.hpp"
#include "body_t16.hpp"
#include "body_t32.hpp"
#include "body_t64.hpp"

namespace qcoll {
namespace {

// Slot s on workgroup b of a launch, a plan of the FFT kernels.
__device__ __forceinline__ void fft_slot(const MultiArgs& m, int s, int64_t b, double2* lds) {
  const KernelArgs& a = m.slot[s];
  const int64_t b0 = b - m.block_start[s], nb = m.block_start[s + 1] - m.block_start[s];
  if (a.tile == 64) {   // one cell (or part of one) per workgroup of four wavefronts
    switch (a.n) {
#define QCOLL_FFT64_BODY(R) \
  case 4 * R: fft64_body<R, false>(a, b0, nb, lds); break;
      QCOLL_FFT64_SIZES(QCOLL_FFT64_BODY)
#undef QCOLL_FFT64_BODY
      default: break;
    }
    return;
  }
  // a wavefront per cell, or in the split form the workgroup's four wavefronts
  const bool split = a.split > 1;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wpb = blockDim.x >> 6;
  double* l = reinterpret_cast<double*>(lds);
  switch (a.n) {
#define QCOLL_FFT_BODY(N)                                                                      \
  case N:                                                                                      \
    fft_body<N, false>(a, split ? b0 : b0 * wpb + w, split ? nb : nb * wpb, split, w,          \
                       l + w * (FftGrid<N>::kWaveBytes / 8));                                  \
    break;
    QCOLL_FFT_SIZES(QCOLL_FFT_BODY)
#undef QCOLL_FFT_BODY
    default: break;
  }
}

// FFT: the launch has slots of the FFT kernels. With their 23 bodies beside the matrix
// bodies the kernel spills (209 registers, 304 bytes of scratch per lane), which the
// transform split of the 64-point matrix form felt most (300 cells of 48 x 48, hard
// spheres, M = 8, four parts each: 381 us, without the FFT bodies 358), so launches of
// matrix slots alone have a kernel without them: 244 registers, no spills.
template <bool FFT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void multi_kernel(MultiArgs m) {
  extern __shared__ double2 lds[];
  const int64_t b = blockIdx.x;
  int s = 0;
#pragma unroll 1
  while (s + 1 < m.nslots && b >= m.block_start[s + 1]) ++s;
  s = __builtin_amdgcn_readfirstlane(s);
  const KernelArgs& a = m.slot[s];
  if constexpr (FFT) {
    if (a.fft) {
      fft_slot(m, s, b, lds);
      return;
    }
  }
  if (a.tile == 64) {  // one cell (or one part of one, in the split form) per workgroup of four wavefronts
    const int64_t first = b - m.block_start[s], stride = m.block_start[s + 1] - m.block_start[s];
    if (a.split > 1) {
      if (a.precision == 4) t64_body<-1, true, true>(a, first, stride, lds);
      else t64_body<-1, false, true>(a, first, stride, lds);
    } else {
      if (a.precision == 4) t64_body<-1, true>(a, first, stride, lds);
      else t64_body<-1, false>(a, first, stride, lds);
    }
    return;
  }
  if (a.split > 1) {  // 32x32 FX16 tiles, one cell per workgroup of four wavefronts sharing its transforms
    half8* eo = reinterpret_cast<half8*>(lds);
    load_eo_table(a, eo);
    fx16_t32_body<-1, true>(a, b - m.block_start[s], m.block_start[s + 1] - m.block_start[s],
                            lds + (kEoLdsBytes + (threadIdx.x >> 6) * kFhatLdsBytes) / 16, eo);
    return;
  }
  const int wpb = blockDim.x >> 6;
  const int64_t first = (b - m.block_start[s]) * wpb + (threadIdx.x >> 6);
  const int64_t stride = (m.block_start[s + 1] - m.block_start[s]) * wpb;
  if (a.tile == 32) {
    if (a.precision == 4) {  // block-uniform branch: the table load's barrier is safe
      half8* eo = reinterpret_cast<half8*>(lds);
      load_eo_table(a, eo);
      fx16_t32_body<-1>(a, first, stride, lds + (kEoLdsBytes + (threadIdx.x >> 6) * kFhatLdsBytes) / 16, eo);
    }
    else fp32_t32_body<-1>(a, first, stride);
  } else {
    if (a.precision == 4) fx16_t16_body<-1>(a, first, stride);
    else fp32_t16_body<-1>(a, first, stride);
  }
}

}  // namespace

int launch_multi(const MultiArgs& args, int waves_per_block, hipStream_t stream) {
  const int64_t blocks = args.block_start[args.nslots];
  if (blocks <= 0) return 0;
  bool t64 = false;
  for (int i = 0; i < args.nslots; ++i) t64 |= args.slot[i].tile == 64;
  if (t64 && waves_per_block != 4) return -4;   // the tile-64 body needs four wavefronts per workgroup
  // dynamic LDS above the 64 KB default: 76 KB for four wavefronts of N <= 32
  // cells (both kernel families), 79 KB for a tile-64 cell of the matrix kernels, 67 KB
  // of the FFT kernels
  constexpr int kT32LdsBytes = kEoLdsBytes + 4 * kFhatLdsBytes;
  static const bool attr_ok = [] {
    int most = kT64LdsBytes > kT32LdsBytes ? kT64LdsBytes : kT32LdsBytes;
    for (int n = 4; n <= 32; n += 2) most = most > 4 * fft_wave_bytes(n) ? most : 4 * fft_wave_bytes(n);
    return hipFuncSetAttribute(reinterpret_cast<const void*>(multi_kernel<true>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, most) == hipSuccess &&
           hipFuncSetAttribute(reinterpret_cast<const void*>(multi_kernel<false>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, most) == hipSuccess;
  }();
  if (!attr_ok) return -3;
  int lds_bytes = 0;
  bool fft = false;
  for (int i = 0; i < args.nslots; ++i) {
    const KernelArgs& a = args.slot[i];
    const int need = a.fft && a.tile == 64 ? Fft64<16>::kLdsBytes
                     : a.fft ? waves_per_block * fft_wave_bytes(a.n)
                     : a.tile == 64 ? kT64LdsBytes
                     : a.tile == 32 && a.precision == 4 ? kEoLdsBytes + kFhatLdsBytes * waves_per_block
                                                        : 0;
    if (need > lds_bytes) lds_bytes = need;
    fft |= a.fft != 0;
  }
  const dim3 grid(static_cast<unsigned>(blocks)), block(64 * waves_per_block);
  if (fft) hipLaunchKernelGGL(multi_kernel<true>, grid, block, lds_bytes, stream, args);
  else hipLaunchKernelGGL(multi_kernel<false>, grid, block, lds_bytes, stream, args);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace qcoll
