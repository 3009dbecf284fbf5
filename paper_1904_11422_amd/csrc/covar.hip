// Device code of the covariance form and its launches.  A code object of its
// own: in one with the others its kernels moved theirs, and the 128 x 128
// image kernel, unchanged instruction for instruction, took 1 % longer (205.4
// -> 207.6 us at 16 channels of 1024 dual-pol antennas, 200 samples).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "covar_launch.hpp"

namespace epic {

// Time splits of V added into the first, so that what follows reads one plane
// per product whatever the split (holding up to four in flight cost the fold and
// the gradient 11 to 29 spilled registers, reloaded behind the prefetch of V).
// Bound: HBM, one pass.  Only calls of few channels split.
__global__ __launch_bounds__(256) void cov_sum_kernel(CovSumArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.total) return;
  const int64_t h = a.n / 2, cl = i / h;
  int4* v = reinterpret_cast<int4*>(a.v + cl * a.n_split * a.n) + i % h;
  int4 s = v[0];
  for (int k = 1; k < a.n_split; ++k) {
    const int4 x = v[k * h];
    s = make_int4(s.x + x.x, s.y + x.y, s.z + x.z, s.w + x.w);
  }
  v[0] = s;
}

namespace covar {
namespace {

// The fold's template for a shape: f(kernel, threads).
template <typename F> void fold_dispatch(const Shape& s, F&& f) {
#define EPIC_CF(PP, WW, KK)                                                                       \
  if (s.n_pol == PP && s.wide == WW && s.kind == KK)                                              \
    f(cov_fold_kernel<PP, WW, KK>, CovFold<PP, WW, KK>::NT);
  EPIC_CF(1, false, kCovPlain) EPIC_CF(1, false, kCovMany) EPIC_CF(1, false, kCovCrowded)
  EPIC_CF(2, false, kCovPlain) EPIC_CF(2, false, kCovMany) EPIC_CF(2, false, kCovCrowded)
  EPIC_CF(1, true, kCovPlain) EPIC_CF(1, true, kCovMany) EPIC_CF(2, true, kCovPlain) EPIC_CF(2, true, kCovMany)
#undef EPIC_CF
}

}  // namespace

int fold_blocks_per_cu(const Shape& s) {
  int nb = 1;
  fold_dispatch(s, [&](auto k, int nt) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, nt, 0) != hipSuccess) nb = 1;
  });
  return std::max(1, nb);
}

void launch_corr(const CovCorrArgs& a, int n_pol, hipStream_t stream) {
  const bool whole = a.n_ant % 4 == 0;
  auto go = [&](auto k) { hipLaunchKernelGGL(k, dim3((unsigned)a.total), dim3(256), 0, stream, a); };
  if (n_pol == 2) {
    if (whole) go(cov_corr_kernel<2, true>);
    else go(cov_corr_kernel<2, false>);
  } else {
    if (whole) go(cov_corr_kernel<1, true>);
    else go(cov_corr_kernel<1, false>);
  }
}

void launch_sum(const CovSumArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(cov_sum_kernel, dim3((unsigned)((a.total + 255) / 256)), dim3(256), 0, stream, a);
}

void launch_fold(const CovFoldArgs& a, const Shape& s, hipStream_t stream) {
  fold_dispatch(s, [&](auto k, int nt) { hipLaunchKernelGGL(k, dim3((unsigned)a.W), dim3(nt), 0, stream, a); });
}

void launch_image(const CovImageArgs& a, int n_pol, int n_chan, hipStream_t stream) {
  if (n_pol == 2) hipLaunchKernelGGL(cov_image_kernel<2>, dim3(3 * n_chan), dim3(512), 0, stream, a);
  else hipLaunchKernelGGL(cov_image_kernel<1>, dim3(n_chan), dim3(512), 0, stream, a);
}

void launch_hat(const CovHatArgs& a, int n_pol, int n_chan, hipStream_t stream) {
  if (n_pol == 2) hipLaunchKernelGGL(cov_hat_kernel<2>, dim3(4 * n_chan), dim3(512), 0, stream, a);
  else hipLaunchKernelGGL(cov_hat_kernel<1>, dim3(n_chan), dim3(512), 0, stream, a);
}

void launch_adjoint(const CovGradArgs& a, const Shape& s, hipStream_t stream) {
  auto go = [&](auto k) { hipLaunchKernelGGL(k, dim3((unsigned)a.total), dim3(64 * kCovGradWaves), 0, stream, a); };
#define EPIC_CG(PP, WW) \
  if (s.n_pol == PP && s.wide == WW) go(cov_adjoint_kernel<PP, WW>);
  EPIC_CG(1, false) EPIC_CG(1, true) EPIC_CG(2, false) EPIC_CG(2, true)
#undef EPIC_CG
}

void launch_grad_sum(const CovGradSumArgs& a, int n_pol, hipStream_t stream) {
  const dim3 grid((unsigned)((a.n + 255) / 256));
  if (n_pol == 2) hipLaunchKernelGGL(cov_grad_sum_kernel<2>, grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL(cov_grad_sum_kernel<1>, grid, dim3(256), 0, stream, a);
}

}  // namespace covar
}  // namespace epic
