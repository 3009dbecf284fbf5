// Launches of the covariance form's kernels (covar.hip), for the host side.
#pragma once
#include "covar.hpp"
#include "covar_adjoint.hpp"

namespace epic {
namespace covar {

// Shape of a launch: polarisations, wide block, kind of fold (kCovPlain, ..).
struct Shape {
  int n_pol;
  bool wide;
  int kind;
};

int fold_blocks_per_cu(const Shape& s);
void launch_corr(const CovCorrArgs& a, int n_pol, hipStream_t stream);
void launch_sum(const CovSumArgs& a, hipStream_t stream);
void launch_fold(const CovFoldArgs& a, const Shape& s, hipStream_t stream);
void launch_image(const CovImageArgs& a, int n_pol, int n_chan, hipStream_t stream);
void launch_hat(const CovHatArgs& a, int n_pol, int n_chan, hipStream_t stream);
void launch_adjoint(const CovGradArgs& a, const Shape& s, hipStream_t stream);
void launch_grad_sum(const CovGradSumArgs& a, int n_pol, hipStream_t stream);

}  // namespace covar
}  // namespace epic
