// FP32 Chebyshev steps (the FP32 multigrid cycle).
#include "chebstep.hpp"

namespace spk {
template int cheb_step<float>(spk_mat *, const ChebStep<float> &, float *, hipStream_t, int *);
}  // namespace spk
