// The FP32 inner iterations of mixed solves.
#include "iterate.hpp"

namespace spk {
template int launch_iterations<float>(spk_mat *, Workspace *, int, hipStream_t);
}  // namespace spk
