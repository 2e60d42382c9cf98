// The FP64 Krylov iterations.
#include "iterate.hpp"

namespace spk {
template int launch_iterations<double>(spk_mat *, Workspace *, int, hipStream_t);
}  // namespace spk
