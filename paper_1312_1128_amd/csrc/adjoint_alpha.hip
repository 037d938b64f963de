// The adjoint walk's kernels: alpha cotangents only (see adjoint_walk.hpp).
#include "adjoint_walk.hpp"

namespace glm {

void launch_adjoint_alpha(const AdjointArgs& a) { launch_adjoint_order<false>(a); }

} // namespace glm
