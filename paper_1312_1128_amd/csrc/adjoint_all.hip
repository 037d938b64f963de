// The adjoint walk's kernels: alpha, kappa and gamma cotangents (see adjoint_walk.hpp).
#include "adjoint_walk.hpp"

namespace glm {

void launch_adjoint_all(const AdjointArgs& a) { launch_adjoint_order<true>(a); }

} // namespace glm
