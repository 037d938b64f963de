// The forward walk's kernels: alpha, kappa and gamma (see walk_fwd.hpp).
#include "walk_fwd.hpp"

namespace glm {

void launch_walk_full(const WalkArgs& a) { launch_walk_order<false, 0, false>(a); }

} // namespace glm
