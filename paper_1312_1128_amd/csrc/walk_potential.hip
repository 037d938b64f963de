// The forward walk's kernels: alpha and the lensing potential (see walk_fwd.hpp).
#include "walk_fwd.hpp"

namespace glm {

void launch_walk_potential(const WalkArgs& a) { launch_walk_order<true, 0, true>(a); }

} // namespace glm
