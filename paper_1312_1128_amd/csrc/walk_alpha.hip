// The forward walk's kernels: alpha only (see walk_fwd.hpp).
#include "walk_fwd.hpp"

namespace glm {

void launch_walk_alpha(const WalkArgs& a) { launch_walk_order<true, 0, false>(a); }

} // namespace glm
