// The forward walk's kernels with per-ray interaction counts (see walk_fwd.hpp).
#include "walk_fwd.hpp"

namespace glm {

void launch_walk_counts(const WalkArgs& a, bool alpha_only)
{
    if (alpha_only) launch_walk_order<true, 1, false>(a);
    else launch_walk_order<false, 1, false>(a);
}

} // namespace glm
