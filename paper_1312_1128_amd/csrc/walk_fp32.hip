// The forward walk's kernels with plain FP32 sums of alpha (debug, see walk_fwd.hpp).
#include "walk_fwd.hpp"

namespace glm {

void launch_walk_fp32(const WalkArgs& a, bool alpha_only)
{
    if (alpha_only) launch_walk_order<true, 2, false>(a);
    else launch_walk_order<false, 2, false>(a);
}

} // namespace glm
