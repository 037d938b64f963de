// Persistent walk over many lenses (Sec. 3.3): every wavefront takes (lens,
// 64-ray group) items from a device counter until the queue is empty.  Lenses
// are ranked by estimated cost, so the largest ray groups start first.
// Six wavefronts per SIMD (80 registers, a few spilled around the far expansion): 24
// lenses 7.93 ms, 8.20 with five, 8.72 with the four that 97 registers leave.
#include <algorithm>

#include "walk_fwd.hpp"

namespace glm {

namespace {

template <int P, bool AONLY, int MODE, int KIND>
__global__ __launch_bounds__(kBlock, 6) void k_walk_batched(const BatchLens* __restrict__ lenses, int nlens,
                                                        const int64_t* __restrict__ gprefix, int* __restrict__ counter,
                                                        const double* __restrict__ xs, const double* __restrict__ ys,
                                                        const uint32_t* __restrict__ perm)
{
    __shared__ __align__(16) char lds[(kBlock / kWave) * solo_lds_bytes(true)];
    const int lane = threadIdx.x & (kWave - 1);
    const TravLds L = solo_lds(lds + (threadIdx.x / kWave) * solo_lds_bytes(true), true);
    const int64_t total = gprefix[nlens];
    for (;;) {
        int it = 0;
        if (lane == 0) it = atomicAdd(counter, 1);
        it = __builtin_amdgcn_readfirstlane(__shfl(it, 0, kWave));
        if (it >= total) break;
        int lo = 0, hi = nlens; // largest l with gprefix[l] <= it
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (gprefix[mid] <= it) lo = mid;
            else hi = mid;
        }
        const BatchLens& B = lenses[lo];
        const int64_t rl = (int64_t)(it - gprefix[lo]) * kWave + lane;
        const bool valid = rl < B.nrays;
        const int64_t gi = B.ray_off + (valid ? rl : 0);
        const double X = valid ? xs[gi] : 0.0, Y = valid ? ys[gi] : 0.0;
        const RayGroup g = ray_group(X, Y, valid, MODE != 2);
        FwdVisitor<P, AONLY, MODE, false, KIND, MODE != 2> v(B.tree, g, X, Y, lane, valid);
        traverse<false, false>(B.tree, v, g, X, Y, lane, 0, 1, L);
        if (g.far) {
            double* words = reinterpret_cast<double*>(L.stkm);
            v.put_words(words);
            wave_lds_sync();
            v.finish(words);
            wave_lds_sync(); // the next item's stack overwrites the words
        }
        if constexpr (!AONLY) join_shear(v.A);
        if (valid) write_out<AONLY, false>(v.A, v.cnt, (int64_t)perm[gi] - B.ray_off, B.out);
    }
}

template <int P, bool AONLY>
void launch(const BatchArgs& a)
{
    const int blocks = (int)std::min<int64_t>((a.items + 3) / 4, 256 * 8);
#define GLM_WALK(MD, KD)                                                                                          \
    hipLaunchKernelGGL((k_walk_batched<P, AONLY, MD, KD>), dim3(blocks), dim3(kBlock), 0, a.st, a.table, a.nlens, \
                       a.gpre, a.counter, a.xs, a.ys, a.perm)
    if (a.kind == kKindNfw) {
        if (a.fp32_alpha) GLM_WALK(2, kKindNfw);
        else GLM_WALK(0, kKindNfw);
    } else {
        if (a.fp32_alpha) GLM_WALK(2, kKindGauss);
        else GLM_WALK(0, kKindGauss);
    }
#undef GLM_WALK
}

} // namespace

void launch_walk_batched(const BatchArgs& a)
{
#define GLM_CASE(PP)                            \
    case PP:                                    \
        if (a.alpha_only) launch<PP, true>(a);  \
        else launch<PP, false>(a);              \
        break;
    switch (a.order) {
        GLM_CASE(0) GLM_CASE(1) GLM_CASE(2) GLM_CASE(3) GLM_CASE(4) GLM_CASE(5) GLM_CASE(6)
        GLM_CASE(7) GLM_CASE(8) GLM_CASE(9) GLM_CASE(10) GLM_CASE(11) GLM_CASE(12)
        default: break;
    }
#undef GLM_CASE
}

} // namespace glm
