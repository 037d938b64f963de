// Ray staging and the forward / adjoint walks.
#pragma once

#include <algorithm>

#include "build.hpp"

namespace glm {

// Outputs of a walk (input order of the rays).
struct WalkOut {
    float *a1, *a2, *k, *g1, *g2;
    int32_t* counts;
    float* psi = nullptr; // potential walk only
    float* td = nullptr;  // time delay |alpha|^2 / 2 - psi (nullable)
};

// One lens of a batched walk (device table entry).
struct BatchLens {
    TreeDev tree;
    int64_t nrays;
    int64_t ray_off;   // offset of its rays in the concatenated staged arrays
    const double* rx;  // the caller's rays (input order)
    const double* ry;
    WalkOut out;
};

// Persistent walk over several lenses; host_table is in queue order (largest
// expected work first), every tree built with the same order.
size_t batch_workspace_bytes(int nlens, int64_t total_rays);
glm_status shoot_batched_device(const BatchLens* host_table, int nlens, int order, uint32_t flags, void* ws,
                                hipStream_t st);

size_t refine_workspace_bytes(int64_t ncells);
glm_status refine_round_device(double* cx, double* cy, double* side, const float* ka, const float* g1,
                               const float* g2, int64_t ncells, int64_t nrefine, int32_t* refined, void* ws,
                               hipStream_t st);
// The two halves of a round: rank the cells (order = cell indices by
// descending score, in ws), then split the first nrefine of them.
glm_status refine_rank_device(const double* side, const float* ka, const float* g1, const float* g2,
                              int64_t ncells, void* ws, const uint32_t** order, hipStream_t st);
glm_status refine_spawn_device(const uint32_t* order, int64_t nrefine, int64_t ncells, double* cx, double* cy,
                               double* side, int32_t* refined, hipStream_t st);

// Interpolation shortcut of refinement (interp.hip): per-cell level and
// integer coordinates plus a (level, i, j) -> cell hash, in a caller buffer.
struct InterpLayout {
    size_t lev, ci, cj, keys, vals, bytes;
    int64_t table_cap;
};
InterpLayout interp_layout(int64_t capacity);
size_t interp_round_workspace_bytes(int64_t ncells, int64_t nrefine);
glm_status interp_init_device(const double* cx, const double* cy, int64_t ncells, double x0, double y0, double h0,
                              int64_t capacity, void* state, hipStream_t st);
glm_status interp_round_device(double* cx, double* cy, double* side, float* a1, float* a2, float* ka, float* g1,
                               float* g2, int64_t ncells, int64_t nrefine, int64_t nbase, float tol, bool deflections,
                               int32_t* refined, int32_t* shoot_idx, int32_t* shoot_count, int64_t capacity,
                               void* state, void* ws, hipStream_t st);
// kappa, gamma of cells idx[0 .. min(*count, max_count)) (idx NULL: cells 0 ..
// max_count; count NULL: max_count) from their three-point magnification matrix.
glm_status interp_estimate_device(const double* cx, const double* cy, const float* a1, const float* a2, float* ka,
                                  float* g1, float* g2, const int32_t* idx, const int32_t* count, int64_t max_count,
                                  int64_t nbase, int64_t capacity, const void* state, hipStream_t st);
size_t shoot_indexed_workspace_bytes(int64_t count);

// Per-ray counts of a walk: boxes visited (opening tests), boxes accepted,
// leaf particles summed, list particles the ray falls inside; then counts of
// its group's wavefronts (the same for all rays of a group): list entries tested
// against the ray group (the search overhead), boxes some lane accepted, leaf
// particles evaluated, list candidates evaluated.  The per-lane counts over the
// wavefront's give the lane use of each phase.
constexpr int kCounts = 8;

// Sums of one ray over one range of boxes.
struct Partial {
    double a1, a2, k, g1, g2, ps;
    int32_t cnt[kCounts];
};

// Byte offsets of the ray workspace pieces.
struct RayLayout {
    size_t k0, k1, v0, v1, xs, ys, hist, part, parts, bytes;
};
RayLayout ray_layout(int64_t nrays);

struct StagedRays {
    const double* xs;
    const double* ys;
    const uint32_t* perm; // sorted -> input position, or null when unsorted
};

// Sort the rays along a Hilbert curve (8 to 16 bits per axis in their bounding square) so that
// each 64-ray group is spatially compact.
glm_status stage_rays(const double* rx, const double* ry, int64_t nrays, void* ws, const RayLayout& L,
                      StagedRays* out, hipStream_t st);
// The staged rays that stage_rays left in the workspace (no launch).
StagedRays staged_rays_view(int64_t nrays, void* ws, const RayLayout& L);

// Rays per group (64 down to 4) and wavefronts that share a group (1 to 16, a
// power of two) of a forward walk.
//  - Few rays: a group of 64 scattered rays covers much of the lens and needs
//    nearly everything that any of them needs, while most of the chip idles;
//    groups of fewer rays (the other lanes idle) need less each.  1,024 rays on
//    1e6 particles: 3.65 ms in 16 groups of 64, 0.45 ms in 256 of 4.  The
//    halving pays up to more groups on larger trees (4,096 rays on 1e4
//    particles: 185 us in 256 groups, 229 in 512; on 1e6 particles 1,168 us in
//    256, 696 in 1,024).
//  - Wavefronts: the most that keep the launch under `fill`.  On a small tree
//    the groups cost alike and more wavefronts only wait for one another; over a
//    large one the groups of the dense core cost many times the others.
//    262,144 rays (4,096 groups) with 1, 2, 4, 8 wavefronts each, in us: on 1e4
//    particles 520, 464, 480, 666; on 6e4 863, 684, 610, 787; on 1e6 -, 2405,
//    1682, 1617.  Each has at least kWaveParticles particles of the lens to share
//    (60 particles: 1e4 rays in their order 25.7 us with 16, 19.5 with one; 2e5 rays 31.7
//    with two, 27.4 with one).
//  - Over an uneven lens (TreeStorage::uneven: a core far denser than the rest) the few groups
//    there are the whole launch's length: four times the `fill`, from kUnevenParticles particles.
//    Equal mass per octave of radius, 3e4 particles, 2.8e5 rays: 2,230 us with one
//    wavefront per group, 1,286 with two, 780 with four; adjoint 3,190, 1,456, 958; 1e5
//    particles, 7e5 rays: adjoint 5,720, 2,618, 1,681.  (NFW halos and patches of stars count as
//    even, and over those the even fill is the better one: 1e5 uniform particles, 3e5 rays
//    424 us with four, 569 with eight; 1.4e5 rays of a refinement over 3e5 particles, 3e4 of them
//    stars in one patch, 564 us with eight, 784 with sixteen.)
constexpr int kMaxGroupRays = 64;
constexpr int kWaveParticles = 64;
constexpr int64_t kUnevenParticles = 2048;
struct WalkShape {
    int rays, waves, split;
};

// Whether a walk opens most of the tree: a box of side d is opened within about d / theta, and
// below this the leaves' opened squares cover most of the lens from everywhere.  Then
// smaller groups need no less each, far boxes are rare, and the work lies evenly along the preorder:
// a launch of few groups splits it into `split` box ranges with workgroups of
// their own (up to kOpenGroups, of kOpenWaves wavefronts), whose sums
// meet in range order.  theta = 0, 60 rays on 3e5 particles: 9.4 ms in groups of 4
// rays, 0.28 in 64 ranges of one group; 5,000 rays 24.9, 2.1.  2e4 rays on 3e4 particles,
// 1,024 workgroups of 8 wavefronts 716 us, 4,096 of 8 616, of 4 593.  The rule goes by r =
// n theta^2 / max(16, leaf size): smaller leaves split no earlier (leaves of 2, 6e4 particles, 1.5e4
// rays at r = 3.4: 3,215 us not split; adjoint of 5,000 particles at 2: 709), large ones a little later,
// half as late with many groups (leaves of 64, 1.5e4 rays, adjoint of 6e4 points at r = 15 370 us not
// split, 832; walk of a core 612, 390).  The fewer the groups, the further it reaches (not
// split and split, leaves of 16: 2e5 particles, 1.5e4 rays at r = 11 1,700, 620; at 17 1.6 to 2.3
// times; 6e4 rays at 11 +-5%, at 17 5e4 particles 0.9 to 1.3 times, beyond less).  The adjoint
// gains less on a small lens (1.2e4 particles, 1.5e4 rays at 11: 0.7 to 1.2 times), and more on an uneven
// one, whose few long groups the ranges even out (1.5e4 rays at 17: 5e4 particles 1,332, 470;
// 2e5 5,500, 1,405; 6e4 rays on 2e5 at 28: 1.3 times).
constexpr int64_t kOpenParticles = 2048;
constexpr int64_t kOpenGroups = 4096;
constexpr int kOpenWaves = 4;
constexpr int64_t kMaxSplit = 64;
inline int64_t full_groups(int64_t nrays) { return (nrays + kMaxGroupRays - 1) / kMaxGroupRays; }
inline bool walk_opens(int64_t nrays, const TreeStorage& ts, bool adjoint = false)
{
    const int64_t groups = full_groups(nrays), n = ts.n;
    double reach = groups < 512 ? 20.0 : 8.0;
    if (adjoint && n < 32768 && groups >= 128) reach = 8.0;
    if (adjoint && ts.uneven && n >= 8192 && groups < 1024) reach = 40.0;
    const double leaf = groups < (adjoint ? 128 : 512) ? ts.params.leaf_size : 0.5 * ts.params.leaf_size;
    return n >= kOpenParticles && n * ts.params.theta * ts.params.theta < reach * std::max(16.0, leaf);
}
// Box ranges of at least 64 boxes that make up to `groups` workgroups.
inline int open_split(int64_t nrays, const TreeStorage& ts, int64_t groups)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>(groups / full_groups(nrays), ts.ncells / 64));
}

inline WalkShape walk_shape(int64_t nrays, const TreeStorage& ts, bool adjoint = false)
{
    const int64_t n = ts.n;
    if (walk_opens(nrays, ts, adjoint) && full_groups(nrays) < kOpenGroups)
        return WalkShape{kMaxGroupRays, kOpenWaves, (int)std::min<int64_t>(kMaxSplit, open_split(nrays, ts, kOpenGroups))};
    const int64_t min_groups = n < 131072 ? 256 : (n < 524288 ? 512 : 1024);
    int64_t fill = n < 32768 ? 8192 : (n < 524288 ? 20480 : 40960);
    if (ts.uneven && n >= kUnevenParticles) fill *= 4;
    WalkShape s{kMaxGroupRays, 1, 1};
    while (s.rays > 4 && nrays < min_groups * s.rays) s.rays /= 2;
    const int64_t groups = (nrays + s.rays - 1) / s.rays;
    while (s.waves < 16 && 2 * s.waves * groups <= fill && s.waves * kWaveParticles < n) s.waves *= 2;
    return s;
}

// Whether a walk expands far boxes over its ray groups (farfield.hpp).  With fewer rays
// than kFarRays the groups of scattered rays are too wide to have many far boxes, and a
// ray's result keeps not depending on its group.  On a small tree a group's few far
// boxes cost less one by one than its expansion's evaluation (2e6 rays: 20 particles 190 us with,
// 181 without; 60 particles 267, 255; 200 particles in 30 to 70 boxes 399, 395; 1,000
// particles 728, 853).
constexpr int64_t kFarRays = 65536;
constexpr int64_t kFarBoxes = 64;
inline bool walk_far(int64_t nrays, const TreeStorage& ts)
{
    return nrays >= kFarRays && ts.ncells >= kFarBoxes && !walk_opens(nrays, ts);
}

// The same for the adjoint walk: at most 8 wavefronts, whose LDS (a ray table
// each) still fits twice on a CU, and fewer on a small lens, where all groups' wavefronts queue on
// the same few particles' atomics, the more so the more rays there are (1, 2, 4, 8 wavefronts, in
// us: 300 particles, 1e4 rays 273, -, 169, -; 1.3e5 rays 344, -, 593, -; 1,200 smoothed
// particles, 1.3e5 rays 295, 397, 400, -).  A walk that opens most of the tree has full ray
// masks, for which one wavefront per range, lanes as rays, is the better particle pass from 128
// groups, or from 320 on a small lens of leaves that fill the lanes (theta = 0: 2e5 rays on 2,500
// particles 2,012 us with four, 1,058 with one; 3,000 rays 115, 206; 1.5e4 rays at r = 6 on 3,000
// particles 120 to 208, 246 to 340, on 1.2e4 223 to 326, 322 to 455, on 5e4 points or halo equal, on
// an uneven lens 632, 511, on 2e5 particles 2,206, 1,588; 3e4 rays, theta = 0.04 on 1.2e4 568,
// 419; leaves of 2, 1.5e4 rays on 1.2e4 particles 585, 341).
constexpr int64_t kOpenSoloGroups = 32768;
inline WalkShape adjoint_shape(int64_t nrays, const TreeStorage& ts)
{
    if (walk_opens(nrays, ts, true) && full_groups(nrays) >= (ts.n < 32768 && ts.params.leaf_size >= 8 ? 320 : 128))
        return WalkShape{kMaxGroupRays, 1, open_split(nrays, ts, kOpenSoloGroups)};
    WalkShape s = walk_shape(nrays, ts, true);
    if (s.split > 1) return s;
    const int64_t share = nrays >= kFarRays && !ts.uneven ? 8 * kWaveParticles : kWaveParticles;
    if (s.waves > 8) s.waves = 8;
    while (s.waves > 1 && s.waves * share > ts.n) s.waves /= 2;
    return s;
}

glm_status shoot_device(const TreeStorage& ts, const double* rx, const double* ry, int64_t nrays, float* a1,
                        float* a2, float* k, float* g1, float* g2, int32_t* counts, uint32_t flags, void* ws,
                        hipStream_t st);

glm_status shoot_indexed_device(const TreeStorage& ts, const double* cx, const double* cy, const int32_t* idx,
                                int64_t count, float* a1, float* a2, float* ka, float* g1, float* g2, uint32_t flags,
                                void* ws, hipStream_t st);

// alpha and the potential psi (and the time delay when td is not NULL) of
// the rays.
glm_status potential_device(const TreeStorage& ts, const double* rx, const double* ry, int64_t nrays, float* a1,
                            float* a2, float* psi, float* td, uint32_t flags, void* ws, hipStream_t st);

// kind: kKindGauss (q = cutoff) or kKindNfw (s = sizes, q = concentration)
glm_status direct_device(const double* x, const double* y, const double* m, const double* s, int64_t n, double q,
                         int kind, const double* rx, const double* ry, int64_t nrays, int fp64, void* const out5[5],
                         hipStream_t st);

// Cotangents: ga1, ga2 = dL/dalpha, gk = dL/dkappa, gg1, gg2 = dL/dgamma (each nullable: zero).
// The workspace holds the ray staging, then the box adjoints and the
// per-particle direct-term sums.
size_t adjoint_workspace_bytes(const TreeStorage& ts, int64_t nrays);
glm_status adjoint_device(const TreeStorage& ts, const double* rx, const double* ry, int64_t nrays, const float* ga1,
                          const float* ga2, const float* gk, const float* gg1, const float* gg2, double* dm,
                          double* dx, double* dy, double* ds, uint32_t flags, void* ws, hipStream_t st);

} // namespace glm
