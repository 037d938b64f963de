// Smoothing lengths on gfx950 (Sec. 3.1): for every particle of a built tree
// the 2D distance to its k-th nearest other particle (the particle itself
// excluded, coincident particles counted at distance 0).
//
// One wavefront serves 64 particles that are neighbours in Morton order (one
// per lane).  Each lane keeps the k smallest squared distances found so far
// (knn_list.hpp), starting from its own k neighbours on either side along the
// Morton order.  (Started from the group's 64 particles, the few lanes on the far
// side of one of the curve's jumps had no bound but the distance across it, and
// their wavefront scanned a good part of the lens: at 1e6 particles, k = 32, half
// a wavefront per SIMD was running on average over 11 ms.)  Then the wave walks
// the tree: it enters a box if some lane's distance to the box square is below
// that lane's current k-th distance, and scans the particles of the leaves it
// reaches.  Every distance is FP64 and formed exactly as in the definition, so
// the result is the k-th smallest FP64 distance.
#include <math.h>

#include "build.hpp"
#include "knn_list.hpp"

namespace glm {

namespace {

__device__ inline double knn_d2(double X, double Y, double px, double py)
{
#pragma clang fp contract(off)
    const double dx = X - px, dy = Y - py;
    return dx * dx + dy * dy;
}

constexpr int kKnnStack = 384;

template <int KC>
__global__ __launch_bounds__(kBlock) void k_knn(TreeDev T, BoxArrays b, double x0, double y0, double S,
                                               double margin, int k, double* __restrict__ s_out)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int n = T.n;
    const int g0 = (blockIdx.x * (kBlock / kWave) + w) * kWave; // first particle of the group
    if (g0 >= n) return;
    const int j = knn_particle(g0, lane, n);
    const bool valid = lane < n - g0;
    const PRec me = T.prt[j];
    const double X = me.x, Y = me.y;
    __shared__ double lds[kBlock / kWave][kKnnQueue * kWave];
    __shared__ int stack[kBlock / kWave][kKnnStack];
    KnnList<KC> L(k, lds[w], lane);

    // each lane's k neighbours along the Morton order on either side first
    for (int o = 1; o <= k; ++o) {
        const KnnSeed sd = knn_seed(j, o, n);
        const PRec &pa = T.prt[sd.before], &pb = T.prt[sd.after];
        const double da = knn_d2(X, Y, pa.x, pa.y), db = knn_d2(X, Y, pb.x, pb.y);
        L.insert(sd.has_before ? da : INFINITY);
        L.insert(sd.has_after ? db : INFINITY);
    }

    // then every box that some lane still needs
    const double gx0 = wave_min(X), gx1 = wave_max(X), gy0 = wave_min(Y), gy1 = wave_max(Y); // (idle lanes: particle g0)
    int* stk = stack[w];
    int top = 1;
    if (lane == 0) stk[0] = 0;
    wave_lds_sync();
    while (top > 0) {
        top = __builtin_amdgcn_readfirstlane(top);
        const int m = knn_take(top, kKnnStack, 4, kMaxLevel);
        top -= m;
        const bool has = lane < m;
        const int c = has ? stk[top + lane] : 0;
        const double side = ldexp(S, -b.level[c]);
        const double cx = x0 + ((double)b.ix[c] + 0.5) * side, cy = y0 + ((double)b.iy[c] + 0.5) * side;
        const double hs = 0.5 * side + margin;
        const int leaf = b.leaf[c], beg = b.beg[c], end = b.end[c];
        const int4 kc = *reinterpret_cast<const int4*>(T.kids + 4 * (size_t)c);
        const double far = wave_max(valid ? L.bound() : 0.0);
        bool keep = has;
        {
            const double dx = fmax(fmax(gx0 - cx, cx - gx1) - hs, 0.0), dy = fmax(fmax(gy0 - cy, cy - gy1) - hs, 0.0);
            keep = keep && dx * dx + dy * dy < far;
        }
        bool push = false;
        uint64_t todo = __ballot(keep);
        while (todo) {
            const int u = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const double h = knn_bcast(hs, u);
            const double dx = fmax(fabs(X - knn_bcast(cx, u)) - h, 0.0), dy = fmax(fabs(Y - knn_bcast(cy, u)) - h, 0.0);
            if (!__any(valid && dx * dx + dy * dy < L.bound())) continue;
            if (!__builtin_amdgcn_readlane(leaf, u)) {
                push = push || lane == u;
                continue;
            }
            const int lb = __builtin_amdgcn_readlane(beg, u), le = __builtin_amdgcn_readlane(end, u);
            for (int base = lb; base < le; base += kWave) { // (a leaf at the depth cap may exceed 64)
                const int p = base + lane;
                const bool in = p < le;
                double px = 0.0, py = 0.0;
                if (in) {
                    px = T.prt[p].x;
                    py = T.prt[p].y;
                }
                const double ex = fmax(fmax(gx0 - px, px - gx1), 0.0), ey = fmax(fmax(gy0 - py, py - gy1), 0.0);
                uint64_t near = __ballot(in && (ex * ex + ey * ey) * (1.0 - 1e-12) < far);
                while (near) {
                    const int v = __ffsll((unsigned long long)near) - 1;
                    near &= near - 1;
                    const int q = base + v;
                    const bool seen = q - j <= k && j - q <= k; // already in this lane's list, or itself
                    const double d2 = knn_d2(X, Y, knn_bcast(px, v), knn_bcast(py, v));
                    L.offer(seen ? INFINITY : d2);
                }
            }
        }
        const int kid[4] = {kc.x, kc.y, kc.z, kc.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool on = push && kid[u] >= 0;
            const uint64_t kb = __ballot(on);
            if (on) stk[top + knn_rank(kb)] = kid[u];
            top += __popcll(kb);
        }
        wave_lds_sync();
    }
    L.flush();
    if (valid) s_out[T.perm[j]] = sqrt(L.bound());
}

} // namespace

glm_status knn_device(const TreeStorage& ts, int k, double* s_out, hipStream_t st)
{
    const int64_t groups = ((int64_t)ts.n + kWave - 1) / kWave;
    const dim3 g(ceil_div(groups, kBlock / kWave)), blk(kBlock);
    // box squares widened by far more than the rounding of the quantisation,
    // so that pruning never drops a particle of the box
    const double margin = 1e-12 * ts.side;
    if (k <= 16)
        hipLaunchKernelGGL((k_knn<16>), g, blk, 0, st, ts.dev, ts.b, ts.x0, ts.y0, ts.side, margin, k, s_out);
    else if (k <= 32)
        hipLaunchKernelGGL((k_knn<32>), g, blk, 0, st, ts.dev, ts.b, ts.x0, ts.y0, ts.side, margin, k, s_out);
    else
        hipLaunchKernelGGL((k_knn<64>), g, blk, 0, st, ts.dev, ts.b, ts.x0, ts.y0, ts.side, margin, k, s_out);
    GLM_HIP(hipGetLastError());
    return GLM_OK;
}

} // namespace glm
