// Adjoint of the forward tree walk: the push-down to the particles and the
// launches.  The walk itself is in adjoint_walk.hpp.
#include <math.h>

#include "adjoint_walk.hpp"

namespace glm {

namespace {

// Box adjoints -> particles.  One thread per particle walks its ancestors,
// then adds the direct-term gradients the walk gathered.  A box holds Abar_0 ..
// Abar_{P+1} (scaled by r_cm^k) and its centre-of-mass adjoint is Bbar =
// sum_{k <= P} (k + 1) Q_k Abar_{k+1} (dF/dz_cm = sum (k + 1) Q_k w^-(k+2)),
// formed here in FP64.
template <int P>
__global__ __launch_bounds__(kBlock) void k_pushdown(TreeDev T, const double* __restrict__ ms,
                                                    const double* __restrict__ abar, const double* __restrict__ pg,
                                                    double* __restrict__ dm, double* __restrict__ dx,
                                                    double* __restrict__ dy, double* __restrict__ ds)
{
    constexpr int NA = 2 * (P + 1) + 2;
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k >= T.n) return;
    const PRec pr = T.prt[k];
    const int32_t i = T.perm[k]; // original index
    const double mi = ms[k];
    double gm = 0.0, gzr = 0.0, gzi = 0.0;
    int c = 0;
    for (int guard = 0; guard <= kMaxLevel && c < T.ncells; ++guard) {
        const double* ab = abar + (size_t)c * NA;
        bool any = false;
#pragma unroll
        for (int q = 0; q < NA; ++q) any |= ab[q] != 0.0;
        const CellHdr h = T.hdr[c];
        if (any) {
            const double M = T.cM[c];
            const double rcm = (double)T.mom[(size_t)c * mom_stride(P) + 1];
            const double* Q = T.cq + (size_t)c * (P + 1) * 2;
            const double dr = pr.x - h.cx, di = pr.y - h.cy;
            double Br = 0.0, Bi = 0.0;
            {
                double irk = 1.0 / rcm; // r_cm^-(k+1)
                const double irc = irk;
                for (int kk = 0; kk <= P; ++kk) {
                    const double Ar = ab[2 * (kk + 1)] * irk, Ai = ab[2 * (kk + 1) + 1] * irk;
                    const double qr = Q[2 * kk], qi = Q[2 * kk + 1];
                    Br += (kk + 1) * (qr * Ar - qi * Ai);
                    Bi += (kk + 1) * (qr * Ai + qi * Ar);
                    irk *= irc;
                }
            }
            // sm = sum_k Abar_k dQ_k/dm + Bbar d/M ; sz = sum_k Abar_k dQ_k/dz + Bbar m/M
            // (one reciprocal of M per box: an FP64 division is a long instruction sequence)
            const double iM = M > 0.0 ? 1.0 / M : 0.0, miM = mi * iM;
            double smr = 0.0, smi = 0.0, szr = 0.0, szi = 0.0;
            double dkr = 1.0, dki = 0.0, dkm1r = 0.0, dkm1i = 0.0; // d^k, d^(k-1)
            double irk = 1.0;                                      // r_cm^-k
            const double irc = 1.0 / rcm;
            for (int kk = 0; kk <= P; ++kk) {
                const double Ar = ab[2 * kk] * irk, Ai = ab[2 * kk + 1] * irk;
                double tmr = dkr, tmi = dki;                     // d^k
                double tzr = kk * mi * dkm1r, tzi = kk * mi * dkm1i; // k m d^(k-1)
                if (M > 0.0 && kk > 0) {
                    const double qr = Q[2 * (kk - 1)], qi = Q[2 * (kk - 1) + 1];
                    // k Q_{k-1} d / M and k Q_{k-1} m / M
                    tmr -= kk * (qr * dr - qi * di) * iM;
                    tmi -= kk * (qr * di + qi * dr) * iM;
                    tzr -= kk * qr * miM;
                    tzi -= kk * qi * miM;
                }
                smr += Ar * tmr - Ai * tmi;
                smi += Ar * tmi + Ai * tmr;
                szr += Ar * tzr - Ai * tzi;
                szi += Ar * tzi + Ai * tzr;
                dkm1r = dkr;
                dkm1i = dki;
                const double nr = dkr * dr - dki * di, ni = dkr * di + dki * dr;
                dkr = nr;
                dki = ni;
                irk *= irc;
            }
            if (M > 0.0) {
                smr += (Br * dr - Bi * di) * iM;
                smi += (Br * di + Bi * dr) * iM;
                szr += Br * miM;
                szi += Bi * miM;
            }
            gm += smr;
            gzr += szr;
            gzi += szi;
        }
        if (h.info & kInfoLeaf) break;
        // descend into the child whose Morton range holds position k (the four
        // children's ranges load together)
        const int4 kc = *reinterpret_cast<const int4*>(T.kids + 4 * (size_t)c);
        const int cu[4] = {kc.x, kc.y, kc.z, kc.w};
        int ch = -1;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (cu[u] >= 0 && k >= T.cbeg[cu[u]] && k < T.cend[cu[u]]) ch = cu[u];
        if (ch < 0) break;
        c = ch;
    }
    // plus the direct terms the walk gathered for this particle
    double q[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < kPgCopies; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) q[j] += pg[(size_t)r * 4 * T.n + 4 * (size_t)k + j];
    if (dm) dm[i] += gm + q[0];
    if (dx) dx[i] += gzr + q[1];
    if (dy) dy[i] += q[2] - gzi;
    if (ds) ds[i] += q[3];
}

__global__ void k_fill_zero(double* p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

// copy 0 of the box adjoints += copies 1 .. kAdjCopies - 1 (n words each)
__global__ void k_sum_copies(double* p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    double s = p[i];
#pragma unroll
    for (int r = 1; r < kAdjCopies; ++r) s += p[(size_t)r * n + i];
    p[i] = s;
}

// FP64 scratch words: kAdjCopies copies of the box adjoints (NA per box),
// then 4 direct-term gradients per particle.
size_t adjoint_scratch_words(const TreeStorage& ts)
{
    const int NA = 2 * (ts.params.order + 1) + 2;
    return (size_t)kAdjCopies * ts.ncells * NA + 4 * (size_t)kPgCopies * ts.n;
}

template <int P>
glm_status launch_adjoint(const TreeStorage& ts, const StagedRays& sr, int64_t nrays, const CotIn& ci, double* dm,
                          double* dx, double* dy, double* ds, double* abar,
                          hipStream_t st)
{
    constexpr int NA = 2 * (P + 1) + 2;
    const size_t words = adjoint_scratch_words(ts);
    const int64_t nbox = (int64_t)ts.ncells * NA;
    double* pg = abar + (size_t)kAdjCopies * nbox;
    hipLaunchKernelGGL(k_fill_zero, dim3(ceil_div((int64_t)words, kBlock)), dim3(kBlock), 0, st, abar, (int64_t)words);
    const AdjointArgs a{ts.dev, sr.xs, sr.ys, sr.perm, nrays, ci, pg, abar, adjoint_shape(nrays, ts), walk_far(nrays, ts), st};
    if (ci.gk || ci.gg1 || ci.gg2) launch_adjoint_all(a);
    else launch_adjoint_alpha(a);
    hipLaunchKernelGGL(k_sum_copies, dim3(ceil_div(nbox, (int64_t)kBlock)), dim3(kBlock), 0, st, abar, nbox);
    hipLaunchKernelGGL((k_pushdown<P>), dim3(ceil_div(ts.n, kBlock)), dim3(kBlock), 0, st, ts.dev, ts.ms, abar, pg, dm,
                       dx, dy, ds);
    GLM_HIP(hipGetLastError());
    return GLM_OK;
}

} // namespace

size_t adjoint_workspace_bytes(const TreeStorage& ts, int64_t nrays)
{
    return ray_layout(nrays).bytes + sizeof(double) * adjoint_scratch_words(ts);
}

glm_status adjoint_device(const TreeStorage& ts, const double* rx, const double* ry, int64_t nrays, const float* ga1,
                          const float* ga2, const float* gk, const float* gg1, const float* gg2, double* dm,
                          double* dx, double* dy, double* ds, uint32_t flags, void* ws, hipStream_t st)
{
    if (nrays == 0) return GLM_OK;
    StagedRays sr{rx, ry, nullptr};
    const RayLayout L = ray_layout(nrays);
    if (flags & GLM_RAYS_STAGED) {
        sr = staged_rays_view(nrays, ws, L); // glm_stage_rays left them at the workspace's start
    } else if (!(flags & GLM_RAYS_ORDERED)) {
        glm_status rc = stage_rays(rx, ry, nrays, ws, L, &sr, st);
        if (rc != GLM_OK) return rc;
    }
    double* abar = reinterpret_cast<double*>(static_cast<char*>(ws) + L.bytes);
#define GLM_CASE(PP)                                                                                              \
    case PP:                                                                                                      \
        return launch_adjoint<PP>(ts, sr, nrays, CotIn{ga1, ga2, gk, gg1, gg2}, dm, dx, dy, ds, abar, st);
    switch (ts.params.order) {
        GLM_CASE(0) GLM_CASE(1) GLM_CASE(2) GLM_CASE(3) GLM_CASE(4) GLM_CASE(5) GLM_CASE(6)
        GLM_CASE(7) GLM_CASE(8) GLM_CASE(9) GLM_CASE(10) GLM_CASE(11) GLM_CASE(12)
        default: return fail(GLM_ESTATE, "unsupported order");
    }
#undef GLM_CASE
}

} // namespace glm
