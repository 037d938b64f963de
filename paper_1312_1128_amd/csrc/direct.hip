// Plain direct summation over every particle (the theta = 0 limit of the
// tree, Sec. 5.1), FP32 terms summed in FP64, or FP64 throughout, for truncated
// Gaussians or truncated NFW halos (and point masses with either).
//
// A workgroup of 16 (or 4) wavefronts serves RB rays.  Particles stream through LDS in
// tiles; lane (ray, sub) of wavefront w takes every kth particle of a tile,
// k = (wavefronts) * 64 / RB, and the partial sums meet at the end (lanes of a ray by
// shuffles, wavefronts in LDS, in wavefront order).  One thread per ray left the
// chip mostly idle below about 500,000 rays: 20,480 validation rays made 80 workgroups
// for 256 compute units.
#include <float.h>
#include <math.h>

#include <algorithm>

#include "eval.hpp"
#include "walk.hpp"

namespace glm {

namespace {

// q: Gaussian cutoff or halo concentration; norm: 1 / C or 1 / g(c)
template <int KIND>
__device__ inline void make_rec(PRec& r, double x, double y, double m, double s, double q, double norm, uint32_t idx)
{
#pragma clang fp contract(off)
    const double qs = KIND == kKindNfw ? s : q * s;
    r.x = x;
    r.y = y;
    r.qs2 = s > 0.0 ? qs * qs : 0.0;
    r.m = (float)m;
    r.mC = (float)(m * norm);
    r.h = s > 0.0 ? (float)(KIND == kKindNfw ? q / s : 1.0 / (2.0 * s * s)) : 0.0f;
    r.meta = idx; // not listed: the profile inside the support, a point outside
}

// Wavefronts of a workgroup (a tile is one particle per thread): 16 where few
// rays share a workgroup; 4 with 64 rays, where there are workgroups enough and
// fewer wavefronts wait for one another at the tiles' barriers (halos, whose
// lanes diverge: 2.62e5 rays and 30,000 halos 23.2 ms with 16 wavefronts).
__host__ __device__ constexpr int dir_waves(int rb) { return rb == kWave ? 4 : 16; }

// Partial sums v[0 .. NV) of the lanes and wavefronts that share the
// workgroup's RB rays, summed into the lanes of wavefront 0 below RB (true there).
template <int RB, int NV>
__device__ inline bool direct_sum(double* v, double* lds)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
    for (int o = kWave / 2; o >= RB; o >>= 1)
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] += __shfl_xor(v[i], o, kWave);
    __syncthreads(); // the tile is free
    if (w > 0 && lane < RB)
#pragma unroll
        for (int i = 0; i < NV; ++i) lds[((w - 1) * NV + i) * RB + lane] = v[i];
    __syncthreads();
    if (w > 0 || lane >= RB) return false;
    for (int u = 0; u < dir_waves(RB) - 1; ++u)
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] += lds[(u * NV + i) * RB + lane];
    return true;
}

// x of the massless records that stand in a tile's places without a particle (a step takes
// several places at once, the last one's may be such): far from every ray, while its square is
// still finite.  (At the origin, 1 / r^2 of a ray next to it overflows, and 0 inf is no number.)
constexpr double kNowhere = 1e100;

template <bool AONLY, int KIND, int RB>
__global__ __launch_bounds__(kWave* dir_waves(RB)) void k_direct32(const double* __restrict__ x, const double* __restrict__ y,
                                                         const double* __restrict__ m, const double* __restrict__ s,
                                                         int n, double q, double norm, const double* __restrict__ rx,
                                                         const double* __restrict__ ry, int64_t nr,
                                                         float* __restrict__ a1, float* __restrict__ a2,
                                                         float* __restrict__ ka, float* __restrict__ g1,
                                                         float* __restrict__ g2)
{
    constexpr int SUB = kWave / RB, NV = AONLY ? 2 : 5, kDirWaves = dir_waves(RB), kDirTile = kWave * kDirWaves;
    __shared__ __align__(16) char lds[sizeof(PRec) * kDirTile];
    static_assert(sizeof(lds) >= sizeof(double) * (kDirWaves - 1) * NV * RB, "the sums fit the tile");
    PRec* tile = reinterpret_cast<PRec*>(lds);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int64_t r = (int64_t)blockIdx.x * RB + lane % RB;
    const double X = r < nr ? rx[r] : 0.0, Y = r < nr ? ry[r] : 0.0;
    Acc A = {};
    for (int64_t base = 0; base < n; base += kDirTile) {
        const int64_t j = base + threadIdx.x;
        PRec t;
        if (j < n) make_rec<KIND>(t, x[j], y[j], m[j], s ? s[j] : 0.0, q, norm, (uint32_t)j);
        else make_rec<KIND>(t, kNowhere, 0.0, 0.0, 0.0, q, norm, 0u);
        __syncthreads(); // the previous tile is done
        tile[threadIdx.x] = t;
        __syncthreads();
        const int cnt = (int)(n - base < kDirTile ? n - base : kDirTile);
        for (int k = w * SUB; k < cnt; k += kDirWaves * SUB)
            leaf_particle<AONLY, true, false, KIND>(tile[k + lane / RB], X, Y, A);
    }
    if constexpr (!AONLY) join_shear(A);
    double v[5] = {alpha1(A), alpha2(A), A.k, A.g1, A.g2};
    if (!direct_sum<RB, NV>(v, reinterpret_cast<double*>(lds)) || r >= nr) return;
    a1[r] = (float)v[0];
    a2[r] = (float)v[1];
    if (!AONLY) {
        ka[r] = (float)v[2];
        g1[r] = (float)v[3];
        g2[r] = (float)v[4];
    }
}

// 1 / v to FP64 rounding (about 1 ulp): the hardware estimate and two Newton
// steps, 5 instructions for a division's dozen; outside the range where the
// steps cannot over- or underflow, the division.
__device__ inline double recip64(double v)
{
    double r = __builtin_amdgcn_rcp(v);
    double e = fma(-v, r, 1.0);
    r = fma(r, e, r);
    e = fma(-v, r, 1.0);
    r = fma(r, e, r);
    if (__any(!(v >= 0x1p-900 && v <= 0x1p900))) r = v >= 0x1p-900 && v <= 0x1p900 ? r : 1.0 / v;
    return r;
}

// FP64: the brute-force sum term by term (Sec. 3.1 kernel or the NFW halo of
// Sec. 3.2 inside the support, Sec. 3.5 point mass outside).  C: the Gaussian
// normalisation 1 - exp(-q^2/2), or g(c) for halos.  FP64 VALU bound: a point
// pair takes one reciprocal of r^2 and about 25 FP64 operations (it took four
// divisions); the profile is evaluated where some lane is inside a support.
// 20,480 rays on 2e5 smoothed particles: 49.3 ms with one thread per ray, 6.5 ms now.
template <bool AONLY, int KIND, int RB>
__global__ __launch_bounds__(kWave* dir_waves(RB)) void k_direct64(const double* __restrict__ x, const double* __restrict__ y,
                                                         const double* __restrict__ m, const double* __restrict__ s,
                                                         int n, double q, double C, const double* __restrict__ rx,
                                                         const double* __restrict__ ry, int64_t nr,
                                                         double* __restrict__ a1, double* __restrict__ a2,
                                                         double* __restrict__ ka, double* __restrict__ g1,
                                                         double* __restrict__ g2)
{
    constexpr int SUB = kWave / RB, NV = AONLY ? 2 : 5, kDirWaves = dir_waves(RB), kDirTile = kWave * kDirWaves;
    __shared__ __align__(16) double sums[5 * kDirTile]; // the tile, then the sums
    double2* txy = reinterpret_cast<double2*>(sums);    // position
    double2* tmq = txy + kDirTile;                      // mass and squared support
    double* ts = sums + 4 * kDirTile;
    static_assert(5 * kDirTile >= (kDirWaves - 1) * NV * RB, "the sums fit the tile");
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int64_t r = (int64_t)blockIdx.x * RB + lane % RB;
    const double X = r < nr ? rx[r] : 0.0, Y = r < nr ? ry[r] : 0.0;
    double sa1 = 0, sa2 = 0, sk = 0, sg1 = 0, sh2 = 0; // sh2: half of -gamma2
    for (int64_t base = 0; base < n; base += kDirTile) {
        const int64_t j = base + threadIdx.x;
        const double sj = (j < n && s) ? s[j] : 0.0;
        double2 xy = make_double2(kNowhere, 0.0), mq = make_double2(0.0, 0.0);
        if (j < n) {
#pragma clang fp contract(off)
            const double qs = KIND == kKindNfw ? sj : q * sj;
            xy = make_double2(x[j], y[j]);
            mq = make_double2(m[j], sj > 0.0 ? qs * qs : 0.0);
        }
        __syncthreads(); // the previous tile is done
        txy[threadIdx.x] = xy;
        tmq[threadIdx.x] = mq;
        ts[threadIdx.x] = sj;
        __syncthreads();
        const int cnt = (int)(n - base < kDirTile ? n - base : kDirTile);
#pragma unroll(KIND == kKindNfw ? 1 : 2)
        for (int k0 = w * SUB; k0 < cnt; k0 += kDirWaves * SUB) {
            const int k = k0 + lane / RB;
            const double2 p = txy[k], mm = tmq[k];
            double d1, d2;
            const double r2 = sqdist(X, Y, p.x, p.y, &d1, &d2);
            const bool inside = r2 < mm.y;
            // (a particle exactly at the ray, or so near that 1 / r^2 overflows, has no deflection)
            const double ir2 = r2 >= DBL_MIN ? recip64(r2) : 0.0;
            double hh = mm.x * ir2, G = hh; // alpha = hh d, gamma = -G (cos 2phi, sin 2phi)
            if (inside) {
                const double sp = ts[k];
                double K;
                if constexpr (KIND == kKindNfw) {
                    const double hs = q / sp, x2 = r2 * (hs * hs);
                    double gx2, f;
                    nfw_shape<double, 17>(x2, x2 - 1.0, 0.1, &gx2, &f);
                    const double mh2 = mm.x / C * (hs * hs);
                    hh = mh2 * gx2;
                    K = r2 > 0.0 ? 0.5 * mh2 * f : 0.0; // a halo's centre gives nothing
                } else {
                    const double u = r2 / (2.0 * sp * sp);
                    hh = mm.x * (-expm1(-u) / C) * ir2;
                    K = mm.x * exp(-u) / (2.0 * sp * sp * C);
                }
                G = hh - K;
                sk += K;
            }
            sa1 = fma(hh, d1, sa1);
            sa2 = fma(hh, d2, sa2);
            if (!AONLY) {
                sg1 = fma(-G, (d1 * d1 - d2 * d2) * ir2, sg1); // (hh ir2 can leave the range of an FP64)
                sh2 = fma(G, d1 * d2 * ir2, sh2);
            }
        }
    }
    double v[5] = {sa1, sa2, sk, sg1, -2.0 * sh2};
    if (!direct_sum<RB, NV>(v, sums) || r >= nr) return;
    a1[r] = v[0];
    a2[r] = v[1];
    if (!AONLY) {
        ka[r] = v[2];
        g1[r] = v[3];
        g2[r] = v[4];
    }
}

// Rays per workgroup: the most that still leave a few workgroups for every
// compute unit (2e5 particles: 4,096 rays 1.8 ms in 1,024 workgroups of 4 rays;
// 262,144 rays on 3e4 particles 17.4 ms in 4,096 of 64, 20.4 in 16,384 of 16).
inline int direct_rays(int64_t nrays)
{
    return nrays >= 64 * 2048 ? 64 : (nrays >= 16 * 512 ? 16 : 4);
}

glm_status launch_direct(const double* x, const double* y, const double* m, const double* s, int64_t n, double q,
                         int kind, const double* rx, const double* ry, int64_t nrays, int rb, int fp64,
                         void* const out5[5], hipStream_t st)
{
    const double C = kind == kKindNfw ? nfw_g_at(q) : -expm1(-0.5 * q * q);
    const bool aonly = !out5[2] || !out5[3] || !out5[4];
    const dim3 g(ceil_div(nrays, rb)), b(kWave * dir_waves(rb));
#define GLM_DIRECT(KERNEL, AO, KD, NORM)                                                                                \
    do {                                                                                                                \
        if (rb == 64)                                                                                                   \
            hipLaunchKernelGGL((KERNEL<AO, KD, 64>), g, b, 0, st, x, y, m, s, (int)n, q, NORM, rx, ry, nrays, o[0], o[1], \
                               o[2], o[3], o[4]);                                                                       \
        else if (rb == 16)                                                                                              \
            hipLaunchKernelGGL((KERNEL<AO, KD, 16>), g, b, 0, st, x, y, m, s, (int)n, q, NORM, rx, ry, nrays, o[0], o[1], \
                               o[2], o[3], o[4]);                                                                       \
        else                                                                                                            \
            hipLaunchKernelGGL((KERNEL<AO, KD, 4>), g, b, 0, st, x, y, m, s, (int)n, q, NORM, rx, ry, nrays, o[0], o[1], \
                               o[2], o[3], o[4]);                                                                       \
    } while (0)
#define GLM_KINDS(KERNEL, NORM)                              \
    do {                                                     \
        if (kind == kKindNfw) {                              \
            if (aonly) GLM_DIRECT(KERNEL, true, kKindNfw, NORM);   \
            else GLM_DIRECT(KERNEL, false, kKindNfw, NORM);        \
        } else {                                             \
            if (aonly) GLM_DIRECT(KERNEL, true, kKindGauss, NORM); \
            else GLM_DIRECT(KERNEL, false, kKindGauss, NORM);      \
        }                                                    \
    } while (0)
    if (fp64) {
        double* o[5];
        for (int k = 0; k < 5; ++k) o[k] = static_cast<double*>(out5[k]);
        GLM_KINDS(k_direct64, C);
    } else {
        float* o[5];
        for (int k = 0; k < 5; ++k) o[k] = static_cast<float*>(out5[k]);
        GLM_KINDS(k_direct32, 1.0 / C);
    }
#undef GLM_KINDS
#undef GLM_DIRECT
    GLM_HIP(hipGetLastError());
    return GLM_OK;
}

// Rays of one launch: a launch has fewer than 2^32 threads, and a ray up to 4 of them
// where there are so many.
constexpr int64_t kDirectLaunch = 1ll << 29;

} // namespace

glm_status direct_device(const double* x, const double* y, const double* m, const double* s, int64_t n, double q,
                         int kind, const double* rx, const double* ry, int64_t nrays, int fp64, void* const out5[5],
                         hipStream_t st)
{
    const int rb = direct_rays(nrays); // for all of its launches
    for (int64_t at = 0; at < nrays; at += kDirectLaunch) {
        void* o[5];
        for (int k = 0; k < 5; ++k) o[k] = out5[k] ? static_cast<char*>(out5[k]) + at * (fp64 ? 8 : 4) : nullptr;
        const glm_status rc = launch_direct(x, y, m, s, n, q, kind, rx + at, ry + at, std::min(nrays - at, kDirectLaunch),
                                            rb, fp64, o, st);
        if (rc != GLM_OK) return rc;
    }
    return GLM_OK;
}

} // namespace glm
