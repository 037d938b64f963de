// Local expansion of far boxes over one 64-ray group.
//
// A box that every ray of the group accepts, with centre of mass at distance d
// from the group's centre, has no singularity of its series nearer than
// d (its sources: d - r_cm), so over the group (radius a) its field is a power
// series in z = delta / a (delta: a ray's offset from the group's centre),
//   alpha1 - i alpha2 = F(w0 + delta) = sum_j L_j z^j,
//   L_j = v e^j sum_k C(k + j, j) u_k,  v = 1 / w0, e = -a v, u_k = (Q_k / r_cm^k) t^k, t = r_cm v,
// the exact re-expansion of the box's own multipole series (order P), cut at
// order kFarOrder.  With a / (d - r_cm) < kFarRatio = 0.3 and order 15 the first
// term left out is at most 0.3^16 = 4e-9 of the field and 16 0.3^15 = 2.3e-7 of
// its derivative, and the rest of the derivative's series sums to 3.4e-7 of it: below FP32
// rounding for alpha, a few roundings for gamma, in the worst direction at the edge of a
// group at the limit.  One box evaluated per ray in FP32 has more
// than that: a clump under a 400^2 grid, rays 18 spacings off (groups at the
// limit), error of gamma over gamma, far boxes and without, rms 1.07e-7 and 1.23e-7, largest
// 3.4e-7 and 3.4e-7; 24 to 40 spacings off 9.4e-8, 1.24e-7; of alpha 3.6e-8, 6.5e-8.  The 1e6-particle
// halo (theta = 0.2, order 12, 400^2 rays against the FP64 direct sum): alpha 2.7e-8, 2.9e-8,
// gamma 6.3e-8, 6.5e-8; ratios of 0.28, 0.27 and 0.25 give the same to 1%.  Every
// ray's decisions are unchanged; only the evaluation of accepted boxes is.
//
// Per ray a box costs about 95 instructions of a wavefront; here the lanes are
// boxes, 64 at a time cost about 600, so a box costs about 10.
#pragma once

#include <float.h>

#include "eval.hpp"
#include "lanesum.hpp"

namespace glm {

constexpr int kFarOrder = 15;
constexpr int kFarWords = 2 * (kFarOrder + 1);
constexpr float kFarRatio = 0.3f;

// One group of 64 rays: its bounding box, the lanes that carry a ray, its
// centre and radius, and whether far boxes are expanded.
struct RayGroup {
    double gx0, gx1, gy0, gy1;
    uint64_t full;
    double ox, oy; // centre
    float a, inva; // radius and its reciprocal
    bool far;
};

__device__ inline RayGroup ray_group(double X, double Y, bool valid, bool far)
{
    RayGroup g{};
    g.gx0 = wave_min(valid ? X : INFINITY);
    g.gx1 = wave_max(valid ? X : -INFINITY);
    g.gy0 = wave_min(valid ? Y : INFINITY);
    g.gy1 = wave_max(valid ? Y : -INFINITY);
    g.full = __ballot(valid);
    g.far = far;
    if (far) {
        g.ox = 0.5 * (g.gx0 + g.gx1);
        g.oy = 0.5 * (g.gy0 + g.gy1);
        const double d1 = X - g.ox, d2 = Y - g.oy;
        g.a = (float)sqrt(wave_max(valid ? d1 * d1 + d2 * d2 : 0.0));
        g.inva = 1.0f / g.a;
        // no scale to expand on with all rays at one point, nor with a ray at infinity (the
        // rays' offsets over the radius would be NaN, also with no box expanded)
        g.far = g.a > 1e-30f && g.a <= FLT_MAX;
    }
    return g;
}

// Whether a box that every ray accepts may go through the local expansion:
// a / (d - r_cm) < kFarRatio, r_cm = theta r_cut.  (Strict, so that a radius or
// distance whose square overflows gives no far boxes.)
__device__ inline bool is_far(const RayGroup& g, const CellHdr& h, float theta)
{
    if (!g.far) return false;
    const float f1 = (float)(g.ox - h.cx), f2 = (float)(g.oy - h.cy);
    const float need = g.a * (1.0f / kFarRatio) + theta * sqrtf((float)h.rcut2);
    return fmaf(f1, f1, f2 * f2) > need * need;
}

__host__ __device__ constexpr float far_binomial(int k, int j)
{
    double r = 1.0;
    for (int i = 1; i <= j; ++i) r = r * (double)(k + i) / (double)i; // C(k + j, j)
    return (float)r;
}

// Offset of the group's centre from box c's centre of mass, per lane: v = 1/w0
// (0 on lanes without a box) and |w0|^2.  v in FP64: its error is the same for every ray
// of the group, and with FP32's the 1e6-particle halo's alpha had 5% more error than with
// every box evaluated per ray; a few instructions of 600.
struct FarOffset {
    double v1, v2;
    float r2;
};
__device__ inline FarOffset far_offset(const TreeDev& T, const RayGroup& g, int c, bool active)
{
    const double2 cm = *reinterpret_cast<const double2*>(&T.hdr[c].cx);
    const double f1 = active ? g.ox - cm.x : 1.0, f2 = active ? g.oy - cm.y : 0.0;
    const double r2 = fma(f1, f1, f2 * f2);
    double inv = __builtin_amdgcn_rcp(r2);
    inv = fma(inv, fma(-r2, inv, 1.0), inv);
    if (!active) inv = 0.0;
    return FarOffset{f1 * inv, -f2 * inv, (float)r2};
}

// One far box per lane: u_k and the running factor v e^j of its words.
template <int P>
struct FarBox {
    float M, r2;
    float u1[P + 1], u2[P + 1]; // u_k, k = 2 .. P
    float p1, p2;               // v e^j, j the next word
    float e1, e2;
    double v1, v2;

    __device__ void load(const TreeDev& T, const RayGroup& g, int c, bool active)
    {
        const FarOffset o = far_offset(T, g, c, active);
        constexpr int ST = mom_stride(P);
        float mo[ST];
        const float4* mp = reinterpret_cast<const float4*>(T.mom + (size_t)c * ST);
#pragma unroll
        for (int i = 0; i < ST / 4; ++i) {
            const float4 q = mp[i];
            mo[4 * i] = q.x;
            mo[4 * i + 1] = q.y;
            mo[4 * i + 2] = q.z;
            mo[4 * i + 3] = q.w;
        }
        M = mo[0];
        r2 = o.r2;
        v1 = o.v1;
        v2 = o.v2;
        p1 = (float)v1;
        p2 = (float)v2;
        const float t1 = mo[1] * p1, t2 = mo[1] * p2;
        float q1 = t1, q2 = t2;
#pragma unroll
        for (int k = 2; k <= P; ++k) {
            const float n1 = fmaf(q1, t1, -q2 * t2), n2 = fmaf(q1, t2, q2 * t1);
            q1 = n1;
            q2 = n2;
            const float a1 = mo[2 + 2 * (k - 2)], a2 = mo[3 + 2 * (k - 2)];
            u1[k] = fmaf(a1, q1, -a2 * q2);
            u2[k] = fmaf(a1, q2, a2 * q1);
        }
        e1 = -g.a * p1;
        e2 = -g.a * p2;
    }

    // Real part of the box's complex potential at the group's centre.
    __device__ float psi0(bool active) const
    {
        float re = 0.0f;
#pragma unroll
        for (int k = P; k >= 2; --k) re = fmaf(u1[k], 1.0f / (float)k, re);
        return active ? fmaf(0.5f * M, __logf(r2), -re) : 0.0f;
    }

    // The words L_J0 .. L_(J0 + kFarOrder / 2) (Re, Im); J0 = 0 first, then the other half.
    // What FP32 rounds off L_0, the field at the centre, is added to (r1, r2).
    template <int J0>
    __device__ void words(float* L, double& r1, double& r2)
    {
#pragma unroll
        for (int j = J0; j <= J0 + kFarOrder / 2; ++j) {
            float s1 = M, s2 = 0.0f;
#pragma unroll
            for (int k = 2; k <= P; ++k) {
                s1 = fmaf(far_binomial(k, j), u1[k], s1);
                s2 = fmaf(far_binomial(k, j), u2[k], s2);
            }
            L[2 * (j - J0)] = fmaf(p1, s1, -p2 * s2);
            L[2 * (j - J0) + 1] = fmaf(p1, s2, p2 * s1);
            if (j == 0) {
                r1 += fma(v1, (double)s1, -v2 * (double)s2) - (double)L[0];
                r2 += fma(v1, (double)s2, v2 * (double)s1) - (double)L[1];
            }
            const float n1 = fmaf(p1, e1, -p2 * e2), n2 = fmaf(p1, e2, p2 * e1);
            p1 = n1;
            p2 = n2;
        }
    }
};

// The group's local expansion at this lane's ray (L: the FP64 words in LDS),
// added to its sums.  L_0 and L_1, the field and its derivative at the centre,
// stay in FP64.
template <bool AONLY, bool PSI>
__device__ inline void far_eval(const RayGroup& g, const double* L, double X, double Y, Acc& A)
{
    const double dz1 = (X - g.ox) * (double)g.inva, dz2 = (Y - g.oy) * (double)g.inva;
    const float z1 = (float)dz1, z2 = (float)dz2;
    // b = sum_{j>=2} L_j z^(j-2), c = b'
    float b1 = (float)L[2 * kFarOrder], b2 = (float)L[2 * kFarOrder + 1], c1 = 0.0f, c2 = 0.0f;
#pragma unroll
    for (int j = kFarOrder - 1; j >= 2; --j) {
        if constexpr (!AONLY) {
            const float m1 = fmaf(c1, z1, fmaf(-c2, z2, b1)), m2 = fmaf(c1, z2, fmaf(c2, z1, b2));
            c1 = m1;
            c2 = m2;
        }
        const float n1 = fmaf(b1, z1, fmaf(-b2, z2, (float)L[2 * j])), n2 = fmaf(b1, z2, fmaf(b2, z1, (float)L[2 * j + 1]));
        b1 = n1;
        b2 = n2;
    }
    // F = L_0 + z (L_1 + z b)
    const float y1 = fmaf(z1, b1, fmaf(-z2, b2, (float)L[2])), y2 = fmaf(z1, b2, fmaf(z2, b1, (float)L[3]));
    A.a1 += L[0] + (double)fmaf(z1, y1, -z2 * y2);
    A.a2 -= L[1] + (double)fmaf(z1, y2, z2 * y1);
    if constexpr (!AONLY) {
        // a F' = L_1 + z (2 b + z c)
        const float x1 = fmaf(z1, c1, fmaf(-z2, c2, 2.0f * b1)), x2 = fmaf(z1, c2, fmaf(z2, c1, 2.0f * b2));
        A.g1 += (L[2] + (double)fmaf(z1, x1, -z2 * x2)) * (double)g.inva;
        A.g2 -= (L[3] + (double)fmaf(z1, x2, z2 * x1)) * (double)g.inva;
    }
    if constexpr (PSI) {
        // a sum_j L_j z^(j+1) / (j + 1), L_0's part in FP64
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int j = kFarOrder; j >= 1; --j) {
            const float q1 = (float)L[2 * j] * (1.0f / (float)(j + 1)), q2 = (float)L[2 * j + 1] * (1.0f / (float)(j + 1));
            const float n1 = fmaf(s1, z1, fmaf(-s2, z2, q1)), n2 = fmaf(s1, z2, fmaf(s2, z1, q2));
            s1 = n1;
            s2 = n2;
        }
        const float w1 = fmaf(z1, z1, -z2 * z2), w2 = 2.0f * z1 * z2;
        A.ps += (double)g.a * (dz1 * L[0] - dz2 * L[1] + (double)fmaf(s1, w1, -s2 * w2));
    }
}

} // namespace glm
