// Adjoint of the forward tree walk: dL/d(m, x, y, s) of the particles for
// cotangents ga = dL/dalpha of the rays, and optionally gk = dL/dkappa and
// gg = dL/dgamma, on the frozen topology and decisions of the forward walk
// (the same traversal runs again and takes the same FP64 decisions).
//
// Direct terms (leaf particles, big-particle corrections) give particle
// gradients directly:
//   dL/dm_i = ga . alpha_i / m_i,  dL/dz_i = -J_i ga  (alpha depends on x - x_i,
//   J_i = [[k + g1, g2], [g2, k - g1]] of the single particle),
//   dL/ds_i = ga . d alpha_i / d s_i = -m (ga . d) e^-u / (s^3 C) inside.
// An accepted box contributes F = alpha1 - i alpha2 = sum_k Q_k w^-(k+1), so
// with g_hat = ga1 + i ga2 the walk accumulates per box
//   Abar_k r_cm^k = sum_r g_hat v t^k   (v = 1/w, t = r_cm v), k = 0 .. P + 1,
// and the centre-of-mass adjoint sum_r g_hat dF/dz_cm = sum_{k <= P} (k + 1) Q_k Abar_{k+1}
// follows from them in the push-down.  A gamma cotangent adds, with gg_hat =
// gg1 + i gg2 (gamma1 - i gamma2 = F'(w)),
//   Abar_k r_cm^k -= (k + 1) gg_hat v^2 t^k,
// and the same sum then gives its centre-of-mass adjoint -gg_hat F''(w) too;
// kappa gets nothing from a box.
// Direct terms of a circular profile, with u = r^2, A = alpha / d, kappa(u):
//   gamma1 - i gamma2 = a conj(w)^2,  a = (kappa - A)/u,  b = u A'' = dkappa/du - 2a,
//   d kappa / d d_j = 2 (dkappa/du) d_j,
//   d gamma1/d d1 = 2 d1 (b c + a), d gamma1/d d2 = 2 d2 (b c - a),
//   d gamma2/d d1 = 2 d2 (b (1 + c) + a), d gamma2/d d2 = 2 d1 (b (1 - c) + a),  c = cos 2phi;
// dkappa/du = -h kappa and d kappa/ds - dA/ds = m e^-x x / (C s^3) for the Gaussian (x = h u).
// A push-down pass gives every particle its share through
//   dQ_k/dm_i = d^k - k Q_{k-1} d / M,  dQ_k/dz_i = k m_i d^(k-1) - k Q_{k-1} m_i / M,
//   dz_cm/dm_i = d / M,  dz_cm/dz_i = m_i / M  (d = z_i - z_cm; all holomorphic).
// Per-lane terms are reduced across the wavefront before one FP64 atomic per
// quantity; the particles' terms are formed and reduced in FP64, so that the
// point-mass parts of big-particle pairs cancel like the forward's balance.
#pragma once

#include <type_traits>

#include "traverse.hpp"

namespace glm {

// The wavefronts add their box adjoints into kAdjCopies copies (wavefront w
// into copy w % kAdjCopies), summed into copy 0 before the push-down: the boxes
// near the root are accepted by nearly every ray group, and with one copy their
// FP64 atomics all queued on the same few lines.
constexpr int kAdjCopies = 8;
// Likewise the per-particle direct-term sums, in kPgCopies copies that the
// push-down adds up.
constexpr int kPgCopies = 4;

// Cotangents of one ray: alpha (g1, g2), kappa (k), gamma (h1, h2).
struct Cot {
    float g1, g2, k, h1, h2;
};

// Gradient words of one particle for this lane, from its profile in unit mass: A, G = A - kappa, K =
// kappa and R = u dkappa/du (u = r^2), ird = 1 / u, offset d, w1 = d1^2 - d2^2, w2 = d1 d2.  With
// J = h1 cos 2phi + h2 sin 2phi,
//   W0 = A (g . d) + k K - G J                                            dL/dm,
//   W1 = [G (g1 w1 + 2 g2 w2) - 2 (d1 V - G (h1 d1 + h2 d2))] / u - K g1  dL/dx / m,
//   W2 = [G (2 g1 w2 - g2 w1) - 2 (d2 V - G (h2 d1 - h1 d2))] / u - K g2  dL/dy / m,
//   W3 = K (g . d) + k (K + R) + J R,     V = k R + (R + 2 G) J           dL/ds / (-m c),
// c as in word_factor: the a, b and dkappa/du of the file's head times u, so that nothing divides by
// u twice.  All of it is linear in (A, G, K, R): a big-particle
// correction takes the point mass off A and G, and its words then cancel those of the leaf to FP64
// rounding.  FP64 throughout: an FP64 FMA issues like an FP32 one here, and the widened cotangents
// and squares are shared by the four words (POINT: K = R = 0); the factors that a particle's rays have in common
// (m, -m c) are left to after the sum over the rays.
template <bool KG, bool POINT>
__device__ inline void grad_words(const Cot& cg, double d1, double d2, double w1, double w2, double ird, double A,
                                  double G, double K, double R, double* W)
{
    const double g1 = (double)cg.g1, g2 = (double)cg.g2, t2 = w2 + w2;
    const double gd = fma(g1, d1, g2 * d2);
    double n1 = fma(g1, w1, g2 * t2), n2 = fma(g1, t2, -g2 * w1), t = G * ird;
    W[0] = A * gd;
    W[3] = POINT ? 0.0 : K * gd;
    if constexpr (KG) {
        const double k = (double)cg.k, h1 = (double)cg.h1, h2 = (double)cg.h2;
        const double J = fma(h1, w1, h2 * t2) * ird;
        double V;
        if constexpr (POINT) {
            W[0] = fma(-G, J, W[0]);
            V = 2.0 * G * J;
        } else {
            W[0] += fma(k, K, -G * J);
            W[3] += fma(k, K + R, J * R);
            V = fma(k, R, fma(2.0, G, R) * J);
        }
        n1 = fma(2.0, fma(h1, d1, h2 * d2), n1);
        n2 = fma(2.0, fma(h2, d1, -h1 * d2), n2);
        V *= -2.0 * ird;
        W[1] = fma(t, n1, d1 * V);
        W[2] = fma(t, n2, d2 * V);
    } else {
        W[1] = t * n1;
        W[2] = t * n2;
    }
    if constexpr (!POINT) {
        W[1] = fma(-K, g1, W[1]);
        W[2] = fma(-K, g2, W[2]);
    }
}

// Words of one particle, by the same cases as the forward's leaf_particle (mode 0) and
// list_particle (mode 1: Gaussian - point inside the support, nothing outside).
template <bool KG, int KIND>
__device__ inline void particle_grad(const PRec& pr, double X, double Y, int mode, const Cot& cg, float invC, double* W)
{
    double d1, d2, w1, w2;
    const double r2 = sqdist_angles(X, Y, pr.x, pr.y, &d1, &d2, &w1, &w2);
    const float r2f = (float)r2;
    // 1 / r^2, finite: at r = 0 every word it enters has a factor 0
    const float ir2 = fminf(__builtin_amdgcn_rcpf(r2f), 3.402823466e38f);
    const double ird = (double)ir2;
    const bool inside = r2 < pr.qs2;
    if (mode == 0) {
        if ((pr.meta >> 31) != 0 || !__any(inside)) { // a listed particle is a point mass here
            grad_words<KG, true>(cg, d1, d2, w1, w2, ird, ird, ird, 0.0, 0.0, W);
            return;
        }
    } else {
        W[0] = W[1] = W[2] = W[3] = 0.0;
        if (!inside) return;
    }
    // per unit mass (invC = 1 / C, or 1 / g(c)): the factors of profile_terms without m
    float A, G, K, R;
    if constexpr (KIND == kKindNfw) {
        const double x2 = r2 * ((double)pr.h * (double)pr.h);
        float gx2, f, dfde;
        nfw_shape32((float)x2, (float)(x2 - 1.0), &gx2, &f, &dfde);
        const float hh2 = (invC * pr.h) * pr.h;
        A = hh2 * gx2;
        K = r2 > 0.0 ? 0.5f * hh2 * f : 0.0f;
        G = A - K;
        R = r2 > 0.0 ? r2f * (0.5f * hh2 * (pr.h * pr.h) * dfde) : 0.0f;
    } else {
        const float u = r2f * pr.h;
        const float e = __expf(-u);
        const float hu = invC * pr.h;
        gauss_terms(u, e, ir2, invC, hu, &A, &G);
        K = hu * e;
        R = -u * K;
    }
    if (mode == 0) {
        A = inside ? A : ir2;
        G = inside ? G : ir2;
        K = inside ? K : 0.0f;
        R = inside ? R : 0.0f;
        grad_words<KG, false>(cg, d1, d2, w1, w2, ird, (double)A, (double)G, (double)K, (double)R, W);
    } else {
        grad_words<KG, false>(cg, d1, d2, w1, w2, ird, (double)A - ird, (double)G - ird, (double)K, (double)R, W);
    }
}

// What word w of a particle is multiplied by: dkappa/ds and d(kappa - A)/ds are -c (kappa + R) and
// -c R of a profile that scales with its size, c = 2 / s (Gaussian: 2 sqrt(2 h)) or 2 / size.
template <int KIND>
__device__ inline double word_factor(const PRec& pr, int w)
{
    if (w == 0) return 1.0;
    if (w < 3) return (double)pr.m;
    const float c = KIND == kKindNfw ? 2.0f * __builtin_amdgcn_rsqf((float)pr.qs2) : 2.0f * __builtin_sqrtf(2.0f * pr.h);
    return -(double)pr.m * (double)c;
}

// Position of the c-th set bit (from 0) of m, for c < popcount(m).
__device__ inline int nth_set_bit(uint64_t m, int c)
{
    int pos = 0;
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
        const int low = __popcll(m & ((1ull << w) - 1));
        if (c >= low) {
            c -= low;
            m >>= w;
            pos += w;
        }
    }
    return pos;
}

// The rays of a wavefront that take part in a particle pass, packed in the
// wavefront's LDS slice: ray slot s (s < popcount(rays)) is the s-th set bit.
struct RayTable {
    double* x;
    double* y;
    float2* g;   // alpha cotangent
    float* k;    // kappa cotangent
    float2* h;   // gamma cotangent
};

__device__ inline RayTable ray_table(float* lds)
{
    RayTable t;
    t.x = reinterpret_cast<double*>(lds);
    t.y = t.x + kWave;
    t.g = reinterpret_cast<float2*>(t.y + kWave);
    t.k = reinterpret_cast<float*>(t.g + kWave);
    t.h = reinterpret_cast<float2*>(t.k + kWave);
    return t;
}
constexpr int kRayTableFloats = 2 * 2 * kWave + 2 * kWave + kWave + 2 * kWave; // 2304 bytes

// Gradient terms of the particles selected by `sel` (bit k: record rec[k])
// for the rays of the wavefront whose bit is set in `rays`, summed over those
// rays into the particles' four FP64 accumulators (m, x, y, s) at
// pg + 4 * (Morton position).  Lanes hold (particle, ray slot) pairs rather
// than rays: the taking-part rays are first packed into the wavefront's LDS
// slice (their positions and cotangents), then a pass takes up to 32
// particles, splits the lanes into G = 64 / count groups, and each lane sums
// its particle's terms over the ray slots g, g + G, ... of the packed table
// (so no pass is spent on rays that do not take part); the G partial sums
// then meet in the lanes of group 0, which add them with one atomic
// instruction per accumulator.
template <bool KG, int KIND>
__device__ inline void particles_grad(const PRec* __restrict__ rec, uint64_t sel, int mode, uint64_t rays, double X,
                                      double Y, const Cot& cg, float invC, double* __restrict__ pg, int lane,
                                      float* lds)
{
    const RayTable tab = ray_table(lds);
    const int nr = __popcll(rays);
    if ((rays >> lane) & 1ull) {
        const int slot = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(rays >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)rays, 0u));
        tab.x[slot] = X;
        tab.y[slot] = Y;
        tab.g[slot] = make_float2(cg.g1, cg.g2);
        if constexpr (KG) {
            tab.k[slot] = cg.k;
            tab.h[slot] = make_float2(cg.h1, cg.h2);
        }
    }
    wave_lds_sync();
    while (sel) {
        const int total = __popcll(sel);
        const int C = total < 32 ? total : 32; // particles in this pass
        const int G = kWave / C;               // ray groups (>= 2)
        const int its = (nr + G - 1) / G;      // ray slots per group
        const int c = lane % C, g = lane / C;
        const PRec pr = rec[nth_set_bit(sel, c)];
        double A[4] = {0.0, 0.0, 0.0, 0.0};
        for (int t = 0; t < its; ++t) {
            const int s = g + G * t;
            if (g >= G || s >= nr) continue;
            Cot cr{};
            const float2 gg = tab.g[s];
            cr.g1 = gg.x;
            cr.g2 = gg.y;
            if constexpr (KG) {
                cr.k = tab.k[s];
                const float2 hh = tab.h[s];
                cr.h1 = hh.x;
                cr.h2 = hh.y;
            }
            double Wt[4];
            particle_grad<KG, KIND>(pr, tab.x[s], tab.y[s], mode, cr, invC, Wt);
#pragma unroll
            for (int w = 0; w < 4; ++w) A[w] += Wt[w];
        }
        // the G ray groups' sums meet in group 0 pairwise, in ceil(log2 G) rounds
        for (int st = 1; st < G; st <<= 1) {
            const bool take = (g & (2 * st - 1)) == 0 && g + st < G;
            const int src = take ? lane + st * C : lane;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const double v = __shfl(A[w], src, kWave);
                if (take) A[w] += v;
            }
        }
        if (g == 0) {
            double* dst = pg + 4 * (size_t)(pr.meta & 0x7fffffffu);
#pragma unroll
            for (int w = 0; w < 4; ++w)
                if (A[w] != 0.0) unsafeAtomicAdd(dst + w, A[w] * word_factor<KIND>(pr, w));
        }
        for (int q = 0; q < C; ++q) sel &= sel - 1; // drop this pass's particles
    }
    wave_lds_sync(); // the slice is written again by the next user
}

// Cotangent arrays of the rays (input order); any may be NULL (zero).
struct CotIn {
    const float *ga1, *ga2, *gk, *gg1, *gg2;
};


// FP32 words of LDS scratch of one wavefront: the words of a far pass (half of
// them at a time) or the ray table of a particle pass, one or the other.
template <int P, bool PAIRS, bool FAR>
constexpr int adj_scratch()
{
    const int far = FAR ? kWave * 2 * ((P + 3) / 2) : 0, pairs = PAIRS ? kRayTableFloats : 0;
    return far > pairs ? far : pairs;
}

// Visitor of the adjoint walk.  A box's contribution to dL/d(moments) is, per
// ray, g_hat v t^k - (k + 1) gg_hat v^2 t^k for k = 0 .. P + 1 (v = 1 / w, t = r_cm v),
// summed over the rays that accept it: 2 P + 4 FP32 words per lane, summed over the
// lanes in registers, one FP64 atomic instruction over adjacent words.  Far
// boxes (farfield.hpp) need only the rays' moments about the group's centre,
//   Lam_j = sum_r (g_hat z^j + gg_hat (j / a) z^(j-1)),   z = delta / a,
// the adjoint of the local expansion's coefficients, from which the box's words
// follow as t^k sum_j C(k + j, j) v e^j Lam_j, with lanes as boxes.
template <int P, bool KG, int KIND, bool FAR, bool PAIRS>
struct AdjVisitor {
    static constexpr bool stats = false;
    static constexpr bool farfield = FAR;
    static constexpr int NA = 2 * (P + 2);
    struct Box {
        float rcm;
    };
    const TreeDev& T;
    const RayGroup& g;
    const double X, Y;
    const int lane;
    const Cot cg;
    double* const abox;
    double* const pg;
    float* const lds;  // adj_scratch words
    float* const lam;  // kFarWords words: Lam_j
    const int wslot;

    __device__ AdjVisitor(const TreeDev& T_, const RayGroup& g_, double X_, double Y_, int lane_, const Cot& cg_,
                          double* abox_, double* pg_, float* lds_, float* lam_)
        : T(T_), g(g_), X(X_), Y(Y_), lane(lane_), cg(cg_), abox(abox_), pg(pg_), lds(lds_), lam(lam_),
          wslot(word_slot<NA>(lane_))
    {
        if (FAR && g.far) ray_moments();
    }

    // Lam_j into LDS, half of them at a time (lanes without a ray have zero cotangents)
    __device__ void ray_moments()
    {
        const bool valid = lane_bit(g.full);
        const float z1 = valid ? (float)((X - g.ox) * (double)g.inva) : 0.0f;
        const float z2 = valid ? (float)((Y - g.oy) * (double)g.inva) : 0.0f;
        float p1 = cg.g1, p2 = cg.g2, q1 = cg.h1 * g.inva, q2 = cg.h2 * g.inva; // g_hat z^j, gg_hat z^(j-1) / a
        const int slot = word_slot<kFarWords / 2>(lane);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            float a[kFarWords / 2];
#pragma unroll
            for (int i = 0; i <= kFarOrder / 2; ++i) {
                const int j = half * (kFarOrder / 2 + 1) + i;
                a[2 * i] = KG && j > 0 ? fmaf((float)j, q1, p1) : p1;
                a[2 * i + 1] = KG && j > 0 ? fmaf((float)j, q2, p2) : p2;
                const float n1 = fmaf(p1, z1, -p2 * z2), n2 = fmaf(p1, z2, p2 * z1);
                p1 = n1;
                p2 = n2;
                if (KG && j > 0) {
                    const float m1 = fmaf(q1, z1, -q2 * z2), m2 = fmaf(q1, z2, q2 * z1);
                    q1 = m1;
                    q2 = m2;
                }
            }
            const double t = word_totals64<kFarWords / 2>(a);
            if (slot >= 0) lam[half * (kFarWords / 2) + slot] = (float)t;
        }
        wave_lds_sync();
    }

    __device__ Box load(int c) const { return Box{uniform_ld(T.mom, (int64_t)c * mom_stride(P) + 1)}; }

    __device__ void box(const Box& b, int c, bool acc, double w1, double w2)
    {
        // every lane forms the words, those that did not accept with zero
        // cotangents and w = (1, 0): exactly 0, with no branch and no clearing
        float a[NA];
        const float f1 = acc ? (float)w1 : 1.0f, f2 = acc ? (float)w2 : 0.0f;
        const float e1 = acc ? cg.g1 : 0.0f, e2 = acc ? cg.g2 : 0.0f;
        const float inv = __builtin_amdgcn_rcpf(f1 * f1 + f2 * f2);
        const float v1 = f1 * inv, v2 = -f2 * inv;
        const float t1 = b.rcm * v1, t2 = b.rcm * v2;
        float p1 = fmaf(e1, v1, -e2 * v2), p2 = fmaf(e1, v2, e2 * v1); // g_hat v t^k
        float q1 = 0.0f, q2 = 0.0f;                                    // gg_hat v^2 t^k
        if constexpr (KG) {
            const float h1 = acc ? cg.h1 : 0.0f, h2 = acc ? cg.h2 : 0.0f;
            const float x1 = fmaf(h1, v1, -h2 * v2), x2 = fmaf(h1, v2, h2 * v1);
            q1 = fmaf(x1, v1, -x2 * v2);
            q2 = fmaf(x1, v2, x2 * v1);
        }
#pragma unroll
        for (int k = 0; k <= P + 1; ++k) {
            a[2 * k] = KG ? fmaf(-(float)(k + 1), q1, p1) : p1;
            a[2 * k + 1] = KG ? fmaf(-(float)(k + 1), q2, p2) : p2;
            const float n1 = fmaf(p1, t1, -p2 * t2), n2 = fmaf(p1, t2, p2 * t1);
            p1 = n1;
            p2 = n2;
            if constexpr (KG) {
                const float m1 = fmaf(q1, t1, -q2 * t2), m2 = fmaf(q1, t2, q2 * t1);
                q1 = m1;
                q2 = m2;
            }
        }
        const float mine = word_totals<NA>(a);
        if (wslot >= 0) unsafeAtomicAdd(abox + (size_t)c * NA + wslot, (double)mine);
    }

    // Words [K0, K1) of the far boxes (complex, lanes as boxes) through LDS to
    // adjacent lanes: as many boxes per atomic instruction as fit the wavefront.
    template <int K0, int K1>
    __device__ void far_add(int c, uint64_t boxes, const float* H, float t1, float t2, float& s1, float& s2)
    {
        constexpr int N = 2 * (K1 - K0);
#pragma unroll
        for (int k = K0; k < K1; ++k) {
            float r1 = 0.0f, r2 = 0.0f;
#pragma unroll
            for (int j = kFarOrder; j >= 0; --j) {
                r1 = fmaf(far_binomial(k, j), H[2 * j], r1);
                r2 = fmaf(far_binomial(k, j), H[2 * j + 1], r2);
            }
            lds[lane * N + 2 * (k - K0)] = fmaf(s1, r1, -s2 * r2);
            lds[lane * N + 2 * (k - K0) + 1] = fmaf(s1, r2, s2 * r1);
            const float n1 = fmaf(s1, t1, -s2 * t2), n2 = fmaf(s1, t2, s2 * t1); // t^(k+1)
            s1 = n1;
            s2 = n2;
        }
        wave_lds_sync();
        constexpr int B = kWave / N; // boxes per pass
        const int nb = __popcll(boxes), u = lane / N, i = lane % N;
        for (int b = 0; b < nb; b += B) {
            const int at = b + u;
            const int ca = __shfl(c, at < nb ? at : 0, kWave);
            if (u < B && at < nb) unsafeAtomicAdd(abox + (size_t)ca * NA + 2 * K0 + i, (double)lds[at * N + i]);
        }
        wave_lds_sync();
    }

    __device__ void far(int c, bool active)
    {
        const FarOffset o = far_offset(T, g, c, active);
        const float rcm = T.mom[(size_t)c * mom_stride(P) + 1];
        float p1 = (float)o.v1, p2 = (float)o.v2;
        const float t1 = rcm * p1, t2 = rcm * p2, e1 = -g.a * p1, e2 = -g.a * p2;
        float H[kFarWords]; // v e^j Lam_j
#pragma unroll
        for (int j = 0; j <= kFarOrder; ++j) {
            const float l1 = lam[2 * j], l2 = lam[2 * j + 1];
            H[2 * j] = fmaf(p1, l1, -p2 * l2);
            H[2 * j + 1] = fmaf(p1, l2, p2 * l1);
            const float n1 = fmaf(p1, e1, -p2 * e2), n2 = fmaf(p1, e2, p2 * e1);
            p1 = n1;
            p2 = n2;
        }
        const uint64_t boxes = __ballot(active); // the first lanes
        float s1 = 1.0f, s2 = 0.0f;
        far_add<0, (P + 2) / 2>(c, boxes, H, t1, t2, s1, s2);
        far_add<(P + 2) / 2, P + 2>(c, boxes, H, t1, t2, s1, s2);
    }

    // One particle's gradient (m, x, y, s) over the rays that `c` has cotangents of: per-ray words in
    // FP64, summed over the wavefront in registers (each 16-lane row ends with one of the
    // four words), one atomic instruction over the four adjacent words.
    __device__ void particle(const PRec& pr, int mode, const Cot& c)
    {
        double W[4];
        particle_grad<KG, KIND>(pr, X, Y, mode, c, T.invC, W);
        const double t = row_word4(W);
        if ((lane & 15) == 0 && t != 0.0)
            unsafeAtomicAdd(pg + 4 * (size_t)(pr.meta & 0x7fffffffu) + (lane >> 4), t * word_factor<KIND>(pr, lane >> 4));
    }

    // The cotangents of the rays in m (the other lanes' are zero).
    __device__ Cot cot_of(uint64_t m) const
    {
        const bool on = lane_bit(m);
        return Cot{on ? cg.g1 : 0.0f, on ? cg.g2 : 0.0f, on ? cg.k : 0.0f, on ? cg.h1 : 0.0f, on ? cg.h2 : 0.0f};
    }

    __device__ void leaf(int pbeg, int pend, uint64_t opn)
    {
        if constexpr (PAIRS) {
            for (int j = pbeg; j < pend; j += kWave) { // a leaf at the depth cap may exceed 64
                const int np = pend - j < kWave ? pend - j : kWave;
                const uint64_t sel = np == kWave ? ~0ull : ((1ull << np) - 1);
                particles_grad<KG, KIND>(T.prt + j, sel, 0, opn, X, Y, cg, T.invC, pg, lane, lds);
            }
        } else {
            const Cot c = cot_of(opn);
            PRec pr = uniform_ld(T.prt, pbeg);
            for (int j = pbeg; j < pend; ++j) {
                int next = j + 1 < pend ? j + 1 : j;
                settle(pr, next);
                const PRec nx = uniform_ld(T.prt, next);
                particle(pr, 0, c);
                pr = nx;
            }
        }
    }

    __device__ void list(int lbeg, int lend, int stride, uint64_t actm)
    {
        const Cot c = PAIRS ? cg : cot_of(actm);
        for (int base = lbeg; base < lend; base += stride) {
            const int j = base + lane;
            bool cand = false;
            if (j < lend) {
                const PRec pr = T.lst[j];
                const double dx = fmax(fmax(g.gx0 - pr.x, pr.x - g.gx1), 0.0);
                const double dy = fmax(fmax(g.gy0 - pr.y, pr.y - g.gy1), 0.0);
                cand = dx * dx + dy * dy < pr.qs2 * (1.0 + 1e-9);
            }
            uint64_t cm = __ballot(cand);
            if (!cm) continue;
            if constexpr (PAIRS) {
                particles_grad<KG, KIND>(T.lst + base, cm, 1, actm, X, Y, cg, T.invC, pg, lane, lds);
            } else {
                PRec pr = uniform_ld(T.lst, base + __ffsll((unsigned long long)cm) - 1);
                while (cm) {
                    const uint64_t rest = cm & (cm - 1);
                    int next = base + __ffsll((unsigned long long)(rest ? rest : cm)) - 1;
                    settle(pr, next);
                    const PRec nx = uniform_ld(T.lst, next);
                    particle(pr, 1, c);
                    pr = nx;
                    cm = rest;
                }
            }
        }
    }
};

// Bytes of LDS of one wavefront besides the traversal's.
template <int P, bool COOP, bool FAR>
constexpr size_t adj_wave_lds() { return 4 * (adj_scratch<P, COOP, FAR>() + kFarWords); }

// Wavefronts of one group: COOP (W = blockDim.x / 64, groups of `rays` rays) or one.
template <int P, bool KG, int KIND, bool COOP, bool FAR>
__global__ __launch_bounds__(COOP ? kWave * kMaxGroupWaves : kWave) void k_adjoint_walk(
    TreeDev T, const double* __restrict__ rxs, const double* __restrict__ rys, const uint32_t* __restrict__ rperm,
    int64_t nrays, CotIn ci, double* __restrict__ pg, double* __restrict__ abar, int rays, int split, bool far)
{
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = COOP ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)) : 0;
    const int W = COOP ? (int)(blockDim.x / kWave) : 1;
    int64_t grp;
    int c0, c1;
    box_range(split, T.ncells, &c0, &c1);
    if (!group_task(blockIdx.x / split, (nrays + rays - 1) / rays, &grp)) return; // (whole workgroups)
    // this wavefront's copies of the box adjoints and of the particle sums (see kAdjCopies)
    const int wid = (int)blockIdx.x * W + w;
    const int64_t r = grp * rays + lane;
    const bool valid = lane < rays && r < nrays;
    const double X = valid ? rxs[r] : 0.0, Y = valid ? rys[r] : 0.0;
    const int64_t o = valid ? (rperm ? (int64_t)rperm[r] : r) : 0;
    Cot cg{0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    if (valid) {
        cg.g1 = ci.ga1 ? ci.ga1[o] : 0.0f;
        cg.g2 = ci.ga2 ? ci.ga2[o] : 0.0f;
        if constexpr (KG) {
            cg.k = ci.gk ? ci.gk[o] : 0.0f;
            cg.h1 = ci.gg1 ? ci.gg1[o] : 0.0f;
            cg.h2 = ci.gg2 ? ci.gg2[o] : 0.0f;
        }
    }
    const RayGroup g = ray_group(X, Y, valid, FAR && far);
    char* own = lds + (COOP ? coop_lds_bytes(W) + w * adj_wave_lds<P, COOP, FAR>() : solo_lds_bytes(true));
    float* scratch = reinterpret_cast<float*>(own);
    AdjVisitor<P, KG, KIND, FAR, COOP> v(T, g, X, Y, lane, cg, abar + (size_t)(wid % kAdjCopies) * T.ncells * (2 * (P + 2)),
                                   pg + (size_t)(wid % kPgCopies) * 4 * T.n, scratch, scratch + adj_scratch<P, COOP, FAR>());
    traverse<COOP, true>(T, v, g, X, Y, lane, w, W, COOP ? coop_lds(lds, W) : solo_lds(lds, true), c0, c1);
}

// Arguments of an adjoint walk launch.
struct AdjointArgs {
    const TreeDev& T;
    const double *rxs, *rys;
    const uint32_t* rperm;
    int64_t nrays;
    CotIn ci;
    double *pg, *abar;
    WalkShape shape;
    bool far;
    hipStream_t st;
};

template <int P, bool KG, int KIND>
void launch_adjoint_kind(const AdjointArgs& a)
{
    const dim3 g((unsigned)(group_grid((a.nrays + a.shape.rays - 1) / a.shape.rays) * a.shape.split));
    const int W = a.shape.waves;
    const auto go = [&](auto coop, auto far) {
        constexpr bool COOP = decltype(coop)::value, FAR = decltype(far)::value;
        const size_t lds = COOP ? coop_lds_bytes(W) + W * adj_wave_lds<P, COOP, FAR>() : solo_lds_bytes(true) + adj_wave_lds<P, COOP, FAR>();
        hipLaunchKernelGGL((k_adjoint_walk<P, KG, KIND, COOP, FAR>), g, dim3(kWave * W), lds, a.st, a.T, a.rxs, a.rys,
                           a.rperm, a.nrays, a.ci, a.pg, a.abar, a.shape.rays, a.shape.split, a.far);
    };
    if (W == 1) go(std::false_type{}, std::true_type{});
    else if (a.far) go(std::true_type{}, std::true_type{});
    else go(std::true_type{}, std::false_type{});
}

template <bool KG>
void launch_adjoint_order(const AdjointArgs& a)
{
#define GLM_CASE(PP)                                                                   \
    case PP:                                                                           \
        if (a.T.kind == kKindNfw) launch_adjoint_kind<PP, KG, kKindNfw>(a);            \
        else launch_adjoint_kind<PP, KG, kKindGauss>(a);                               \
        break;
    switch (a.T.order) {
        GLM_CASE(0) GLM_CASE(1) GLM_CASE(2) GLM_CASE(3) GLM_CASE(4) GLM_CASE(5) GLM_CASE(6)
        GLM_CASE(7) GLM_CASE(8) GLM_CASE(9) GLM_CASE(10) GLM_CASE(11) GLM_CASE(12)
        default: break;
    }
#undef GLM_CASE
}

// One translation unit each (they compile side by side).
void launch_adjoint_alpha(const AdjointArgs& a); // cotangents of alpha only
void launch_adjoint_all(const AdjointArgs& a);   // and of kappa and gamma

} // namespace glm
