// Forward walk of one 64-ray group: the visitor of the traversal (lanes as
// rays), the kernels over all groups, and their launch.  Evaluation is FP32:
// the multipole series is a Horner scheme in t = r_cm / w on moments normalised
// by M r_cm^k; the terms are summed in FP64.
#pragma once

#include <type_traits>

#include "traverse.hpp"

namespace glm {

// MODE: 0 = the product walk, 1 = the same plus interaction counts, 2 = plain
// FP32 sum of the alpha terms (debug).
template <int P, bool AONLY, int MODE, bool PSI, int KIND, bool FAR>
struct FwdVisitor {
    using Box = BoxMoments<P>;
    static constexpr bool f64a = MODE != 2;
    static constexpr bool stats = MODE == 1;
    static constexpr bool farfield = FAR;
    const TreeDev& T;
    const RayGroup& g;
    const double X, Y;
    const int lane;
    const bool valid;
    Acc A{};
    int cnt[stats ? kCounts : 1] = {};
    double flo = 0.0, fhi = 0.0; // this lane's words of the two halves of the group's local expansion (see word_slot)
    double fpsi = 0.0; // this lane's boxes' potential at the group's centre

    __device__ FwdVisitor(const TreeDev& T_, const RayGroup& g_, double X_, double Y_, int lane_, bool valid_)
        : T(T_), g(g_), X(X_), Y(Y_), lane(lane_), valid(valid_)
    {
    }

    __device__ void visited(int full) { if constexpr (stats) cnt[0] += valid ? full : 0; }
    __device__ void visited_some(bool act) { if constexpr (stats) cnt[0] += act; }

    __device__ void accepted(int far)
    {
        if constexpr (stats) {
            cnt[1] += valid ? far : 0;
            cnt[5] += far;
        }
    }

    __device__ void far(int c, bool active)
    {
        FarBox<P> b;
        b.load(T, g, c, active);
        if constexpr (PSI) fpsi += (double)b.psi0(active);
        // half of the words at a time: fewer registers
        float L[kFarWords / 2];
        double r1 = 0.0, r2 = 0.0;
        b.template words<0>(L, r1, r2);
        A.a1 += wave_sum(r1);
        A.a2 -= wave_sum(r2);
        flo += word_totals64<kFarWords / 2>(L);
        b.template words<kFarOrder / 2 + 1>(L, r1, r2);
        fhi += word_totals64<kFarWords / 2>(L);
    }

    // This lane's words of the local expansion into `words` (kFarWords doubles of LDS).
    __device__ void put_words(double* words) const
    {
        const int slot = word_slot<kFarWords / 2>(lane);
        if (slot >= 0) {
            words[slot] = flo;
            words[kFarWords / 2 + slot] = fhi;
        }
    }

    // The local expansion at the rays.
    __device__ void finish(const double* words)
    {
        far_eval<AONLY, PSI>(g, words, X, Y, A);
        if constexpr (PSI) A.ps += wave_sum(fpsi);
    }

    __device__ Box load(int c) const { return uniform_ld(reinterpret_cast<const Box*>(T.mom), c); }

    __device__ void box(const Box& mo, int, bool acc, double w1, double w2)
    {
        if constexpr (stats) {
            cnt[1] += acc;
            ++cnt[5];
        }
        if (acc) eval_box<P, AONLY, f64a, PSI>(mo, w1, w2, A);
    }

    __device__ void leaf(int pbeg, int pend, uint64_t opn)
    {
        const bool act = lane_bit(opn);
        if constexpr (stats) {
            if (act) cnt[2] += pend - pbeg;
            cnt[6] += pend - pbeg;
        }
        int j = pbeg;
        PRec even = uniform_ld(T.prt, j), odd;
        // one particle of the leaf: `now` is here, `then` is loaded behind the work on it
        const auto step = [&](PRec& now, PRec& then) {
            int next = j + 1 < pend ? j + 1 : j;
            settle(now, next);
            then = uniform_ld(T.prt, next);
            if (act) leaf_particle<AONLY, f64a, PSI, KIND>(now, X, Y, A, T.psiK, T.einTerms, T.invC);
            return ++j < pend;
        };
        while (step(even, odd) && step(odd, even)) {
        }
    }

    // List entries lbeg .. lend - 1 in chunks of 64, `stride` apart.
    __device__ void list(int lbeg, int lend, int stride, uint64_t actm)
    {
        const bool act = lane_bit(actm);
        int hits = 0;
        for (int base = lbeg; base < lend; base += stride) {
            const int j = base + lane;
            bool cand = false;
            if (j < lend) {
                const PRec me = T.lst[j];
                const double dx = fmax(fmax(g.gx0 - me.x, me.x - g.gx1), 0.0);
                const double dy = fmax(fmax(g.gy0 - me.y, me.y - g.gy1), 0.0);
                cand = dx * dx + dy * dy < me.qs2 * (1.0 + 1e-9);
            }
            uint64_t cm = __ballot(cand);
            if constexpr (stats) {
                cnt[4] += base + kWave < lend ? kWave : lend - base;
                cnt[7] += __popcll(cm);
            }
            if (!cm) continue;
            PRec even = uniform_ld(T.lst, base + __ffsll((unsigned long long)cm) - 1), odd;
            const auto step = [&](PRec& now, PRec& then) {
                const uint64_t rest = cm & (cm - 1);
                int next = base + __ffsll((unsigned long long)(rest ? rest : cm)) - 1;
                settle(now, next);
                then = uniform_ld(T.lst, next);
                if (act) list_particle<AONLY, f64a, PSI, KIND>(now, X, Y, A, hits, T.psiK, T.einTerms, T.invC);
                cm = rest;
                return cm != 0;
            };
            while (step(even, odd) && step(odd, even)) {
            }
        }
        if constexpr (stats) cnt[3] += hits;
    }
};

template <bool AONLY, bool STATS, bool PSI = false>
__device__ inline void write_out(const Acc& A, const int* cnt, int64_t o, const WalkOut& out)
{
    const double a1 = alpha1(A), a2 = alpha2(A);
    out.a1[o] = (float)a1;
    out.a2[o] = (float)a2;
    if constexpr (PSI) {
        out.psi[o] = (float)A.ps;
        if (out.td) out.td[o] = (float)(0.5 * (a1 * a1 + a2 * a2) - A.ps); // Sec. 3.2: |alpha|^2 / 2 - psi
    }
    if (!AONLY) {
        if (out.k) out.k[o] = (float)A.k;
        if (out.g1) out.g1[o] = (float)A.g1;
        if (out.g2) out.g2[o] = (float)A.g2;
    }
    if (STATS && out.counts)
        for (int i = 0; i < kCounts; ++i) out.counts[kCounts * o + i] = cnt[i];
}

// Wavefronts per SIMD that the walk's kernels are held to: `most`, but four for the halos' potential,
// whose FP64 logarithms and arctangent take 128 registers (with the 80 of six it spilled 100:
// 1e5 halos, 1e6 rays 25.6 ms, 17.6 with four).
template <bool PSI, int KIND>
constexpr int walk_waves(int most) { return PSI && KIND == kKindNfw ? 4 : most; }

// One wavefront (and workgroup) per ray group.
template <int P, bool AONLY, int MODE, bool PSI, int KIND, bool FAR>
__global__ __launch_bounds__(kWave, (walk_waves<PSI, KIND>(6))) void k_walk(TreeDev T, const double* __restrict__ rxs,
                                               const double* __restrict__ rys, const uint32_t* __restrict__ rperm,
                                               int64_t nrays, WalkOut out)
{
    __shared__ __align__(16) char lds[solo_lds_bytes(FAR)];
    const int lane = threadIdx.x;
    int64_t grp;
    if (!group_task(blockIdx.x, (nrays + kWave - 1) / kWave, &grp)) return;
    const int64_t r = grp * kWave + lane;
    const bool valid = r < nrays;
    const double X = valid ? rxs[r] : 0.0, Y = valid ? rys[r] : 0.0;
    const RayGroup g = ray_group(X, Y, valid, FAR);
    FwdVisitor<P, AONLY, MODE, PSI, KIND, FAR> v(T, g, X, Y, lane, valid);
    traverse<false, false>(T, v, g, X, Y, lane, 0, 1, solo_lds(lds, FAR));
    if (FAR && g.far) {
        double* words = reinterpret_cast<double*>(lds);
        v.put_words(words);
        wave_lds_sync();
        v.finish(words);
    }
    if constexpr (!AONLY) join_shear(v.A);
    if (valid) write_out<AONLY, MODE == 1, PSI>(v.A, v.cnt, rperm ? (int64_t)rperm[r] : r, out);
}

// FP64 words per ray that the wavefronts of a group sum up at the end.
template <bool AONLY, bool PSI>
constexpr int coop_words() { return 2 + (AONLY ? 0 : 3) + (PSI ? 1 : 0); }

// LDS of k_walk_coop: the traversal's; reused by the final sums.
template <bool AONLY, bool PSI, bool STATS>
constexpr size_t walk_coop_lds(int W)
{
    const size_t sums = (size_t)(W - 1) * kWave * (8 * coop_words<AONLY, PSI>() + (STATS ? 4 * kCounts : 0));
    return coop_lds_bytes(W) > sums ? coop_lds_bytes(W) : sums;
}

// W = blockDim.x / 64 wavefronts per group of `rays` (up to 64) rays; their sums meet in wavefront
// order in LDS.
template <int P, bool AONLY, int MODE, bool PSI, int KIND, bool FAR>
__global__ __launch_bounds__(kWave* kMaxGroupWaves, (walk_waves<PSI, KIND>(5))) void k_walk_coop(TreeDev T, const double* __restrict__ rxs,
                                                                    const double* __restrict__ rys,
                                                                    const uint32_t* __restrict__ rperm, int64_t nrays,
                                                                    WalkOut out, int rays, int split, Partial* __restrict__ parts)
{
    extern __shared__ __align__(16) char lds[];
    constexpr bool STATS = MODE == 1;
    constexpr int NW = coop_words<AONLY, PSI>();
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), W = blockDim.x / kWave;
    int64_t grp;
    int c0, c1;
    const int part = box_range(split, T.ncells, &c0, &c1);
    if (!group_task(blockIdx.x / split, (nrays + rays - 1) / rays, &grp)) return; // (whole workgroups)
    const int64_t r = grp * rays + lane;
    const bool valid = lane < rays && r < nrays;
    const double X = valid ? rxs[r] : 0.0, Y = valid ? rys[r] : 0.0;
    const RayGroup g = ray_group(X, Y, valid, FAR);
    FwdVisitor<P, AONLY, MODE, PSI, KIND, FAR> v(T, g, X, Y, lane, valid);
    traverse<true, true>(T, v, g, X, Y, lane, w, W, coop_lds(lds, W), c0, c1);
    Acc& A = v.A;
    if constexpr (!AONLY) join_shear(A);
    __syncthreads(); // the traversal's LDS is free
    double* sums = reinterpret_cast<double*>(lds);
    if (FAR && g.far) { // the wavefronts' local expansions, summed into one
        v.put_words(sums + w * kFarWords);
        __syncthreads();
        if (w == 0) {
            double t = 0.0;
            if (lane < kFarWords)
                for (int u = 0; u < W; ++u) t += sums[u * kFarWords + lane];
            wave_lds_sync();
            if (lane < kFarWords) sums[lane] = t;
            wave_lds_sync();
            v.finish(sums);
        } else if constexpr (PSI) {
            A.ps += wave_sum(v.fpsi);
        }
        __syncthreads();
    }
    int* csum = reinterpret_cast<int*>(sums + (size_t)(W - 1) * NW * kWave);
    if (w > 0) {
        double* p = sums + (size_t)(w - 1) * NW * kWave + lane;
        p[0] = alpha1(A);
        p[kWave] = alpha2(A);
        if constexpr (!AONLY) {
            p[2 * kWave] = A.k;
            p[3 * kWave] = A.g1;
            p[4 * kWave] = A.g2;
        }
        if constexpr (PSI) p[(NW - 1) * kWave] = A.ps;
        if constexpr (STATS)
            for (int i = 0; i < kCounts; ++i) csum[((w - 1) * kCounts + i) * kWave + lane] = v.cnt[i];
    }
    __syncthreads();
    if (w > 0 || !valid) return;
    for (int u = 0; u < W - 1; ++u) {
        const double* p = sums + (size_t)u * NW * kWave + lane;
        A.a1 += p[0];
        A.a2 += p[kWave];
        if constexpr (!AONLY) {
            A.k += p[2 * kWave];
            A.g1 += p[3 * kWave];
            A.g2 += p[4 * kWave];
        }
        if constexpr (PSI) A.ps += p[(NW - 1) * kWave];
        if constexpr (STATS)
            for (int i = 0; i < kCounts; ++i) v.cnt[i] += csum[(u * kCounts + i) * kWave + lane];
    }
    if (split == 1) {
        write_out<AONLY, STATS, PSI>(A, v.cnt, rperm ? (int64_t)rperm[r] : r, out);
        return;
    }
    Partial q{};
    q.a1 = alpha1(A);
    q.a2 = alpha2(A);
    q.k = A.k;
    q.g1 = A.g1;
    q.g2 = A.g2;
    q.ps = A.ps;
    if constexpr (STATS)
        for (int i = 0; i < kCounts; ++i) q.cnt[i] = v.cnt[i];
    parts[(int64_t)part * nrays + r] = q;
}

// Arguments of a walk launch.
struct WalkArgs {
    const TreeDev& T;
    const double *rxs, *rys;
    const uint32_t* rperm;
    int64_t nrays;
    WalkOut out;
    WalkShape shape;
    bool far;  // expand far boxes over the groups
    Partial* parts; // of shape.split box ranges per ray
    hipStream_t st;
};

template <int P, bool AONLY, int MODE, bool PSI, int KIND>
void launch_walk_kind(const WalkArgs& a)
{
    const dim3 g((unsigned)(group_grid((a.nrays + a.shape.rays - 1) / a.shape.rays) * a.shape.split));
    const auto launch = [&](auto far) {
        constexpr bool FAR = decltype(far)::value;
        if (a.shape.waves == 1 && a.shape.rays == kWave && a.shape.split == 1)
            hipLaunchKernelGGL((k_walk<P, AONLY, MODE, PSI, KIND, FAR>), g, dim3(kWave), 0, a.st, a.T, a.rxs, a.rys, a.rperm,
                               a.nrays, a.out);
        else
            hipLaunchKernelGGL((k_walk_coop<P, AONLY, MODE, PSI, KIND, FAR>), g, dim3(kWave * a.shape.waves),
                               (walk_coop_lds<AONLY, PSI, MODE == 1>(a.shape.waves)), a.st, a.T, a.rxs, a.rys, a.rperm,
                               a.nrays, a.out, a.shape.rays, a.shape.split, a.parts);
    };
    if constexpr (MODE != 2) {
        if (a.far) return launch(std::true_type{});
    }
    launch(std::false_type{});
}

template <bool AONLY, int MODE, bool PSI>
void launch_walk_order(const WalkArgs& a)
{
#define GLM_CASE(PP)                                                                            \
    case PP:                                                                                    \
        if (a.T.kind == kKindNfw) launch_walk_kind<PP, AONLY, MODE, PSI, kKindNfw>(a);          \
        else launch_walk_kind<PP, AONLY, MODE, PSI, kKindGauss>(a);                             \
        break;
    switch (a.T.order) {
        GLM_CASE(0) GLM_CASE(1) GLM_CASE(2) GLM_CASE(3) GLM_CASE(4) GLM_CASE(5) GLM_CASE(6)
        GLM_CASE(7) GLM_CASE(8) GLM_CASE(9) GLM_CASE(10) GLM_CASE(11) GLM_CASE(12)
        default: break;
    }
#undef GLM_CASE
}

// One translation unit each (they compile side by side).
void launch_walk_full(const WalkArgs& a);      // alpha, kappa, gamma
void launch_walk_alpha(const WalkArgs& a);     // alpha only
void launch_walk_potential(const WalkArgs& a); // alpha and psi
void launch_walk_counts(const WalkArgs& a, bool alpha_only);
void launch_walk_fp32(const WalkArgs& a, bool alpha_only);

// Arguments of a batched launch (device table, host sizes).
struct BatchArgs {
    const BatchLens* table;
    int nlens;
    const int64_t* gpre;
    int* counter;
    const double *xs, *ys;
    const uint32_t* perm;
    int64_t items;
    int order, kind;
    bool alpha_only, fp32_alpha;
    hipStream_t st;
};
void launch_walk_batched(const BatchArgs& a);

} // namespace glm
