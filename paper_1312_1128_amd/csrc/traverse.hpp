// Lane-parallel tree traversal of one 64-ray group, shared by the forward walk
// and its adjoint.
//
// The traversal keeps a stack of (box, mask) items in LDS, the mask naming the
// rays of the group that have accepted no ancestor of the box.  A round takes
// many items, one per lane, and tests each box against the group's bounding
// box: either every ray accepts it, or none does, or the decision differs
// between rays (about one box in three) and is taken ray by ray, with lanes as
// rays.  The bounding-box distances round monotonically (the same FP64
// operations as the per-ray test, no contraction), so the decisions are
// exactly those of a per-ray walk.  The boxes' work then goes to a visitor:
//   box(b, c, acc, w1, w2)   rays `acc` accept box c (b = load(c), offset w per ray)
//   leaf(pbeg, pend, opn)    rays `opn` sum these particles
//   list(lbeg, lend, act)    rays `act` check these big-particle list entries
// with wave-uniform arguments and lanes as rays.  A box that every ray of the
// group accepts, far enough from the group, goes to
//   far(c, active)           lanes as boxes
// instead: its field over the group is a local expansion (farfield.hpp).
//
// A stackless preorder walk with lanes as rays (one box at a time, every box
// tested per ray) spent a fifth of its instructions on the traversal, and a
// dependent scalar load per box made it slow wherever few wavefronts run.
//
// One wavefront serves a group (SOLO), or W wavefronts of one workgroup do: they
// share the stack, take interleaved items, and deal the resulting work among
// themselves through LDS queues, so that a group with much work (the centre
// of a halo, seen by few scattered rays) is not left to one wavefront.
#pragma once

#include "farfield.hpp"
#include "walk.hpp"

namespace glm {

// Stack room that a descent box by box can need: three siblings per level.
constexpr int kStackReserve = 3 * kMaxLevel;
// Items of a SOLO stack.  (Without far boxes the kernels need few enough registers for eight
// wavefronts per SIMD, which 5 KB of LDS each allow.)
__host__ __device__ constexpr int solo_stack(bool far) { return far ? 448 : 400; }
constexpr int kMaxGroupWaves = 16;
constexpr int kFarQueue = 2 * kWave; // far boxes waiting for their pass

// Items to take off a stack of `top` items: as many as leave the reserve after
// their (at most four) children went on; one by one when there is no such room
// (a depth-first descent then stays inside the reserve).
__device__ inline int take_count(int top, int cap, int most)
{
    int n = (cap - top - kStackReserve) / 3;
    n = n < 1 ? 1 : n;
    n = n < most ? n : most;
    return n < top ? n : top;
}

// LDS of one group (device pointers into dynamic LDS; queues only with W > 1).
struct TravLds {
    uint64_t* stkm;
    uint64_t* qm;   // three queues of `qcap` masks: accepted boxes, open leaves, lists
    int* stkb;
    int* qb;        // the queues' boxes, or first particles or entries
    int* qe;        // the last two queues' ends of those
    int* cnt;       // 3 x kMaxGroupWaves item counts of a round
    int* fq;        // far boxes
    int cap, qcap;
};

__host__ __device__ constexpr int coop_stack(int W) { return W <= 2 ? 512 : (W == 4 ? 768 : (W == 8 ? 1280 : 2048)); }
__host__ __device__ constexpr int coop_queue(int W)
{
    const int by_stack = (coop_stack(W) - kStackReserve) / 3;
    return kWave * W < by_stack ? kWave * W : by_stack;
}
__host__ __device__ constexpr size_t solo_lds_bytes(bool far)
{
    return 12ull * solo_stack(far) + (far ? 4ull * kFarQueue : 0);
}
__host__ __device__ constexpr size_t coop_lds_bytes(int W)
{
    return 12ull * coop_stack(W) + 48ull * coop_queue(W) + 16ull * kMaxGroupWaves + 4ull * kWave;
}

__device__ inline TravLds solo_lds(char* base, bool far)
{
    TravLds L{};
    L.cap = solo_stack(far);
    L.stkm = reinterpret_cast<uint64_t*>(base);
    L.stkb = reinterpret_cast<int*>(base + 8 * L.cap);
    L.fq = L.stkb + L.cap;
    return L;
}

__device__ inline TravLds coop_lds(char* base, int W)
{
    TravLds L;
    L.cap = coop_stack(W);
    L.qcap = coop_queue(W);
    L.stkm = reinterpret_cast<uint64_t*>(base);
    L.qm = L.stkm + L.cap;
    L.stkb = reinterpret_cast<int*>(L.qm + 3 * L.qcap);
    L.qb = L.stkb + L.cap;
    L.qe = L.qb + 3 * L.qcap;
    L.cnt = L.qe + 2 * L.qcap;
    L.fq = L.cnt + 4 * kMaxGroupWaves; // one round's boxes after fewer than 64 left over
    return L;
}

__device__ inline uint64_t readlane64(uint64_t v, int k)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), k);
    return ((uint64_t)hi << 32) | lo;
}
__device__ inline double readlane_f64(double v, int k)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), k), hi = __builtin_amdgcn_readlane(__double2hiint(v), k);
    return __hiloint2double(hi, lo);
}
__device__ inline uint64_t uniform64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}
// lanes below this one whose bit is set in m
__device__ inline int rank_in(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// this lane's bit of a wave-uniform mask
__device__ inline bool lane_bit(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// A box's header and what its visitor needs of it, loaded together.
template <class B>
struct HdrBox {
    CellHdr h;
    B box;
};

// Smallest and largest FP64 squared distance of a point to the group's
// bounding box; both round like the per-ray sqdist, so they bound its value for
// every ray of the group.
__device__ inline void box_dist2(const RayGroup& g, double cx, double cy, double* dn2, double* df2)
{
#pragma clang fp contract(off)
    const double xa = g.gx0 - cx, xb = g.gx1 - cx, ya = g.gy0 - cy, yb = g.gy1 - cy;
    const double nx = fmax(fmax(xa, -xb), 0.0), ny = fmax(fmax(ya, -yb), 0.0);
    const double fx = fmax(fabs(xa), fabs(xb)), fy = fmax(fabs(ya), fabs(yb));
    *dn2 = nx * nx + ny * ny;
    *df2 = fx * fx + fy * fy;
}

// The traversal (see the file comment).  Every lane of the group's W
// wavefronts calls it; X, Y is the lane's ray (the same in every wavefront).
// RANGE: only the boxes [c0, c1) of the preorder go to the visitor, their
// ancestors are passed through (a group's work over several workgroups).
template <bool COOP, bool RANGE, class V>
__device__ inline void traverse(const TreeDev& T, V& v, const RayGroup& g, double X, double Y, int lane, int w, int W,
                                const TravLds& L, int c0 = 0, int c1 = 0)
{
    int top = 1;
    if (w == 0 && lane == 0) {
        L.stkb[0] = 0;
        L.stkm[0] = g.full;
    }
    if constexpr (COOP) __syncthreads();
    int rot = 0; // which wavefront takes the next queue item
    int nf = 0;  // far boxes queued
    while (top > 0) {
        if constexpr (V::farfield && !COOP)
            if (nf >= kWave) {
                nf -= kWave;
                v.far(L.fq[nf + lane], true);
            }
        top = __builtin_amdgcn_readfirstlane(top);
        const int n = take_count(top, L.cap, COOP ? (kWave * W < L.qcap ? kWave * W : L.qcap) : kWave);
        const int idx = COOP ? lane * W + w : lane; // interleaved, so that every wavefront gets a share
        const bool has = idx < n;
        top -= n;
        int c = 0;
        uint64_t m = 0;
        if (has) {
            c = L.stkb[top + idx];
            m = L.stkm[top + idx];
        }
        const CellHdr h = T.hdr[c];
        const bool in = RANGE ? has && h.next > c0 && c < c1 : has;
        const bool own = RANGE ? in && c >= c0 : has;
        const uint64_t ownm = RANGE && !COOP ? __ballot(own) : 0;
        double dn2, df2;
        box_dist2(g, h.cx, h.cy, &dn2, &df2);
        const bool all = in && dn2 > h.rcut2;
        const bool mixed = in && !all && df2 > h.rcut2;
        const bool leaf = (h.info & kInfoLeaf) != 0;
        bool fa = false;
        if constexpr (V::farfield) {
            fa = own && all && m == g.full && is_far(g, h, T.theta);
            const uint64_t fb = __ballot(fa);
            if constexpr (!COOP) {
                if (fa) L.fq[nf + rank_in(fb)] = c;
                nf += __popcll(fb);
            }
            if constexpr (V::stats) v.accepted(__popcll(fb));
        }
        if constexpr (V::stats) v.visited(__popcll(__ballot(own && m == g.full)));
        // the boxes that only some rays accept, and (SOLO) all the work of the accepted ones
        uint64_t am = all ? m : 0ull;
        uint64_t todo = COOP ? __ballot(mixed) : __ballot(mixed || (own && all && !fa));
        if constexpr (COOP) {
            while (todo) {
                const int k = __ffsll((unsigned long long)todo) - 1;
                todo &= todo - 1;
                const bool act = lane_bit(readlane64(m, k));
                double w1, w2;
                const double d2 = sqdist(X, Y, readlane_f64(h.cx, k), readlane_f64(h.cy, k), &w1, &w2);
                const uint64_t ak = __ballot(act && d2 > readlane_f64(h.rcut2, k));
                if (lane == k) am = ak;
            }
        } else if (todo) {
            int k = __ffsll((unsigned long long)todo) - 1, ck = __builtin_amdgcn_readlane(c, k);
            typename V::Box even = v.load(ck), odd;
            // one box of the round: `now` is here, `then` is loaded behind the work on it (two
            // records that take turns, no copies: the loop issues as many scalar instructions
            // as vector ones)
            const auto step = [&](typename V::Box& now, typename V::Box& then) {
                todo &= todo - 1;
                const int kn = todo ? __ffsll((unsigned long long)todo) - 1 : k;
                int cn = __builtin_amdgcn_readlane(c, kn);
                settle(now, cn);
                then = v.load(cn);
                const bool act = lane_bit(readlane64(m, k));
                double w1, w2;
                const double d2 = sqdist(X, Y, readlane_f64(h.cx, k), readlane_f64(h.cy, k), &w1, &w2);
                const bool acc = act && d2 > readlane_f64(h.rcut2, k);
                const uint64_t ak = __ballot(acc);
                if (ak && (!RANGE || ((ownm >> k) & 1))) v.box(now, ck, acc, w1, w2);
                if (lane == k) am = ak;
                const bool more = kn != k;
                k = kn;
                ck = cn;
                return more;
            };
            while (step(even, odd) && step(odd, even)) {
            }
        }
        if constexpr (V::stats) {
            uint64_t part = __ballot(own && m != g.full);
            while (part) {
                const int k = __ffsll((unsigned long long)part) - 1;
                part &= part - 1;
                v.visited_some(lane_bit(readlane64(m, k)));
            }
        }
        const uint64_t om = m & ~am; // the rays that open the box
        bool lr = false;
        if (own && (h.info & kInfoList)) {
            const double* q = T.lreach + 4 * (size_t)c;
            lr = (g.gx1 >= q[0]) & (g.gx0 <= q[1]) & (g.gy1 >= q[2]) & (g.gy0 <= q[3]);
        }
        const bool opl = own && leaf && om != 0;
        CellExt e{};
        if (lr || opl) e = T.ext[c];
        if constexpr (!COOP) {
            uint64_t lt = __ballot(lr);
            while (lt) {
                const int k = __ffsll((unsigned long long)lt) - 1;
                lt &= lt - 1;
                v.list(__builtin_amdgcn_readlane(e.lbeg, k), __builtin_amdgcn_readlane(e.lend, k), kWave,
                       readlane64(m, k));
            }
            uint64_t lf = __ballot(opl);
            while (lf) {
                const int k = __ffsll((unsigned long long)lf) - 1;
                lf &= lf - 1;
                v.leaf(__builtin_amdgcn_readlane(e.pbeg, k), __builtin_amdgcn_readlane(e.pend, k), readlane64(om, k));
            }
        }
        // children of the opened boxes
        const bool push = in && !leaf && om != 0;
        int4 kc = make_int4(-1, -1, -1, -1);
        if (push) kc = *reinterpret_cast<const int4*>(T.kids + 4 * (size_t)c);
        const int kid[4] = {kc.x, kc.y, kc.z, kc.w};
        uint64_t kb[4];
        int nk = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            kb[u] = __ballot(kid[u] >= 0);
            nk += __popcll(kb[u]);
        }
        int at = top; // where this wavefront's children go
        if constexpr (COOP) {
            const uint64_t qa[4] = {__ballot(own && am != 0 && !fa), __ballot(opl), __ballot(lr), __ballot(fa)};
            // counts of this wavefront, two to a word (a round's are below 2^16)
            const int pk[2] = {(int)(__popcll(qa[0]) | (__popcll(qa[1]) << 16)),
                               (int)(__popcll(qa[2]) | (__popcll(qa[3]) << 16))};
            if (lane == 0) {
                L.cnt[w] = nk;
                L.cnt[kMaxGroupWaves + w] = pk[0];
                L.cnt[2 * kMaxGroupWaves + w] = pk[1];
            }
            __syncthreads();
            // lane 16 q + u: word q of wavefront u; inclusive sums along each row of 16
            int cv = (lane & 15) < W && lane < 3 * kMaxGroupWaves ? L.cnt[lane] : 0;
#pragma unroll
            for (int o = 1; o < kMaxGroupWaves; o <<= 1) {
                const int t = __shfl_up(cv, o, kMaxGroupWaves);
                if ((lane & 15) >= o) cv += t;
            }
            at += __builtin_amdgcn_readlane(cv, w) - nk;
            top += __builtin_amdgcn_readlane(cv, 15);
            int qn[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int word = q >> 1, sh = 16 * (q & 1);
                const int off = ((__builtin_amdgcn_readlane(cv, 16 * (word + 1) + w) - pk[word]) >> sh) & 0xffff;
                qn[q] = (__builtin_amdgcn_readlane(cv, 16 * (word + 1) + 15) >> sh) & 0xffff;
                if (lane_bit(qa[q])) {
                    if (q == 3) {
                        L.fq[nf + off + rank_in(qa[q])] = c;
                    } else {
                        const int p = q * L.qcap + off + rank_in(qa[q]);
                        L.qb[p] = q == 0 ? c : (q == 1 ? e.pbeg : e.lbeg);
                        if (q > 0) L.qe[p - L.qcap] = q == 1 ? e.pend : e.lend;
                        L.qm[p] = q == 0 ? am : (q == 1 ? om : m);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (kid[u] >= 0) {
                    const int p = at + rank_in(kb[u]);
                    L.stkb[p] = kid[u];
                    L.stkm[p] = om;
                }
                at += __popcll(kb[u]);
            }
            __syncthreads();
            // the round's work, dealt item by item (W is a power of two); far
            // boxes 64 at a time, the rest wait for the next round
            if constexpr (V::farfield) {
                nf += qn[3];
                while (nf >= kWave) {
                    nf -= kWave;
                    if (((w - rot++) & (W - 1)) == 0) v.far(L.fq[nf + lane], true);
                }
            }
            int i = (w - rot) & (W - 1);
            if (i < qn[0]) {
                int ck = __builtin_amdgcn_readfirstlane(L.qb[i]);
                uint64_t mk = uniform64(L.qm[i]);
                HdrBox<typename V::Box> even{uniform_ld(T.hdr, ck), v.load(ck)}, odd;
                const auto step = [&](HdrBox<typename V::Box>& now, HdrBox<typename V::Box>& then) {
                    i += W;
                    const int in = i < qn[0] ? i : i - W;
                    int cn = __builtin_amdgcn_readfirstlane(L.qb[in]);
                    const uint64_t mn = uniform64(L.qm[in]);
                    settle(now, cn);
                    then = {uniform_ld(T.hdr, cn), v.load(cn)};
                    v.box(now.box, ck, lane_bit(mk), X - now.h.cx, Y - now.h.cy);
                    ck = cn;
                    mk = mn;
                    return i < qn[0];
                };
                while (step(even, odd) && step(odd, even)) {
                }
            }
            rot += qn[0];
            for (i = (w - rot) & (W - 1); i < qn[1]; i += W) {
                const int p = L.qcap + i;
                v.leaf(__builtin_amdgcn_readfirstlane(L.qb[p]), __builtin_amdgcn_readfirstlane(L.qe[i]),
                       uniform64(L.qm[p]));
            }
            rot += qn[1];
            // the 64-entry chunks of all lists in turn
            for (i = 0; i < qn[2]; ++i) {
                const int p = 2 * L.qcap + i;
                const int lb = __builtin_amdgcn_readfirstlane(L.qb[p]);
                const int le = __builtin_amdgcn_readfirstlane(L.qe[L.qcap + i]);
                const int my = (w - rot) & (W - 1), chunks = (le - lb + kWave - 1) / kWave;
                rot += chunks;
                if (my < chunks) v.list(lb + my * kWave, le, kWave * W, uniform64(L.qm[p]));
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (kid[u] >= 0) {
                    const int p = at + rank_in(kb[u]);
                    L.stkb[p] = kid[u];
                    L.stkm[p] = om;
                }
                at += __popcll(kb[u]);
            }
            top = at;
        }
    }
    if constexpr (V::farfield) {
        if (COOP && ((w - rot) & (W - 1)) != 0) return; // (fewer than 64 left: one wavefront's pass)
        while (nf > 0) {
            const int n = nf < kWave ? nf : kWave;
            nf -= n;
            v.far(lane < n ? L.fq[nf + lane] : 0, lane < n);
        }
    }
}

} // namespace glm
