// Shared by the two nearest-neighbour kernels: the k smallest values seen by a
// lane, and the pieces of their traversal.
//
// One wavefront serves 64 particles, one per lane.  Boxes wait on a stack in LDS;
// a round takes many, one per lane, drops those farther from the wavefront's
// bounding box than the largest k-th distance of its lanes, and tests the others
// lane by lane with their bounds broadcast from the lane that loaded them, so
// that a round pays one load latency for up to 64 boxes.  (A stackless walk with a
// dependent scalar load per box spent most of its time waiting for them.)
#pragma once

#include "lanesum.hpp"

namespace glm {

// An ascending list of KC values in registers, whose first KC - k slots hold -inf,
// so that the k-th smallest always sits in the last slot; and a queue in LDS
// of values below it that are not in the list yet.  A list insertion costs 2 KC FP64
// instructions of the whole wavefront whichever lanes need it, and with lanes at
// different particles nearly every candidate is needed by some lane but only by
// a few.  The queue lets each lane collect its own; when some lane has kKnnQueue of
// them, all lanes insert what they have, one per round.  The bound a lane tests
// against is then a little old, never too small.  1e6 particles of an NFW halo,
// k = 32: 8.7-11.5 ms with a stackless walk and one insertion per candidate, 1.7 ms
// with the queue and the stack (3D: 11.5 against 4.5 ms); what remains is FP64
// arithmetic of the insertions at two wavefronts per SIMD (the list's registers).
constexpr int kKnnQueue = 8;

// Smaller and larger of two values, neither a NaN.  (fmin and fmax first
// quiet their operands: 32 more instructions in an insertion of a list of 32.)
__device__ inline double min_nonan(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline double max_nonan(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

template <int KC>
struct KnnList {
    double h[KC];
    double* q; // kKnnQueue x 64 doubles of LDS, this lane's column
    int cnt = 0;

    __device__ KnnList(int k, double* lds, int lane) : q(lds + lane)
    {
#pragma unroll
        for (int i = 0; i < KC; ++i) h[i] = i < KC - k ? -INFINITY : INFINITY;
    }

    __device__ double bound() const { return h[KC - 1]; }

    // v into the list (the largest entry drops out): h[i] <- max(h[i-1], min(v, h[i])).
    __device__ void insert(double v)
    {
#pragma unroll
        for (int i = KC - 1; i > 0; --i) h[i] = max_nonan(h[i - 1], min_nonan(v, h[i]));
        h[0] = min_nonan(v, h[0]);
    }

    // Every lane of the wavefront offers a value (INFINITY for none).
    __device__ void offer(double v)
    {
        const bool need = v < bound();
        if (need) q[cnt * kWave] = v;
        cnt += need;
        if (__any(cnt == kKnnQueue)) flush();
    }

    __device__ void flush()
    {
        for (int i = 0; __any(i < cnt); ++i) insert(i < cnt ? q[i * kWave] : INFINITY);
        cnt = 0;
    }
};

// The particle of lane `lane` of the wavefront that serves g0 .. g0 + 63 of n
// particles: its own, or g0 for the idle lanes of the last wavefront.
__host__ __device__ inline int knn_particle(int g0, int lane, int n) { return lane < n - g0 ? g0 + lane : g0; }

// Particle j's neighbours o places before and after it along the sorted order
// of n particles, j itself where there is none.  (No sum of the two that could
// pass 2^31.)
struct KnnSeed {
    int before, after;
    bool has_before, has_after;
};
__host__ __device__ inline KnnSeed knn_seed(int j, int o, int n)
{
    KnnSeed s;
    s.has_before = j >= o;
    s.has_after = n - 1 - j >= o;
    s.before = s.has_before ? j - o : j;
    s.after = s.has_after ? j + o : j;
    return s;
}

__device__ inline double knn_bcast(double v, int k)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), k), hi = __builtin_amdgcn_readlane(__double2hiint(v), k);
    return __hiloint2double(hi, lo);
}

// Position of this lane among the set bits of m.
__device__ inline int knn_rank(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Items to take off a stack of `top` items with room for `cap`, each of which
// may put `fan` on: as many as leave (fan - 1) `levels` free (what a descent one by
// one can need), at least one.
__device__ inline int knn_take(int top, int cap, int fan, int levels)
{
    int n = (cap - top - (fan - 1) * levels) / (fan - 1);
    n = n < 1 ? 1 : (n < kWave ? n : kWave);
    return n < top ? n : top;
}

} // namespace glm
