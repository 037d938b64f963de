// Ray staging, and the launches of the forward walk (Sec. 3.2) and of the
// batched walk of many lenses.  The walk itself is in traverse.hpp and
// walk_fwd.hpp.
#include <math.h>

#include <algorithm>
#include <vector>

#include "walk_fwd.hpp"

namespace glm {

namespace {

// ------------------------------------------------------------ ray staging

// blocks of the first pass of the ray bounding box (enough waves in flight to
// stream the coordinates at full bandwidth)
constexpr int kRayBboxBlocks = 1024;

__global__ __launch_bounds__(kBlock) void k_ray_bbox(const double* __restrict__ x, const double* __restrict__ y,
                                                    int64_t n, double* __restrict__ part)
{
    __shared__ double red[4][kBlock];
    double x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        x0 = fmin(x0, x[i]);
        x1 = fmax(x1, x[i]);
        y0 = fmin(y0, y[i]);
        y1 = fmax(y1, y[i]);
    }
    red[0][threadIdx.x] = x0;
    red[1][threadIdx.x] = x1;
    red[2][threadIdx.x] = y0;
    red[3][threadIdx.x] = y1;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            red[0][threadIdx.x] = fmin(red[0][threadIdx.x], red[0][threadIdx.x + o]);
            red[1][threadIdx.x] = fmax(red[1][threadIdx.x], red[1][threadIdx.x + o]);
            red[2][threadIdx.x] = fmin(red[2][threadIdx.x], red[2][threadIdx.x + o]);
            red[3][threadIdx.x] = fmax(red[3][threadIdx.x], red[3][threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int k = 0; k < 4; ++k) part[blockIdx.x * 4 + k] = red[k][0];
}

// Position of cell (x, y) along the Hilbert curve over 2^bits x 2^bits cells
// (quadrant by quadrant from the top: the curve's four quadrants in order,
// then the frame of the one entered, transposed or turned).  64 rays in a row
// along it always form one compact patch; along the Morton curve, which jumps,
// a third of the groups of a grid that is not a power of two across straddled a
// jump, and walking such a group costs several times a compact one: 837^2 rays
// on 1e6 particles took 4.0 ms against 2.6 ms for the 1024^2 rays of an aligned grid.
__device__ inline uint32_t hilbert_key(uint32_t x, uint32_t y, int bits)
{
    uint32_t d = 0;
    for (int s = bits - 1; s >= 0; --s) {
        const uint32_t rx = (x >> s) & 1u, ry = (y >> s) & 1u;
        d = (d << 2) | ((3u * rx) ^ ry);
        const uint32_t flip = (ry == 0u && rx != 0u) ? ~0u : 0u;
        const uint32_t fx = x ^ flip, fy = y ^ flip;
        x = ry == 0u ? fy : fx;
        y = ry == 0u ? fx : fy;
    }
    return d;
}

// bounding box of the rays from the per-block partials
__global__ __launch_bounds__(kBlock) void k_ray_root(const double* __restrict__ part, int nb, double* __restrict__ bb)
{
    __shared__ double red[4][kBlock];
    double v[4] = {INFINITY, -INFINITY, INFINITY, -INFINITY};
    for (int b = threadIdx.x; b < nb; b += kBlock) {
        v[0] = fmin(v[0], part[b * 4 + 0]);
        v[1] = fmax(v[1], part[b * 4 + 1]);
        v[2] = fmin(v[2], part[b * 4 + 2]);
        v[3] = fmax(v[3], part[b * 4 + 3]);
    }
    for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            red[0][threadIdx.x] = fmin(red[0][threadIdx.x], red[0][threadIdx.x + o]);
            red[1][threadIdx.x] = fmax(red[1][threadIdx.x], red[1][threadIdx.x + o]);
            red[2][threadIdx.x] = fmin(red[2][threadIdx.x], red[2][threadIdx.x + o]);
            red[3][threadIdx.x] = fmax(red[3][threadIdx.x], red[3][threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x < 4) bb[threadIdx.x] = red[threadIdx.x][0];
}

// Hilbert keys of the rays in their bounding square, `bits` (<= 16) per axis
__global__ __launch_bounds__(kBlock) void k_ray_keys(const double* __restrict__ x, const double* __restrict__ y,
                                                    int64_t n, const double* __restrict__ bb, int bits,
                                                    uint32_t* __restrict__ key, uint32_t* __restrict__ val)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double bx0 = bb[0], by0 = bb[2];
    double ext = fmax(bb[1] - bx0, bb[3] - by0);
    if (!(ext > 0.0)) ext = 1.0;
    const double top = (double)((1u << bits) - 1u);
    const double sc = top / ext;
    const uint32_t qx = (uint32_t)fmin(fmax((x[i] - bx0) * sc, 0.0), top);
    const uint32_t qy = (uint32_t)fmin(fmax((y[i] - by0) * sc, 0.0), top);
    key[i] = hilbert_key(qx, qy, bits);
    val[i] = (uint32_t)i;
}

__global__ __launch_bounds__(kBlock) void k_ray_gather(const uint32_t* __restrict__ perm, const double* __restrict__ x,
                                                      const double* __restrict__ y, int64_t n, double* __restrict__ xs,
                                                      double* __restrict__ ys)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    xs[k] = x[perm[k]];
    ys[k] = y[perm[k]];
}

} // namespace

// Slots for the sums of a split walk, growing with nrays (a workspace for a launch also serves
// every smaller one).
static int64_t split_slots(int64_t nrays)
{
    const int64_t groups = (nrays + kWave - 1) / kWave;
    return kWave * std::min(kMaxSplit * groups, kOpenGroups);
}

RayLayout ray_layout(int64_t nrays)
{
    RayLayout L;
    Arena a;
    L.k0 = a.take(4ull * nrays);
    L.k1 = a.take(4ull * nrays);
    L.v0 = a.take(4ull * nrays);
    L.v1 = a.take(4ull * nrays);
    L.xs = a.take(8ull * nrays);
    L.ys = a.take(8ull * nrays);
    L.hist = a.take(4ull * radix_hist_words(nrays));
    L.part = a.take(sizeof(double) * 4 * (kRayBboxBlocks + 1));
    L.parts = a.take(sizeof(Partial) * (size_t)split_slots(nrays));
    L.bytes = a.size;
    return L;
}

// Bits per axis of the ray sort key.  The key only forms the ray groups (a ray's
// decisions do not depend on them, and where far boxes are expanded its values do by rounding):
// about four cells per ray suffice, 8 to 16 bits per axis.
static int ray_key_bits(int64_t nrays)
{
    int bits = 8;
    while (bits < 16 && (1ll << (2 * bits)) < 4 * nrays) ++bits;
    return bits;
}

glm_status stage_rays(const double* rx, const double* ry, int64_t nrays, void* ws, const RayLayout& L,
                      StagedRays* out, hipStream_t st)
{
    char* W = static_cast<char*>(ws);
    uint32_t* k0 = reinterpret_cast<uint32_t*>(W + L.k0);
    uint32_t* k1 = reinterpret_cast<uint32_t*>(W + L.k1);
    uint32_t* v0 = reinterpret_cast<uint32_t*>(W + L.v0);
    uint32_t* v1 = reinterpret_cast<uint32_t*>(W + L.v1);
    double* xs = reinterpret_cast<double*>(W + L.xs);
    double* ys = reinterpret_cast<double*>(W + L.ys);
    uint32_t* hist = reinterpret_cast<uint32_t*>(W + L.hist);
    double* part = reinterpret_cast<double*>(W + L.part);
    const int nbb = kRayBboxBlocks;
    const int g = ceil_div(nrays, kBlock);
    hipLaunchKernelGGL(k_ray_bbox, dim3(nbb), dim3(kBlock), 0, st, rx, ry, nrays, part);
    hipLaunchKernelGGL(k_ray_root, dim3(1), dim3(kBlock), 0, st, part, nbb, part + 4 * nbb);
    const int bits = ray_key_bits(nrays);
    hipLaunchKernelGGL(k_ray_keys, dim3(g), dim3(kBlock), 0, st, rx, ry, nrays, part + 4 * nbb, bits, k0, v0);
    const int w = radix_sort_u32(k0, v0, k1, v1, nrays, (2 * bits + 7) / 8, hist, st);
    const uint32_t* perm = w ? v1 : v0;
    hipLaunchKernelGGL(k_ray_gather, dim3(g), dim3(kBlock), 0, st, perm, rx, ry, nrays, xs, ys);
    GLM_HIP(hipGetLastError());
    *out = staged_rays_view(nrays, ws, L);
    return GLM_OK;
}

StagedRays staged_rays_view(int64_t nrays, void* ws, const RayLayout& L)
{
    char* W = static_cast<char*>(ws);
    // the sort ends in (k1, v1) after an odd number of passes (radix_sort_u32)
    const int passes = (2 * ray_key_bits(nrays) + 7) / 8;
    const uint32_t* perm = reinterpret_cast<const uint32_t*>(W + ((passes & 1) ? L.v1 : L.v0));
    return StagedRays{reinterpret_cast<const double*>(W + L.xs), reinterpret_cast<const double*>(W + L.ys), perm};
}

// ------------------------------------------------------------ batched walk

namespace {

constexpr int kBboxSplit = 32; // blocks per lens for the ray bounding boxes

__global__ __launch_bounds__(kBlock) void k_batch_bbox(const BatchLens* __restrict__ lenses, double* __restrict__ part)
{
    __shared__ double red[4][kBlock];
    const BatchLens& L = lenses[blockIdx.x];
    double v[4] = {INFINITY, -INFINITY, INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.y * kBlock + threadIdx.x; i < L.nrays; i += (int64_t)kBlock * kBboxSplit) {
        const double x = L.rx[i], y = L.ry[i];
        v[0] = fmin(v[0], x);
        v[1] = fmax(v[1], x);
        v[2] = fmin(v[2], y);
        v[3] = fmax(v[3], y);
    }
    for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            red[0][threadIdx.x] = fmin(red[0][threadIdx.x], red[0][threadIdx.x + o]);
            red[1][threadIdx.x] = fmax(red[1][threadIdx.x], red[1][threadIdx.x + o]);
            red[2][threadIdx.x] = fmin(red[2][threadIdx.x], red[2][threadIdx.x + o]);
            red[3][threadIdx.x] = fmax(red[3][threadIdx.x], red[3][threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x < 4) part[((size_t)blockIdx.x * kBboxSplit + blockIdx.y) * 4 + threadIdx.x] = red[threadIdx.x][0];
}

__global__ void k_batch_bbox_final(const double* __restrict__ part, int nlens, double* __restrict__ bb)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 4 * nlens) return;
    const int l = t / 4, k = t % 4;
    double v = (k & 1) ? -INFINITY : INFINITY;
    for (int b = 0; b < kBboxSplit; ++b) {
        const double p = part[((size_t)l * kBboxSplit + b) * 4 + k];
        v = (k & 1) ? fmax(v, p) : fmin(v, p);
    }
    bb[t] = v;
}

__device__ inline int find_lens(const int64_t* __restrict__ roff, int nlens, int64_t gi)
{
    int lo = 0, hi = nlens;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (roff[mid] <= gi) lo = mid;
        else hi = mid;
    }
    return lo;
}

// key = lens rank << 2 bits | Hilbert key in the lens's ray box
__global__ __launch_bounds__(kBlock) void k_batch_keys(const BatchLens* __restrict__ lenses, int nlens,
                                                      const int64_t* __restrict__ roff, const double* __restrict__ bb,
                                                      int64_t total, int bits, uint64_t* __restrict__ key,
                                                      uint32_t* __restrict__ val)
{
    const int64_t gi = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (gi >= total) return;
    const int l = find_lens(roff, nlens, gi);
    const int64_t i = gi - roff[l];
    const double bx0 = bb[4 * l], by0 = bb[4 * l + 2];
    double ext = fmax(bb[4 * l + 1] - bx0, bb[4 * l + 3] - by0);
    if (!(ext > 0.0)) ext = 1.0;
    const double top = (double)((1u << bits) - 1u);
    const double sc = top / ext;
    const uint32_t qx = (uint32_t)fmin(fmax((lenses[l].rx[i] - bx0) * sc, 0.0), top);
    const uint32_t qy = (uint32_t)fmin(fmax((lenses[l].ry[i] - by0) * sc, 0.0), top);
    key[gi] = ((uint64_t)l << (2 * bits)) | (uint64_t)hilbert_key(qx, qy, bits);
    val[gi] = (uint32_t)gi;
}

__global__ __launch_bounds__(kBlock) void k_batch_gather(const BatchLens* __restrict__ lenses,
                                                        const int64_t* __restrict__ roff,
                                                        const uint64_t* __restrict__ key,
                                                        const uint32_t* __restrict__ val, int64_t total, int bits,
                                                        double* __restrict__ xs, double* __restrict__ ys)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= total) return;
    const int l = (int)(key[k] >> (2 * bits));
    const int64_t i = (int64_t)val[k] - roff[l];
    xs[k] = lenses[l].rx[i];
    ys[k] = lenses[l].ry[i];
}

__global__ void k_zero_int(int* p) { *p = 0; }

struct BatchLayout {
    size_t table, roff, gpre, bb, bbpart, counter, k0, k1, v0, v1, xs, ys, hist, bytes;
};

BatchLayout batch_layout(int nlens, int64_t total)
{
    BatchLayout B;
    Arena a;
    B.table = a.take(sizeof(BatchLens) * (size_t)nlens);
    B.roff = a.take(8ull * (nlens + 1));
    B.gpre = a.take(8ull * (nlens + 1));
    B.bb = a.take(32ull * nlens);
    B.bbpart = a.take(32ull * nlens * kBboxSplit);
    B.counter = a.take(64);
    B.k0 = a.take(8ull * total);
    B.k1 = a.take(8ull * total);
    B.v0 = a.take(4ull * total);
    B.v1 = a.take(4ull * total);
    B.xs = a.take(8ull * total);
    B.ys = a.take(8ull * total);
    B.hist = a.take(4ull * radix_hist_words(total));
    B.bytes = a.size;
    return B;
}

} // namespace

size_t batch_workspace_bytes(int nlens, int64_t total) { return batch_layout(nlens, total).bytes; }

glm_status shoot_batched_device(const BatchLens* host_table, int nlens, int order, uint32_t flags, void* ws,
                                hipStream_t st)
{
    int64_t total = 0, items = 0;
    std::vector<int64_t> roff(nlens + 1), gpre(nlens + 1);
    for (int l = 0; l < nlens; ++l) {
        roff[l] = total;
        gpre[l] = items;
        total += host_table[l].nrays;
        items += (host_table[l].nrays + kWave - 1) / kWave;
    }
    roff[nlens] = total;
    gpre[nlens] = items;
    if (total == 0) return GLM_OK;
    std::vector<BatchLens> tab(host_table, host_table + nlens);
    for (int l = 0; l < nlens; ++l) tab[l].ray_off = roff[l];
    const BatchLayout B = batch_layout(nlens, total);
    char* W = static_cast<char*>(ws);
    BatchLens* dtab = reinterpret_cast<BatchLens*>(W + B.table);
    int64_t* droff = reinterpret_cast<int64_t*>(W + B.roff);
    int64_t* dgpre = reinterpret_cast<int64_t*>(W + B.gpre);
    double* bb = reinterpret_cast<double*>(W + B.bb);
    int* counter = reinterpret_cast<int*>(W + B.counter);
    uint64_t* k0 = reinterpret_cast<uint64_t*>(W + B.k0);
    uint64_t* k1 = reinterpret_cast<uint64_t*>(W + B.k1);
    uint32_t* v0 = reinterpret_cast<uint32_t*>(W + B.v0);
    uint32_t* v1 = reinterpret_cast<uint32_t*>(W + B.v1);
    double* xs = reinterpret_cast<double*>(W + B.xs);
    double* ys = reinterpret_cast<double*>(W + B.ys);
    uint32_t* hist = reinterpret_cast<uint32_t*>(W + B.hist);
    GLM_HIP(hipMemcpyAsync(dtab, tab.data(), sizeof(BatchLens) * nlens, hipMemcpyHostToDevice, st));
    GLM_HIP(hipMemcpyAsync(droff, roff.data(), 8ull * (nlens + 1), hipMemcpyHostToDevice, st));
    GLM_HIP(hipMemcpyAsync(dgpre, gpre.data(), 8ull * (nlens + 1), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, st, counter);
    double* bbpart = reinterpret_cast<double*>(W + B.bbpart);
    hipLaunchKernelGGL(k_batch_bbox, dim3(nlens, kBboxSplit), dim3(kBlock), 0, st, dtab, bbpart);
    hipLaunchKernelGGL(k_batch_bbox_final, dim3(ceil_div(4 * nlens, 64)), dim3(64), 0, st, bbpart, nlens, bb);
    const int g = ceil_div(total, kBlock);
    // per lens, about four cells per ray (the largest lens sets the width)
    int64_t most = 0;
    for (int l = 0; l < nlens; ++l) most = std::max(most, host_table[l].nrays);
    int bits = 8;
    while (bits < 16 && (1ll << (2 * bits)) < 4 * most) ++bits;
    hipLaunchKernelGGL(k_batch_keys, dim3(g), dim3(kBlock), 0, st, dtab, nlens, droff, bb, total, bits, k0, v0);
    int lens_bits = 0;
    while ((1 << lens_bits) < nlens) ++lens_bits;
    const int passes = (2 * bits + lens_bits + 7) / 8;
    const int w = radix_sort_u64(k0, v0, k1, v1, total, passes, hist, st);
    const uint64_t* ks = w ? k1 : k0;
    const uint32_t* perm = w ? v1 : v0;
    hipLaunchKernelGGL(k_batch_gather, dim3(g), dim3(kBlock), 0, st, dtab, droff, ks, perm, total, bits, xs, ys);
    // every lens of a batch has the same order and particle kind
    launch_walk_batched(BatchArgs{dtab, nlens, dgpre, counter, xs, ys, perm, items, order, host_table[0].tree.kind,
                                  (flags & GLM_ALPHA_ONLY) != 0, (flags & GLM_FP32_ALPHA) != 0, st});
    GLM_HIP(hipGetLastError());
    return GLM_OK;
}

namespace {

// Per ray, the sums of its box ranges in range order.
__global__ __launch_bounds__(kBlock) void k_walk_merge(const Partial* __restrict__ parts, int split, int64_t nrays,
                                                      const uint32_t* __restrict__ rperm, WalkOut out)
{
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= nrays) return;
    Partial s = parts[r];
    for (int k = 1; k < split; ++k) {
        const Partial& q = parts[(int64_t)k * nrays + r];
        s.a1 += q.a1;
        s.a2 += q.a2;
        s.k += q.k;
        s.g1 += q.g1;
        s.g2 += q.g2;
        s.ps += q.ps;
        for (int i = 0; i < kCounts; ++i) s.cnt[i] += q.cnt[i];
    }
    const int64_t o = rperm ? (int64_t)rperm[r] : r;
    out.a1[o] = (float)s.a1;
    out.a2[o] = (float)s.a2;
    if (out.k) out.k[o] = (float)s.k;
    if (out.g1) out.g1[o] = (float)s.g1;
    if (out.g2) out.g2[o] = (float)s.g2;
    if (out.psi) out.psi[o] = (float)s.ps;
    if (out.td) out.td[o] = (float)(0.5 * (s.a1 * s.a1 + s.a2 * s.a2) - s.ps);
    if (out.counts)
        for (int i = 0; i < kCounts; ++i) out.counts[kCounts * o + i] = s.cnt[i];
}

void merge_parts(const WalkArgs& a)
{
    if (a.shape.split > 1)
        hipLaunchKernelGGL(k_walk_merge, dim3(ceil_div(a.nrays, kBlock)), dim3(kBlock), 0, a.st, a.parts, a.shape.split,
                           a.nrays, a.rperm, a.out);
}

} // namespace

glm_status shoot_device(const TreeStorage& ts, const double* rx, const double* ry, int64_t nrays, float* a1,
                        float* a2, float* k, float* g1, float* g2, int32_t* counts, uint32_t flags, void* ws,
                        hipStream_t st)
{
    if (nrays == 0) return GLM_OK;
    StagedRays sr{rx, ry, nullptr};
    const RayLayout L = ray_layout(nrays);
    if (flags & GLM_RAYS_STAGED) {
        sr = staged_rays_view(nrays, ws, L); // glm_stage_rays left them in the workspace
    } else if (!(flags & GLM_RAYS_ORDERED)) {
        glm_status rc = stage_rays(rx, ry, nrays, ws, L, &sr, st);
        if (rc != GLM_OK) return rc;
    }
    const bool aonly = (flags & GLM_ALPHA_ONLY) != 0;
    if (aonly) k = g1 = g2 = nullptr;
    Partial* parts = reinterpret_cast<Partial*>(static_cast<char*>(ws) + L.parts);
    const WalkArgs a{ts.dev, sr.xs, sr.ys, sr.perm, nrays, WalkOut{a1, a2, k, g1, g2, counts}, walk_shape(nrays, ts),
                     walk_far(nrays, ts), parts, st};
    // the product walk with counters where counts are asked for, else the product or the plain-FP32 walk
    if (counts) launch_walk_counts(a, aonly);
    else if (flags & GLM_FP32_ALPHA) launch_walk_fp32(a, aonly);
    else if (aonly) launch_walk_alpha(a);
    else launch_walk_full(a);
    merge_parts(a);
    GLM_HIP(hipGetLastError());
    return GLM_OK;
}

glm_status potential_device(const TreeStorage& ts, const double* rx, const double* ry, int64_t nrays, float* a1,
                            float* a2, float* psi, float* td, uint32_t flags, void* ws, hipStream_t st)
{
    if (nrays == 0) return GLM_OK;
    StagedRays sr{rx, ry, nullptr};
    const RayLayout L = ray_layout(nrays);
    if (!(flags & GLM_RAYS_ORDERED)) {
        glm_status rc = stage_rays(rx, ry, nrays, ws, L, &sr, st);
        if (rc != GLM_OK) return rc;
    }
    WalkOut out{a1, a2, nullptr, nullptr, nullptr, nullptr};
    out.psi = psi;
    out.td = td;
    Partial* parts = reinterpret_cast<Partial*>(static_cast<char*>(ws) + L.parts);
    const WalkArgs a{ts.dev, sr.xs, sr.ys, sr.perm, nrays, out, walk_shape(nrays, ts), walk_far(nrays, ts), parts, st};
    launch_walk_potential(a);
    merge_parts(a);
    GLM_HIP(hipGetLastError());
    return GLM_OK;
}

} // namespace glm
