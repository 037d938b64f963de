// Stable LSD radix sort (8-bit digits) and exclusive scan for gfx950.
//
// Sort pass = histogram per 2048-key tile -> per digit, an exclusive scan of
// its counts over the tiles (and the digit's total) -> scatter, where each
// tile takes its digit bases from the digit totals, ranks its keys stably
// (rank_tile), reorders them by digit in LDS and writes each
// digit's run with consecutive lanes.  Loads and stores are coalesced.
// Up to kFewTiles tiles the scatter adds the tiles' counts up itself, and up
// to kOneBlock keys one workgroup does all passes in LDS: at these sizes the time is
// launches and latency, not bytes.
#include "lanesum.hpp"

namespace glm {

namespace {

constexpr int kItems = 8;                  // keys per thread per tile
constexpr int kTile = kBlock * kItems;     // 2048
constexpr int kScanItems = 16;
constexpr int kScanTile = kBlock * kScanItems; // 4096

__device__ inline uint32_t wave_incl_scan(uint32_t v, int lane)
{
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// exclusive scan over the threads of a block (256, or WAVES wavefronts); returns the block total in *tot
template <int WAVES = kBlock / kWave>
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t* lds_w, uint32_t* tot)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const uint32_t inc = wave_incl_scan(v, lane);
    if (lane == kWave - 1) lds_w[w] = inc;
    __syncthreads();
    uint32_t off = 0, all = 0;
#pragma unroll
    for (int k = 0; k < WAVES; ++k) {
        const uint32_t x = lds_w[k];
        off += (k < w) ? x : 0u;
        all += x;
    }
    __syncthreads();
    *tot = all;
    return off + inc - v;
}

__global__ __launch_bounds__(kBlock) void k_scan_reduce(const int32_t* in, int64_t n, uint32_t* part)
{
    __shared__ uint32_t lw[kBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t i = base + (int64_t)j * kBlock + threadIdx.x;
        if (i < n) s += (uint32_t)in[i];
    }
    uint32_t tot;
    block_excl_scan(s, lw, &tot);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// single block: exclusive scan of nb partials, total into out[n]
__global__ __launch_bounds__(1024) void k_scan_partials(uint32_t* part, int nb, int32_t* out, int64_t n)
{
    __shared__ uint32_t lw[1024 / kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const int per = (nb + 1023) / 1024;
    const int b0 = t * per;
    uint32_t s = 0;
    for (int k = 0; k < per; ++k)
        if (b0 + k < nb) s += part[b0 + k];
    const uint32_t inc = wave_incl_scan(s, lane);
    if (lane == kWave - 1) lw[w] = inc;
    __syncthreads();
    uint32_t off = 0, all = 0;
    for (int k = 0; k < 1024 / kWave; ++k) {
        off += (k < w) ? lw[k] : 0u;
        all += lw[k];
    }
    uint32_t run = off + inc - s;
    for (int k = 0; k < per; ++k)
        if (b0 + k < nb) {
            const uint32_t x = part[b0 + k];
            part[b0 + k] = run;
            run += x;
        }
    if (t == 0) out[n] = (int32_t)all;
}

__global__ __launch_bounds__(kBlock) void k_scan_apply(const int32_t* in, int32_t* out, int64_t n,
                                                      const uint32_t* part)
{
    __shared__ uint32_t lw[kBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t i = base + j;
        v[j] = i < n ? (uint32_t)in[i] : 0u;
        s += v[j];
    }
    uint32_t tot;
    uint32_t run = block_excl_scan(s, lw, &tot) + part[blockIdx.x];
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t i = base + j;
        if (i < n) out[i] = (int32_t)run;
        run += v[j];
    }
}

// Digit counts of one tile into hist[d * nb + tile], or hist[256 * tile + d] (FEW).
template <class K, bool FEW>
__global__ __launch_bounds__(kBlock) void k_radix_hist(const K* keys, int64_t n, int shift, uint32_t* hist,
                                                      int nb)
{
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kTile;
    // all of the thread's keys in flight together, then the counts
    K k[kItems];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t i = base + (int64_t)j * kBlock + threadIdx.x;
        k[j] = i < n ? keys[i] : (K)0;
    }
#pragma unroll
    for (int j = 0; j < kItems; ++j)
        if (base + (int64_t)j * kBlock + threadIdx.x < n) atomicAdd(&h[(uint32_t)(k[j] >> shift) & 255u], 1u);
    __syncthreads();
    hist[FEW ? (int64_t)blockIdx.x * 256 + threadIdx.x : (int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// One block per digit d: exclusive scan of hist[d * nb .. d * nb + nb) over
// the tiles into pre[], and the digit's total into dtot[d].
__global__ __launch_bounds__(kBlock) void k_radix_rowscan(const uint32_t* __restrict__ hist, int nb,
                                                         uint32_t* __restrict__ pre, uint32_t* __restrict__ dtot)
{
    __shared__ uint32_t lw[kBlock / kWave];
    const int d = blockIdx.x, t = threadIdx.x;
    const int per = (nb + kBlock - 1) / kBlock;
    const int64_t row = (int64_t)d * nb;
    const int b0 = t * per;
    uint32_t sum = 0;
    for (int k = 0; k < per; ++k)
        if (b0 + k < nb) sum += hist[row + b0 + k];
    uint32_t tot;
    uint32_t run = block_excl_scan(sum, lw, &tot);
    for (int k = 0; k < per; ++k)
        if (b0 + k < nb) {
            const uint32_t c = hist[row + b0 + k];
            pre[row + b0 + k] = run;
            run += c;
        }
    if (t == 0) dtot[d] = tot;
}

// Stable order by digit of a workgroup's keys: lane l's item j of wavefront w
// is tile position (w ITEMS + j) 64 + l, valid below m.  pos[j] becomes its position in digit
// order and the return value (threads t < 256) the first position of digit t.
// A wavefront ranks its items one after the other against its own counts in
// LDS, with no barrier between them (8 ballots give the lanes holding the same digit; a
// barrier per 256 keys and step made a pass of any size take
// 7 us; 4e6 keys 19.8 -> 16.4 us per pass); two barriers then add up the wavefronts' counts.
template <class K, int WAVES, int ITEMS>
__device__ inline uint32_t rank_tile(const K* keys, int shift, int m, uint32_t (*wcnt)[256], uint32_t* lw, uint32_t* pos)
{
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    for (int i = lane; i < 256; i += kWave) wcnt[w][i] = 0;
    wave_lds_sync();
    const uint64_t lt = __lanemask_lt();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const bool valid = (w * ITEMS + j) * kWave + lane < m;
        const uint32_t d = (uint32_t)(keys[j] >> shift) & 255u;
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            same &= bit ? bb : ~bb;
        }
        const uint32_t lrank = (uint32_t)__popcll(same & lt), before = wcnt[w][d];
        pos[j] = before + lrank;
        wave_lds_sync();
        if (valid && lrank == 0) wcnt[w][d] = before + (uint32_t)__popcll(same);
        wave_lds_sync();
    }
    __syncthreads();
    uint32_t cnt = 0;
    if (t < 256)
        for (int k = 0; k < WAVES; ++k) {
            const uint32_t c = wcnt[k][t];
            wcnt[k][t] = cnt;
            cnt += c;
        }
    uint32_t tot;
    const uint32_t first = block_excl_scan<WAVES>(cnt, lw, &tot);
    if (t < 256)
        for (int k = 0; k < WAVES; ++k) wcnt[k][t] += first;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) pos[j] += wcnt[w][(uint32_t)(keys[j] >> shift) & 255u];
    return first;
}

// Scatter of one tile: the keys are placed in LDS in digit order,
// then written out slot by slot, so that consecutive lanes write consecutive
// addresses of the same digit's run.  The tile's run of digit d starts at
// (keys of digits below d) + (keys of digit d in the tiles before): dtot and pre, or
// the sums of all tiles' counts (FEW).
template <class K, bool FEW>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(const K* kin, const uint32_t* vin, K* kout,
                                                         uint32_t* vout, int64_t n, int shift,
                                                         const uint32_t* __restrict__ hist,
                                                         const uint32_t* __restrict__ pre,
                                                         const uint32_t* __restrict__ dtot, int nb)
{
    constexpr int WAVES = kBlock / kWave;
    __shared__ K sk[kTile];
    __shared__ uint32_t sv[kTile];
    __shared__ uint32_t gbase[256]; // global position of slot 0 for digit d's run
    __shared__ uint32_t wcnt[WAVES][256];
    __shared__ uint32_t lw[WAVES];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    // the thread's keys and values of the whole tile are loaded up front, so
    // their latency overlaps the digit bases' loads and is paid once per tile
    const int64_t base = (int64_t)blockIdx.x * kTile;
    const int m = (int)(n - base < (int64_t)kTile ? n - base : (int64_t)kTile);
    K keys[kItems];
    uint32_t vals[kItems], pos[kItems];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int i = (w * kItems + j) * kWave + lane;
        keys[j] = i < m ? kin[base + i] : (K)0;
        vals[j] = i < m ? vin[base + i] : 0u;
    }
    uint32_t total = 0, mine = 0; // of digit t
    if constexpr (FEW) {
        for (int b0 = 0; b0 < nb; b0 += 16) { // 16 loads in flight
            uint32_t c[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) c[k] = hist[(b0 + k < nb ? b0 + k : 0) * 256 + t];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                total += b0 + k < nb ? c[k] : 0u;
                mine += b0 + k < (int)blockIdx.x ? c[k] : 0u;
            }
        }
    } else {
        total = dtot[t];
        mine = pre[(int64_t)t * nb + blockIdx.x];
    }
    uint32_t all;
    const uint32_t below = block_excl_scan(total, lw, &all); // keys of the digits below t
    const uint32_t first = rank_tile<K, WAVES, kItems>(keys, shift, m, wcnt, lw, pos);
    gbase[t] = below + mine - first;
#pragma unroll
    for (int j = 0; j < kItems; ++j)
        if ((w * kItems + j) * kWave + lane < m) {
            sk[pos[j]] = keys[j];
            sv[pos[j]] = vals[j];
        }
    __syncthreads();
    for (int q = t; q < m; q += kBlock) {
        const K key = sk[q];
        const uint32_t at = gbase[(uint32_t)(key >> shift) & 255u] + (uint32_t)q;
        kout[at] = key;
        vout[at] = sv[q];
    }
}

// All passes of up to 1024 ITEMS keys in one workgroup; the keys stay in
// registers and cross over in LDS.
constexpr int kOneWaves = 16;
template <class K, int ITEMS>
__global__ __launch_bounds__(kWave* kOneWaves) void k_radix_one(const K* kin, const uint32_t* vin, K* kout,
                                                               uint32_t* vout, int n, int first, int passes)
{
    __shared__ K sk[kWave * kOneWaves * ITEMS];
    __shared__ uint32_t sv[kWave * kOneWaves * ITEMS];
    __shared__ uint32_t wcnt[kOneWaves][256];
    __shared__ uint32_t lw[kOneWaves];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    K keys[ITEMS];
    uint32_t vals[ITEMS], pos[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int i = (w * ITEMS + j) * kWave + lane;
        keys[j] = i < n ? kin[i] : (K)0;
        vals[j] = i < n ? vin[i] : 0u;
    }
    for (int p = 0; p < passes; ++p) {
        rank_tile<K, kOneWaves, ITEMS>(keys, 8 * (first + p), n, wcnt, lw, pos);
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if ((w * ITEMS + j) * kWave + lane < n) {
                sk[pos[j]] = keys[j];
                sv[pos[j]] = vals[j];
            }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int i = (w * ITEMS + j) * kWave + lane;
            if (i < n) {
                keys[j] = sk[i];
                vals[j] = sv[i];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int i = (w * ITEMS + j) * kWave + lane;
        if (i < n) {
            kout[i] = keys[j];
            vout[i] = vals[j];
        }
    }
}

// Where the lines lie, by the time to order rays (two to four passes and their
// keys): one workgroup 17.8 us against 25.6 at 1000 keys and 21.5 against 27.1 at 4096, but
// 27.7 against 27.9 at 8192 with eight keys per thread; tiles that add up all counts 39.4 us
// against 44.8 at 40,000 keys and 44.6 against 46.4 at 131,072, but 52.1 against 49.9 at 200,000.
constexpr int64_t kOneBlock = 4096;
constexpr int kFewTiles = 64;

template <class K>
int radix_sort_impl(K* k0, uint32_t* v0, K* k1, uint32_t* v1, int64_t n, int first, int passes, uint32_t* hist,
                    hipStream_t s)
{
    if (n <= 1 || passes <= 0) return 0;
    if (n <= kOneBlock) {
        K* ko = (passes & 1) ? k1 : k0; // (all keys are in registers before the first is written)
        uint32_t* vo = (passes & 1) ? v1 : v0;
        const dim3 one(1), thr(kWave * kOneWaves);
        if (n <= 1024) hipLaunchKernelGGL((k_radix_one<K, 1>), one, thr, 0, s, k0, v0, ko, vo, (int)n, first, passes);
        else hipLaunchKernelGGL((k_radix_one<K, 4>), one, thr, 0, s, k0, v0, ko, vo, (int)n, first, passes);
        return (passes & 1) ? 1 : 0;
    }
    const int nb = ceil_div(n, kTile);
    const int64_t hn = (int64_t)256 * nb;
    uint32_t* pre = hist + hn;
    uint32_t* dtot = pre + hn; // 256 digit totals
    K* ki = k0;
    uint32_t* vi = v0;
    K* ko = k1;
    uint32_t* vo = v1;
    for (int p = 0; p < passes; ++p) {
        const int shift = 8 * (first + p);
        if (nb <= kFewTiles) {
            hipLaunchKernelGGL((k_radix_hist<K, true>), dim3(nb), dim3(kBlock), 0, s, ki, n, shift, hist, nb);
            hipLaunchKernelGGL((k_radix_scatter<K, true>), dim3(nb), dim3(kBlock), 0, s, ki, vi, ko, vo, n, shift, hist,
                               pre, dtot, nb);
        } else {
            hipLaunchKernelGGL((k_radix_hist<K, false>), dim3(nb), dim3(kBlock), 0, s, ki, n, shift, hist, nb);
            hipLaunchKernelGGL(k_radix_rowscan, dim3(256), dim3(kBlock), 0, s, hist, nb, pre, dtot);
            hipLaunchKernelGGL((k_radix_scatter<K, false>), dim3(nb), dim3(kBlock), 0, s, ki, vi, ko, vo, n, shift, hist,
                               pre, dtot, nb);
        }
        K* tk = ki; ki = ko; ko = tk;
        uint32_t* tv = vi; vi = vo; vo = tv;
    }
    return (passes & 1) ? 1 : 0;
}

} // namespace

size_t scan_scratch_words(int64_t n) { return (size_t)ceil_div(n > 0 ? n : 1, kScanTile) + 1; }

void exclusive_scan_i32(const int32_t* in, int32_t* out, int64_t n, int32_t* scratch, hipStream_t s)
{
    const int nb = ceil_div(n > 0 ? n : 1, kScanTile);
    uint32_t* part = reinterpret_cast<uint32_t*>(scratch);
    hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kBlock), 0, s, in, n, part);
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, s, part, nb, out, n);
    hipLaunchKernelGGL(k_scan_apply, dim3(nb), dim3(kBlock), 0, s, in, out, n, part);
}

size_t radix_hist_words(int64_t n)
{
    const int64_t hn = (int64_t)256 * ceil_div(n > 0 ? n : 1, kTile);
    return 2 * (size_t)hn + 256; // counts, their per-digit prefixes, digit totals
}

int radix_sort_u64(uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1, int64_t n, int passes,
                   uint32_t* hist, hipStream_t s)
{
    return radix_sort_impl<uint64_t>(k0, v0, k1, v1, n, 0, passes, hist, s);
}

int radix_sort_u64_digits(uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1, int64_t n, int first, int passes,
                          uint32_t* hist, hipStream_t s)
{
    return radix_sort_impl<uint64_t>(k0, v0, k1, v1, n, first, passes, hist, s);
}

int radix_sort_u32(uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, int64_t n, int passes,
                   uint32_t* hist, hipStream_t s)
{
    return radix_sort_impl<uint32_t>(k0, v0, k1, v1, n, 0, passes, hist, s);
}

} // namespace glm
