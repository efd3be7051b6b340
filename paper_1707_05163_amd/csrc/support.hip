// support.hip -- particle bookkeeping and snapshot conversion kernels:
//   * wavefront compaction of the active-particle list (ballot + mbcnt prefix,
//     one atomic per wave);
//   * counting sorts of the active particles by grid tile (and level in 3D), in LDS
//     where the bins fit, which also drop particles that are no longer active;
//   * conversion of float32 / float64 snapshots into the interleaved node layout
//     of a device slot, including bfloat16 (round to nearest even) and float16
//     with a power-of-two scale per (level, variable).
#include "lp_internal.h"

namespace lp {

namespace {

__global__ void k_fill_u32(uint32_t *p, uint32_t v, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_iota(uint32_t *p, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = (uint32_t)i;
}

uint32_t grid_blocks(size_t n, uint32_t threads, uint32_t cap = 1u << 16)
{
    size_t b = (n + threads - 1) / threads;
    if (b == 0)
        b = 1;
    return (uint32_t)(b > cap ? cap : b);
}

// Keep the ids whose status is still 0.  Each wave finds its survivors with a
// ballot and ranks them with mbcnt; the waves of a block add up their counts in LDS
// and the block reserves room in the output with a single atomic.  A thread takes
// kCompactItems entries, kCompactThreads apart, so that a block covers 4096 entries
// per atomic: atomics on the one counter serialise (about 12 ns each here), and with
// one per 1024 entries they were most of the kernel's time.  Survivors keep their
// order within a block (entry, then wave, then lane).
constexpr int kCompactThreads = 1024, kCompactItems = 4;

__global__ __launch_bounds__(kCompactThreads) void k_compact(const uint32_t *order_in,
                                                             const uint32_t *n_in,
                                                             const uint8_t *status,
                                                             uint32_t *order_out,
                                                             uint32_t *n_out)
{
    constexpr int W = kCompactThreads / 64;
    __shared__ uint32_t wcount[kCompactItems * W];
    __shared__ uint32_t block_base;
    const uint32_t n = *n_in;
    const size_t base = (size_t)blockIdx.x * kCompactThreads * kCompactItems;
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t id[kCompactItems], rank[kCompactItems];
    bool keep[kCompactItems];
#pragma unroll
    for (int j = 0; j < kCompactItems; ++j) {
        const size_t k = base + (size_t)j * kCompactThreads + threadIdx.x;
        id[j] = 0;
        keep[j] = false;
        if (k < n) {
            id[j] = order_in[k];
            keep[j] = status[id[j]] == 0;
        }
        const uint64_t mask = __ballot(keep[j]);
        rank[j] = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        if (lane == 0)
            wcount[j * W + wid] = (uint32_t)__popcll(mask);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tot = 0;
        for (int w = 0; w < kCompactItems * W; ++w) {
            const uint32_t c = wcount[w];
            wcount[w] = tot;
            tot += c;
        }
        block_base = tot ? atomicAdd(n_out, tot) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kCompactItems; ++j)
        if (keep[j])
            order_out[block_base + wcount[j * W + wid] + rank[j]] = id[j];
}

// Runs of equal keys inside a wave (the order is nearly sorted already): each lane
// learns the lane that starts its run and the run length, so one lane per run can
// do the atomic for the whole run.
__device__ inline void wave_runs(uint32_t key, bool valid, int &start, uint32_t &len)
{
    const int lane = threadIdx.x & 63;
    const uint32_t prev = __shfl_up(key, 1, 64);
    const bool prev_valid = __shfl_up(valid ? 1 : 0, 1, 64) != 0;
    const bool is_start = valid && (lane == 0 || !prev_valid || prev != key);
    // lanes that are not valid also end runs
    const uint64_t starts = __ballot(is_start) | __ballot(!valid);
    const uint64_t below = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
    const uint64_t at_or_below = starts & below;
    start = at_or_below ? 63 - __clzll((long long)at_or_below) : lane;
    const uint64_t above = starts & ~below;
    const int next = above ? __ffsll((unsigned long long)above) - 1 : 64;
    len = (uint32_t)(next - lane);  // meaningful on the start lane
}

// the cell to look at first for coordinate x
__device__ inline int cell_guess(const AxisDev &a, double x)
{
    int g = (int)((x - a.lo) * a.ginv);
    if (!a.uniform) {
        g = g < kGuessBins - 1 ? g : kGuessBins - 1;
        g = a.guess[g < 0 ? 0 : g];
    }
    return g < 0 ? 0 : (g > a.n - 2 ? a.n - 2 : g);
}

// the cell of x from a guess g and its two faces
__device__ inline int cell_settle(const AxisDev &a, double x, int g, double lo, double hi)
{
    while (g > 0 && lo > x) {
        --g;
        hi = lo;
        lo = a.c[g];
    }
    while (g < a.n - 2 && hi <= x) {
        ++g;
        hi = a.c[g + 1];
    }
    return g;
}

__device__ inline int cell_of(const AxisDev &a, double x)
{
    const int g = cell_guess(a, x);
    return cell_settle(a, x, g, a.c[g], a.c[g + 1]);
}

// Sort key: tile index (16 x 16 cells, row-major over tiles), times the level in
// 3D; with `cells` (2D) the tile index times 256 plus the cell's row-major index in its
// tile, so that a wave's particles share cells, not only a tile.  Inactive particles get
// no key and are dropped by the sort.
__device__ inline uint32_t sort_key(const GridDev &g, int i, int j, int kk, bool cells)
{
    const uint32_t ntx = (uint32_t)(g.ax.n - 2) / kTile + 1;
    uint32_t key = (uint32_t)(j / kTile) * ntx + (uint32_t)(i / kTile);
    if (cells)
        key = key * (uint32_t)(kTile * kTile) + (uint32_t)((j % kTile) * kTile + i % kTile);
    return g.az.n ? key * (uint32_t)(g.az.n - 1) + (uint32_t)kk : key;
}

__global__ __launch_bounds__(256) void k_sort_keys(GridDev g, const double *x, const double *y,
                                                   const double *z, const uint8_t *status,
                                                   const uint32_t *order, const uint32_t *n_in,
                                                   uint32_t *keys, uint32_t *hist, bool cells)
{
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t n = *n_in;
    uint32_t key = 0xFFFFFFFFu;
    if (k < n) {
        const uint32_t id = order[k];
        if (status[id] == 0)
            key = sort_key(g, cell_of(g.ax, x[id]), cell_of(g.ay, y[id]),
                           g.az.n ? cell_of(g.az, z[id]) : 0, cells);
        keys[k] = key;
    }
    const bool valid = key != 0xFFFFFFFFu;
    int start;
    uint32_t len;
    wave_runs(key, valid, start, len);
    if (valid && start == (int)(threadIdx.x & 63))
        atomicAdd(&hist[key], len);
}

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanChunk = kScanThreads * kScanItems;

// block-wide exclusive scan of one value per thread; returns the block total
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t &excl)
{
    __shared__ uint32_t wsum[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t incl = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, 64);
        if (lane >= off)
            incl += t;
    }
    if (lane == 63)
        wsum[wid] = incl;
    __syncthreads();
    uint32_t wbase = 0, total = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) {
        if (w < wid)
            wbase += wsum[w];
        total += wsum[w];
    }
    __syncthreads();
    excl = wbase + incl - v;
    return total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_partial(const uint32_t *hist,
                                                               uint32_t nbins,
                                                               uint32_t *blocksums)
{
    const size_t base = (size_t)blockIdx.x * kScanChunk + (size_t)threadIdx.x * kScanItems;
    uint32_t s = 0;
    for (int q = 0; q < kScanItems; ++q)
        if (base + q < nbins)
            s += hist[base + q];
    uint32_t excl;
    const uint32_t tot = block_exclusive_scan(s, excl);
    if (threadIdx.x == 0)
        blocksums[blockIdx.x] = tot;
}

// single block: exclusive scan of the block sums in place; total -> *n_out
__global__ __launch_bounds__(kScanThreads) void k_scan_top(uint32_t *blocksums, uint32_t nblk,
                                                           uint32_t *n_out)
{
    uint32_t carry = 0;
    for (uint32_t base = 0; base < nblk; base += kScanThreads) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t v = i < nblk ? blocksums[i] : 0u;
        uint32_t excl;
        const uint32_t tot = block_exclusive_scan(v, excl);
        if (i < nblk)
            blocksums[i] = carry + excl;
        carry += tot;
    }
    if (threadIdx.x == 0)
        *n_out = carry;
}

// hist -> exclusive offsets (in place)
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(uint32_t *hist, uint32_t nbins,
                                                             const uint32_t *blocksums)
{
    const size_t base = (size_t)blockIdx.x * kScanChunk + (size_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
    for (int q = 0; q < kScanItems; ++q) {
        v[q] = base + q < nbins ? hist[base + q] : 0u;
        s += v[q];
    }
    uint32_t excl;
    block_exclusive_scan(s, excl);
    uint32_t run = blocksums[blockIdx.x] + excl;
    for (int q = 0; q < kScanItems; ++q) {
        if (base + q < nbins)
            hist[base + q] = run;
        run += v[q];
    }
}

__global__ __launch_bounds__(256) void k_sort_scatter(const uint32_t *order_in,
                                                      const uint32_t *n_in, const uint32_t *keys,
                                                      uint32_t *offsets, uint32_t *order_out)
{
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t n = *n_in;
    const uint32_t key = k < n ? keys[k] : 0xFFFFFFFFu;
    const bool valid = key != 0xFFFFFFFFu;
    int start;
    uint32_t len;
    wave_runs(key, valid, start, len);
    const int lane = threadIdx.x & 63;
    uint32_t base = 0;
    if (valid && start == lane)
        base = atomicAdd(&offsets[key], len);
    base = __shfl(base, start, 64);
    if (valid)
        order_out[base + (uint32_t)(lane - start)] = order_in[k];
}

// ---------------------------------------------------------------- sorts in LDS
// With up to kSortBins bins (2D grids up to about 1250 x 1250 nodes) a block counts its
// part of the list in LDS and no global atomic is taken: k_sort_hist writes one row of
// counts per block, k_sort_columns turns each bin's column into offsets, and k_sort_apply
// scans the totals, each block for itself, and hands out places from LDS counters.  Bound
// by the chain of reads order -> position -> cell faces, once per thread until there are
// 256 blocks (with two particles a thread k_sort_hist took 10.9 us for 20k particles, not
// 6.6: half the blocks, and twice the code for each to fetch).  7 + 3 + 5 us for 20k
// particles in 4050 bins, 13 + 5 + 8 for 500k.
// The six launches above take one global atomic per particle, which on lists with many
// particles a bin, or all in one, cost up to 1.4 ms; but they do not read and write a row
// of bins per block.  The line is where evenly spread lists take as long either way (16
// steps with a sort before each, LDS against atomics): 0.61 and 0.63 ms for 20k particles in
// 4050 bins, 0.61 and 0.64 in 6072, 0.65 and 0.65 in 7497, 0.67 and 0.65 in 14875; 1.22 and
// 1.24 for 400k in 6072, 1.28 and 1.22 in 7497.
constexpr uint32_t kSortBins = 6144, kSortThreads = 1024;
constexpr uint32_t kSortGroups = 16;  // row groups of k_sort_columns

__host__ __device__ inline uint32_t sort_parts(uint32_t n)
{
    const uint32_t parts = (n + kSortThreads - 1) / kSortThreads;  // at most 256 blocks
    return parts < 256 ? (parts ? parts : 1) : 256;
}

__host__ __device__ inline uint32_t sort_chunk(uint32_t n)
{
    const uint32_t parts = sort_parts(n);
    return ((n + parts - 1) / parts + kSortThreads - 1) / kSortThreads * kSortThreads;
}

// The key of list entry `id`, with its reads overlapped (0xFFFFFFFF: not active).
__device__ inline uint32_t sort_load(const GridDev &g, const double *x, const double *y,
                                     const double *z, const uint8_t *status, uint32_t id,
                                     bool cells)
{
    const AxisDev *ax[3] = {&g.ax, &g.ay, &g.az};
    const uint8_t st = status[id];
    const double p[3] = {x[id], y[id], g.az.n ? z[id] : 0.0};
    double lo[3], up[3];
    int c[3] = {0, 0, 0};
#pragma unroll
    for (int v = 0; v < 3; ++v)
        if (v < 2 || g.az.n)
            c[v] = cell_guess(*ax[v], p[v]);
#pragma unroll
    for (int v = 0; v < 3; ++v)
        if (v < 2 || g.az.n) {
            lo[v] = ax[v]->c[c[v]];
            up[v] = ax[v]->c[c[v] + 1];
        }
#pragma unroll
    for (int v = 0; v < 3; ++v)
        if (v < 2 || g.az.n)
            c[v] = cell_settle(*ax[v], p[v], c[v], lo[v], up[v]);
    return st == 0 ? sort_key(g, c[0], c[1], c[2], cells) : 0xFFFFFFFFu;
}

__global__ __launch_bounds__(kSortThreads) void k_sort_hist(
    GridDev g, const double *x, const double *y, const double *z, const uint8_t *status,
    const uint32_t *order, const uint32_t *n_in, uint32_t chunk, uint32_t nbins, uint32_t *keys,
    uint32_t *rows, bool cells)
{
    extern __shared__ uint32_t bins[];
    for (uint32_t b = threadIdx.x; b < nbins; b += kSortThreads)
        bins[b] = 0u;
    __syncthreads();
    const uint32_t n = *n_in, lo = blockIdx.x * chunk;
    const uint32_t hi = lo + chunk < n ? lo + chunk : n;
    for (uint32_t k = lo + threadIdx.x; k < hi; k += kSortThreads) {
        const uint32_t key = sort_load(g, x, y, z, status, order[k], cells);
        if (key != 0xFFFFFFFFu)
            atomicAdd(&bins[key], 1u);
        keys[k] = key;
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < nbins; b += kSortThreads)
        rows[(size_t)blockIdx.x * nbins + b] = bins[b];
}

// each bin's counts over the blocks -> offsets within the bin; its total to totals
// (64 bins x kSortGroups groups of rows a block, at most 16 rows a thread)
__global__ __launch_bounds__(64 * kSortGroups) void k_sort_columns(uint32_t *rows, uint32_t nbins,
                                                                   uint32_t parts,
                                                                   uint32_t *totals)
{
    __shared__ uint32_t sum[kSortGroups][64];
    const uint32_t lane = threadIdx.x & 63u, grp = threadIdx.x >> 6;
    const uint32_t b = blockIdx.x * 64u + lane;
    const uint32_t per = (parts + kSortGroups - 1) / kSortGroups, p0 = grp * per;
    constexpr int kRows = 256 / kSortGroups;
    uint32_t v[kRows], mine = 0;
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
        const bool in = (uint32_t)q < per && p0 + q < parts && b < nbins;
        v[q] = in ? rows[(size_t)(p0 + q) * nbins + b] : 0u;
    }
#pragma unroll
    for (int q = 0; q < kRows; ++q)
        mine += v[q];
    sum[grp][lane] = mine;
    __syncthreads();
    uint32_t run = 0, total = 0;
#pragma unroll
    for (uint32_t w = 0; w < kSortGroups; ++w) {
        run += w < grp ? sum[w][lane] : 0u;
        total += sum[w][lane];
    }
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
        if ((uint32_t)q < per && p0 + q < parts && b < nbins)
            rows[(size_t)(p0 + q) * nbins + b] = run;
        run += v[q];
    }
    if (grp == 0 && b < nbins)
        totals[b] = total;
}

// exclusive scan of the nbins values at v (LDS) by one block; returns their sum
__device__ inline uint32_t scan_bins(uint32_t *v, uint32_t nbins)
{
    __shared__ uint32_t wsum[kSortThreads / 64];
    const uint32_t per = (nbins + kSortThreads - 1) / kSortThreads, lo = threadIdx.x * per;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t s = 0;
    for (uint32_t b = lo; b < lo + per && b < nbins; ++b)
        s += v[b];
    uint32_t incl = s;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, 64);
        if (lane >= off)
            incl += t;
    }
    if (lane == 63)
        wsum[wid] = incl;
    __syncthreads();
    uint32_t run = incl - s, total = 0;
    for (int w = 0; w < (int)(kSortThreads / 64); ++w) {
        run += w < wid ? wsum[w] : 0u;
        total += wsum[w];
    }
    for (uint32_t b = lo; b < lo + per && b < nbins; ++b) {
        const uint32_t c = v[b];
        v[b] = run;
        run += c;
    }
    return total;
}

__global__ __launch_bounds__(kSortThreads) void k_sort_apply(const uint32_t *order_in,
                                                             const uint32_t *n_in, uint32_t chunk,
                                                             uint32_t nbins, const uint32_t *keys,
                                                             const uint32_t *rows,
                                                             const uint32_t *totals,
                                                             uint32_t *order_out, uint32_t *n_out)
{
    extern __shared__ uint32_t bins[];
    // (every read of the totals and of the block's row goes out before any is used: in a
    // loop over the bins each waited for the one before, 12.9 us in place of 7.2 for 14875)
    constexpr int kPer = kSortBins / kSortThreads;
    uint32_t tot[kPer], row[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const uint32_t b = threadIdx.x + (uint32_t)q * kSortThreads;
        if ((uint32_t)q * kSortThreads < nbins) {
            tot[q] = b < nbins ? totals[b] : 0u;
            row[q] = b < nbins ? rows[(size_t)blockIdx.x * nbins + b] : 0u;
        }
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const uint32_t b = threadIdx.x + (uint32_t)q * kSortThreads;
        if (b < nbins)
            bins[b] = tot[q];
    }
    __syncthreads();
    const uint32_t total = scan_bins(bins, nbins);
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *n_out = total;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const uint32_t b = threadIdx.x + (uint32_t)q * kSortThreads;
        if (b < nbins)
            bins[b] += row[q];
    }
    __syncthreads();
    const uint32_t n = *n_in, lo = blockIdx.x * chunk;
    const uint32_t hi = lo + chunk < n ? lo + chunk : n;
    for (uint32_t k = lo + threadIdx.x; k < hi; k += kSortThreads) {
        const uint32_t key = keys[k], id = order_in[k];
        if (key != 0xFFFFFFFFu)
            order_out[atomicAdd(&bins[key], 1u)] = id;
    }
}

// ---------------------------------------------------------------- snapshot conversion
__device__ inline uint32_t bf16_rne(float f)
{
    uint32_t b = __float_as_uint(f);
    if ((b & 0x7F800000u) == 0x7F800000u && (b & 0x007FFFFFu))
        return (b >> 16) | 0x40u;  // quiet NaN
    b += 0x7FFFu + ((b >> 16) & 1u);
    return b >> 16;
}

__device__ inline uint32_t f16_bits(float f)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)f);
}

// Power-of-two scale s = 2^(ceil(log2 m) - 14) for a level whose largest
// magnitude is m (so |F / s| <= 2^14), or 1 when the level is all zeros.
__device__ inline float f16_scale(float m)
{
    if (!(m > 0.f))
        return 1.f;
    int e;
    const float fr = frexpf(m, &e);  // m = fr * 2^e, fr in [0.5, 1)
    const int c = (fr == 0.5f) ? e - 1 : e;
    return ldexpf(1.f, c - 14);
}

// max |F| of every level of two or three variables, out[variable * nzl + level] (cleared
// before).  Bound by the read of the planes, so each level is split over `parts` blocks,
// enough to fill the chip; non-negative floats order as their bits do, so the blocks'
// maxima meet in an integer atomic.  Three variables of 50 levels of 3600 x 1800 values:
// 0.81 ms a snapshot, 4.8 TB/s (with one block a level the pushes held the benchmark's 3D
// run with this storage up: 196 ms then, 177 now).
struct LevelPlanes {
    const float *f[3];
};

__global__ __launch_bounds__(256) void k_level_absmax(LevelPlanes F, size_t plane, uint32_t nzl,
                                                      uint32_t parts, uint32_t *out)
{
    const uint32_t part = blockIdx.x % parts, k = blockIdx.x / parts;
    const float *p = F.f[k / nzl] + (size_t)(k % nzl) * plane;
    const size_t step = (size_t)parts * 256;
    float m = 0.f;
    size_t i = (size_t)part * 256 + threadIdx.x;
    for (; i + 3 * step < plane; i += 4 * step)
        m = fmaxf(fmaxf(fmaxf(m, fabsf(p[i])), fmaxf(fabsf(p[i + step]), fabsf(p[i + 2 * step]))),
                  fabsf(p[i + 3 * step]));
    for (; i < plane; i += step)
        m = fmaxf(m, fabsf(p[i]));
    for (int off = 32; off > 0; off >>= 1)
        m = fmaxf(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0 && m > 0.f)
        atomicMax(out + k, __float_as_uint(m));
}

template <int ST, bool IS3D>
__global__ void k_convert(const float *U, const float *V, const float *W, const double *U64,
                          const double *V64, const double *W64, size_t plane, int nzl,
                          void *slot, const float *scales)
{
    const size_t total = plane * (size_t)nzl;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        if constexpr (ST == kF64) {
            const double u = U64 ? U64[i] : (double)U[i];
            const double v = V64 ? V64[i] : (double)V[i];
            if constexpr (IS3D) {
                const double w = W64 ? W64[i] : (double)W[i];
                static_cast<double4 *>(slot)[i] = make_double4(u, v, w, 0.0);
            } else {
                static_cast<double2 *>(slot)[i] = make_double2(u, v);
            }
        } else if constexpr (ST == kF32) {
            if constexpr (IS3D)
                static_cast<float4 *>(slot)[i] = make_float4(U[i], V[i], W[i], 0.f);
            else
                static_cast<float2 *>(slot)[i] = make_float2(U[i], V[i]);
        } else if constexpr (ST == kBF16) {
            const uint32_t a = bf16_rne(U[i]) | (bf16_rne(V[i]) << 16);
            if constexpr (IS3D)
                static_cast<uint2 *>(slot)[i] = make_uint2(a, bf16_rne(W[i]));
            else
                static_cast<uint32_t *>(slot)[i] = a;
        } else {
            const size_t k = i / plane;
            const float *sc = scales + k * 3;
            const uint32_t a = f16_bits(U[i] / sc[0]) | (f16_bits(V[i] / sc[1]) << 16);
            if constexpr (IS3D)
                static_cast<uint2 *>(slot)[i] = make_uint2(a, f16_bits(W[i] / sc[2]));
            else
                static_cast<uint32_t *>(slot)[i] = a;
        }
    }
}

// turn the per-(level, variable) maxima into scales, in place
__global__ void k_scales_from_max(float *s, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        s[i] = f16_scale(s[i]);
}

// gather per-level maxima [var][level] into [level][var]
__global__ void k_interleave_max(const float *m, int nzl, int nvar, float *s)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nzl * 3) {
        const int k = i / 3, v = i % 3;
        s[i] = v < nvar ? m[v * nzl + k] : 0.f;
    }
}

}  // namespace

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_blocks(n, 256, 4096)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_iota(uint32_t *p, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_iota, dim3(grid_blocks(n, 256, 4096)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_compact(const uint32_t *order_in, const uint32_t *n_in, const uint8_t *status,
                          uint32_t *order_out, uint32_t *n_out, uint32_t n_launch,
                          hipStream_t s)
{
    hipError_t e = launch_fill_u32(n_out, 0u, 1, s);
    if (e != hipSuccess || n_launch == 0)
        return e;
    constexpr uint32_t kPerBlock = kCompactThreads * kCompactItems;
    hipLaunchKernelGGL(k_compact, dim3((n_launch + kPerBlock - 1) / kPerBlock),
                       dim3(kCompactThreads), 0, s, order_in, n_in, status, order_out, n_out);
    return hipGetLastError();
}

uint32_t sort_bins(const GridDev &g, bool cells)
{
    const uint32_t ntx = (uint32_t)(g.ax.n - 2) / kTile + 1;
    const uint32_t nty = (uint32_t)(g.ay.n - 2) / kTile + 1;
    uint32_t nb = ntx * nty;
    if (g.az.n)
        nb *= (uint32_t)(g.az.n - 1);
    else if (cells)
        nb *= (uint32_t)(kTile * kTile);
    return nb;
}

size_t sort_blocksums(uint32_t nbins)
{
    return nbins <= kSortBins ? nbins : (nbins + kScanChunk - 1) / kScanChunk;
}

size_t sort_hist(uint32_t nbins, size_t n)
{
    return nbins <= kSortBins ? (size_t)nbins * sort_parts((uint32_t)n) : nbins;
}

hipError_t launch_sort(const GridDev &g, const double *x, const double *y, const double *z,
                       const uint8_t *status, const uint32_t *order_in, const uint32_t *n_in,
                       uint32_t n_launch, uint32_t *keys, uint32_t *hist, uint32_t nbins,
                       uint32_t *blocksums, uint32_t *order_out, uint32_t *n_out,
                       hipStream_t s, bool cells)
{
    cells = cells && !g.az.n;
    if (nbins <= kSortBins) {
        const size_t lds = (size_t)nbins * sizeof(uint32_t);
        const dim3 blk(kSortThreads);
        const uint32_t parts = sort_parts(n_launch), chunk = sort_chunk(n_launch);
        hipLaunchKernelGGL(k_sort_hist, dim3(parts), blk, lds, s, g, x, y, z, status, order_in,
                           n_in, chunk, nbins, keys, hist, cells);
        hipLaunchKernelGGL(k_sort_columns, dim3((nbins + 63) / 64), dim3(64 * kSortGroups), 0, s,
                           hist, nbins, parts, blocksums);
        hipLaunchKernelGGL(k_sort_apply, dim3(parts), blk, lds, s, order_in, n_in, chunk, nbins,
                           keys, hist, blocksums, order_out, n_out);
        return hipGetLastError();
    }
    hipError_t e = launch_fill_u32(hist, 0u, nbins, s);
    if (e != hipSuccess)
        return e;
    const uint32_t nb = (n_launch + 255) / 256;
    if (nb)
        hipLaunchKernelGGL(k_sort_keys, dim3(nb), dim3(256), 0, s, g, x, y, z, status, order_in,
                           n_in, keys, hist, cells);
    const uint32_t nblk = (uint32_t)sort_blocksums(nbins);
    hipLaunchKernelGGL(k_scan_partial, dim3(nblk), dim3(kScanThreads), 0, s, hist, nbins,
                       blocksums);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kScanThreads), 0, s, blocksums, nblk, n_out);
    hipLaunchKernelGGL(k_scan_apply, dim3(nblk), dim3(kScanThreads), 0, s, hist, nbins,
                       blocksums);
    if (nb)
        hipLaunchKernelGGL(k_sort_scatter, dim3(nb), dim3(256), 0, s, order_in, n_in, keys, hist,
                           order_out);
    return hipGetLastError();
}

static hipError_t launch_level_absmax(const float *U, const float *V, const float *W, int nvar,
                                      size_t plane, int nzl, float *out, hipStream_t s)
{
    uint32_t *bits = reinterpret_cast<uint32_t *>(out);
    const hipError_t e = launch_fill_u32(bits, 0u, (size_t)nzl * nvar, s);
    if (e != hipSuccess)
        return e;
    // at least 8192 values a block, at most 4096 blocks unless there are more levels
    const size_t levels = (size_t)nzl * nvar;
    const size_t fill = levels < 4096 ? 4096 / levels : 1, most = (plane + 8191) / 8192;
    const uint32_t parts = (uint32_t)(fill < most ? fill : most);
    hipLaunchKernelGGL(k_level_absmax, dim3((uint32_t)(levels * parts)), dim3(256), 0, s,
                       LevelPlanes{{U, V, W}}, plane, (uint32_t)nzl, parts, bits);
    return hipGetLastError();
}

hipError_t launch_convert_snapshot(int store, bool is3d, const float *U, const float *V,
                                   const float *W, const double *U64, const double *V64,
                                   const double *W64, size_t plane, int nzl, void *slot,
                                   float *scales, float *tmp, hipStream_t s)
{
    const size_t total = plane * (size_t)nzl;
    const dim3 grid(grid_blocks(total, 256, 1u << 15)), blk(256);
    if (store == kF16S) {
        // scales[level*3 + var] from the per-level maxima of each variable (tmp: 3*nzl)
        float *m = scales;
        const hipError_t e = launch_level_absmax(U, V, W, is3d ? 3 : 2, plane, nzl, tmp, s);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(k_interleave_max, dim3((nzl * 3 + 255) / 256), dim3(256), 0, s, tmp,
                           nzl, is3d ? 3 : 2, m);
        hipLaunchKernelGGL(k_scales_from_max, dim3((nzl * 3 + 255) / 256), dim3(256), 0, s, m,
                           nzl * 3);
    }
#define LP_CONV(ST, D3)                                                                       \
    hipLaunchKernelGGL((k_convert<ST, D3>), grid, blk, 0, s, U, V, W, U64, V64, W64, plane,   \
                       nzl, slot, scales)
    switch (store) {
    case kF64: if (is3d) LP_CONV(kF64, true); else LP_CONV(kF64, false); break;
    case kF32: if (is3d) LP_CONV(kF32, true); else LP_CONV(kF32, false); break;
    case kBF16: if (is3d) LP_CONV(kBF16, true); else LP_CONV(kBF16, false); break;
    case kF16S: if (is3d) LP_CONV(kF16S, true); else LP_CONV(kF16S, false); break;
    default: return hipErrorInvalidValue;
    }
#undef LP_CONV
    return hipGetLastError();
}

}  // namespace lp
