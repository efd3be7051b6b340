// results.hip -- how results come back to host arrays, and the blocks of device and
// pinned memory that particle sets hand on to the next ones.
//
// Results go through pinned staging: a kernel writes each piece of the arrays into a
// pinned chunk over PCIe, and host threads copy the chunks into the caller's (pageable)
// arrays while the next pieces arrive.  A plain copy to pageable memory runs at 18 GB/s
// here, a copy to pinned memory at 57.
#include <algorithm>
#include <atomic>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>
#include <unordered_map>
#include <vector>

#include "lp_internal.h"
#include "lp_objects.h"

namespace {

// ---------------------------------------------------------------- blocks kept for reuse
// Programs make and destroy particle sets of the same size over and over (a release a day,
// the runs of an ensemble), and a hipMalloc and hipFree pair costs 13 us at 8 MB and 320 us
// at 80 MB.  Freed blocks stay in lists by device and kind, at most kKeepDevice and
// kKeepHost bytes of them, while any field set lives; they are given back when the last one
// is destroyed, and when any allocation of the library fails (lp_malloc).  A block is freed
// only when no work on it is pending, so the next owner may use it on any stream.  One lock
// guards it all.
constexpr size_t kKeepDevice = (size_t)1 << 30, kKeepHost = (size_t)64 << 20;

struct Pool {
    struct Block {
        int dev;  // device, or -1: pinned host memory
        size_t bytes;
    };
    std::mutex mu;
    std::unordered_map<void *, Block> live;
    std::map<int, std::multimap<size_t, void *>> kept;
    size_t kept_bytes[2] = {0, 0};  // device, host
    int users = 0;
};

Pool &pool()
{
    static Pool *p = new Pool();  // never destroyed: the runtime may be gone by then
    return *p;
}

void release(int dev, void *p)
{
    if (dev < 0)
        (void)hipHostFree(p);
    else
        (void)hipFree(p);
}

void purge_locked(Pool &P)
{
    for (auto &l : P.kept)
        for (auto &b : l.second)
            release(l.first, b.second);
    P.kept.clear();
    P.kept_bytes[0] = P.kept_bytes[1] = 0;
}

// Chunks of pinned memory for results: a set of 16 MB at most (2 MB for small results), so
// kKeepHost keeps up to four of them.
constexpr size_t kChunk = (size_t)1 << 20;
constexpr int kThreads = 8;  // host threads, two chunks each

}  // namespace

void *lp_pool_alloc(size_t bytes, bool host, hipError_t *err)
{
    *err = hipSuccess;
    bytes = (bytes + 255) & ~(size_t)255;
    int dev = -1;
    if (!host && (*err = hipGetDevice(&dev)) != hipSuccess)
        return nullptr;
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    try {
        auto &list = P.kept[dev];
        auto it = list.lower_bound(bytes);  // the smallest that fits, not much too large
        if (it != list.end() && it->first <= bytes + bytes / 4) {
            void *p = it->second;
            const size_t n = it->first;
            P.live[p] = {dev, n};
            list.erase(it);
            P.kept_bytes[host] -= n;
            return p;
        }
        void *p = nullptr;
        for (int k = 0; k < 2; ++k) {
            *err = host ? hipHostMalloc(&p, bytes, hipHostMallocDefault) : hipMalloc(&p, bytes);
            if (*err == hipSuccess) {
                P.live[p] = {dev, bytes};
                return p;
            }
            (void)hipGetLastError();
            if (P.kept_bytes[0] + P.kept_bytes[1] == 0)
                break;
            purge_locked(P);
        }
    } catch (const std::exception &) {
        *err = hipErrorOutOfMemory;
    }
    return nullptr;
}

void lp_pool_free(void *p)
{
    if (!p)
        return;
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    auto it = P.live.find(p);
    if (it == P.live.end())
        return;
    const Pool::Block b = it->second;
    P.live.erase(it);
    const int host = b.dev < 0;
    if (P.users > 0 && P.kept_bytes[host] + b.bytes <= (host ? kKeepHost : kKeepDevice)) {
        try {
            P.kept[b.dev].emplace(b.bytes, p);
            P.kept_bytes[host] += b.bytes;
            return;
        } catch (const std::exception &) {
        }
    }
    release(b.dev, p);
}

void lp_pool_purge(void)
{
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    purge_locked(P);
}

hipError_t lp_malloc(void **p, size_t bytes, bool host)
{
    hipError_t e = hipSuccess;
    for (int k = 0; k < 2; ++k) {
        *p = nullptr;
        e = host ? hipHostMalloc(p, bytes, hipHostMallocDefault) : hipMalloc(p, bytes);
        if (e == hipSuccess)
            return e;
        (void)hipGetLastError();
        if (k == 0)
            lp_pool_purge();
    }
    *p = nullptr;
    return e;
}

void lp_pool_user(int change)
{
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    P.users += change;
    if (P.users <= 0)
        purge_locked(P);
}

namespace {

// ---------------------------------------------------------------- arrays to the host
// Segments of device arrays into a pinned chunk, in 16-byte words (segments start at
// 16-byte boundaries on both sides; the last bytes of one go singly).
constexpr int kMaxSegs = 10;
struct ToHost {
    const char *src[kMaxSegs];
    uint32_t off[kMaxSegs], bytes[kMaxSegs];
    int32_t n;
    char *dst;
};

__global__ __launch_bounds__(256) void k_to_host(ToHost a)
{
    const uint32_t t = blockIdx.x * 256u + threadIdx.x, step = gridDim.x * 256u;
    for (int s = 0; s < a.n; ++s) {
        const uint32_t w = a.bytes[s] / 16;
        const uint4 *src = reinterpret_cast<const uint4 *>(a.src[s]);
        uint4 *dst = reinterpret_cast<uint4 *>(a.dst + a.off[s]);
        for (uint32_t i = t; i < w; i += step)
            dst[i] = src[i];
        for (uint32_t i = 16 * w + t; i < a.bytes[s]; i += step)
            a.dst[a.off[s] + i] = a.src[s][i];
    }
}

// What one launch brings: a chunk's worth of segments and where they go.
struct Piece {
    ToHost k{};
    char *to[kMaxSegs];
    uint32_t used = 0;
};

}  // namespace

static hipError_t copy_plain(hipStream_t stream, const lp_readback *segs, int nsegs)
{
    hipError_t e = hipStreamSynchronize(stream);
    for (int s = 0; s < nsegs && e == hipSuccess; ++s)
        if (segs[s].bytes)
            e = hipMemcpy(segs[s].dst, segs[s].src, segs[s].bytes, hipMemcpyDeviceToHost);
    return e;
}

hipError_t lp_read_back(int dev, hipStream_t stream, const lp_readback *segs, int nsegs)
{
    hipError_t err = hipSuccess;
    char *stage = nullptr;
    std::vector<std::thread> th;
    try {
        std::vector<Piece> pieces;
        size_t total = 0;
        for (int s = 0; s < nsegs; ++s) {
            total += segs[s].bytes;
            for (size_t at = 0; at < segs[s].bytes;) {
                if (pieces.empty() || pieces.back().used >= kChunk ||
                    pieces.back().k.n == kMaxSegs)
                    pieces.emplace_back();
                Piece &p = pieces.back();
                const size_t n = std::min(segs[s].bytes - at, kChunk - p.used);
                const int q = p.k.n++;
                p.k.src[q] = (const char *)segs[s].src + at;
                p.k.off[q] = p.used;
                p.k.bytes[q] = (uint32_t)n;
                p.to[q] = (char *)segs[s].dst + at;
                p.used = (uint32_t)((p.used + n + 15) & ~(size_t)15);
                at += n;
            }
        }
        if (pieces.empty())
            return hipSuccess;
        // a thread for every 4 MB: below that starting one costs more than it copies
        const int T = (int)std::min<size_t>(kThreads, std::max<size_t>(1, total >> 22));
        const size_t chunks = std::min<size_t>(2 * T, pieces.size());
        stage = (char *)lp_pool_alloc(chunks <= 2 ? 2 * kChunk : 2 * kThreads * kChunk, true, &err);
        if (!stage)  // no pinned memory left: plain copies
            return copy_plain(stream, segs, nsegs);
        // thread t takes pieces t, t + T, ...: its next piece arrives in one of its chunks
        // while it copies the other one out
        std::atomic<int> bad{hipSuccess};
        auto work = [&](int t) {
            int old = dev;
            hipError_t e = hipGetDevice(&old);
            if (e == hipSuccess && old != dev)
                e = hipSetDevice(dev);
            hipEvent_t ev[2] = {nullptr, nullptr};
            for (auto &x : ev)
                if (e == hipSuccess)
                    e = hipEventCreateWithFlags(&x, hipEventDisableTiming);
            auto start = [&](size_t i, int c) {
                Piece &p = pieces[i];
                p.k.dst = stage + (size_t)(2 * t + c) * kChunk;
                const uint32_t blocks = std::min<uint32_t>(64, p.used / 4096 + 1);
                hipLaunchKernelGGL(k_to_host, dim3(blocks), dim3(256), 0, stream, p.k);
                const hipError_t x = hipGetLastError();
                return x == hipSuccess ? hipEventRecord(ev[c], stream) : x;
            };
            int c = 0;
            if (e == hipSuccess && (size_t)t < pieces.size())
                e = start(t, 0);
            for (size_t i = t; i < pieces.size() && e == hipSuccess; i += T, c ^= 1) {
                if (i + T < pieces.size())
                    e = start(i + T, c ^ 1);
                if (e == hipSuccess)
                    e = hipEventSynchronize(ev[c]);
                if (e != hipSuccess)
                    break;
                const Piece &p = pieces[i];
                for (int q = 0; q < p.k.n; ++q)
                    std::memcpy(p.to[q], p.k.dst + p.k.off[q], p.k.bytes[q]);
            }
            for (auto &x : ev)
                if (x)
                    (void)hipEventDestroy(x);
            if (old != dev)
                (void)hipSetDevice(old);
            if (e != hipSuccess)
                bad = (int)e;
        };
        int started = 1;
        try {
            for (; started < T; ++started)
                th.emplace_back(work, started);
        } catch (const std::exception &) {  // no more threads: this one takes their pieces
        }
        work(0);
        for (int t = started; t < T; ++t)
            work(t);
        for (auto &x : th)
            x.join();
        err = (hipError_t)bad.load();
        if (err != hipSuccess)
            (void)hipStreamSynchronize(stream);  // nothing writes the chunks any more
    } catch (const std::exception &) {  // (thrown before anything was queued)
        err = copy_plain(stream, segs, nsegs);
    }
    lp_pool_free(stage);
    return err;
}

namespace lp {
namespace {

// Counts over the status bytes (active, out of bounds, land, deleted) and the sums of the
// particle-step and retry counters' slots, added to out[0 .. 5].
__global__ __launch_bounds__(256) void k_count_status(const uint8_t *st, size_t n,
                                                      const unsigned long long *steps,
                                                      unsigned long long *out)
{
    uint32_t c[4] = {0, 0, 0, 0};
    for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const uint32_t s = st[i];
        c[0] += s == 0;
        c[1] += s & 1u;
        c[2] += (s >> 1) & 1u;
        c[3] += (s >> 2) & 1u;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        for (int off = 32; off > 0; off >>= 1)
            c[q] += __shfl_xor(c[q], off, 64);
        if ((threadIdx.x & 63) == 0 && c[q])
            atomicAdd(&out[q], (unsigned long long)c[q]);
    }
    if (blockIdx.x == 0 && threadIdx.x < 2 * kCountSlots) {
        const unsigned long long v =
            steps[(threadIdx.x / kCountSlots) * (size_t)kCountWords +
                  (threadIdx.x % kCountSlots) * (size_t)kCountStride];
        if (v)
            atomicAdd(&out[4 + threadIdx.x / kCountSlots], v);
    }
}

__global__ void k_clear(unsigned long long *p, int n)
{
    if ((int)threadIdx.x < n)
        p[threadIdx.x] = 0ull;
}

}  // namespace

hipError_t launch_count_status(const uint8_t *st, size_t n, const unsigned long long *steps,
                               unsigned long long *out, hipStream_t s)
{
    const size_t blocks = std::min<size_t>(256, (n + 4095) / 4096 + 1);
    hipLaunchKernelGGL(k_clear, dim3(1), dim3(64), 0, s, out, 6);
    hipLaunchKernelGGL(k_count_status, dim3((uint32_t)blocks), dim3(256), 0, s, st, n, steps, out);
    return hipGetLastError();
}

}  // namespace lp
