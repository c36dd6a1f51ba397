// Error reporting, allocation and a device-wide prefix sum.
#include <cstdarg>
#include <cstdio>
#include <algorithm>
#include <cstdlib>
#include <map>
#include <mutex>
#include <new>

#include "fea_internal.h"

namespace fea {

static thread_local std::string g_error;

int set_error(int code, const char *fmt, ...)
{
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_error = buf;
    return code;
}

void clear_error() { g_error.clear(); }

// Allocation-failure injection for tests of the error path: when the
// environment variable FEA_FAIL_ALLOC_AT=n is set, the allocation of the
// n-th device array of the process (1-based) fails.
static long g_alloc_count = 0;

static bool alloc_injected()
{
    static const char *fail_at = getenv("FEA_FAIL_ALLOC_AT");
    ++g_alloc_count;
    return fail_at && atol(fail_at) == g_alloc_count;
}

int dalloc(void **p, size_t bytes)
{
    *p = nullptr;
    if (alloc_injected())
        return set_error(FEA_ENOMEM, "device allocation of %zu bytes failed (injected)", bytes);
    if (bytes == 0) bytes = 8;
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) {  // once more with the pool given back
        int dev = 0;
        (void)hipGetLastError();
        if (hipGetDevice(&dev) == hipSuccess) pool_flush(dev);
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return set_error(FEA_ENOMEM, "device allocation of %zu bytes failed: %s", bytes,
                         hipGetErrorString(e));
    }
    return FEA_OK;
}

// ------------------------------------------------------------------ pool
// Freed device memory that the next allocation may take instead of the
// driver's: a program that rebuilds its graph for every new mesh allocates
// and frees the same sizes each time, and the driver clears what is freed.
// 48^3 hybrid mesh (0.4 GB a build, assembly and destruction): 4.9 ms or,
// once the driver is behind with its clearing, 16.6 ms a pass without the
// pool, 3.2 ms with it.
// Bounded: at most kPoolBytes and kPoolBlocks unused a device; the longest
// unused goes back to the driver first, and also one that kPoolAge later
// allocations have passed over; all of them do before an allocation fails, and
// when the caller says so (fea_release_memory).
// A block enters the pool with no work on it pending: pool_free takes the
// result of the wait for that work and hands the block to the driver if the
// wait failed (hipFree then waits itself, or refuses). Any stream and thread may
// have it next.
namespace {

constexpr size_t kPoolBytes = size_t(1) << 30;
constexpr size_t kPoolBlocks = 16;
constexpr uint64_t kPoolAge = 64;

struct PoolBlock {
    void *p;
    size_t bytes;
    int device;
    uint64_t stamp;
};

struct Pool {
    std::mutex mtx;
    std::vector<PoolBlock> idle;   // oldest first
    std::map<void *, PoolBlock> used;
    uint64_t clock = 0;
};

Pool &pool()
{
    // never destroyed: graphs may outlive static objects
    alignas(Pool) static unsigned char mem[sizeof(Pool)];
    static Pool *p = new (mem) Pool;
    return *p;
}

// With the lock held: unlists blocks of the device, oldest first, while
// `more` says so.
template <typename F>
void pool_drop(Pool &q, int device, std::vector<PoolBlock> &out, F &&more)
{
    for (size_t i = 0; i < q.idle.size();) {
        if (q.idle[i].device == device && more(q.idle[i])) {
            out.push_back(q.idle[i]);
            q.idle.erase(q.idle.begin() + (ptrdiff_t)i);
        } else {
            ++i;
        }
    }
}

// Unlisted blocks to the driver; those that it refuses (under a capture) are
// listed again. Returns whether it took all of them.
bool pool_give_back(Pool &q, const std::vector<PoolBlock> &old)
{
    bool all = true;
    for (const PoolBlock &b : old) {
        if (hipFree(b.p) == hipSuccess) continue;
        (void)hipGetLastError();
        all = false;
        try {
            std::lock_guard<std::mutex> lock(q.mtx);
            q.idle.insert(q.idle.begin(), b);
        } catch (...) {
        }
    }
    return all;
}

}  // namespace

hipError_t pool_alloc(void **p, size_t bytes)
{
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    constexpr size_t G = size_t(2) << 20;
    if (bytes >= G) bytes = (bytes + G - 1) / G * G;
    Pool &q = pool();
    std::vector<PoolBlock> old;
    try {
        std::lock_guard<std::mutex> lock(q.mtx);
        old.reserve(q.idle.size());
        ++q.clock;
        size_t best = q.idle.size();
        for (size_t i = 0; i < q.idle.size(); ++i) {
            const PoolBlock &b = q.idle[i];
            // no more than half of a block unused
            if (b.device == dev && b.bytes >= bytes && b.bytes / 2 <= bytes &&
                (best == q.idle.size() || b.bytes < q.idle[best].bytes))
                best = i;
        }
        if (best < q.idle.size()) {
            const PoolBlock b = q.idle[best];
            q.used[b.p] = b;
            q.idle.erase(q.idle.begin() + (ptrdiff_t)best);
            *p = b.p;
        }
        pool_drop(q, dev, old, [&](const PoolBlock &b) { return q.clock - b.stamp > kPoolAge; });
    } catch (...) {
        return hipErrorOutOfMemory;
    }
    pool_give_back(q, old);
    if (*p) return hipSuccess;
    e = hipMalloc(p, bytes);
    if (e != hipSuccess) {  // once more with the pool given back
        (void)hipGetLastError();
        pool_flush(dev);
        e = hipMalloc(p, bytes);
        if (e != hipSuccess) {
            *p = nullptr;
            return e;
        }
    }
    try {
        std::lock_guard<std::mutex> lock(q.mtx);
        q.used[*p] = PoolBlock{*p, bytes, dev, 0};
    } catch (...) {  // not listed: pool_free hands it to hipFree
    }
    return hipSuccess;
}

bool pool_flush(int device)
{
    Pool &q = pool();
    std::vector<PoolBlock> old;
    {
        std::lock_guard<std::mutex> lock(q.mtx);
        try {
            old.reserve(q.idle.size());
        } catch (...) {
            return false;
        }
        pool_drop(q, device, old, [](const PoolBlock &) { return true; });
    }
    return pool_give_back(q, old);
}

void pool_free(void *p, hipError_t waited)
{
    if (!p) return;
    if (waited != hipSuccess) {
        dfree(p);
        (void)hipGetLastError();  // of the wait, or of a free refused under a capture
        return;
    }
    Pool &q = pool();
    std::vector<PoolBlock> old;
    bool kept = false;
    try {
        std::lock_guard<std::mutex> lock(q.mtx);
        auto it = q.used.find(p);
        if (it != q.used.end()) {
            PoolBlock b = it->second;
            q.used.erase(it);
            if (b.bytes <= kPoolBytes) {
                size_t bytes = b.bytes, blocks = 1;
                for (const PoolBlock &o : q.idle)
                    if (o.device == b.device) {
                        bytes += o.bytes;
                        ++blocks;
                    }
                old.reserve(q.idle.size());
                q.idle.reserve(q.idle.size() + 1);
                pool_drop(q, b.device, old, [&](const PoolBlock &o) {
                    const bool go = bytes > kPoolBytes || blocks > kPoolBlocks;
                    if (go) {
                        bytes -= o.bytes;
                        --blocks;
                    }
                    return go;
                });
                b.stamp = q.clock;
                q.idle.push_back(b);
                kept = true;
            }
        }
    } catch (...) {
    }
    pool_give_back(q, old);
    if (!kept) (void)hipFree(p);
}

int dalloc_pool(void **p, size_t bytes)
{
    *p = nullptr;
    if (alloc_injected()) return set_error(FEA_ENOMEM, "device allocation of %zu bytes failed (injected)", bytes);
    hipError_t e = pool_alloc(p, bytes ? bytes : 8);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return set_error(FEA_ENOMEM, "device allocation of %zu bytes failed: %s", bytes, hipGetErrorString(e));
    }
    return FEA_OK;
}

int dalloc_arrays(void **base, const DevArray *arrays, size_t n)
{
    *base = nullptr;
    size_t total = 0;
    bool injected = false;
    auto room = [](const DevArray &a) { return (std::max<size_t>(a.bytes, 1) + 255) / 256 * 256; };
    for (size_t i = 0; i < n; ++i) {
        const DevArray &a = arrays[i];
        *a.p = nullptr;
        injected = alloc_injected() || injected;
        total += room(a);
    }
    if (injected) return set_error(FEA_ENOMEM, "device allocation of %zu bytes failed (injected)", total);
    hipError_t e = pool_alloc(base, total);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return set_error(FEA_ENOMEM, "device allocation of %zu bytes failed: %s", total, hipGetErrorString(e));
    }
    char *at = (char *)*base;
    for (size_t i = 0; i < n; ++i) {
        *arrays[i].p = at;
        at += room(arrays[i]);
    }
    return FEA_OK;
}

void dfree(void *p)
{
    if (!p) return;
    {
        std::lock_guard<std::mutex> lock(pool().mtx);
        pool().used.erase(p);
    }
    (void)hipFree(p);
}

// ------------------------------------------------------------------ scan
// Three passes: per-tile sums, a single-workgroup scan of the tile sums,
// then per-tile rescans with the tile offset. 256 threads x 8 items.
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

int64_t scan_tmp_elems(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

__device__ inline int64_t block_exclusive_scan(int64_t v, int64_t *total)
{
    __shared__ int64_t s[kScanThreads];
    int t = threadIdx.x;
    s[t] = v;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        int64_t add = (t >= off) ? s[t - off] : 0;
        __syncthreads();
        s[t] += add;
        __syncthreads();
    }
    int64_t incl = s[t];
    *total = s[kScanThreads - 1];
    __syncthreads();
    return incl - v;
}

template <typename T>
__global__ void __launch_bounds__(kScanThreads) k_scan_partials(const T *in, int64_t n, int64_t *part)
{
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int64_t sum = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i)
        if (base + i < n) sum += (int64_t)in[base + i];
    int64_t total;
    block_exclusive_scan(sum, &total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_tiles(int64_t *part, int64_t ntiles)
{
    int64_t carry = 0;
    for (int64_t b = 0; b < ntiles; b += kScanThreads) {
        int64_t i = b + threadIdx.x;
        int64_t v = (i < ntiles) ? part[i] : 0;
        int64_t total;
        int64_t ex = block_exclusive_scan(v, &total);
        if (i < ntiles) part[i] = carry + ex;
        carry += total;
        __syncthreads();
    }
}

template <typename T>
__global__ void __launch_bounds__(kScanThreads) k_scan_final(const T *in, int64_t n, const int64_t *part,
                                                            int64_t *ptr)
{
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int64_t v[kScanItems];
    int64_t sum = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        v[i] = (base + i < n) ? (int64_t)in[base + i] : 0;
        sum += v[i];
    }
    int64_t total;
    int64_t run = block_exclusive_scan(sum, &total) + part[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        run += v[i];
        if (base + i < n) ptr[base + i + 1] = run;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) ptr[0] = 0;
}

template <typename T>
static int scan_impl(const T *in, int64_t n, int64_t *ptr, int64_t *tmp, hipStream_t s)
{
    if (n <= 0) {
        FEA_HIP(hipMemsetAsync(ptr, 0, sizeof(int64_t), s));
        return FEA_OK;
    }
    int64_t ntiles = (n + kScanTile - 1) / kScanTile;
    k_scan_partials<T><<<(unsigned)ntiles, kScanThreads, 0, s>>>(in, n, tmp);
    k_scan_tiles<<<1, kScanThreads, 0, s>>>(tmp, ntiles);
    k_scan_final<T><<<(unsigned)ntiles, kScanThreads, 0, s>>>(in, n, tmp, ptr);
    FEA_HIP(hipGetLastError());
    return FEA_OK;
}

int scan_to_ptr_u8(const uint8_t *in, int64_t n, int64_t *ptr, int64_t *tmp, hipStream_t s)
{
    return scan_impl(in, n, ptr, tmp, s);
}
int scan_to_ptr_i32(const int32_t *in, int64_t n, int64_t *ptr, int64_t *tmp, hipStream_t s)
{
    return scan_impl(in, n, ptr, tmp, s);
}
int scan_to_ptr_i64(const int64_t *in, int64_t n, int64_t *ptr, int64_t *tmp, hipStream_t s)
{
    return scan_impl(in, n, ptr, tmp, s);
}

}  // namespace fea

extern "C" int fea_release_memory(void)
{
    fea::clear_error();
    int dev = 0;
    FEA_HIP(hipGetDevice(&dev));
    if (!fea::pool_flush(dev)) return fea::set_error(FEA_EHIP, "the driver did not take back all unused memory");
    return FEA_OK;
}

extern "C" const char *fea_last_error(void) { return fea::g_error.c_str(); }

extern "C" const char *fea_version(void) { return "fea-gfx950 0.1"; }
