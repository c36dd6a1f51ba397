// The library's host paths on the CPU: this program defines the runtime calls
// that libfea.so makes (device memory is host memory, kernels do nothing, waits
// and allocations fail on demand), loads the library and goes through its C
// entry points with meshes of nodes without elements. Checks where freed
// device memory goes and what a graph can be loaded from. Usage: host_paths_check LIBFEA CHECK DIRECTORY; exit status 0 on
// success.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <sys/stat.h>

#include <csignal>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "../../include/fea.h"

// ------------------------------------------------------------ the runtime
static std::mutex mtx;
static std::map<void *, size_t> live;  // device memory the driver has given out
static int n_malloc = 0, fail_malloc = 0;
static size_t largest_freed = 0;
static bool fail_device_wait = false, fail_stream_wait = false, refuse_free = false;

extern "C" {
hipError_t hipMalloc(void **p, size_t n)
{
    std::lock_guard<std::mutex> lock(mtx);
    *p = nullptr;
    if (fail_malloc > 0) {
        --fail_malloc;
        return hipErrorOutOfMemory;
    }
    ++n_malloc;
    *p = calloc(1, n);
    live[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> lock(mtx);
    if (refuse_free) return hipErrorStreamCaptureUnsupported;
    auto it = live.find(p);
    if (it == live.end()) return p ? hipErrorInvalidValue : hipSuccess;
    if (it->second > largest_freed) largest_freed = it->second;
    live.erase(it);
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof(*p));
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return fail_device_wait ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return fail_stream_wait ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }  // memory starts as zeros
hipError_t hipMemcpyToSymbol(const void *, const void *, size_t, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static char symbol[64];
    *p = symbol;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
}

// ------------------------------------------------------------- the library
static decltype(&fea_graph_build) graph_build;
static decltype(&fea_graph_destroy) graph_destroy;
static decltype(&fea_graph_save) graph_save;
static decltype(&fea_graph_load) graph_load;
static decltype(&fea_last_error) last_error;
static decltype(&fea_release_memory) release_memory;

static int failures = 0;
#define CHECK(c)                                                              \
    do {                                                                      \
        if (!(c)) {                                                           \
            std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); \
            ++failures;                                                       \
        }                                                                     \
    } while (0)

static fea_graph *build(int64_t nodes, int expect = FEA_OK)
{
    fea_graph *g = nullptr;
    const int rc = graph_build(nodes, 0, nullptr, nullptr, nullptr, nullptr, &g);
    CHECK(rc == expect);
    return g;
}

static size_t live_bytes()
{
    size_t n = 0;
    for (const auto &b : live) n += b.second;
    return n;
}

constexpr int64_t M = 1000000;

// The memory of a destroyed graph serves the next one only if the wait for
// the work on it succeeded.
static void check_waits()
{
    graph_destroy(build(M));
    int before = n_malloc;
    fea_graph *g = build(M);
    CHECK(n_malloc == before);  // all of it from freed blocks
    largest_freed = 0;
    fail_device_wait = true;
    graph_destroy(g);
    fail_device_wait = false;
    CHECK(largest_freed >= 16 * (size_t)M);  // its two tables of M + 1 offsets went to the driver
    before = n_malloc;
    g = build(M);
    CHECK(n_malloc > before);
    graph_destroy(g);
    // a build whose waits fail: neither its scratch memory nor its arrays stay
    const size_t have = live.size();
    CHECK(have > 0);
    fail_device_wait = fail_stream_wait = true;
    build(M, FEA_EHIP);
    fail_device_wait = fail_stream_wait = false;
    before = n_malloc;
    graph_destroy(build(M));
    CHECK(n_malloc > before);
}

constexpr size_t GiB = (size_t)1 << 30;

// Unused memory is bounded in bytes and blocks, and what later allocations pass
// over goes back.
static void check_bounds()
{
    std::vector<fea_graph *> g;
    for (int k = 0; k < 6; ++k) g.push_back(build((20 + 3 * k) * M));  // 0.3 to 0.6 GB and as much scratch each
    CHECK(live_bytes() > 2 * GiB);
    for (fea_graph *x : g) graph_destroy(x);
    CHECK(live_bytes() <= GiB && live_bytes() > GiB / 4);
    g.clear();
    for (int k = 0; k < 40; ++k) g.push_back(build((1 + k) * M / 20));
    for (fea_graph *x : g) graph_destroy(x);
    CHECK(live.size() <= 16 && live_bytes() <= GiB);
    graph_destroy(build(80 * M));  // one block beyond the bound: not kept
    CHECK(live_bytes() <= GiB);
    graph_destroy(build(30 * M));
    CHECK(live_bytes() > GiB / 4);
    for (int k = 0; k < 40; ++k) graph_destroy(build(10));
    CHECK(live_bytes() < GiB / 64);
}

// Before an allocation fails, the unused memory goes back; after one that does
// the library goes on.
static void check_full()
{
    graph_destroy(build(30 * M));
    CHECK(live_bytes() > GiB / 4);
    fail_malloc = 1;
    fea_graph *g = build(M);  // too small for the blocks kept: new memory, on the second try
    CHECK(fail_malloc == 0 && live_bytes() < GiB / 4);
    graph_destroy(g);
    fail_malloc = 1000;
    build(10 * M, FEA_ENOMEM);
    fail_malloc = 0;
    graph_destroy(build(10 * M));
}

// fea_release_memory gives back what no graph uses, and nothing else; memory
// that the driver does not take (under a capture) stays in use.
static void check_release()
{
    fea_graph *g = build(M);
    const size_t used = live_bytes();
    graph_destroy(build(2 * M));
    CHECK(live_bytes() > used);
    CHECK(release_memory() == FEA_OK);
    CHECK(live_bytes() <= used && live_bytes() >= 16 * (size_t)M);
    graph_destroy(g);
    CHECK(live_bytes() > 0);
    const size_t kept = live_bytes();
    refuse_free = true;
    CHECK(release_memory() == FEA_EHIP);
    refuse_free = false;
    CHECK(live_bytes() == kept);
    const int before = n_malloc;
    g = build(M / 2 + M / 4);
    CHECK(n_malloc < before + 4);  // not all of it new
    graph_destroy(g);
    CHECK(release_memory() == FEA_OK);
    CHECK(live.empty());
}

// A graph cache is read from a file and from a pipe (which cannot seek); a
// truncated one is refused either way.
static void check_pipe(const std::string &dir)
{
    const std::string file = dir + "/graph", pipe = dir + "/pipe";
    fea_graph *g = build(1000);
    CHECK(graph_save(g, file.c_str()) == FEA_OK);
    graph_destroy(g);
    std::vector<char> data;
    FILE *f = fopen(file.c_str(), "rb");
    for (int c; (c = fgetc(f)) != EOF;) data.push_back((char)c);
    fclose(f);
    CHECK(mkfifo(pipe.c_str(), 0600) == 0);
    auto load = [&](const std::string &from, size_t bytes) {
        std::thread writer([&] {
            FILE *w = fopen(from.c_str(), "wb");
            fwrite(data.data(), 1, bytes, w);  // may end early: the reader gives up
            fclose(w);
        });
        if (from == file) writer.join();
        fea_graph *h = nullptr;
        const int rc = graph_load(from.c_str(), 1000, 0, nullptr, nullptr, nullptr, nullptr, &h);
        if (rc != FEA_OK) std::printf("%zu bytes: %s\n", bytes, last_error());
        if (writer.joinable()) writer.join();
        if (h) graph_destroy(h);
        return rc;
    };
    for (const std::string &from : {file, pipe}) {
        CHECK(load(from, data.size()) == FEA_OK);
        CHECK(load(from, data.size() - 1) == FEA_EINVAL);
        CHECK(load(from, data.size() / 2) == FEA_EINVAL);
    }
}

// A header that no build writes is refused before anything is sized by it:
// more colours than there can be, sizes and family offsets that are not the mesh's.
static void check_header(const std::string &dir)
{
    const std::string file = dir + "/graph";
    fea_graph *g = build(1000);
    CHECK(graph_save(g, file.c_str()) == FEA_OK);
    graph_destroy(g);
    std::vector<char> data;
    FILE *f = fopen(file.c_str(), "rb");
    for (int c; (c = fgetc(f)) != EOF;) data.push_back((char)c);
    fclose(f);
    // header: magic 8, version 4, colours 4, arch 64, then int64: nodes, elements, blocks, map and connectivity
    // lengths, fingerprint, 3 x 5 family offsets, length of the colour buckets
    auto load = [&](size_t at32, int32_t v32, size_t at64, int64_t v64) {
        std::vector<char> d = data;
        if (at32) memcpy(d.data() + at32, &v32, 4);
        if (at64) memcpy(d.data() + at64, &v64, 8);
        FILE *w = fopen(file.c_str(), "wb");
        fwrite(d.data(), 1, d.size(), w);
        fclose(w);
        fea_graph *h = nullptr;
        const int before = n_malloc, rc = graph_load(file.c_str(), 1000, 0, nullptr, nullptr, nullptr, nullptr, &h);
        CHECK(rc == FEA_OK || n_malloc <= before + 1);  // (the mesh check's scratch memory)
        if (h) graph_destroy(h);
        release_memory();
        return rc;
    };
    const int32_t many = 0x7ffffffe;
    CHECK(load(0, 0, 0, 0) == FEA_OK);
    CHECK(load(12, many, 248, 4 * ((int64_t)many + 1)) == FEA_EINVAL);
    CHECK(load(12, 257, 248, 4 * 258) == FEA_EINVAL);
    CHECK(load(0, 0, 104, 1) == FEA_EINVAL);   // map length
    CHECK(load(0, 0, 112, 1) == FEA_EINVAL);   // connectivity length
    for (size_t k = 0; k < 15; ++k) CHECK(load(0, 0, 128 + 8 * k, 1) == FEA_EINVAL);
}

int main(int argc, char **argv)
{
    if (argc != 4) return 2;
    void *lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
    if (!lib) {
        std::fprintf(stderr, "%s\n", dlerror());
        return 2;
    }
    graph_build = (decltype(graph_build))dlsym(lib, "fea_graph_build");
    graph_destroy = (decltype(graph_destroy))dlsym(lib, "fea_graph_destroy");
    graph_save = (decltype(graph_save))dlsym(lib, "fea_graph_save");
    graph_load = (decltype(graph_load))dlsym(lib, "fea_graph_load");
    last_error = (decltype(last_error))dlsym(lib, "fea_last_error");
    release_memory = (decltype(release_memory))dlsym(lib, "fea_release_memory");
    signal(SIGPIPE, SIG_IGN);
    const std::string what = argv[2], dir = argv[3];
    if (what == "waits") check_waits();
    else if (what == "pipe") check_pipe(dir);
    else if (what == "header") check_header(dir);
    else if (what == "bounds") check_bounds();
    else if (what == "full") check_full();
    else if (what == "release") check_release();
    else return 2;
    return failures ? 1 : 0;
}
