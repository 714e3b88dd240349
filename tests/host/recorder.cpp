// A stand-in for the HIP runtime, for tests of libptrt's host code without a
// GPU.  Loaded with RTLD_GLOBAL before libptrt.so, its symbols take the place
// of libamdhip64's: device memory is host memory, kernels do not run, every
// launch is recorded (also those of replayed graphs), and allocations can be
// made to fail.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <cxxabi.h>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <sys/mman.h>
#include <vector>

namespace {

struct Dim3 {
    unsigned x, y, z;
};
struct Launch {
    std::string name;
    Dim3 grid, block;
    int pointers[8]; // of the first arguments (below): not null
};
struct Graph {
    std::vector<Launch> launches;
};

std::mutex g_mutex;
std::map<const void *, std::string> g_kernels;
std::vector<Launch> g_log;
std::map<void *, size_t> g_blocks;
Graph *g_capture = nullptr;
int g_fail_device = 0, g_fail_host = 0; // the n-th allocation from now on fails
int g_fail_new = 0;
int g_last_error = 0;
size_t g_host_most = 0, g_host_now = 0;
size_t g_host_limit = ~(size_t)0; // larger pinned allocations fail
std::vector<size_t> g_device_sizes; // asked for since the last reset
thread_local struct {
    Dim3 grid, block;
    size_t shared;
    void *stream;
} t_call;

thread_local int t_inside = 0; // allocations of the recorder itself do not count
struct Inside {
    Inside() { ++t_inside; }
    ~Inside() { --t_inside; }
};

constexpr int INVALID_VALUE = 1, OUT_OF_MEMORY = 2, INVALID_CONFIGURATION = 9;

int allocate(void **p, size_t bytes)
{
    void *m = mmap(nullptr, bytes ? bytes : 1, PROT_READ | PROT_WRITE,
                   MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return g_last_error = OUT_OF_MEMORY;
    g_blocks[m] = bytes ? bytes : 1;
    *p = m;
    return 0;
}

size_t release(void *p)
{
    auto it = g_blocks.find(p);
    if (it == g_blocks.end()) return 0;
    const size_t bytes = it->second;
    munmap(p, bytes);
    g_blocks.erase(it);
    return bytes;
}

} // namespace

// the library's own allocations (it finds these before libstdc++'s)
void *operator new(size_t bytes)
{
    if (!t_inside && g_fail_new > 0 && --g_fail_new == 0) throw std::bad_alloc();
    if (void *p = std::malloc(bytes ? bytes : 1)) return p;
    throw std::bad_alloc();
}
void *operator new(size_t bytes, const std::nothrow_t &) noexcept
{
    if (!t_inside && g_fail_new > 0 && --g_fail_new == 0) return nullptr;
    return std::malloc(bytes ? bytes : 1);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {

// ------------------------------------------------------------ the recorder
void rec_fail_new(int n) { g_fail_new = n; } // the n-th `new` from now on fails
void rec_reset()
{
    std::lock_guard<std::mutex> lock(g_mutex);
    g_log.clear();
    g_device_sizes.clear();
}
int rec_launches() { return (int)g_log.size(); }
const char *rec_name(int k) { return g_log[k].name.c_str(); }
void rec_shape(int k, unsigned *out)
{
    const Launch &l = g_log[k];
    const unsigned v[6] = {l.grid.x, l.grid.y, l.grid.z, l.block.x, l.block.y, l.block.z};
    std::memcpy(out, v, sizeof(v));
}
// argument k of a k_tile_2d launch that is a pointer is not null
int rec_pointer(int k, int arg) { return g_log[k].pointers[arg]; }
void rec_fail_device(int n) { g_fail_device = n; }
void rec_fail_host(int n) { g_fail_host = n; }
void rec_limit_host(size_t bytes) { g_host_limit = bytes; }
int rec_device_allocations() { return (int)g_device_sizes.size(); }
size_t rec_device_size(int k) { return g_device_sizes[k]; }
size_t rec_host_now() { return g_host_now; }
size_t rec_host_most() { return g_host_most; }
int rec_blocks() { return (int)g_blocks.size(); }

// ------------------------------------------------------- kernels, launches
void **__hipRegisterFatBinary(const void *)
{
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *,
                           void *, void *, int *)
{
    int status = 0;
    char *name = abi::__cxa_demangle(device, nullptr, nullptr, &status);
    g_kernels[host] = name ? name : device;
    std::free(name);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream)
{
    t_call = {grid, block, shared, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream)
{
    *grid = t_call.grid;
    *block = t_call.block;
    *shared = t_call.shared;
    *stream = t_call.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3 block, void **args, size_t, void *)
{
    const Inside inside;
    std::lock_guard<std::mutex> lock(g_mutex);
    // what the runtime refuses: no threads, over 1024 a block, 2^32 threads
    // or more along an axis
    const unsigned g[3] = {grid.x, grid.y, grid.z}, b[3] = {block.x, block.y, block.z};
    bool ok = (unsigned long long)block.x * block.y * block.z <= 1024;
    for (int k = 0; k < 3; ++k) ok = ok && g[k] && b[k] && (unsigned long long)g[k] * b[k] < (1ull << 32);
    if (!ok) return g_last_error = INVALID_CONFIGURATION;
    Launch l{g_kernels[f], grid, block, {}};
    if (l.name.find("k_tile_2d<") != std::string::npos)
        for (int k = 0; k < 5; ++k) l.pointers[k] = *(void **)args[k] != nullptr;
    (g_capture ? g_capture->launches : g_log).push_back(l);
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 2;
    return 0;
}

// ------------------------------------------------------------------ memory
int hipMalloc(void **p, size_t bytes)
{
    const Inside inside;
    std::lock_guard<std::mutex> lock(g_mutex);
    *p = nullptr;
    g_device_sizes.push_back(bytes);
    if (g_fail_device > 0 && --g_fail_device == 0) return g_last_error = OUT_OF_MEMORY;
    return allocate(p, bytes);
}
int hipFree(void *p)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    release(p);
    return 0;
}
int hipHostMalloc(void **p, size_t bytes, unsigned)
{
    const Inside inside;
    std::lock_guard<std::mutex> lock(g_mutex);
    *p = nullptr;
    if ((g_fail_host > 0 && --g_fail_host == 0) || bytes > g_host_limit) return g_last_error = OUT_OF_MEMORY;
    g_host_now += bytes;
    if (g_host_now > g_host_most) g_host_most = g_host_now;
    return allocate(p, bytes);
}
int hipHostFree(void *p)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    g_host_now -= release(p);
    return 0;
}
int hipMemset(void *p, int v, size_t bytes)
{
    // fresh memory is zero; large lattices stay untouched
    if (v != 0 || bytes <= (64u << 20)) std::memset(p, v, bytes);
    return 0;
}
int hipMemcpy(void *to, const void *from, size_t bytes, int)
{
    std::memcpy(to, from, bytes);
    return 0;
}
int hipMemcpyAsync(void *to, const void *from, size_t bytes, int, void *)
{
    std::memcpy(to, from, bytes);
    return 0;
}
int hipGetSymbolAddress(void **p, const void *)
{
    *p = nullptr;
    return INVALID_VALUE;
}

// ------------------------------------------------ devices, streams, events
int hipGetDevice(int *d)
{
    *d = 0;
    return 0;
}
int hipDeviceGetAttribute(int *v, int, int)
{
    *v = 256;
    return 0;
}
int hipStreamCreateWithFlags(void **s, unsigned)
{
    *s = std::malloc(1);
    return 0;
}
int hipStreamDestroy(void *s)
{
    std::free(s);
    return 0;
}
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipEventCreate(void **e)
{
    *e = std::malloc(1);
    return 0;
}
int hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void *e)
{
    std::free(e);
    return 0;
}
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventQuery(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *)
{
    *ms = 1.0f;
    return 0;
}
int hipGetLastError()
{
    const int e = g_last_error;
    g_last_error = 0;
    return e;
}
const char *hipGetErrorString(int e) { return e == OUT_OF_MEMORY ? "out of memory" : "stand-in error"; }

// ------------------------------------------------------------------ graphs
int hipStreamBeginCapture(void *, int)
{
    const Inside inside;
    g_capture = new Graph;
    return 0;
}
int hipStreamEndCapture(void *, void **graph)
{
    *graph = g_capture;
    g_capture = nullptr;
    return 0;
}
int hipGraphInstantiate(void **exec, void *graph, void *, char *, size_t)
{
    const Inside inside;
    *exec = new Graph(*static_cast<Graph *>(graph));
    return 0;
}
int hipGraphDestroy(void *graph)
{
    delete static_cast<Graph *>(graph);
    return 0;
}
int hipGraphExecDestroy(void *exec)
{
    delete static_cast<Graph *>(exec);
    return 0;
}
int hipGraphLaunch(void *exec, void *)
{
    const Inside inside;
    const Graph *g = static_cast<Graph *>(exec);
    g_log.insert(g_log.end(), g->launches.begin(), g->launches.end());
    return 0;
}

} // extern "C"
