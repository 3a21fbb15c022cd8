// Stand-in for the HIP runtime calls that the library's host code makes: nothing runs, every call that orders work on
// streams is recorded.  Loaded ahead of the library, it shows on a machine without a GPU which stream waits for what.
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <cxxabi.h>
#include <map>
#include <mutex>
#include <string>
#include <vector>

struct Entry {
    int kind;                 // 0 launch or copy, 1 event recorded, 2 wait for an event
    const void *stream, *event;
    const void *kernel;       // of a launch
    unsigned blocks, threads;
};
static std::mutex g_mu;
static std::vector<Entry> g_log;
static char g_symbol[256];
static void add(int kind, const void *stream, const void *event, const void *kernel = nullptr, unsigned blocks = 0,
                unsigned threads = 0)
{
    std::lock_guard<std::mutex> g(g_mu);
    g_log.push_back({kind, stream, event, kernel, blocks, threads});
}
// the kernels the library brings along, by the address that a launch names
static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}

extern "C" {
size_t stub_log_size() { return g_log.size(); }
void stub_log_get(size_t i, int *kind, const void **stream, const void **event)
{
    *kind = g_log[i].kind;
    *stream = g_log[i].stream;
    *event = g_log[i].event;
}
void stub_log_clear() { g_log.clear(); }
// the kernel of entry i and its launch shape; an empty name for anything else
const char *stub_log_kernel(size_t i, unsigned *blocks, unsigned *threads)
{
    *blocks = g_log[i].blocks;
    *threads = g_log[i].threads;
    const auto it = names().find(g_log[i].kernel);
    return it == names().end() ? "" : it->second.c_str();
}
size_t stub_kernel_count() { return names().size(); }
const char *stub_kernel_name(size_t i)
{
    auto it = names().begin();
    while (i--) ++it;
    return it->second.c_str();
}

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    int rc;
    char *s = abi::__cxa_demangle(device, nullptr, nullptr, &rc);
    names()[host] = rc == 0 ? s : device;
    std::free(s);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPopCallConfiguration(void *, void *, size_t *, void *) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipMalloc(void **p, size_t n) { *p = std::malloc(n); return *p ? 0 : 2; }
int hipFree(void *p) { std::free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *stream) { add(0, stream, nullptr); return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = g_symbol; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 1; return 0; }
struct Dim3 { unsigned x, y, z; };
int hipLaunchKernel(const void *kernel, Dim3 grid, Dim3 block, void **, size_t, void *stream)
{
    add(0, stream, nullptr, kernel, grid.x, block.x);
    return 0;
}
int hipStreamCreateWithFlags(void **s, unsigned) { *s = std::malloc(16); return 0; }
int hipStreamDestroy(void *s) { std::free(s); return 0; }
int hipStreamIsCapturing(void *, int *status) { *status = 0; return 0; }
int hipStreamWaitEvent(void *stream, void *event, unsigned) { add(2, stream, event); return 0; }
int hipEventCreate(void **e) { *e = std::malloc(16); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void *e) { std::free(e); return 0; }
int hipEventRecord(void *event, void *stream) { add(1, stream, event); return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0.f; return 0; }
}
