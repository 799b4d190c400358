// A HIP runtime without a device: the host side of libspkv.so runs against it and every kernel
// launch is written down (kernel, grid, block) in place of being executed.  "Device" memory is the
// address the caller hands over; copies to the host deliver the bytes the test has set.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <dlfcn.h>
#include <map>
#include <new>
#include <string>
#include <vector>

struct Dim3 {
    uint32_t x, y, z;
};

static std::map<const void*, std::string> g_kernel;       // host stub -> mangled device name
static std::vector<std::string> g_log;
static std::vector<unsigned char> g_device_bytes;         // what copies to the host deliver
static int g_sync_error = 0;                              // what waiting for a stream returns
static int g_prompt_lengths = 0;                          // do the lengths that a prompt sends arrive?
static int g_capture_status = 0, g_capture_error = 0, g_last_error = 0, g_event_ready = 1;
static std::string g_watch;                               // kernels whose argument is read ...
static int g_watch_arg, g_watch_at;                       // ... the int at this byte of this argument
static Dim3 g_grid, g_block;
static size_t g_shared;
static void* g_stream;
static int deliver(void* dst, size_t n) {
    memset(dst, 0, n);
    memcpy(dst, g_device_bytes.data(), n < g_device_bytes.size() ? n : g_device_bytes.size());
    return 0;
}

// Allocations of the library (not of this file), by who calls.
static int g_news = 0;
void* operator new(size_t n) {
    Dl_info at;
    if (dladdr(__builtin_return_address(0), &at) != 0 && at.dli_fname != nullptr && strstr(at.dli_fname, "libspkv") != nullptr) g_news += 1;
    void* p = malloc(n > 0 ? n : 1);
    if (p == nullptr) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {

// ---- what the test sets and reads
int rec_news() {                                          // since the last such question
    const int n = g_news;
    g_news = 0;
    return n;
}
void rec_device_bytes(const void* p, size_t n) {
    g_device_bytes.assign(static_cast<const unsigned char*>(p), static_cast<const unsigned char*>(p) + n);
}
void rec_capture(int status, int error) { g_capture_status = status, g_capture_error = error; }
void rec_event_ready(int ready) { g_event_ready = ready; }
void rec_prompt_lengths(int arrive) { g_prompt_lengths = arrive; }
void rec_sync_error(int e) { g_sync_error = e; }
void rec_watch(const char* kernel, int arg, int at) { g_watch = kernel, g_watch_arg = arg, g_watch_at = at; }
int rec_take(char* buf, int cap) {                        // the oldest entry; -1: none
    if (g_log.empty()) return -1;
    std::string s = g_log.front();
    g_log.erase(g_log.begin());
    const int n = (int)s.size() < cap ? (int)s.size() : cap - 1;
    memcpy(buf, s.data(), n);
    buf[n] = 0;
    return n;
}

// ---- registration and launches
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    g_kernel[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
    g_grid = grid, g_block = block, g_shared = shared, g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
    *grid = g_grid, *block = g_block, *shared = g_shared, *stream = g_stream;
    return 0;
}
int hipLaunchKernel(const void* host, Dim3 grid, Dim3 block, void** args, size_t, void*) {
    if (!g_watch.empty() && g_kernel[host].find(g_watch) != std::string::npos) {
        int v;
        memcpy(&v, static_cast<char*>(args[g_watch_arg]) + g_watch_at, 4);
        g_log.push_back("watched " + std::to_string(v) + " 0 0");
    }
    if (g_kernel[host].find("spkv_copy_lengths") != std::string::npos && g_event_ready) {
        const int n = *static_cast<int*>(args[1]);         // (lengths, n, where to, ticket)
        int* to = *static_cast<int**>(args[2]);
        deliver(to, 4 * (size_t)n);
        to[n] = *static_cast<int*>(args[3]);
    }
    if (g_kernel[host].find("spkv_bulk_scatter") != std::string::npos && g_prompt_lengths) {
        const int ordered = *static_cast<int*>(args[8]) > 0;   // (..., order of spans, {where to, ticket})
        struct { int* to; int ticket; } copy;
        memcpy(&copy, args[9], sizeof(copy));
        const int n = (int)grid.y - ordered;
        if (copy.to != nullptr) deliver(copy.to, 4 * (size_t)n), copy.to[n] = copy.ticket;
    }
    g_log.push_back(g_kernel[host] + " " + std::to_string(grid.x) + " " + std::to_string(grid.y) + " " + std::to_string(block.x));
    return 0;
}

// ---- the rest of what the library calls
int hipGetLastError() {
    const int e = g_last_error;
    g_last_error = 0;
    return e;
}
int hipStreamIsCapturing(void*, int* status) {
    *status = g_capture_status;
    if (g_capture_error != 0) g_last_error = g_capture_error;
    return g_capture_error;
}
int hipGetDevice(int* d) {
    *d = 0;
    return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {              // compute units are all that is asked for
    *v = 256;
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* host, int block, size_t) {
    const std::string& name = g_kernel[host];              // as the gfx950 build reports it
    const bool d64 = name.find("ILi64E") != std::string::npos;
    if (name.find("chunk_split") != std::string::npos) {
        const bool one = name.find("ELi1E") != std::string::npos, two = name.find("ELi2E") != std::string::npos;
        *n = one ? (d64 ? 16 : 8) : two ? (d64 ? 8 : 4) : 4;
    } else {
        *n = (d64 ? 16 : 12) * 64 / block;
    }
    return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
    static unsigned char scratch[256];
    *p = scratch;
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
    *p = calloc(1, n);
    return 0;
}
int hipHostFree(void* p) {
    g_log.push_back("host_free 0 0 0");
    free(p);
    return 0;
}
int hipMemcpy(void* dst, const void*, size_t n, int) { return deliver(dst, n); }
int hipMemcpyAsync(void* dst, const void*, size_t n, int, void*) {
    g_log.push_back("copy " + std::to_string(n) + " 0 0");
    return deliver(dst, n);
}
int hipStreamSynchronize(void*) { return g_sync_error; }
int hipEventCreate(void** e) {
    *e = malloc(1);
    return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e) {
    free(e);
    return 0;
}
int hipEventElapsedTime(float* ms, void*, void*) {
    *ms = 0.f;
    return 0;
}
int hipEventQuery(void*) {
    g_log.push_back("event_query 0 0 0");
    if (g_event_ready) return 0;
    return g_last_error = 600;                             // hipErrorNotReady
}
int hipEventRecord(void*, void*) {
    g_log.push_back("event_record 0 0 0");
    return 0;
}
int hipDeviceSynchronize() {
    g_log.push_back("device_sync 0 0 0");
    return 0;
}
int hipEventSynchronize(void*) { return 0; }
}
