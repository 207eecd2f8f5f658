// A host-memory stand-in for the HIP calls of librlbm.so's host code, for CPU
// tests of its error paths: "device" memory is host memory, kernels do nothing,
// asynchronous copies stay queued until their stream is waited for.  Loaded
// with RTLD_GLOBAL before the library, whose calls then bind here.
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

namespace {
struct Copy {
    void* dst;
    const void* src;
    size_t n;
};
std::vector<Copy> queued;
std::map<void*, size_t> pinned;
size_t pinned_bytes = 0, pinned_peak = 0, pinned_limit = (size_t)-1;
long frees = 0, waits = 0, launches = 0, blocks = 0, replays = 0, fail_at = -1;
int last_error = 0;
constexpr int OUT_OF_MEMORY = 2, LAUNCH_FAILURE = 719;

void drain() {
    for (const Copy& c : queued) std::memmove(c.dst, c.src, c.n);
    queued.clear();
    ++waits;
}
}  // namespace

struct Dim3 {
    unsigned x, y, z;
};
static Dim3 pushed[2];

extern "C" {

// what a test sets and reads
void stub_pinned_limit(size_t bytes) { pinned_limit = bytes; }          // hipHostMalloc fails beyond
void stub_fail_launch(long n) { fail_at = n < 0 ? -1 : launches + n; }  // the n-th launch from now fails
long stub_queued() { return (long)queued.size(); }
long stub_waits() { return waits; }
long stub_frees() { return frees; }
long stub_blocks() { return blocks; }      // of all launches
long stub_replays() { return replays; }    // of graphs
size_t stub_pinned() { return pinned_bytes; }

int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "stub error"; }
int hipThreadExchangeStreamCaptureMode(int*) { return 0; }

int hipHostMalloc(void** p, size_t n, unsigned) {
    if (n > pinned_limit) return OUT_OF_MEMORY;
    *p = std::aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    pinned[*p] = n;
    pinned_bytes += n;
    return 0;
}
int hipHostFree(void* p) {
    ++frees;
    pinned_bytes -= pinned.at(p);
    pinned.erase(p);
    std::free(p);
    return 0;
}
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }

int hipMemcpy(void* dst, const void* src, size_t n, int) {
    drain();
    std::memmove(dst, src, n);
    return 0;
}
int hipMemcpy2D(void* dst, size_t dp, const void* src, size_t sp, size_t w, size_t h, int) {
    drain();
    for (size_t r = 0; r < h; ++r) std::memmove((char*)dst + r * dp, (const char*)src + r * sp, w);
    return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t n, int, void*) {
    queued.push_back({dst, src, n});
    return 0;
}
int hipMemcpy2DAsync(void* dst, size_t dp, const void* src, size_t sp, size_t w, size_t h, int, void*) {
    for (size_t r = 0; r < h; ++r) queued.push_back({(char*)dst + r * dp, (const char*)src + r * sp, w});
    return 0;
}
int hipStreamSynchronize(void*) { drain(); return 0; }

int hipEventCreateWithFlags(void** e, unsigned) { *e = nullptr; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = nullptr; return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { *g = nullptr; return 0; }
int hipGraphInstantiate(void** x, void*, void*, char*, size_t) { *x = &pushed; return 0; }
int hipGraphLaunch(void*, void*) { ++replays; return 0; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
int hipGetSymbolAddress(void** p, const void*) {
    static char device_array[1 << 20];
    *p = device_array;
    return 0;
}

int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t, void*) {
    pushed[0] = g;
    pushed[1] = b;
    return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, void** st) {
    *g = pushed[0];
    *b = pushed[1];
    *s = 0;
    *st = nullptr;
    return 0;
}
int hipLaunchKernel(const void*, Dim3 g, Dim3, void**, size_t, void*) {
    blocks += (long)g.x * g.y * g.z;
    if (launches++ == fail_at) return last_error = LAUNCH_FAILURE;
    return 0;
}
}
