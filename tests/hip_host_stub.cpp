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
long frees = 0, waits = 0, launches = 0, fail_at = -1;
int last_error = 0;
constexpr int OUT_OF_MEMORY = 2, LAUNCH_FAILURE = 719;

void drain() {
    for (const Copy& c : queued) std::memmove(c.dst, c.src, c.n);
    queued.clear();
    ++waits;
}
}  // namespace

extern "C" {
struct Dim3 {
    unsigned x, y, z;
};

// what a test sets and reads
void stub_pinned_limit(size_t bytes) { pinned_limit = bytes; }          // hipHostMalloc fails beyond
void stub_fail_launch(long n) { fail_at = n < 0 ? -1 : launches + n; }  // the n-th launch from now fails
long stub_queued() { return (long)queued.size(); }
long stub_waits() { return waits; }
long stub_frees() { return frees; }
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

int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, void** st) {
    *g = *b = Dim3{1, 1, 1};
    *s = 0;
    *st = nullptr;
    return 0;
}
int hipLaunchKernel(const void*, Dim3, Dim3, void**, size_t, void*) {
    if (launches++ == fail_at) return last_error = LAUNCH_FAILURE;
    return 0;
}
}
