// A HIP runtime without a device, for tests of the library's host code on the
// CPU: device memory is zeroed host memory, copies and clears happen at once,
// and kernel launches do nothing but count.  Loaded globally before
// libwnnc.so, its functions take the place of the HIP runtime's.
#include <cstdio>
#include <cstdlib>
#include <cstring>

namespace {
int fail_at = 0;        // the allocation that fails, counted from 1 (0: none)
long long launches = 0; // kernels launched
int pending = 0;        // operations queued since the last wait
struct Dim3 {
    unsigned x, y, z;
};
struct Config {
    Dim3 grid, block;
    size_t shared;
    void *stream;
} config;
int queued() {
    ++pending;
    return 0;
}
int launched() {
    ++launches;
    return queued();
}
int waited() {
    pending = 0;
    return 0;
}
}  // namespace

extern "C" {
// the tests' side
void host_fail_allocation(int k) { fail_at = k; }
long long host_launches() { return launches; }
int host_pending() { return pending; }

// the library's side
void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *,
                           void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t s, void *st) {
    config = {g, b, s, st};
    return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *s, void **st) {
    *g = config.grid, *b = config.block, *s = config.shared, *st = config.stream;
    return 0;
}
int hipLaunchKernel(const void *, Dim3, Dim3, void **, size_t, void *) { return launched(); }
int hipExtLaunchKernel(const void *, Dim3, Dim3, void **, size_t, void *, void *, void *, int) {
    return launched();
}
int hipMalloc(void **p, size_t n) {
    *p = nullptr;
    if (fail_at > 0 && --fail_at == 0) return 2;  // out of memory
    *p = calloc(1, n ? n : 1);
    return *p ? 0 : 2;
}
int hipFree(void *p) {
    free(p);
    return waited();
}
int hipMemcpy(void *d, const void *s, size_t n, int) {
    memcpy(d, s, n);
    return waited();
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) {
    memcpy(d, s, n);
    return queued();
}
int hipMemsetAsync(void *d, int v, size_t n, void *) {
    memset(d, v, n);
    return queued();
}
int hipStreamSynchronize(void *) { return waited(); }
int hipEventCreate(void **e) {
    *e = malloc(1);
    return 0;
}
int hipEventDestroy(void *e) {
    free(e);
    return 0;
}
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return waited(); }
int hipEventElapsedTime(float *ms, void *, void *) {
    *ms = 0.f;
    return 0;
}
int hipGetDevice(int *d) {
    *d = 0;
    return 0;
}
int hipGetDeviceCount(int *n) {
    *n = 1;
    return 0;
}
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }
int hipGetSymbolAddress(void **p, const void *) {
    static char scratch[64];
    *p = scratch;
    return 0;
}
}
