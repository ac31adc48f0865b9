// A stand-in for the HIP runtime that runs nothing: device memory is host
// memory, and every kernel launch is noted by name with its grid and block.
// Loaded (RTLD_GLOBAL) before libsas.so, it lets a process without a GPU make
// plans and see what a call would launch.  Kernels do not run, so no result
// of a call may be read.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 {
    uint32_t x, y, z;
};
struct Launch {
    std::string name;
    Dim3 grid, block;
};
std::map<const void *, std::string> &kernels() {
    static std::map<const void *, std::string> k;
    return k;
}
std::vector<Launch> launches;
struct Config {
    Dim3 grid, block;
    size_t lds;
    void *stream;
} config;
}  // namespace

extern "C" {
int64_t recorder_count() { return (int64_t)launches.size(); }
void recorder_clear() { launches.clear(); }
// Mangled name of launch i; dims: grid x, y, z, block x, y, z.
const char *recorder_launch(int64_t i, uint32_t *dims) {
    const Launch &l = launches[(size_t)i];
    std::memcpy(dims, &l.grid, sizeof(Dim3));
    std::memcpy(dims + 3, &l.block, sizeof(Dim3));
    return l.name.c_str();
}

int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream) {
    config = Config{grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream) {
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *stream = config.stream;
    return 0;
}
void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
    kernels()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3 block, void **, size_t, void *) {
    launches.push_back(Launch{kernels()[f], grid, block});
    return 0;
}
int hipMalloc(void **p, size_t n) {
    *p = std::aligned_alloc(256, (n + 255) / 256 * 256 + 256);
    return *p ? 0 : 2;
}
int hipFree(void *p) {
    std::free(p);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) {
    std::memcpy(d, s, n);
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) {
    std::memcpy(d, s, n);
    return 0;
}
int hipMemset(void *d, int v, size_t n) {
    std::memset(d, v, n);
    return 0;
}
int hipMemsetAsync(void *d, int v, size_t n, void *) {
    std::memset(d, v, n);
    return 0;
}
int hipGetSymbolAddress(void **p, const void *) {
    static void *mem = std::aligned_alloc(256, 64 << 20);
    *p = mem;
    return 0;
}
int hipGetDevice(int *d) {
    *d = 0;
    return 0;
}
int hipDeviceGetAttribute(int *v, int, int) {
    *v = 256;  // compute units are all that the library asks for
    return 0;
}
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipEventCreate(void **e) {
    *e = nullptr;
    return 0;
}
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *t, void *, void *) {
    *t = 0.0f;
    return 0;
}
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "recorded"; }
int hipStreamSynchronize(void *) { return 0; }
int hipDeviceSynchronize() { return 0; }
}
