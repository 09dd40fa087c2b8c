// launch_recorder.cpp -- a stand-in for the HIP runtime calls of libsslbm.so
// that records what would run, for tests on a machine without a GPU. Loaded
// with RTLD_GLOBAL before the library, its definitions are the ones the
// library binds to: device memory is host memory, every launch and copy is
// written down in order, and events read a clock that advances by a price per
// launch. Launched kernels do not run.
#include <cxxabi.h>
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

namespace {

struct Record {
    std::string name;  // demangled kernel, or "copy"
    unsigned grid = 0, block = 0;
    void *in = nullptr, *out = nullptr;  // first two arguments (a copy: source, destination)
    std::vector<unsigned char> args[12];
};

std::map<const void *, std::string> names;
std::vector<Record> records;
std::vector<std::pair<std::string, double>> prices;  // part of a name, ms a launch
double now_ms = 0.0;
bool device = true;  // device queries succeed
std::map<hipEvent_t, double> stamps;
int last_error = 0;
int queries = 0;  // of the current device

struct Config {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
};
std::vector<Config> configs;

}  // namespace

extern "C" {

// ---- what a test asks ------------------------------------------------------
int rec_count() { return (int)records.size(); }
const char *rec_name(int i) { return records[i].name.c_str(); }
unsigned rec_grid(int i) { return records[i].grid; }
unsigned rec_block(int i) { return records[i].block; }
void *rec_in(int i) { return records[i].in; }
void *rec_out(int i) { return records[i].out; }
void rec_clear() { records.clear(); }
void rec_price(const char *part, double ms) { prices.emplace_back(part, ms); }
void rec_device(int there) { device = there != 0; }
int rec_last_error() { return last_error; }
int rec_queries() { return std::exchange(queries, 0); }
// The 32-bit word at byte offset `at` of argument a of launch i.
int rec_arg(int i, int a, int at) {
    int v = 0;
    std::memcpy(&v, records[i].args[a].data() + at, 4);
    return v;
}
void *rec_arg_ptr(int i, int a) {
    void *v = nullptr;
    std::memcpy(&v, records[i].args[a].data(), 8);
    return v;
}

// ---- the runtime -----------------------------------------------------------
void __hipRegisterFunction(void **modules, const void *host, char *device_name, const char *name,
                           unsigned limit, void *tid, void *bid, void *block, void *grid,
                           int *size) {
    int status = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    names[host] = status == 0 ? d : name;
    std::free(d);
    using F = void (*)(void **, const void *, char *, const char *, unsigned, void *, void *,
                       void *, void *, int *);
    static const F real = (F)dlsym(RTLD_NEXT, "__hipRegisterFunction");
    if (real)
        real(modules, host, device_name, name, limit, tid, bid, block, grid, size);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
    configs.push_back({grid, block, shared, stream});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared,
                                     hipStream_t *stream) {
    const Config c = configs.back();
    configs.pop_back();
    *grid = c.grid;
    *block = c.block;
    *shared = c.shared;
    *stream = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t,
                           hipStream_t) {
    Record r;
    r.name = names.count(f) ? names[f] : "?";
    r.grid = grid.x * grid.y;
    r.block = block.x;
    std::memcpy(&r.in, args[0], 8);
    std::memcpy(&r.out, args[1], 8);
    // The arguments a test looks at: pointers among the first four, then
    // (the march) rows per wavefront, strips and wavefronts as integers.
    const int count = r.name.find("sslbm_march_kernel") != std::string::npos ? 7
                      : r.name.find("ensemble_") != std::string::npos        ? 4
                                                                             : 2;
    for (int a = 0; a < count; ++a)
        r.args[a].assign((unsigned char *)args[a], (unsigned char *)args[a] + (a < 4 ? 8 : 4));
    for (const auto &p : prices)
        if (r.name.find(p.first) != std::string::npos)
            now_ms += p.second;
    records.push_back(std::move(r));
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t, hipMemcpyKind, hipStream_t) {
    Record r;
    r.name = "copy";
    r.in = const_cast<void *>(src);
    r.out = dst;
    records.push_back(std::move(r));
    return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) {
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    ++queries;
    if (!device)
        last_error = hipErrorNoDevice;
    return device ? hipSuccess : hipErrorNoDevice;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 256;
    return device ? hipSuccess : hipErrorNoDevice;
}
// Registers of a march kernel, near enough for its wavefronts per SIMD.
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *f) {
    std::memset(a, 0, sizeof *a);
    char type[8] = "";
    int K = 0, V = 0;
    const std::string &name = names[f];
    const size_t at = name.find('<');
    if (at == std::string::npos ||
        std::sscanf(name.c_str() + at, "<%7[a-z], %d, %*[a-z], %d>", type, &K, &V) != 3)
        return hipErrorInvalidValue;
    const int words = type[0] == 'd' ? 2 : 1, regs = words * V * (15 * K + 35);
    a->numRegs = regs < 256 ? regs : 256;
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const int e = last_error;
    last_error = 0;
    return (hipError_t)e;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = (hipStream_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    std::free((void *)s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    stamps.erase(e);
    std::free((void *)e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
    stamps[e] = now_ms;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) {
    *ms = (float)(stamps[b] - stamps[a]);
    return hipSuccess;
}

}  // extern "C"
