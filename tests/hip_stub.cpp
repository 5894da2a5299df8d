// A stand-in for the HIP runtime, for tests of the library's host code on the CPU: device
// memory is host memory, kernels do not run, and every launch is written down.  Loaded
// with global symbols before the library, so that the library's calls come here.
#include <cstdint>
#include <cstdio>
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
    uint32_t grid, block;
    size_t lds;
    void *out;  // reduce_kernel: where it writes
    int levels; // kernels over one graph: levels of its table of tau0 ancestors
};
std::map<const void *, std::string> &names() {
    static std::map<const void *, std::string> m;
    return m;
}
std::vector<Launch> launches;
std::map<const void *, size_t> lds_limit;  // hipFuncAttributeMaxDynamicSharedMemorySize
std::string failing;                       // the call that fails next
Dim3 c_grid, c_block;
size_t c_lds;
void *c_stream;
size_t free_bytes = 64ull << 30;
int per_cu = 4;

int fails(const char *call) {
    if (failing != call) return 0;
    failing.clear();
    return 1;
}
}  // namespace

extern "C" {
// ---- for the tests
void stub_fail(const char *call) { failing = call; }
void stub_clear() { launches.clear(); }
void stub_set(size_t free_b, int blocks_per_cu) { free_bytes = free_b; per_cu = blocks_per_cu; }
int stub_launches() { return (int)launches.size(); }
const char *stub_name(int i) { return launches[(size_t)i].name.c_str(); }
int stub_grid(int i) { return (int)launches[(size_t)i].grid; }
int stub_levels(int i) { return launches[(size_t)i].levels; }
int stub_block(int i) { return (int)launches[(size_t)i].block; }
size_t stub_lds(int i) { return launches[(size_t)i].lds; }
size_t stub_limit(const char *kernel) {  // the dynamic LDS it may take (of one whose name holds this)
    for (const auto &l : lds_limit)
        if (names()[l.first].find(kernel) != std::string::npos) return l.second;
    return 0;
}
void *stub_out(int i) { return launches[(size_t)i].out; }

// ---- the runtime (0: hipSuccess, 1: hipErrorInvalidValue)
void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
    names()[host] = name;
}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void *s) {
    c_grid = g; c_block = b; c_lds = lds; c_stream = s;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *lds, void **s) {
    *g = c_grid; *b = c_block; *lds = c_lds; *s = c_stream;
    return 0;
}
static int last_error = 0;
int hipLaunchKernel(const void *f, Dim3 g, Dim3 b, void **args, size_t lds, void *) {
    Launch l{names()[f], g.x, b.x, lds, nullptr, -1};
    for (const char *k : {"tree_kernel", "frontier_kernel", "persistent_kernel"})  // GraphDev comes first, its last word
        if (l.name.find(k) != std::string::npos) memcpy(&l.levels, static_cast<char *>(args[0]) + 104, 4);
    if (l.name.find("reduce_kernel") != std::string::npos) l.out = *static_cast<void **>(args[4]);
    launches.push_back(l);
    if (lds > (64u << 10) && lds > lds_limit[f]) last_error = 1;
    return last_error;
}
int hipGetLastError() {
    const int e = last_error;
    last_error = 0;
    return e;
}
const char *hipGetErrorString(int e) { return e ? "stub error" : "no error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipGetDevicePropertiesR0600(void *, int) { return 1; }
int hipFuncSetAttribute(const void *f, int, int v) { lds_limit[f] = (size_t)v; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int, size_t) {
    // the one-wavefront kernels of the chain sampler are bound by their table's LDS
    const std::string &k = names()[f];
    *n = k.find("frontier") != std::string::npos || k.find("tree_kernel") != std::string::npos ? per_cu : 10;
    return 0;
}
int hipMemGetInfo(size_t *f, size_t *t) { *f = free_bytes; *t = free_bytes; return 0; }
int hipMalloc(void **p, size_t n) {
    if (fails("hipMalloc")) return 2;
    return (*p = calloc(1, n)) ? 0 : 2;
}
int hipMallocAsync(void **p, size_t n, void *) { return hipMalloc(p, n); }
int hipFree(void *p) { free(p); return 0; }
int hipFreeAsync(void *p, void *) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) {
    if (fails("hipHostMalloc")) return 2;
    return (*p = calloc(1, n)) ? 0 : 2;
}
int hipHostFree(void *p) { free(p); return 0; }
int hipHostGetDevicePointer(void **d, void *h, unsigned) {
    *d = nullptr;
    if (fails("hipHostGetDevicePointer")) return 1;
    *d = h;
    return 0;
}
int hipGetSymbolAddress(void **p, const void *) {
    static void *scratch = calloc(1, 256ull << 20);
    *p = scratch;
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { memcpy(d, s, n); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *) { memset(d, v, n); return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = nullptr; return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { *g = nullptr; return 0; }
int hipGraphInstantiate(void **e, void *, void *, void *, size_t) { *e = nullptr; return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipGraphLaunch(void *, void *) { return 0; }
}
