// The HIP runtime calls that the library makes, as a recorder without a GPU:
// built as a libamdhip64.so.7 that a test process loads before the library, it
// keeps the name and grid of every launch, hands out addresses that nothing
// reads, and refuses what the test asks it to refuse.  For tests of the host
// side (dispatch rules, scratch sizes, error paths).
#include <cxxabi.h>

#include <cstdint>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>

struct Dim3 {
    uint32_t x, y, z;
};

namespace {
struct Launch {
    std::string name;
    Dim3 grid, block;
};
std::vector<Launch> launches;
std::map<const void*, std::string> kernels;
std::vector<std::pair<Dim3, Dim3>> configs;
std::vector<size_t> config_shm;
long refuse_at = -1;       // index of the launch to refuse
uint64_t malloc_limit = ~0ull, malloc_next = 1ull << 44;
int capture = 0, occupancy = 1;
constexpr int kErrorMemory = 2, kErrorLaunch = 719;
}  // namespace

extern "C" {
void rec_reset() { launches.clear(); refuse_at = -1; malloc_limit = ~0ull; capture = 0; }
void rec_refuse_launch(long i) { refuse_at = i; }
void rec_malloc_limit(uint64_t b) { malloc_limit = b; }
void rec_capture(int on) { capture = on; }
void rec_occupancy(int blocks) { occupancy = blocks; }
long rec_count() { return (long)launches.size(); }
const char* rec_name(long i) { return launches[i].name.c_str(); }
void rec_grid(long i, uint32_t* g) { g[0] = launches[i].grid.x, g[1] = launches[i].grid.y, g[2] = launches[i].block.x; }

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) {
    int st = 0;
    char* d = abi::__cxa_demangle(device, nullptr, nullptr, &st);
    kernels[host] = st == 0 && d ? d : device;
    free(d);
}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shm, void*) {
    configs.push_back({g, b});
    config_shm.push_back(shm);
    return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* shm, void** stream) {
    *g = configs.back().first, *b = configs.back().second, *shm = config_shm.back(), *stream = nullptr;
    configs.pop_back();
    config_shm.pop_back();
    return 0;
}
static int last_error = 0;
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void**, size_t, void*) {
    const bool no = (long)launches.size() == refuse_at;
    launches.push_back({no ? "refused" : kernels[f], g, b});
    return last_error = no ? kErrorLaunch : 0;
}
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = occupancy; return 0; }
int hipMalloc(void** p, size_t bytes) {
    if (bytes > malloc_limit) return last_error = kErrorMemory;
    *p = (void*)malloc_next;
    malloc_next += (bytes + 0xfffff) & ~(uint64_t)0xfffff;
    return 0;
}
int hipFree(void*) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)(1ull << 43); return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, int, void*) { return 0; }
int hipStreamIsCapturing(void*, int* st) { *st = capture; return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipExtStreamCreateWithCUMask(void** s, uint32_t, const uint32_t*) { *s = (void*)(1ull << 42); return 0; }
}
