// A device that lives in host memory, for tests of the library's host path on
// a machine without a GPU: the HIP calls libaq.so makes, with allocations in
// (lazily committed) host memory and launches that are checked against the
// launch limits but run nothing.  Loaded into the global symbol
// scope before libaq.so, its functions are the ones the library binds to.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>

#include <sys/mman.h>

namespace {

struct Dim {
    uint32_t x, y, z;
};
struct Launch {
    uint32_t grid[3], block[3];
    uint64_t lds;
};

constexpr int kOk = 0, kInvalidValue = 1, kInvalidConfiguration = 9, kOutOfMemory = 2;

std::map<void*, size_t> g_live;
size_t g_live_bytes = 0;
int64_t g_news = 0;
Launch g_launch[64];         // the first ones since the last reset
int64_t g_launches = 0;
int g_error = 0;          // what the next hipGetLastError reports
struct Config {
    Dim grid, block;
    size_t lds;
    void* stream;
} g_config;

}  // namespace

extern "C" {

int64_t host_live_bytes() { return (int64_t)g_live_bytes; }
int64_t host_news() { return g_news; }
int64_t host_launches() { return g_launches; }
void host_reset_launches() { g_launches = 0; }
void host_launch(int64_t i, uint64_t* out) {   // grid, block, dynamic LDS
    const Launch& l = g_launch[i & 63];
    for (int k = 0; k < 3; ++k) {
        out[k] = l.grid[k];
        out[3 + k] = l.block[k];
    }
    out[6] = l.lds;
}

int hipGetDeviceCount(int* n) { *n = 1; return kOk; }
int hipGetDevice(int* d) { *d = 0; return kOk; }
int hipGetLastError() {
    const int e = g_error;
    g_error = kOk;
    return e;
}
int hipDeviceSynchronize() { return kOk; }
const char* hipGetErrorString(int e) {
    return e == kInvalidConfiguration ? "invalid configuration" : e == kOutOfMemory ? "out of memory" : "host device error";
}
int hipMalloc(void** p, size_t bytes) {
    *p = nullptr;
    if (bytes == 0) return kOk;
    void* m = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return kOutOfMemory;
    g_live[m] = bytes;
    g_live_bytes += bytes;
    *p = m;
    return kOk;
}
int hipFree(void* p) {
    if (!p) return kOk;
    auto it = g_live.find(p);
    if (it == g_live.end()) return kInvalidValue;
    g_live_bytes -= it->second;
    munmap(p, it->second);
    g_live.erase(it);
    return kOk;
}
int hipMemcpy(void* dst, const void* src, size_t n, int) { std::memcpy(dst, src, n); return kOk; }
int hipMemset(void* dst, int v, size_t n) { std::memset(dst, v, n); return kOk; }
int hipFuncSetAttribute(const void*, int, int value) { return value <= 160 * 1024 ? kOk : kInvalidValue; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t lds) {
    *n = lds > 80 * 1024 ? 1 : 2;
    return kOk;
}
int hipEventRecordWithFlags(void*, void*, unsigned) { return kOk; }
int hipStreamIsCapturing(void*, int* status) { *status = 0; return kOk; }
int hipGetSymbolAddress(void** p, const void*) {
    static void* scratch = mmap(nullptr, size_t(64) << 20, PROT_READ | PROT_WRITE,
                                MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    *p = scratch;
    return kOk;
}

void** __hipRegisterFatBinary(const void*) {
    static void* module = nullptr;
    return &module;
}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void* stream) {
    g_config = Config{grid, block, lds, stream};
    return kOk;
}
int __hipPopCallConfiguration(Dim* grid, Dim* block, size_t* lds, void** stream) {
    *grid = g_config.grid;
    *block = g_config.block;
    *lds = g_config.lds;
    *stream = g_config.stream;
    return kOk;
}
int hipLaunchKernel(const void*, Dim grid, Dim block, void**, size_t lds, void*) {
    // the limits of a launch: threads of a block, threads along x, blocks along y and z, LDS
    if (!grid.x || !grid.y || !grid.z || block.x * block.y * block.z > 1024 ||
        (uint64_t)grid.x * block.x >= (uint64_t(1) << 32) || grid.y > 65536 || grid.z > 65536 || lds > 160 * 1024)
        return g_error = kInvalidConfiguration;
    if (g_launches < 64) g_launch[g_launches] = Launch{{grid.x, grid.y, grid.z}, {block.x, block.y, block.z}, lds};
    ++g_launches;
    return kOk;
}

}  // extern "C"

// host allocations of the library (it takes its operator new from here too)
void* operator new(size_t n) {
    ++g_news;
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void* operator new(size_t n, const std::nothrow_t&) noexcept {
    ++g_news;
    return std::malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
void operator delete(void* p, const std::nothrow_t&) noexcept { std::free(p); }
