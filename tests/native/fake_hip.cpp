// A HIP runtime without a device, for tests of what the library asks of one:
// loaded with RTLD_GLOBAL ahead of the library it takes the place of the real
// runtime's calls.  Device memory is host memory that starts as zeros, copies
// are copies, and no kernel runs: a launch is only recorded.  It keeps two of
// the runtime's rules: a grid holds fewer than 2^32 threads in x, and the
// error of a failed call stays the thread's last error until it is asked for.
#include <sys/mman.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {

enum { kOk = 0, kInvalidValue = 1, kOutOfMemory = 2, kInvalidConfiguration = 9 };
struct Dim {
    uint32_t x, y, z;
};
struct Launch {
    std::string name;
    Dim grid, block;
    size_t shared;
};

std::recursive_mutex mu;
std::map<const void *, std::string> names;
std::vector<Launch> launches;
std::map<void *, size_t> blocks;
size_t limit = 0, in_use = 0, most = 0;  // limit: device bytes there are (0: any number)
uint32_t pack_amax = 0;                  // what k_pack16 finds as its rows' largest |element| (bits)
thread_local int last = kOk;
thread_local struct {
    Dim grid, block;
    size_t shared;
    void *stream;
} call;

int fail(int e) {
    last = e;
    return e;
}

int device_alloc(void **p, size_t bytes) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    *p = nullptr;
    if (limit && in_use + bytes > limit) return fail(kOutOfMemory);
    void *m = mmap(nullptr, bytes ? bytes : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return fail(kOutOfMemory);
    blocks[m] = bytes;
    in_use += bytes;
    if (in_use > most) most = in_use;
    *p = m;
    return kOk;
}

int device_free(void *p) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    auto it = blocks.find(p);
    if (!p) return kOk;
    if (it == blocks.end()) return fail(kInvalidValue);
    munmap(p, it->second ? it->second : 1);
    in_use -= it->second;
    blocks.erase(it);
    return kOk;
}

}  // namespace

extern "C" {

// for the test
void fake_limit(uint64_t bytes) { limit = bytes; }
void fake_amax(float v) { std::memcpy(&pack_amax, &v, 4); }
uint64_t fake_in_use() { return in_use; }
uint64_t fake_most() { return most; }
void fake_reset() {
    launches.clear();
    most = in_use;
}
int64_t fake_launches() { return (int64_t)launches.size(); }
const char *fake_launch(int64_t i, uint64_t *grid, uint64_t *block) {
    const Launch &l = launches[(size_t)i];
    *grid = (uint64_t)l.grid.x * l.grid.y * l.grid.z;
    *block = (uint64_t)l.block.x * l.block.y * l.block.z;
    return l.name.c_str();
}
uint64_t fake_shared(int64_t i) { return launches[(size_t)i].shared; }

// for the library
void **__hipRegisterFatBinary(const void *) {
    static void *module = nullptr;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t shared, void *stream) {
    call = {grid, block, shared, stream};
    return kOk;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *shared, void **stream) {
    *grid = call.grid;
    *block = call.block;
    *shared = call.shared;
    *stream = call.stream;
    return kOk;
}
int hipLaunchKernel(const void *f, Dim grid, Dim block, void **args, size_t shared, void *) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if ((uint64_t)grid.x * block.x >= 1ull << 32 || grid.x == 0 || block.x == 0) return fail(kInvalidConfiguration);
    launches.push_back({names[f], grid, block, shared});
    if (pack_amax && names[f].find("k_pack16") != std::string::npos)
        // its last argument, a PackStats: the largest |element| is the third word
        (*static_cast<uint32_t **>(args[10]))[2] = pack_amax;
    return kOk;
}
int hipMalloc(void **p, size_t bytes) { return device_alloc(p, bytes); }
int hipMallocAsync(void **p, size_t bytes, void *) { return device_alloc(p, bytes); }
int hipFree(void *p) { return device_free(p); }
int hipFreeAsync(void *p, void *) { return device_free(p); }
int hipHostMalloc(void **p, size_t bytes, unsigned) {
    *p = std::malloc(bytes ? bytes : 1);
    return *p ? kOk : fail(kOutOfMemory);
}
int hipHostFree(void *p) {
    std::free(p);
    return kOk;
}
int hipMemcpy(void *d, const void *s, size_t n, int) {
    std::memcpy(d, s, n);
    return kOk;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) {
    std::memcpy(d, s, n);
    return kOk;
}
int hipMemsetAsync(void *d, int v, size_t n, void *) {
    std::memset(d, v, n);
    return kOk;
}
int hipGetSymbolAddress(void **, const void *) { return fail(kInvalidValue); }
int hipDeviceGetAttribute(int *v, int, int) {
    *v = 256;
    return kOk;
}
int hipFuncSetAttribute(const void *, int, int) { return kOk; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *v, const void *, int, size_t shared) {
    // one wavefront each, five on a SIMD, 160 KB
    *v = (int)std::min<size_t>(20, (160u << 10) / std::max<size_t>(shared, 1));
    return kOk;
}
int hipGetDevice(int *d) {
    *d = 0;
    return kOk;
}
int hipSetDevice(int) { return kOk; }
int hipGetLastError() {
    const int e = last;
    last = kOk;
    return e;
}
const char *hipGetErrorString(int e) {
    return e == kOutOfMemory ? "out of memory" : e == kInvalidConfiguration ? "invalid configuration" : "error";
}
int hipEventCreate(void **e) {
    *e = nullptr;
    return kOk;
}
int hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void *) { return kOk; }
int hipEventElapsedTime(float *ms, void *, void *) {
    *ms = 1.f;
    return kOk;
}
int hipEventRecord(void *, void *) { return kOk; }
int hipEventSynchronize(void *) { return kOk; }
int hipStreamCreate(void **s) {
    *s = nullptr;
    return kOk;
}
int hipStreamDestroy(void *) { return kOk; }
int hipStreamSynchronize(void *) { return kOk; }

}  // extern "C"
