// A device that has no room for some buffers, for tests: loaded with
// RTLD_GLOBAL ahead of the HIP runtime, hipMalloc passes every request on to
// it, but one of more than the limit (or of the one size refused) as one that
// no device can grant, so that the runtime itself reports (and remembers) the
// failure.
#include <dlfcn.h>

#include <cstddef>
#include <cstdint>
#include <initializer_list>

namespace {
size_t limit = 0, refused = 0;  // bytes; 0: none
int64_t times = -1;              // how often the one size is refused; below 0: always
int64_t failed = 0;
}  // namespace

extern "C" {

void alloc_limit(uint64_t bytes) { limit = bytes; }
void alloc_refuse(uint64_t bytes, int64_t often) {
    refused = bytes;
    times = often;
}
int64_t alloc_failed() { return failed; }

int hipMalloc(void **p, size_t bytes) {
    using Fn = int (*)(void **, size_t);
    static const Fn real = [] {
        void *h = nullptr;
        for (const char *so : {"libamdhip64.so.7", "libamdhip64.so"})
            if (!h) h = dlopen(so, RTLD_NOLOAD | RTLD_LAZY);
        return h ? reinterpret_cast<Fn>(dlsym(h, "hipMalloc")) : nullptr;
    }();
    if (!real) return 3;  // not initialized
    const bool one = refused && bytes == refused && times != 0;
    if ((!limit || bytes <= limit) && !one) return real(p, bytes);
    if (one) --times;
    ++failed;
    const int rc = real(p, (size_t)1 << 60);
    if (rc == 0) *p = nullptr;
    return rc ? rc : 2;
}

}  // extern "C"
