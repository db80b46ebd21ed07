// hipMalloc that reports out of memory above a size or at one call, and hipHostMalloc above a size, for a process that loads this library before
// the solver's (its symbols are found first). No GPU code.
#include <dlfcn.h>

#include <cstddef>

static size_t limit = ~size_t(0);
static int refused = 0, refuse_call = 0;

extern "C" void shim_limit(size_t bytes) { limit = bytes; }
extern "C" void shim_refuse_call(int k) { refuse_call = k; }  // the k-th from now (0: none)
extern "C" int shim_refused() { return refused; }

extern "C" int hipMalloc(void** p, size_t bytes) {
    static auto real = reinterpret_cast<int (*)(void**, size_t)>(dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY), "hipMalloc"));
    if (bytes > limit || (refuse_call > 0 && --refuse_call == 0)) {
        ++refused;
        return 2;  // hipErrorOutOfMemory
    }
    return real(p, bytes);
}

static size_t host_limit = ~size_t(0);

extern "C" void shim_host_limit(size_t bytes) { host_limit = bytes; }

extern "C" int hipHostMalloc(void** p, size_t bytes, unsigned flags) {
    static auto real = reinterpret_cast<int (*)(void**, size_t, unsigned)>(dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY), "hipHostMalloc"));
    if (bytes > host_limit) {
        ++refused;
        return 2;
    }
    return real(p, bytes, flags);
}
