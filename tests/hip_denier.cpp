// Loaded ahead of liblbm.so in a process of its own, refuses pinned host memory
// or new host threads while it is told to, as a machine without them would.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <system_error>

static int pinned = 0, threads = 0, refused = 0;

extern "C" {
void deny(int no_pinned, int no_threads)
{
    pinned = no_pinned;
    threads = no_threads;
}
int denied() { return refused; }

hipError_t hipHostMalloc(void **p, size_t n, unsigned flags)
{
    if (pinned) return ++refused, hipErrorOutOfMemory;
    using Fn = hipError_t (*)(void **, size_t, unsigned);
    static const Fn next = (Fn)dlsym(dlopen("libamdhip64.so.7", RTLD_NOW | RTLD_NOLOAD), "hipHostMalloc");
    return next(p, n, flags);
}

// std::thread's start
void _ZNSt6thread15_M_start_threadESt10unique_ptrINS_6_StateESt14default_deleteIS1_EEPFvvE(void *self, void *state,
                                                                                         void (*depend)())
{
    if (threads) {
        ++refused;
        throw std::system_error(EAGAIN, std::generic_category());
    }
    using Fn = void (*)(void *, void *, void (*)());
    static const Fn next =
        (Fn)dlsym(RTLD_NEXT, "_ZNSt6thread15_M_start_threadESt10unique_ptrINS_6_StateESt14default_deleteIS1_EEPFvvE");
    next(self, state, depend);
}
}
