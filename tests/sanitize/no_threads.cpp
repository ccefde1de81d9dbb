// Preloaded into a test's process: once refuse_threads(1) is called, pthread_create fails as it does at
// the limit of processes.  Test infrastructure only.
#include <dlfcn.h>
#include <pthread.h>

#include <cerrno>

static bool g_refuse = false;

extern "C" void refuse_threads(int on) { g_refuse = on != 0; }

extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* x) {
    using Create = int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*);
    static const Create real = (Create)dlsym(RTLD_NEXT, "pthread_create");
    return g_refuse ? EAGAIN : real(t, a, f, x);
}
