#include "runtime.h"

#include <dlfcn.h>
#include <errno.h>
#include <pthread.h>

#include <cstdlib>
#include <cstring>
#include <new>

#include "flat.h"

// the launchers that these checks look at, in place of those that report a failure
#define slos_launch_select no_launch_select
#define slos_launch_layer no_launch_layer
#define slos_prepare_batch_kernels no_prepare_batch_kernels
#include "stubs.cpp"
#undef slos_launch_select
#undef slos_launch_layer
#undef slos_prepare_batch_kernels

FakeRuntime fake;
static constexpr size_t kHead = 64;

int slos_launch_select(const SelectParams &p, int, void *)
{
    fake.select = p;
    ++fake.selects;
    return 0;
}
int slos_launch_layer(const LayerParams &, const LayerLaunch &, void *) { return 0; }
int slos_prepare_batch_kernels() { return 0; }

// host memory that runs out once
void *operator new(size_t n)
{
    if (fake.news.load(std::memory_order_relaxed) >= 0 && fake.news.fetch_sub(1) == 0) throw std::bad_alloc();
    if (void *p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void *operator new(size_t n, const std::nothrow_t &) noexcept
{
    try {
        return operator new(n);
    } catch (std::bad_alloc &) {
        return nullptr;
    }
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

extern "C" {

// std::thread's, so that a system without room for another thread can be had
int pthread_create(pthread_t *t, const pthread_attr_t *a, void *(*f)(void *), void *arg)
{
    if (fake.no_threads) return EAGAIN;
    typedef int (*Create)(pthread_t *, const pthread_attr_t *, void *(*)(void *), void *);
    static const Create create = (Create)dlsym(RTLD_NEXT, "pthread_create");
    return create(t, a, f, arg);
}

hipError_t hipMalloc(void **p, size_t bytes)
{
    *p = nullptr;
    if (bytes > fake.budget || fake.used > fake.budget - bytes) return hipErrorOutOfMemory;
    size_t *head = (size_t *)malloc(bytes + kHead);  // its size goes before the block
    if (!head) return hipErrorOutOfMemory;
    *head = bytes;
    *p = (char *)head + kHead;
    fake.used += bytes;
    fake.peak = fake.peak < fake.used ? fake.used : fake.peak;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    size_t *head = (size_t *)((char *)p - kHead);
    fake.used -= *head;
    free(head);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned)
{
    return (*p = malloc(bytes)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    fake.copied = n;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n)
{
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDeviceCount(int *n)
{
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "stand-in runtime"; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

// not reached by the checks
hipError_t hipEventCreate(hipEvent_t *) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipErrorNotSupported; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }

} // extern "C"
