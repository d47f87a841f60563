// hip_runtime.h -- the part of the HIP API that libkvio.so uses, on the CPU:
// the library's sources, kernels included, compile against it unchanged (but
// for the inline-asm stores, which the test rewrites as plain stores), so their
// address arithmetic runs where an access out of bounds is a plain fault.
//
// Streams are synchronous.  A kernel runs wave by wave; the 64 lanes of a wave
// are coroutines that meet at every cross-lane operation, and it is an error if
// they do not all arrive at the same one.  Every allocation lies against an
// inaccessible page.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <functional>
#include <new>

#define __device__
#define __host__
#define __global__
#define __constant__
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (x)
#define HIP_DYNAMIC_SHARED(type, name) type *name = static_cast<type *>(emu_lds());
#define __builtin_amdgcn_fence(...) ((void)0)

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
extern thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;

typedef enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 } hipError_t;
typedef struct ihipStream_t *hipStream_t;
typedef struct ihipEvent_t *hipEvent_t;
typedef void *hipDeviceptr_t;
typedef enum { hipMemoryTypeHost = 0, hipMemoryTypeDevice = 2 } hipMemoryType;
typedef enum { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2, hipMemcpyDefault = 4 } hipMemcpyKind;
struct hipPointerAttribute_t {
    hipMemoryType type;
    int device;
    void *devicePointer, *hostPointer;
};
enum { hipEventDisableTiming = 2, hipStreamNonBlocking = 1 };
enum { hipHostMallocPortable = 1, hipHostMallocMapped = 2, hipHostMallocCoherent = 0x40000000 };
enum : unsigned { hipHostMallocNonCoherent = 0x80000000u };

extern "C" {
void *emu_alloc(size_t bytes, int device, int at_end);
void emu_free(void *p);
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p);
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p);
hipError_t hipMalloc(void **p, size_t n);
hipError_t hipFree(void *p);
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags);
hipError_t hipHostFree(void *p);
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k);
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st);
hipError_t hipMemset(void *d, int v, size_t n);
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char *hipGetErrorString(hipError_t) { return "error"; }
inline const char *hipGetErrorName(hipError_t) { return "hipError"; }
inline hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(new char);
    return hipSuccess;
}
inline hipError_t hipExtStreamCreateWithCUMask(hipStream_t *s, uint32_t, const uint32_t *) {
    return hipStreamCreateWithFlags(s, 0);
}
inline hipError_t hipStreamDestroy(hipStream_t s) { delete reinterpret_cast<char *>(s); return hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(new char);
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<char *>(e); return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
template <class T>
hipError_t hipGetSymbolAddress(void **p, T &sym) { *p = (void *)&sym; return hipSuccess; }

// ---------------------------------------------------------------- the device
void emu_launch(dim3 grid, dim3 block, size_t lds, const std::function<void()> &lane, const void *arg, size_t bytes);
uint64_t emu_exchange(uint64_t v, int from, const char *what);   // `from` < 0: every lane must bring the same
uint64_t emu_ballot(bool v, const char *what);
void *emu_kernarg();
void *emu_lds();

template <class First, class... Rest>
void emu_run(void (*k)(First, Rest...), dim3 grid, dim3 block, size_t lds, const First &first, const Rest &...rest) {
    emu_launch(grid, block, lds, [&] { k(first, rest...); }, &first, sizeof first);
}
#define hipLaunchKernelGGL(k, grid, block, lds, stream, ...) \
    emu_run(k, grid, block, lds, __VA_ARGS__)

inline int __shfl(int v, int lane) { return (int)emu_exchange((uint32_t)v, lane & 63, "shfl"); }
inline long long __shfl(long long v, int lane) { return (long long)emu_exchange((uint64_t)v, lane & 63, "shfl64"); }
inline uint32_t __builtin_amdgcn_readlane(uint32_t v, int lane) { return (uint32_t)emu_exchange(v, lane & 63, "readlane"); }
inline uint32_t __builtin_amdgcn_readfirstlane(uint32_t v) { return (uint32_t)emu_exchange(v, -1, "readfirstlane"); }
inline uint64_t __ballot(bool v) { return emu_ballot(v, "ballot"); }
inline void __builtin_amdgcn_wave_barrier() { emu_ballot(true, "wave_barrier"); }
inline bool __any(bool v) { return emu_ballot(v, "any") != 0; }
inline bool __all(bool v) { return emu_ballot(v, "all") == ~uint64_t(0); }
inline void __builtin_amdgcn_s_sleep(int) {}
inline void __builtin_amdgcn_s_barrier() {}      // waves run one after another and share nothing
inline void *__builtin_amdgcn_kernarg_segment_ptr() { return emu_kernarg(); }
template <class T>
T atomicCAS(T *p, T cmp, T val) { T old = *p; if (old == cmp) *p = val; return old; }
template <class T>
T atomicAdd(T *p, T val) { T old = *p; *p = old + val; return old; }
