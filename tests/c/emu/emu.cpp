// emu.cpp -- memory and waves of the CPU build (see hip/hip_runtime.h).
#include <hip/hip_runtime.h>

#include <setjmp.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <ucontext.h>

#include <map>

#include "kvio_internal.h"

thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;

namespace {

constexpr size_t kPage = 4096;
struct Region {
    char *map;
    size_t mapped, bytes;
    int device;
};
std::map<uintptr_t, Region> &regions() {
    static std::map<uintptr_t, Region> r;
    return r;
}
const std::pair<const uintptr_t, Region> *find(const void *p) {
    auto it = regions().upper_bound(reinterpret_cast<uintptr_t>(p));
    if (it == regions().begin()) return nullptr;
    --it;
    return reinterpret_cast<uintptr_t>(p) < it->first + it->second.bytes ? &*it : nullptr;
}
[[noreturn]] void die(const char *why, const char *what) {
    fprintf(stderr, "emulated wave: %s at %s\n", why, what);
    abort();
}

}  // namespace

extern "C" {

// `bytes` of memory with an inaccessible page on both sides, as close to the
// one behind (at_end) or the one before it as 16-byte alignment allows.
void *emu_alloc(size_t bytes, int device, int at_end) {
    const size_t room = (bytes + kPage - 1) / kPage * kPage, mapped = room + 2 * kPage;
    char *m = static_cast<char *>(mmap(nullptr, mapped, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
    if (m == MAP_FAILED || mprotect(m + kPage, room, PROT_READ | PROT_WRITE) != 0) return nullptr;
    char *p = m + kPage + (at_end ? (room - bytes) / 16 * 16 : 0);
    regions()[reinterpret_cast<uintptr_t>(p)] = {m, mapped, bytes, device};
    return p;
}
void emu_free(void *p) {
    auto it = regions().find(reinterpret_cast<uintptr_t>(p));
    if (it == regions().end()) return;
    munmap(it->second.map, it->second.mapped);
    regions().erase(it);
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    const auto *r = find(p);
    if (r == nullptr) return hipErrorInvalidValue;
    a->type = r->second.device ? hipMemoryTypeDevice : hipMemoryTypeHost;
    a->devicePointer = const_cast<void *>(p);
    a->hostPointer = r->second.device ? nullptr : const_cast<void *>(p);
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p) {
    const auto *r = find(p);
    if (r == nullptr) return hipErrorInvalidValue;
    *base = reinterpret_cast<void *>(r->first);
    *size = r->second.bytes;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return (*p = emu_alloc(n, 1, 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { emu_free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return (*p = emu_alloc(n, 0, 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { emu_free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return hipSuccess; }

}  // extern "C"

namespace {

// One wave: 64 coroutines on stacks of their own, each entered once with
// makecontext and switched with setjmp / longjmp (no system call).
constexpr int kLanes = 64;
constexpr size_t kStack = 64 << 10;
struct Wave {
    ucontext_t start[kLanes], home;
    jmp_buf at[kLanes], back;
    char *stacks = nullptr;
    bool fresh[kLanes], done[kLanes];
    const char *what[kLanes];
    uint64_t value[2][kLanes];
    int phase[kLanes];
    int lane = 0;
    const std::function<void()> *body = nullptr;
    unsigned first_thread = 0;
};
Wave w;
void *kernarg = nullptr, *shared = nullptr;

void enter() {
    (*w.body)();
    w.done[w.lane] = true;
    _longjmp(w.back, 1);
}

void meet(const char *what) {
    w.what[w.lane] = what;
    if (_setjmp(w.at[w.lane]) == 0) _longjmp(w.back, 1);
}

void run_wave() {
    for (int l = 0; l < kLanes; ++l) {
        w.fresh[l] = true;
        w.done[l] = false;
        w.phase[l] = 0;
    }
    for (;;) {
        int ended = 0;
        for (int l = 0; l < kLanes; ++l) {
            w.lane = l;
            threadIdx.x = w.first_thread + static_cast<unsigned>(l);
            if (_setjmp(w.back) == 0) {
                if (w.fresh[l]) {
                    w.fresh[l] = false;
                    getcontext(&w.start[l]);
                    w.start[l].uc_stack.ss_sp = w.stacks + size_t(l) * kStack;
                    w.start[l].uc_stack.ss_size = kStack;
                    w.start[l].uc_link = nullptr;
                    makecontext(&w.start[l], enter, 0);
                    setcontext(&w.start[l]);
                } else {
                    _longjmp(w.at[l], 1);
                }
            }
            ended += w.done[l];
        }
        if (ended == kLanes) return;
        if (ended != 0) die("some lanes ended while others wait", w.what[w.done[0] ? 63 : 0]);
        for (int l = 1; l < kLanes; ++l)
            if (strcmp(w.what[l], w.what[0]) != 0 || w.phase[l] != w.phase[0]) die("lanes wait at different operations", w.what[l]);
    }
}

}  // namespace

uint64_t emu_exchange(uint64_t v, int from, const char *what) {
    const int p = w.phase[w.lane]++ & 1;
    w.value[p][w.lane] = v;
    meet(what);
    if (from >= 0) return w.value[p][from];
    for (int l = 1; l < kLanes; ++l)
        if (w.value[p][l] != w.value[p][0]) die("a value taken as wave-uniform is not", what);
    return w.value[p][0];
}

uint64_t emu_ballot(bool v, const char *what) {
    const int p = w.phase[w.lane]++ & 1;
    w.value[p][w.lane] = v;
    meet(what);
    uint64_t m = 0;
    for (int l = 0; l < kLanes; ++l) m |= w.value[p][l] << l;
    return m;
}

void *emu_kernarg() { return kernarg; }
void *emu_lds() { return shared; }

namespace {
int64_t launches = 0, last_tiles = 0, last_block = 0, last_waves = 0, last_pause = 0;
}
extern "C" int64_t emu_launches() { return launches; }
extern "C" int64_t emu_last_tiles() { return last_tiles; }    // of the last copy kernel
extern "C" int64_t emu_last_block() { return last_block; }
extern "C" int64_t emu_last_waves() { return last_waves; }
extern "C" int64_t emu_last_pause() { return last_pause; }    // behind a step of 256 vectors, in 64 cycles
// KiB that a default load of `bytes` (rows that fill their steps) keeps in flight.
extern "C" int64_t emu_default_load_kib(int64_t bytes, int layout) {
    const kvio::Shape s = kvio::default_shape(kvio::kLoad, bytes, layout, kvio::kTransposeBelow, 8, 256);
    return int64_t(s.workgroups) * (s.threads / 64) * s.tile_kib;
}

void emu_launch(dim3 grid, dim3 block, size_t lds, const std::function<void()> &lane, const void *arg, size_t bytes) {
    if (block.x == 0 || block.x % kLanes != 0 || grid.x == 0) die("launch shape", "launch");
    ++launches;
    if (bytes == sizeof(kvio::CopyArgs)) {
        const auto &a = *static_cast<const kvio::CopyArgs *>(arg);
        const int64_t one_layer = 2 * a.head_groups;
        last_tiles = a.total_tiles;
        last_block = block.x;
        last_waves = a.waves;
        last_pause = int64_t(a.pause) * 256 >> 16;
        if (a.planes > kvio::kMaxPlanes && a.planes > one_layer) die("more planes than a launch counts", "launch");
    }
    if (w.stacks == nullptr) w.stacks = static_cast<char *>(malloc(kLanes * kStack));
    kernarg = emu_alloc(bytes, 1, 1);
    memcpy(kernarg, arg, bytes);
    if (lds > 64 << 10) die("too much LDS", "launch");
    shared = lds ? emu_alloc(lds, 1, 1) : nullptr;
    gridDim = grid;
    blockDim = block;
    w.body = &lane;
    // The workgroups run last to first: nothing may depend on their order.
    for (unsigned b = grid.x; b-- > 0;)
        for (unsigned t = 0; t < block.x; t += kLanes) {
            blockIdx.x = b;
            w.first_thread = t;
            run_wave();
        }
    emu_free(kernarg);
    if (shared) emu_free(shared);
    kernarg = shared = nullptr;
}
