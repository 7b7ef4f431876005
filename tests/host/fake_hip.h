// A stand-in for the HIP runtime, for checks of the library's host code on a
// machine without a GPU: a program that includes this file once defines the
// runtime's functions itself, so the library it is linked to calls these.  Device
// memory is host memory whose addresses are never handed out twice; no kernel
// runs (but for the head counts that the GPU build's host part goes on with);
// every launch is checked for pointers into memory that has been freed.
#pragma once

#include <cxxabi.h>
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace fake {

struct Block {
    size_t bytes;
    int dev;
    bool live;
};

std::map<char *, Block> blocks;              // by address
// host stub -> demangled name, __device__ variable -> its memory (the library
// registers them before this program's own objects are constructed)
std::map<const void *, std::string> &kernels() { static std::map<const void *, std::string> m; return m; }
std::map<const void *, void *> &vars() { static std::map<const void *, void *> m; return m; }
size_t limit = (size_t)1 << 40, live_bytes = 0;
int device = 0, stale = 0, mallocs = 0, frees = 0, launches = 0;
bool capturing = false;                      // streams are being captured: nothing may wait
bool pending[2] = {};                        // work of a device that nothing has waited for
dim3 grid, block;                            // of the last launch
std::string last_stale;

const Block *find(const void *p)
{
    auto it = blocks.upper_bound((char *)p);
    if (it == blocks.begin()) return nullptr;
    --it;
    return (char *)p < it->first + it->second.bytes ? &it->second : nullptr;
}

// `p` is handed to what `who` names: it may not be in memory that has been freed
void check(const void *p, const std::string &who)
{
    const Block *b = find(p);
    if (!b || b->live) return;
    ++stale;
    last_stale = who;
}

// the kernel's arguments that its signature says are pointers
void check_args(const std::string &name, void **args)
{
    const size_t open = name.rfind('(');
    int depth = 0, i = 0;
    std::string one;
    for (size_t c = open + 1; c < name.size(); ++c) {
        const char ch = name[c];
        if ((ch == ',' || ch == ')') && depth == 0) {
            if (one.find('*') != std::string::npos) check(*(void **)args[i], name + " argument " + std::to_string(i));
            one.clear();
            ++i;
            if (ch == ')') break;
            continue;
        }
        depth += ch == '<' ? 1 : ch == '>' ? -1 : 0;
        one += ch;
    }
}

}  // namespace fake

extern "C" {

hipError_t hipMalloc(void **p, size_t bytes)
{
    if (fake::capturing) return hipErrorStreamCaptureUnsupported;
    if (fake::live_bytes + bytes > fake::limit) return hipErrorOutOfMemory;
    const size_t map = (bytes + 4096) / 4096 * 4096;
    *p = mmap(nullptr, map, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (*p == MAP_FAILED) abort();
    fake::blocks[(char *)*p] = {bytes, fake::device, true};
    fake::live_bytes += bytes;
    ++fake::mallocs;
    return hipSuccess;
}

hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    auto it = fake::blocks.find((char *)p);
    if (it == fake::blocks.end() || !it->second.live) {
        fprintf(stderr, "hipFree of what is not allocated\n");
        abort();
    }
    it->second.live = false;
    fake::live_bytes -= it->second.bytes;
    fake::pending[it->second.dev] = false;   // waits for the block's device
    madvise(p, (it->second.bytes + 4096) / 4096 * 4096, MADV_DONTNEED);
    ++fake::frees;
    return hipSuccess;
}

hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { *p = calloc(1, bytes); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    fake::check(d, "copy to");
    fake::check(s, "copy from");
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t)
{
    fake::pending[fake::device] = true;
    return hipMemcpy(d, s, n, k);
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    fake::check(d, "memset");
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize()
{
    if (fake::capturing) return hipErrorStreamCaptureUnsupported;
    fake::pending[fake::device] = false;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    if (fake::capturing) return hipErrorStreamCaptureUnsupported;
    fake::pending[fake::device] = false;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = fake::device; return hipSuccess; }
hipError_t hipSetDevice(int d) { fake::device = d; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st)
{
    *st = fake::capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)1; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }

hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, hipStream_t)
{
    const std::string &name = fake::kernels()[f];
    fake::check_args(name, args);
    fake::pending[fake::device] = true;
    fake::grid = grid;
    fake::block = block;
    ++fake::launches;
    if (name.find("tiles_kernel(") != std::string::npos && name.find("seg_tile") == std::string::npos) {
        // head counts of a tensor of one segment: hb[0] = 0, then 1
        const int64_t ntiles = *(int64_t *)args[3];
        int32_t *hb = *(int32_t **)args[4];
        for (int64_t t = 0; t <= ntiles; ++t) hb[t] = t > 0;
    }
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *sym)
{
    void *&a = fake::vars()[sym];
    if (!a) (void)hipMalloc(&a, (size_t)64 << 20);
    *p = a;
    return hipSuccess;
}

// what compiled device code registers at load, and a launch's configuration
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, uint3 *, uint3 *, dim3 *,
                           dim3 *, int *)
{
    int st = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    fake::kernels()[host] = st == 0 ? d : name;
    free(d);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
namespace fake_cfg { static dim3 g, b; static size_t sh; static hipStream_t st; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t st)
{
    fake_cfg::g = g; fake_cfg::b = b; fake_cfg::sh = sh; fake_cfg::st = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *st)
{
    *g = fake_cfg::g; *b = fake_cfg::b; *sh = fake_cfg::sh; *st = fake_cfg::st;
    return hipSuccess;
}

}  // extern "C"
