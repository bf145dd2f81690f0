// A runtime of which nothing is real, for the library without a GPU: "device" memory is host memory, kernels do nothing, one value
// read back from the device is 3, longer reads give what is there (zeros).  The program's definitions take the place of the
// runtime's in the library.  From the call that `fail_from` counts down to on, everything that can fail does.
#pragma once

#include "fm.h"

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

static long fail_from = -1, launches = 0, failed = 0, captures = 0, replays = 0;
static bool capture_fails = false;
static std::map<void*, size_t> live;
static int last = 0;

static int can_fail()
{
    if (fail_from < 0 || --fail_from >= 0) return last = 0;
    fail_from = 0;  // and every call from here on
    ++failed;
    return last = 2;
}

struct Dim3 {
    uint32_t x, y, z;
};
extern "C" {
int hipGetDevice(int* d) { return *d = 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { const int e = last; last = 0; return e; }
const char* hipGetErrorString(int) { return "as the test wants"; }
int hipMalloc(void** p, size_t n)
{
    if (can_fail()) return 2;
    *p = calloc(n, 1);
    live[*p] = n;
    return 0;
}
int hipFree(void* p)
{
    if (live.erase(p) != 1) printf("freed twice\n"), abort();
    free(p);
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) { return (*p = calloc(n, 1)) == nullptr; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void*)
{
    if (can_fail()) return 2;
    const int64_t three = 3;
    memcpy(d, kind == 2 && n == 8 ? (const void*)&three : s, n);
    return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*)
{
    if (can_fail()) return 2;
    memset(d, v, n);
    return 0;
}
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void*) { return can_fail(); }
int hipStreamIsCapturing(void*, int* s) { return *s = 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*)
{
    static char block[1 << 16];
    *p = block;
    return 0;
}
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, void** st)
{
    *g = *b = Dim3{1, 1, 1};
    *s = 0;
    *st = nullptr;
    return 0;
}
int hipLaunchKernel(const void*, Dim3, Dim3, void**, size_t, void*)
{
    if (can_fail()) return 2;
    ++launches;
    return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g)
{
    ++captures;
    *g = capture_fails ? nullptr : malloc(1);
    return capture_fails ? 901 : 0;
}
int hipGraphInstantiate(void** x, void*, void**, char*, size_t) { *x = malloc(1); return 0; }
int hipGraphDestroy(void* g) { free(g); return 0; }
int hipGraphExecDestroy(void* x) { free(x); return 0; }
int hipGraphLaunch(void*, void*) { ++replays; return 0; }
}
