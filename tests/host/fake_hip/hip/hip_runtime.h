// A stand-in for the HIP runtime, for CPU tests of the library's host code.
// Device allocations are numbers without memory behind them, streams count the
// work put on them since they were last waited for, and any call that can fail
// may be made to: the one numbered fake::fail_at.
#pragma once

#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#define __device__
#define __host__
#define __align__(n) __attribute__((aligned(n)))
#define __forceinline__ inline
#define __shared__ static

// Device intrinsics of the elementary functions: a block of one thread, and the
// hardware's estimates of 1 / x and 1 / sqrt(x) off by fake::estimate_error.
namespace fake {
inline double estimate_error = 0;
inline double bits(uint64_t b)
{
    double x;
    memcpy(&x, &b, 8);
    return x;
}
inline uint64_t bits(double x)
{
    uint64_t b;
    memcpy(&b, &x, 8);
    return b;
}
} // namespace fake
struct FakeDim {
    unsigned x, y, z;
};
static const FakeDim threadIdx = {0, 0, 0};
inline void __syncthreads() {}
inline int __double2hiint(double x) { return (int)(fake::bits(x) >> 32); }
inline int __double2loint(double x) { return (int)(uint32_t)fake::bits(x); }
inline double __hiloint2double(int hi, int lo)
{
    return fake::bits((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
}
inline double fake_rcp(double x) { return (double)(1.0L / x * (1.0L + fake::estimate_error)); }
inline double fake_rsq(double x) { return (double)(1.0L / sqrtl(x) * (1.0L + fake::estimate_error)); }
// v_cvt_i32_f64 saturates and takes NaN to 0
inline double fake_ldexp(double x, double n)
{
    return n != n ? x : ldexp(x, (int)fmin(fmax(n, -2147483648.0), 2147483647.0));
}
#define __builtin_amdgcn_rcp fake_rcp
#define __builtin_amdgcn_rsq fake_rsq
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_ldexp(x, n) fake_ldexp(x, (double)(n))

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
typedef struct FakeStream *hipStream_t;
typedef struct FakeEvent *hipEvent_t;
constexpr unsigned hipStreamNonBlocking = 1;

namespace fake {
inline long calls = 0, fail_at = -1;
inline std::map<hipStream_t, int> pending; // work since the stream was last waited for
inline std::vector<std::string> faults;
inline uintptr_t next = 1u << 20;

inline hipError_t step() { return calls++ == fail_at ? hipErrorUnknown : hipSuccess; }
inline hipError_t work(hipStream_t s)
{
    const hipError_t e = step();
    if (e == hipSuccess)
        ++pending[s];
    return e;
}
inline void no_work(const char *what)
{
    for (auto &p : pending)
        if (p.second)
            faults.push_back(std::string(what) + " while a stream has work");
}
template <class P> inline hipError_t handle(P *out)
{
    const hipError_t e = step();
    if (e == hipSuccess)
        *out = (P)(next += 4096);
    return e;
}
} // namespace fake

inline const char *hipGetErrorString(hipError_t) { return "fake error"; }
inline hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
inline hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipMalloc(void **p, size_t) { return fake::handle(p); }
inline hipError_t hipFree(void *) { return fake::no_work("hipFree"), hipSuccess; }
inline hipError_t hipHostMalloc(void **p, size_t n)
{
    const hipError_t e = fake::step();
    if (e == hipSuccess)
        *p = calloc(1, n);
    return e;
}
inline hipError_t hipHostFree(void *p) { return fake::no_work("hipHostFree"), free(p), hipSuccess; }
inline hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned)
{
    const hipError_t e = fake::step();
    if (e == hipSuccess)
        *d = h;
    return e;
}
#define HIP_SYMBOL(x) (&(x))
inline hipError_t hipGetSymbolAddress(void **p, const void *) { return fake::handle(p); }
inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return fake::handle(s); }
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t s) { return fake::pending[s] = 0, hipSuccess; }
inline hipError_t hipEventCreate(hipEvent_t *e) { return fake::handle(e); }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t s) { return fake::work(s); }
inline hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 0, fake::step(); }
inline hipError_t hipMemcpyAsync(void *dst, const void *, size_t n, hipMemcpyKind k, hipStream_t s)
{
    const hipError_t e = fake::work(s);
    if (e == hipSuccess && k == hipMemcpyDeviceToHost)
        memset(dst, 0, n);
    return e;
}
