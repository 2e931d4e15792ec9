#include "_fake_hip.h"

#include <cxxabi.h>

#include <cstdlib>
#include <cstring>
#include <map>

namespace fake {
std::vector<Launch> launches;
std::vector<Limit> limits;
std::vector<size_t> mallocs;
int device = 0;

static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
std::vector<std::string> kernels()
{
    std::vector<std::string> all;
    for (auto &n : names()) all.push_back(n.second);
    return all;
}
static std::string name_of(const void *fn)
{
    auto it = names().find(fn);
    return it == names().end() ? "?" : it->second;
}
static hipError_t record(const void *fn, dim3 g, dim3 b, size_t lds)
{
    launches.push_back({name_of(fn), g, b, lds, device});
    return hipSuccess;
}
static struct { dim3 g, b; size_t lds; hipStream_t s; } pushed;
}  // namespace fake

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *dev, unsigned, void *, void *, dim3 *, dim3 *, int *)
{
    int st = 0;
    char *d = abi::__cxa_demangle(dev, nullptr, nullptr, &st);
    fake::names()[host] = d ? d : dev;
    std::free(d);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s)
{
    fake::pushed = {g, b, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s)
{
    *g = fake::pushed.g; *b = fake::pushed.b; *lds = fake::pushed.lds; *s = fake::pushed.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t) { return fake::record(f, g, b, lds); }
hipError_t hipExtLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t, hipEvent_t, hipEvent_t, int)
{
    return fake::record(f, g, b, lds);
}
hipError_t hipLaunchCooperativeKernel(const void *f, dim3 g, dim3 b, void **, unsigned lds, hipStream_t) { return fake::record(f, g, b, lds); }

hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v)
{
    fake::limits.push_back({fake::name_of(f), v, fake::device});
    return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) { *a = {}; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 2; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = fake::device; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 1;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }

hipError_t hipMalloc(void **p, size_t n)
{
    fake::mallocs.push_back(n);
    *p = std::calloc(n ? n : 1, 1);
    return hipSuccess;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(n, 1); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static double m[1 << 20]; *p = m; return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }

hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0.f; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "fake"; }
}
