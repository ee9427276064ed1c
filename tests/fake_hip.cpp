// Stand-in for the HIP runtime calls that the library makes, for tests without a GPU: nothing is allocated on a device or
// launched; every launch's dynamic LDS is checked against what was asked for the kernel with hipFuncSetAttribute last, and what was
// launched can be asked for.
#include <hip/hip_runtime.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

static std::map<const void *, std::string> &names()      // (the library registers its kernels while it is loaded)
{
    static std::map<const void *, std::string> m;
    return m;
}
static std::string launched;
static std::map<const void *, int> limits;
static int launches, big_launches, over_limit;
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } config;

extern "C" {

int fake_launches() { return launches; }              // since the library was loaded
int fake_big_launches() { return big_launches; }      // with more than the 64 KiB that need no request
int fake_over_limit() { return over_limit; }          // with more than was requested

const char *fake_launched()                           // since the last call: name/bytes of dynamic LDS, a blank behind each
{
    static std::string last;
    last.swap(launched);
    launched.clear();
    return last.c_str();
}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *) { names()[f] = name; }

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return posix_memalign(p, 4096, n) ? hipErrorOutOfMemory : hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = nullptr; return hipErrorInvalidSymbol; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v) { limits[f] = v; return hipSuccess; }

hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { config = {g, b, lds, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s)
{
    *g = config.grid; *b = config.block; *lds = config.lds; *s = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t lds, hipStream_t)
{
    ++launches;
    launched += names()[f] + '/' + std::to_string(lds) + ' ';
    if (lds <= 64 * 1024) return hipSuccess;
    ++big_launches;
    const auto it = limits.find(f);
    over_limit += it == limits.end() || lds > (size_t)it->second;
    return hipSuccess;
}

}
