// A stand-in for the HIP runtime, for tests of the library's host code on a
// machine without a GPU: two devices whose memory is the host's, streams that
// know their device, kernels that are recorded and not run.  Loaded before
// libile.so into the global scope, its functions take the runtime's place.
// As in the runtime, a launch on a stream of another device than the current
// one fails.  Any call can be made to fail (si_fail); every call is a line of
// si_log: name, current device, the stream's device (-1 for none, the current
// device for the null stream), then what the call adds.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Stream {
    int dev;
};

int g_dev = 0;
std::string g_log;
std::map<std::string, int> g_fail;                  // calls until the failing one
std::map<const void *, std::string> g_kernel;
std::map<const void *, size_t> g_size;

int dev_of(hipStream_t s) { return s ? reinterpret_cast<Stream *>(s)->dev : g_dev; }

// Records the call; the error it was told to give, else success.
hipError_t call(const char *name, int sdev, const std::string &more = "")
{
    char b[64];
    snprintf(b, sizeof(b), " %d %d ", g_dev, sdev);
    g_log += name + std::string(b) + more + "\n";
    auto it = g_fail.find(name);
    if (it == g_fail.end() || --it->second > 0) return hipSuccess;
    g_fail.erase(it);
    return hipErrorUnknown;
}

std::string num(size_t n) { return std::to_string(n); }

struct Conf {
    dim3 g, b;
    size_t lds;
    hipStream_t st;
} g_conf;

}  // namespace

extern "C" {

void si_fail(const char *name, int nth) { g_fail[name] = nth; }
const char *si_log() { return g_log.c_str(); }
void si_clear()
{
    g_log.clear();
    g_fail.clear();
}

void **__hipRegisterFatBinary(const void *)
{
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *)
{
    g_kernel[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st)
{
    g_conf = Conf{g, b, lds, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *st)
{
    *g = g_conf.g;
    *b = g_conf.b;
    *lds = g_conf.lds;
    *st = g_conf.st;
    return hipSuccess;
}
static hipError_t g_last = hipSuccess;
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3, void **args, size_t, hipStream_t st)
{
    const std::string &n = g_kernel[f];
    std::string more = n + " " + num(g.x);
    // the reductions' last argument: where the result goes
    if (n.find("k_red_small") != std::string::npos)
        more += *(void **)args[7] ? " result" : " none";
    else if (n.find("k_red_final") != std::string::npos)
        more += *(void **)args[5] ? " result" : " none";
    // the window starts' first argument: the geometry, n_q and s_max its words 4, 5
    else if (n.find("k_prep") != std::string::npos)
        more += " " + num(((const int *)args[0])[4]) + " " + num(((const int *)args[0])[5]);
    g_last = call("hipLaunchKernel", dev_of(st), more);
    if (g_last == hipSuccess && dev_of(st) != g_dev) g_last = hipErrorInvalidHandle;
    return g_last;
}
hipError_t hipGetLastError()
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }

hipError_t hipGetDeviceCount(int *n)
{
    *n = 2;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = g_dev;
    return hipSuccess;
}
hipError_t hipSetDevice(int d)
{
    if (d < 0 || d > 1) return hipErrorInvalidDevice;
    g_dev = d;
    return call("hipSetDevice", -1);
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 160 * 1024;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof(*p));
    strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = 160 * 1024;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static void *mem = calloc(1, (size_t)64 << 20);
    *p = mem;
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n)
{
    hipError_t e = call("hipMalloc", -1, num(n));
    if (e != hipSuccess) return hipErrorOutOfMemory;
    *p = calloc(1, n);
    g_size[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    hipError_t e = call("hipFree", -1, num(g_size[p]));
    free(p);
    return e;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = calloc(1, n);
    return call("hipHostMalloc", -1, num(n));
}
hipError_t hipHostFree(void *p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    hipError_t e = call("hipMemcpy", g_dev, num(n));
    if (e == hipSuccess) memcpy(d, s, n);
    return e;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    hipError_t e = call("hipMemcpyAsync", dev_of(st), num(n));
    if (e == hipSuccess) memcpy(d, s, n);
    return e;
}
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h,
                            hipMemcpyKind, hipStream_t st)
{
    hipError_t e = call("hipMemcpy2DAsync", dev_of(st), num(w * h));
    for (size_t i = 0; i < h && e == hipSuccess; i++)
        memcpy((char *)d + i * dp, (const char *)s + i * sp, w);
    return e;
}
hipError_t hipMemset(void *p, int v, size_t n)
{
    hipError_t e = call("hipMemset", g_dev, num(n));
    if (e == hipSuccess) memset(p, v, n);
    return e;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t st)
{
    hipError_t e = call("hipMemsetAsync", dev_of(st), num(n));
    if (e == hipSuccess) memset(p, v, n);
    return e;
}

hipError_t hipStreamCreate(hipStream_t *s)
{
    *s = reinterpret_cast<hipStream_t>(new Stream{g_dev});
    return call("hipStreamCreate", g_dev);
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    delete reinterpret_cast<Stream *>(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { return call("hipStreamSynchronize", dev_of(s)); }
hipError_t hipEventCreate(hipEvent_t *e)
{
    *e = reinterpret_cast<hipEvent_t>(new int(0));
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete reinterpret_cast<int *>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) { return call("hipEventRecord", dev_of(s)); }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.f;
    return hipSuccess;
}

hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { return call("hipStreamBeginCapture", dev_of(s)); }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g)
{
    *g = reinterpret_cast<hipGraph_t>(new int(0));
    return call("hipStreamEndCapture", dev_of(s));
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *x = reinterpret_cast<hipGraphExec_t>(new int(0));
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return call("hipGraphLaunch", dev_of(s)); }
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete reinterpret_cast<int *>(g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x)
{
    delete reinterpret_cast<int *>(x);
    return hipSuccess;
}

}  // extern "C"
