// The part of the HIP runtime that libhqr's host code calls, for tests without
// a GPU: device memory is host memory, nothing runs, and every launch, event
// and stream operation is written to a log.  One launch can be made to fail.
#include <hip/hip_runtime_api.h>

#include <cxxabi.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

std::string &text() { static std::string s; return s; }
std::map<const void *, std::string> &kernels() { static std::map<const void *, std::string> m; return m; }
std::map<const void *, int> &ids() { static std::map<const void *, int> m; return m; }
std::string fail_name;
int fail_nth = 0, fail_seen = 0;
hipError_t last = hipSuccess;

// streams and events by small numbers, in order of appearance; the null stream is 0
std::string id(const void *h)
{
    if (!h) return "0";
    auto it = ids().emplace(h, (int)ids().size() + 1).first;
    return std::to_string(it->second);
}

void say(const std::string &s) { text() += s + "\n"; }

} // namespace

extern "C" {

const char *host_log() { return text().c_str(); }
void host_clear() { text().clear(); }
// the nth launch (1 ..) of a kernel whose name contains `name` fails; nth 0: none
void host_fail(const char *name, int nth)
{
    fail_name = name;
    fail_nth = nth;
    fail_seen = 0;
}

void **__hipRegisterFatBinary(const void *) { static void *p; return &p; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *)
{
    int st = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    std::string s = d ? d : name;
    free(d);
    const size_t a = s.find("hqr::");
    s = s.substr(a == std::string::npos ? 0 : a + 5);
    kernels()[host] = s.substr(0, s.find('('));
}

static thread_local struct { dim3 g, b; size_t sh; hipStream_t s; } cfg;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s)
{
    cfg = {g, b, sh, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *s)
{
    *g = cfg.g;
    *b = cfg.b;
    *sh = cfg.sh;
    *s = cfg.s;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t, hipStream_t s)
{
    const std::string &k = kernels()[f];
    if (fail_nth && k.find(fail_name) != std::string::npos && ++fail_seen == fail_nth) {
        say("failed " + k);
        return last = hipErrorLaunchFailure;
    }
    std::string l = "launch " + k + " stream=" + id(s) + " grid=" + std::to_string(g.x) + " block=" + std::to_string(b.x);
    if (k.find("wg_batched") != std::string::npos) {
        // descriptors begin with (m, n): 88 bytes each
        const char *d = *(const char **)args[0];
        l += " rows=";
        for (int i = 0; i < *(const int *)args[1]; ++i) l += (i ? "," : "") + std::to_string(*(const int64_t *)(d + 88 * i));
        l += " head=" + std::to_string(*(const uintptr_t *)args[2]);
    }
    if (k.find("batched_lsq") != std::string::npos) l += " head=" + std::to_string(((const uintptr_t *)args[0])[2]);
    say(l);
    return hipSuccess;
}

hipError_t hipGetLastError()
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    say("wait stream=" + id(s) + " event=" + id(e));
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    say("record stream=" + id(s) + " event=" + id(e));
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0.0f; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t s)
{
    *p = malloc(n);
    say("alloc stream=" + id(s));
    return hipSuccess;
}
hipError_t hipFreeAsync(void *p, hipStream_t s)
{
    free(p);
    say("free stream=" + id(s));
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, hipMemcpyKind, hipStream_t)
{
    for (size_t i = 0; i < h; ++i) memcpy((char *)d + i * dp, (const char *)s + i * sp, w);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = malloc(1); return hipSuccess; }

} // extern "C"
