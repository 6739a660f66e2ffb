// The HIP runtime functions that libhc.so calls, without a GPU: memory is host memory, a launch is written to a log, and one
// launch can be made to fail.  For tests of the host side: loaded (RTLD_GLOBAL) before libhc.so in a process of its own.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

static std::map<const void*, std::string> names;
static std::string log_text;
static std::map<std::string, size_t> first_size;             // of a kernel's first argument, where the test has said so
static std::vector<std::string> first_args;                  // of the launches in the log
static long fail_at = 0, taken = 0;
static hipError_t last_error = hipSuccess;
static struct { dim3 grid, block; size_t shared; hipStream_t stream; } config;

static hipError_t launch(const void* fn, dim3 g, dim3 b, void** args, size_t shared, hipStream_t st)
{
    if (fail_at > 0 && --fail_at == 0) return last_error = hipErrorLaunchFailure;
    log_text += names[fn] + " " + std::to_string(g.x) + " " + std::to_string(g.y) + " " + std::to_string(g.z) + " " + std::to_string(b.x) + " " +
                std::to_string(shared) + " " + std::to_string((size_t)st) + "\n";
    first_args.emplace_back((const char*)args[0], first_size.count(names[fn]) ? first_size[names[fn]] : 0);
    return hipSuccess;
}

extern "C" {
const char* fake_log() { return log_text.c_str(); }
void fake_reset(long fail) { log_text.clear(); first_args.clear(); fail_at = fail; last_error = hipSuccess; }
long fake_bytes() { return taken; }
void fake_first_size(const char* kernel, long bytes) { first_size[kernel] = (size_t)bytes; }
long fake_first_arg(long launch, void* to) { memcpy(to, first_args[launch].data(), first_args[launch].size()); return (long)first_args[launch].size(); }

void** __hipRegisterFatBinary(const void*) { return (void**)calloc(1, 8); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) { names[host] = device; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shared, hipStream_t st) { config = {g, b, shared, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shared, hipStream_t* st)
{
    *g = config.grid; *b = config.block; *shared = config.shared; *st = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 g, dim3 b, void** args, size_t shared, hipStream_t st) { return launch(fn, g, b, args, shared, st); }
hipError_t hipExtLaunchKernel(const void* fn, dim3 g, dim3 b, void** args, size_t shared, hipStream_t st, hipEvent_t, hipEvent_t, int) { return launch(fn, g, b, args, shared, st); }
hipError_t hipGetLastError() { const hipError_t e = last_error; last_error = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipMalloc(void** p, size_t n) { taken += (long)n; return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)calloc(1, 8); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) { memset(a, 0, sizeof(*a)); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char room[8 << 20]; *p = room; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) { memset(p, 0, sizeof(*p)); p->multiProcessorCount = 256; return hipSuccess; }
}
