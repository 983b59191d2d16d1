// A HIP runtime that runs nothing and writes down what it was asked, so that the library's host side can be
// tested without a device: loaded into a process ahead of the real runtime, it takes the library's calls.
// One line per call in the log; handles are checked; a launch that the hardware cannot describe (2^32 threads
// or more) fails as it does there.
#include <cxxabi.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

#include <hip/hip_runtime_api.h>

namespace {
std::string g_log, g_fail;
int g_fail_after = -1;
long g_next = 1;
hipError_t g_last = hipSuccess;
void* g_capturing = nullptr;
std::map<const void*, std::string> g_kernels;
std::set<const void*> g_live;
struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} g_config;

void note(const std::string& s) { g_log += s + "\n"; }
std::string id(const void* h) { return h ? std::to_string(reinterpret_cast<long>(h)) : "0"; }
template <typename T>
T make() {
    T h = reinterpret_cast<T>(g_next++);
    g_live.insert(h);
    return h;
}
void check(const void* h) {
    if (h && !g_live.count(h) && h != g_capturing && reinterpret_cast<long>(h) < 1000000) {
        std::fprintf(stderr, "handle %s is not alive\n", id(h).c_str());
        std::abort();
    }
}
// Whether this call of `what` is the one to fail.
bool fails(const char* what) {
    if (g_fail != what || g_fail_after < 0 || g_fail_after-- > 0) return false;
    g_last = hipErrorUnknown;
    return true;
}
}  // namespace

extern "C" {

const char* stub_log() { return g_log.c_str(); }
void stub_clear() { g_log.clear(); }
void stub_fail(const char* what, int after) { g_fail = what, g_fail_after = after; }
void stub_capturing(void* stream) { g_capturing = stream; }

void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(&g_config); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
    int st = 0;
    char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    std::string n = d ? d : name;
    std::free(d);
    size_t open = n.size();  // of the argument list
    for (int depth = 0; open > 0;) {
        --open;
        depth += (n[open] == ')') - (n[open] == '(');
        if (depth <= 0) break;
    }
    n.resize(open);
    if (n.compare(0, 5, "void ") == 0) n = n.substr(5);
    for (const char* ns : {"st::", "march_k::", "(anonymous namespace)::"})
        for (size_t p; (p = n.find(ns)) != std::string::npos;) n.erase(p, std::strlen(ns));
    for (size_t p; (p = n.find(' ')) != std::string::npos;) n.erase(p, 1);
    g_kernels[host] = n;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    g_config = {grid, block, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = g_config.grid, *block = g_config.block, *lds = g_config.lds, *s = g_config.stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void**, size_t, hipStream_t s) {
    check(s);
    if (fails("launch")) return g_last;
    if (uint64_t(grid.x) * block.x > 0xffffffffull) return g_last = hipErrorInvalidConfiguration;
    note("launch " + g_kernels[fn] + " " + std::to_string(grid.x) + " " + std::to_string(block.x) + " " + id(s));
    return hipSuccess;
}
hipError_t hipLaunchCooperativeKernel(const void* fn, dim3 grid, dim3 block, void** a, unsigned l, hipStream_t s) {
    return hipLaunchKernel(fn, grid, block, a, l, s);
}
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256
         : a == hipDeviceAttributeSharedMemPerBlockOptin || a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 163840 : 0;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int threads, size_t) {
    return *n = 1024 / threads > 0 ? 1024 / threads : 1, hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static char block[256];
    return *p = block, hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t st) {
    check(st);
    note("copy " + std::to_string(int(kind)) + " " + std::to_string(n) + " " + id(st));
    if (kind != hipMemcpyDeviceToDevice) std::memcpy(d, s, n);
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    if (fails("stream")) return g_last;
    *s = make<hipStream_t>();
    note("stream " + id(*s));
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    check(s);
    g_live.erase(s);
    note("stream- " + id(s));
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { return check(s), note("sync " + id(s)), hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    *st = s && s == g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    check(s), check(e);
    if (fails("wait")) return g_last;
    note("wait " + id(s) + " " + id(e));
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = make<hipEvent_t>();
    note("event " + id(*e));
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
    check(e);
    g_live.erase(e);
    note("event- " + id(e));
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    check(e), check(s);
    note("record " + id(e) + " " + id(s));
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { return check(e), hipSuccess; }
// (each interval a little shorter than the one before: a tuner keeps the last candidate it times)
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    static float t = 1000.0f;
    return *ms = t -= 0.01f, hipSuccess;
}

hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { return check(s), note("capture " + id(s)), hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
    check(s);
    *g = make<hipGraph_t>();
    note("captured " + id(s));
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
    check(g);
    *x = make<hipGraphExec_t>();
    note("exec " + id(*x));
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return check(g), g_live.erase(g), hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { return check(x), g_live.erase(x), note("exec- " + id(x)), hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) { return check(x), check(s), note("replay " + id(x) + " " + id(s)), hipSuccess; }

}  // extern "C"
